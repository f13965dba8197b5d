// Instantiations of the column mapping (evolve_cols.hpp): 8 lanes per term.
#include "evolve_cols.hpp"

namespace chsim {

hipError_t launch_evolve_c8(int cols, const EvolveJob& J, const DGate* gates, uint32_t n_gates, bool from_zero,
                             uint32_t* err, hipStream_t st) {
  switch (cols) {
#define CHSIM_COLS(C) \
  case C:             \
    return launch_cols_t<8, C>(J, gates, n_gates, from_zero, err, st);
    CHSIM_COLS(1) CHSIM_COLS(2) CHSIM_COLS(3) CHSIM_COLS(4)
    CHSIM_COLS(5) CHSIM_COLS(6) CHSIM_COLS(7) CHSIM_COLS(8)
#undef CHSIM_COLS
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace chsim
