// Instantiations of the column mapping (evolve_cols.hpp): 4 lanes per term, 11 to 16 columns per lane.
#include "evolve_cols.hpp"

namespace chsim {

hipError_t launch_evolve_c4b(int cols, const EvolveJob& J, const DGate* gates, uint32_t n_gates, bool from_zero,
                             uint32_t* err, hipStream_t st) {
  switch (cols) {
#define CHSIM_COLS(C) \
  case C:             \
    return launch_cols_t<4, C>(J, gates, n_gates, from_zero, err, st);
    CHSIM_COLS(11) CHSIM_COLS(12) CHSIM_COLS(13) CHSIM_COLS(14)
    CHSIM_COLS(15) CHSIM_COLS(16)
#undef CHSIM_COLS
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace chsim
