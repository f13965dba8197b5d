// Masks and three-input bitwise operations of the evolution kernels.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace chsim {

// All ones if bit b (< 32) of x is set, else zero.
__device__ __forceinline__ uint32_t bit_mask(uint32_t x, uint32_t b) {
  return (uint32_t)__builtin_amdgcn_sbfe((int)x, b, 1u);
}

// Three-input bitwise operations by truth table (operands A, B, C; the table
// is the function's value on A = 0xF0, B = 0xCC, C = 0xAA).  On gfx950 these
// issue faster than selects, bit-field extracts and and-or, which the compiler
// would otherwise pick for masks derived from booleans.
enum : uint32_t {
  kSel = 0xCA,     // A ? B : C (bitwise)
  kAndXor = 0x6A,  // (A & B) ^ C
  kAnd3 = 0x80,    // A & B & C
  kAndOr = 0xEA    // (A & B) | C
};
template <uint32_t TT>
__device__ __forceinline__ uint32_t bop3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, TT);
}

}  // namespace chsim
