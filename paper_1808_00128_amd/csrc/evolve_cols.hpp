// CH-form evolution with the tableau columns in registers (step (a) of the hot
// path; the same gates and rules as evolve_kernel.hpp, another mapping).
//
// A term is a group of LPT adjacent lanes (64 / LPT terms per wave) and lane li
// of a term holds the columns li C .. li C + C - 1 of F, G and M, C =
// ceil(n / LPT): bit p of a column is the entry of row p.  The gate's qubits
// are uniform, so a left rule is a masked XOR at a uniform bit position of
// every column, and the right rules of the Hadamard update's V_C (Prop. H),
// whose qubits differ from term to term, act on whole columns.  With d = t + u,
// V_0 = d & ~v, V_1 = d & v, q the lowest bit of V_0 if V_0 != 0, else of V_1,
// and W the rest of that set, V_C is, over the n-bit words of columns (i a
// column),
//   V_1 case:  G_i ^= G_q, M_i ^= M_q for i in W;  F_q ^= XOR_{i in W} F_i;
//   V_0 case:  F_i ^= F_q for i in W, M_i ^= F_q for i in V_1;
//              G_q ^= XOR_{i in W} G_i;
//              M_q ^= XOR_{i in W} M_i + XOR_{i in V_1} F_i;
//              gamma += 2 F_q & XOR_{i in V_1} F_i;
//   then R[S_q] if a:  M_q ^= F_q, gamma -= F_q (the new F_q).
// No parity per row is left: a column costs a few three-input operations.
// Every register index is a compile-time constant, and nothing of the state
// is in LDS (it only serves the bit transpose at a span's ends, since the
// term store keeps rows).  gamma is held as two n-bit planes in every lane of
// the term; v and s as the C bits of the lane's columns.
//
// Row q of a matrix, one bit per column, is gathered into C bits per lane
// (rotate and select), so that t, u, alpha, beta and the choice of q cost a
// few operations on one word per lane; counts and bits are combined over the
// term's lanes by DPP moves within a row of 16 lanes.
//
// What bounds it: VALU issue, about 24 C + 65 instructions per Hadamard, 8 C per
// CX, 4 C per CZ, C per S, each for the wave's 64 / LPT terms.  On gfx950 a lone
// wave issues one VALU instruction per 8.6 cycles and two waves of a SIMD one
// per 4.4; from four waves on, XOR and three-input operations on registers take
// 2.6 cycles, bit-field extracts, rotates, counts, DPP moves and anything with a
// scalar register operand 4.4 (independent chains of one instruction each).  Four
// lanes per term do the least work per term (the part of a Hadamard outside
// the columns is shared by 16 terms); more lanes shorten a gate's chain for
// few terms.  Two lanes per term would leave two waves per SIMD.
//
// Measured (n = 50, 65536 terms, per gate; rows in LDS before, 8 lanes): H 3.3 us,
// CX 0.89 (0.95), CZ 0.47 (0.77), S 0.25 (0.78).  The last span of the n = 50
// workload, 65536 terms: 1.12 ms against 1.37 ms under the profiler.
#pragma once

#include <type_traits>

#include "bitops.hpp"
#include "device_common.hpp"
#include "internal.hpp"

namespace chsim {
namespace {

constexpr uint32_t kColWaves = 4;  // waves per workgroup

// The rows in LDS are written and read as 64-bit words and transposed as 32-bit
// halves: both views may alias.
typedef uint32_t __attribute__((may_alias)) lds_u32;
typedef uint64_t __attribute__((may_alias)) lds_u64;

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xF, 0xF, true);
}
// Combine x over the LPT lanes of a term (the result in every lane): quads by
// lane ^ 1 and lane ^ 2, then half-row and row mirrors.
template <int LPT, typename Op>
__device__ __forceinline__ uint32_t group_all(uint32_t x, Op op) {
  x = op(x, dpp32<0xB1>(x));
  x = op(x, dpp32<0x4E>(x));
  if (LPT >= 8) x = op(x, dpp32<0x141>(x));
  if (LPT >= 16) x = op(x, dpp32<0x140>(x));
  return x;
}
template <int LPT>
__device__ __forceinline__ uint32_t group_or(uint32_t x) {
  return group_all<LPT>(x, [](uint32_t a, uint32_t b) { return a | b; });
}
template <int LPT>
__device__ __forceinline__ uint32_t group_xor(uint32_t x) {
  return group_all<LPT>(x, [](uint32_t a, uint32_t b) { return a ^ b; });
}
template <int LPT>
__device__ __forceinline__ uint32_t group_add(uint32_t x) {
  return group_all<LPT>(x, [](uint32_t a, uint32_t b) { return a + b; });
}

// All ones if x != 0 (x < 2^31).
__device__ __forceinline__ uint32_t nonzero_mask(uint32_t x) { return (uint32_t)((int32_t)(0u - x) >> 31); }

// a[k] bit c -> a[c] bit k.
__device__ __forceinline__ void transpose32(uint32_t (&a)[32]) {
  uint32_t m = 0x0000FFFFu;
#pragma unroll
  for (int j = 16; j != 0; j >>= 1) {
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      if (k & j) continue;
      const uint32_t t = ((a[k] >> j) ^ a[k + j]) & m;
      a[k] ^= t << j;
      a[k + j] ^= t;
    }
    m ^= m << (j >> 1);
  }
}

// Bit transpose of a term's matrix in LDS (Rt[0 .. 32 KW), bits 0 .. 32 KW):
// lane li < KW^2 of the term takes one 32 x 32 block and writes it where another
// lane's was, after every lane's reads.
template <int KW>
__device__ __forceinline__ void transpose_lds(lds_u64* Rt, uint32_t li) {
  if (li < (uint32_t)(KW * KW)) {
    const uint32_t rh = li % KW, ch = li / KW;
    lds_u32* const w = reinterpret_cast<lds_u32*>(Rt);
    uint32_t a[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) a[k] = w[(32u * rh + (uint32_t)k) * 2u + ch];
    transpose32(a);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 32; ++k) w[(32u * ch + (uint32_t)k) * 2u + rh] = a[k];
  }
  wave_sync();
}

// Words of LDS per term: its rows and one of padding, so that the terms of a
// wave start in different banks.
template <int KW>
constexpr uint32_t col_pitch() {
  return 32u * KW + 1u;
}

template <int LPT, int C, int KW>
struct Cols {
  uint32_t w[KW][C];  // half, column

  __device__ __forceinline__ void load(lds_u64* Rt, uint32_t li, uint32_t n, const uint64_t* src, uint64_t rs) {
    for (uint32_t p = li; p < 32u * KW; p += LPT) Rt[p] = p < n ? src[(uint64_t)p * rs] : 0ull;
    wave_sync();
    transpose_lds<KW>(Rt, li);
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const lds_u32* const x = reinterpret_cast<const lds_u32*>(Rt + li * C + j);
#pragma unroll
      for (int k = 0; k < KW; ++k) w[k][j] = x[k];
    }
    wave_sync();
  }
  __device__ __forceinline__ void store(lds_u64* Rt, uint32_t li, uint32_t n, uint64_t* dst, uint64_t rs, bool live) {
    for (uint32_t p = LPT * C + li; p < 32u * KW; p += LPT) Rt[p] = 0ull;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      lds_u32* const x = reinterpret_cast<lds_u32*>(Rt + li * C + j);
      x[0] = w[0][j];
      x[1] = KW == 2 ? w[KW - 1][j] : 0u;
    }
    wave_sync();
    transpose_lds<KW>(Rt, li);
    if (live)
      for (uint32_t p = li; p < n; p += LPT) dst[(uint64_t)p * rs] = Rt[p];
    wave_sync();
  }
};

// f(half) with half = 0 or 1 as a compile-time constant (wave-uniform hi).
template <int KW, typename Fn>
__device__ __forceinline__ void with_half(bool hi, Fn f) {
  if constexpr (KW == 1) {
    f(std::integral_constant<int, 0>{});
  } else {
    if (hi) f(std::integral_constant<int, 1>{});
    else f(std::integral_constant<int, 0>{});
  }
}

template <int LPT, int C>
constexpr int col_waves() {
  return evolve_cols_waves(LPT, C);
}

template <int LPT, int C>
__global__ __launch_bounds__(256, (col_waves<LPT, C>())) void k_evolve_cols(EvolveJob J, const DGate* __restrict__ gates, uint32_t n_gates,
                                                     uint32_t from_zero, uint32_t* __restrict__ err) {
  constexpr uint32_t T = 64 / LPT;  // terms per wave
  constexpr int KW = LPT * C > 32 ? 2 : 1;
  const uint64_t count = J.count_dev ? (uint64_t)*J.count_dev : J.count;
  const uint32_t lane = threadIdx.x & 63u, wave = uniform32(threadIdx.x >> 6);
  const uint64_t wave0 = ((uint64_t)blockIdx.x * kColWaves + wave) * T;
  if (wave0 >= count) return;  // whole waves; no barrier follows
  constexpr uint32_t pitch = col_pitch<KW>();
  __shared__ uint64_t lds_rows[kColWaves * T * pitch];
  const uint32_t n = J.dst.n;
  const uint32_t tw = lane / LPT, li = lane % LPT;
  lds_u64* const Rt = lds_rows + (wave * T + tw) * pitch;
  const uint64_t item = wave0 + tw;
  const bool live = item < count;
  // Groups past the last term evolve a copy of item 0 and store nothing.
  const uint64_t it = live ? item : 0;
  const uint64_t sa = J.src_idx ? (uint64_t)J.src_idx[it] : it;  // input state
  const uint64_t ba = J.br_idx ? (uint64_t)J.br_idx[it] : it;    // branch choices
  const uint64_t chb = J.chi_br;
  const uint8_t* __restrict__ branch = J.branch;

  Cols<LPT, C, KW> F, G, M;
  uint32_t glo[KW], ghi[KW];
  uint32_t v, s, w, e = 0u;
#pragma unroll
  for (int k = 0; k < KW; ++k) glo[k] = ghi[k] = 0u;
  if (from_zero) {
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const uint32_t i = li * C + j;
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        F.w[k][j] = G.w[k][j] = i < n && (i >> 5) == (uint32_t)k ? 1u << (i & 31u) : 0u;
        M.w[k][j] = 0u;
      }
    }
    v = s = w = 0u;
  } else {
    F.load(Rt, li, n, J.src.F + sa * J.src_is, J.src_rs);
    G.load(Rt, li, n, J.src.G + sa * J.src_is, J.src_rs);
    M.load(Rt, li, n, J.src.M + sa * J.src_is, J.src_rs);
    for (uint32_t p = li; p < n; p += LPT) {
      const uint32_t g = J.src.gamma[(uint64_t)p * J.src_rs + sa * J.src_is], b = p & 31u;
#pragma unroll
      for (int k = 0; k < KW; ++k)
        if ((p >> 5) == (uint32_t)k) {
          glo[k] |= (g & 1u) << b;
          ghi[k] |= ((g >> 1) & 1u) << b;
        }
    }
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      glo[k] = group_or<LPT>(glo[k]);
      ghi[k] = group_or<LPT>(ghi[k]);
    }
    const uint32_t cm = (1u << C) - 1u;  // C <= 16
    v = (uint32_t)(J.src.v[sa] >> (li * C < 64u ? li * C : 0u)) & (li * C < 64u ? cm : 0u);
    s = (uint32_t)(J.src.s[sa] >> (li * C < 64u ? li * C : 0u)) & (li * C < 64u ? cm : 0u);
    w = (uint32_t)J.src.omega[sa];
  }
  const uint32_t lane_bit = 1u << li;

  // Hadamard on qubit p: Eqs. (H2), (H4), the t = u case, Prop. H.  A term for
  // which the gate is off (onm zero) takes it with a zero row, which changes nothing
  // (no branch per term: the loop's control flow stays uniform).
  auto hadamard = [&](uint32_t p, uint32_t onm) {
    // Row p, one bit per column of the lane, and gamma_p.
    uint32_t Fb = 0u, Gb = 0u, Mb = 0u, gp = 0u;
    with_half<KW>(p >= 32u, [&](auto half) {
      constexpr int h = decltype(half)::value;
      const uint32_t b = p & 31u;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const uint32_t r = b - (uint32_t)j;  // rotates bit b to bit j
        Fb = bop3<kAndOr>(__builtin_amdgcn_alignbit(F.w[h][j], F.w[h][j], r), 1u << j, Fb);
        Gb = bop3<kAndOr>(__builtin_amdgcn_alignbit(G.w[h][j], G.w[h][j], r), 1u << j, Gb);
        Mb = bop3<kAndOr>(__builtin_amdgcn_alignbit(M.w[h][j], M.w[h][j], r), 1u << j, Mb);
      }
      gp = ((glo[h] >> b) & 1u) | (((ghi[h] >> b) & 1u) << 1);
    });
    Fb &= onm;
    Gb &= onm;
    Mb &= onm;
    // t = s + G_p v, u = s + F_p ~v + M_p v: d = t + u is F_p on ~v (V_0) and
    // G_p + M_p on v (V_1); alpha = G_p ~v s, alpha + beta = (G_p + M_p) ~v s +
    // F_p v (M_p + s) (mod 2).  Four counts over the term in one word.
    const uint32_t GM = Gb ^ Mb;
    const uint32_t V0 = Fb & ~v, V1 = GM & v, t = s ^ (Gb & v), nvs = ~v & s;
    uint32_t R = (uint32_t)__popc(Gb & nvs) + ((uint32_t)__popc((GM & nvs) ^ (Fb & v & (Mb ^ s))) << 8) +
                 ((uint32_t)__popc(V0) << 16) + ((uint32_t)__popc(V1) << 24);
    R = group_add<LPT>(R);
    // From here every condition is a mask (all ones or zero): selects on VCC
    // cost up to 16 cycles each when several follow one compare.
    const uint32_t u0 = nonzero_mask(R & 0x00FF0000u);  // V_0 case
    const uint32_t some = nonzero_mask(R >> 16);        // t != u
    const uint32_t alpha = R & 1u;
    const uint32_t d0 = bit_mask(gp, 0u), d1 = bit_mask(gp, 1u) ^ bit_mask(R, 8u);  // delta's bits
    // q, the lowest column of X: eq is its bit in the lane that holds it, else 0.
    const uint32_t X = bop3<kSel>(u0, V0, V1), d = V0 | V1;
    const uint32_t holders = group_or<LPT>(nonzero_mask(X) & lane_bit);
    const uint32_t eq = X & (0u - X) & ~nonzero_mask(holders & (lane_bit - 1u));
    const uint32_t tq = nonzero_mask(group_or<LPT>(t & eq));
    // H^{v_q}(|y_q> + i^delta |1 - y_q>) = 2^{1/2} e^{i pi dw/4} S^a H^b |c> with
    // v_q = 1 in the V_1 case and 0 in the V_0 case.  For y_q = 1, i^delta is
    // factored out and delta negated: its bits become d0 and p1.
    //   V_0: b = 1, a = d0, c = p1;  V_1: b = a = d0, c = p1 + d0 and a further
    //   e^{+-i pi/4} for odd delta.  With t = u (e_q = 0) only the phase
    //   e^{+-i pi/4} = 2^{-1/2} (1 + i^delta) stays, delta odd.
    const uint32_t p1 = d1 ^ (d0 & tq);
    const uint32_t am = d0 & some;
    const uint32_t bm = u0 | d0, ccm = p1 ^ (d0 & ~u0);
    const uint32_t dw = onm & ((tq & ((d0 & 2u) + (d1 & 4u))) + (~u0 & d0 & (1u | (p1 & 6u))));
    e |= onm & ~some & ~d0;
    const uint32_t W = X & ~eq, W0 = W & u0;
    uint32_t X1 = bop3<kSel>(u0, V1, W), eqb = eq;
    if (__ballot(some != 0u) != 0ull) {
      const bool general = __ballot(W0 != 0u) != 0ull;  // some term's V_0 case has a batch W
      // Columns q of G, F and of F (V_0) or M (V_1), to every lane of the term.
      uint32_t Fq[KW], Gq[KW], Mq[KW], A1[KW];
#pragma unroll
      for (int k = 0; k < KW; ++k) Fq[k] = Gq[k] = Mq[k] = A1[k] = 0u;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const uint32_t em = bit_mask(eq, j), xm = bit_mask(X1, j);
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          Fq[k] = bop3<kAndOr>(em, F.w[k][j], Fq[k]);
          Gq[k] = bop3<kAndOr>(em, G.w[k][j], Gq[k]);
          Mq[k] = bop3<kAndOr>(em, M.w[k][j], Mq[k]);
          A1[k] = bop3<kAndXor>(xm, F.w[k][j], A1[k]);  // XOR over W (V_1) or V_1 (V_0) of F
        }
      }
      uint32_t S[KW], Z[KW], AF[KW];
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        Fq[k] = group_or<LPT>(Fq[k]);
        Gq[k] = group_or<LPT>(Gq[k]);
        Mq[k] = group_or<LPT>(Mq[k]);
        A1[k] = group_xor<LPT>(A1[k]);
        S[k] = bop3<kSel>(u0, Fq[k], Mq[k]);
        Z[k] = A1[k];
      }
      if (general) {
        uint32_t A0[KW], AG[KW];
#pragma unroll
        for (int k = 0; k < KW; ++k) A0[k] = AG[k] = 0u;
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const uint32_t wm = bit_mask(W0, j);
#pragma unroll
          for (int k = 0; k < KW; ++k) {
            AG[k] = bop3<kAndXor>(wm, G.w[k][j], AG[k]);
            A0[k] = bop3<kAndXor>(wm, M.w[k][j], A0[k]);
            F.w[k][j] = bop3<kAndXor>(wm, Fq[k], F.w[k][j]);
          }
        }
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          AG[k] = group_xor<LPT>(AG[k]);
          Z[k] ^= group_xor<LPT>(A0[k]);
        }
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const uint32_t em = bit_mask(eq, j);
#pragma unroll
          for (int k = 0; k < KW; ++k) G.w[k][j] = bop3<kAndXor>(em, AG[k], G.w[k][j]);
        }
      }
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        Gq[k] &= ~u0;                                // G gains G_q on W in the V_1 case only
        AF[k] = A1[k] & ~u0;                         // F_q gains this
        const uint32_t f1 = am & (Fq[k] ^ AF[k]);    // R[S_q]
        Z[k] = bop3<kAndXor>(u0, Z[k], f1);          // M_q gains this
        ghi[k] ^= bop3<kAnd3>(u0, Fq[k], A1[k]);     // gamma += 2
        ghi[k] ^= f1 & ~glo[k];                      // gamma -= 1
        glo[k] ^= f1;
      }
      // The column masks are formed again: kept, they would take 2 C registers.
      asm("" : "+v"(eqb), "+v"(X1));
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const uint32_t em = bit_mask(eqb, j), xm = bit_mask(X1, j);
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          G.w[k][j] = bop3<kAndXor>(xm, Gq[k], G.w[k][j]);
          M.w[k][j] = bop3<kAndXor>(xm, S[k], M.w[k][j]);
          M.w[k][j] = bop3<kAndXor>(em, Z[k], M.w[k][j]);
          F.w[k][j] = bop3<kAndXor>(em, AF[k], F.w[k][j]);
        }
      }
    }
    // s' = y with bit q set to c, y = t, or u + e_q when t_q = 1 (y agrees with
    // t + t_q d off bit q); v' = v with bit q set to b.
    s = bop3<kSel>(eq, ccm, t ^ (tq & d));
    v = bop3<kSel>(eq, bm, v);
    w = (w + 4u * alpha + dw) & 7u;
  };

  // gamma_q += a (mod 4); qb: the qubit's bit (zero where the gate does not act).
  auto gamma_add = [&](auto half, uint32_t qb, uint32_t a) {
    constexpr int h = decltype(half)::value;
    const uint32_t a0 = (a & 1u) ? qb : 0u, a1 = (a & 2u) ? qb : 0u;
    ghi[h] ^= a1 ^ (a0 & glo[h]);
    glo[h] ^= a0;
  };

  const uint2* __restrict__ g2 = reinterpret_cast<const uint2*>(gates);
  const uint32_t* __restrict__ seq = J.slot_seq;
  const uint32_t n_occ = J.n_occ;
  uint32_t next_b = n_occ ? (uint32_t)branch[(uint64_t)seq[0] * chb + ba] : 0u;
  uint32_t cur_b = 0u, occ = 1u;
  // Gates are two 32-bit words read on the scalar unit, the next one in flight
  // while the current one is applied (the device list has one padding entry
  // past its last gate, so the read past a span's end is in bounds).
  uint2 nxt = n_gates ? g2[0] : make_uint2(0u, 0u);
  for (uint32_t i = 0; i < n_gates; ++i) {
    const uint32_t w0 = uniform32(nxt.x), w1 = uniform32(nxt.y);
    nxt = g2[i + 1];
    const uint32_t op = w0 & 0xffu, q = (w0 >> 8) & 0xffu, r = (w0 >> 16) & 0xffu;
    const uint32_t cond = (w1 >> 16) & 0xffu;
    if (cond & kSlotStart) {
      cur_b = next_b;
      if (occ < n_occ) next_b = (uint32_t)branch[(uint64_t)seq[occ] * chb + ba];
      ++occ;
    }
    bool on = true;  // per term: the branch choice decides a conditional gate
    if (cond & kCondApply) on = ((w1 >> 24) >> cur_b & 1u) != 0u;
    if (op == OP_H) {
      hadamard(q, on ? ~0u : 0u);
      continue;
    }
    const uint32_t qb = on ? 1u << (q & 31u) : 0u, rb = on ? 1u << (r & 31u) : 0u;
    if (op == OP_CX) {
      // gamma_q += gamma_r + 2 (M_q . F_r); G_r ^= G_q; F_q ^= F_r; M_q ^= M_r.
      with_half<KW>(q >= 32u, [&](auto hq) {
        with_half<KW>(r >= 32u, [&](auto hr) {
          constexpr int a = decltype(hq)::value, b = decltype(hr)::value;
          const uint32_t qs = q & 31u, rs = r & 31u;
          uint32_t dot = 0u;
#pragma unroll
          for (int j = 0; j < C; ++j) {
            const uint32_t fr = bit_mask(F.w[b][j], rs), mr = bit_mask(M.w[b][j], rs);
            const uint32_t mq = bit_mask(M.w[a][j], qs), gq = bit_mask(G.w[a][j], qs);
            dot = bop3<kAndXor>(mq, fr, dot);
            F.w[a][j] = bop3<kAndXor>(fr, qb, F.w[a][j]);
            M.w[a][j] = bop3<kAndXor>(mr, qb, M.w[a][j]);
            G.w[b][j] = bop3<kAndXor>(gq, rb, G.w[b][j]);
          }
          dot = group_xor<LPT>(dot);
          const uint32_t gr = ((glo[b] >> rs) & 1u) | (((ghi[b] >> rs) & 1u) << 1);
          gamma_add(hq, qb, gr + 2u * (dot & 1u));
        });
      });
    } else if (op == OP_CZ) {
      // M_q ^= G_r, M_r ^= G_q.
      with_half<KW>(q >= 32u, [&](auto hq) {
        with_half<KW>(r >= 32u, [&](auto hr) {
          constexpr int a = decltype(hq)::value, b = decltype(hr)::value;
          const uint32_t qs = q & 31u, rs = r & 31u;
#pragma unroll
          for (int j = 0; j < C; ++j) {
            const uint32_t gr = bit_mask(G.w[b][j], rs), gq = bit_mask(G.w[a][j], qs);
            M.w[a][j] = bop3<kAndXor>(gr, qb, M.w[a][j]);
            M.w[b][j] = bop3<kAndXor>(gq, rb, M.w[b][j]);
          }
        });
      });
    } else {
      // S^pw on q: M_q ^= G_q pw times, gamma_q -= pw.
      uint32_t pw = 1u;
      if (op == OP_SLOT_SPOW) pw = ((w0 >> 16) >> (2u * cur_b)) & 3u;
      else if (op == OP_SPOW) pw = w0 >> 24;
      with_half<KW>(q >= 32u, [&](auto hq) {
        constexpr int a = decltype(hq)::value;
        const uint32_t mb = (pw & 1u) ? qb : 0u;
#pragma unroll
        for (int j = 0; j < C; ++j) M.w[a][j] = bop3<kAndXor>(G.w[a][j], mb, M.w[a][j]);
        gamma_add(hq, qb, (4u - pw) & 3u);
      });
    }
  }

  F.store(Rt, li, n, J.dst.F + item * J.dst_is, J.dst_rs, live);
  G.store(Rt, li, n, J.dst.G + item * J.dst_is, J.dst_rs, live);
  M.store(Rt, li, n, J.dst.M + item * J.dst_is, J.dst_rs, live);
  const uint64_t at = (uint64_t)li * C;
  const uint64_t v64 = at < 64u ? (uint64_t)v << at : 0ull, s64 = at < 64u ? (uint64_t)s << at : 0ull;
  const uint32_t vl = group_or<LPT>((uint32_t)v64), vh = group_or<LPT>((uint32_t)(v64 >> 32));
  const uint32_t sl = group_or<LPT>((uint32_t)s64), sh = group_or<LPT>((uint32_t)(s64 >> 32));
  if (live) {
    for (uint32_t p = li; p < n; p += LPT) {
      uint32_t g = 0u;
#pragma unroll
      for (int k = 0; k < KW; ++k)
        if ((p >> 5) == (uint32_t)k) g = ((glo[k] >> (p & 31u)) & 1u) | (((ghi[k] >> (p & 31u)) & 1u) << 1);
      J.dst.gamma[(uint64_t)p * J.dst_rs + item * J.dst_is] = (uint8_t)g;
    }
    if (li == 0) {
      J.dst.v[item] = ((uint64_t)vh << 32) | vl;
      J.dst.s[item] = ((uint64_t)sh << 32) | sl;
      J.dst.omega[item] = (uint8_t)w;
      if (e & 1u) atomicOr(err, 1u);
    }
  }
}

template <int LPT, int C>
hipError_t launch_cols_t(const EvolveJob& J, const DGate* gates, uint32_t n_gates, bool from_zero, uint32_t* err,
                         hipStream_t st) {
  constexpr uint32_t per = kColWaves * 64u / LPT;  // terms per workgroup
  const uint64_t blocks = (J.count + per - 1) / per;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_evolve_cols<LPT, C>), dim3((uint32_t)blocks), dim3(256), 0, st, J, gates, n_gates,
                     from_zero ? 1u : 0u, err);
  return hipGetLastError();
}

}  // namespace
}  // namespace chsim
