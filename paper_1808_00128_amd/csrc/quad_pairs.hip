// Pairs of a term and a state by bit-sliced elimination: sums
//   sum_x i^{-x A x^T} [F_w x = s_w for all w] <x|phi_alpha>
// over a CH term's support, for many states (A, F_w, s_w) at once.  An
// equatorial state has no constraints w; the amplitude of a CH form (a "bra") is a
// Z_4 quadratic form on the solutions of x F = s outside v, and a constraint
// enters as 1/2 sum_{w = 0, 1} (-1)^{w (F_w x + s_w)}, one more variable.
//
// Method.  The support is x1 + span(columns of G in v).  The prologue brings the
// columns to reduced echelon form (any basis of the span gives the same sum): each
// column c has a row p_c in which it is the only one, and only the other rows N
// (m = n - |v| of them) hold further bits H.  With Y = A_N. D, D = [I; H],
//   S_fg = A_{pf,pg} + sum_{i in N} (H_if Y_ig + A_{pf,i} H_ig)
// is the form on the support in n (n - |v|)-like work instead of n^2 + n |v|, with
// x1 as one more column (column 0) that yields the linear and constant parts; the
// term's own form is added from its record.  Constraint variables are columns with
// no bits in N.  The Z_4 form is lifted to Z_2 (Eq. (Q)) with column 0 reused for
// the extra variable, and pairs of variables are eliminated (Eqs. (identity),
// (eq5)).
//
// Mapping: bit-sliced, a word holds one matrix entry of 32 states.  A wave holds
// one term and 4 words (128 states): 16 lanes per word, columns Q j + q on lane j,
// rows in registers.  An entry that all columns of a row need is broadcast within
// the 16 lanes by DPP.  Each step takes the next variable a in order and, state by
// state, the first b with S_ab = 1: b's row is the sum of the rows under the
// first-set masks; states in which a has no partner left take part with zeros (an
// eliminated variable's row and column come out zero by themselves).  Every step is
// code of its own (33, 125 and 240 KB for Q = 2, 3, 4: the waves of a compute unit
// run through it about together, so that it need not fit the instruction cache).
// One bit operation serves 2048 pairs'
// entries of a wave where the lane-per-state form (one 32-bit row of one state per
// lane) serves 64 rows; selection and pivoting cost nothing for divergence.
//
// VALU issue bounds it.  Against one state per lane with its form's rows in LDS
// (equatorial) and one wave per pair (bras), whole calls: n = 40, |v| = 20..22,
// chi = 2^18, 1024 states 73.6 -> 37.0 ms (the pair kernel 67.2 -> 27.3 where the
// clock holds); n = 45, |v| = 41..43, chi = 60000, 500 states 47.0 -> 7.4; n = 50,
// |v| = 46..49, 1000 states 117 -> 38.2; 256 bras n = 40, chi = 2^16 34.1 -> 4.4,
// n = 50, chi = 60000, 200 bras 49.8 -> 12.0.  Loops that moved the rows down and the
// lanes along after every Q steps instead: 30.3 ms (27.3), and 3.17 against 2.82 for
// the 44-variable kernel of the 256 bras.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "bitops.hpp"
#include "device_common.hpp"
#include "internal.hpp"

namespace chsim {

namespace {

template <class F, int... I>
__device__ __forceinline__ void sfor_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(0), ..., f(N - 1) with compile-time indices.
template <int N, class F>
__device__ __forceinline__ void sfor(F&& f) {
  sfor_impl(std::make_integer_sequence<int, N>{}, f);
}

// Lane `kLane` of each row of 16 lanes, in all of them.
template <int kLane>
__device__ __forceinline__ uint32_t row_bcast(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x150 + kLane, 0xF, 0xF, true);
}
// XOR over the 16 lanes of a row, in all of them.
__device__ __forceinline__ uint32_t row_xor(uint32_t x) {
  x ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);
  x ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true);
  x ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, true);
  x ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x140, 0xF, 0xF, true);
  return x;
}
// A & ~B, A | B, (A & ~B) | C as builtins.  What went wrong with plain operators is
// the running mask of the pivot search kept as its complement (none &= ~s1, the pick
// s1 & none, over all rows of an unrolled step): the chain of complements was merged
// into three-input operations with wrong truth tables.  Masks that one step hands to
// the next stay in these forms; the edge tests fail for the other.
enum : uint32_t { kAndNot = 0x30, kOr = 0xFC, kAndNotOr = 0xBA };
__device__ __forceinline__ uint32_t and_xor(uint32_t a, uint32_t b, uint32_t c) { return bop3<kAndXor>(a, b, c); }

// Record of a term (8-byte words): header (|v|, m, omega), the form's diagonal
// planes over the columns (bit 0: the constant), rows of H (m, two zero rows
// after them), p_c and the list N as 32-bit words (N padded by two n's: the zero
// row), then per column c = 0 .. |v|: H_c, the form's column, p_c.
struct RecLayout {
  uint32_t hrow, p, nlist, cols, words;
};
__host__ __device__ constexpr RecLayout rec_layout(uint32_t n) {
  RecLayout r{};
  r.hrow = 3u;
  r.p = r.hrow + n + 2u;
  r.nlist = r.p + (n + 3u) / 2u;
  r.cols = r.nlist + (n + 3u) / 2u;
  r.words = r.cols + 3u * (n + 1u);
  return r;
}

__device__ __forceinline__ uint64_t gather_bits(uint64_t x, uint64_t m) {
  uint64_t out = 0;
  for (uint32_t k = 0; m; m &= m - 1ull, ++k) out |= ((x >> __builtin_ctzll(m)) & 1ull) << k;
  return out;
}

constexpr uint32_t kPrepWaves = 4;

// One wave per term, lane = row, then lane = column.  Counts 0, 1: max |v|, max
// (64 - |v|), unless stat is null (one launch takes every term).
__global__ __launch_bounds__(64 * kPrepWaves) void k_quad_prep(TermsView T, uint64_t count, uint64_t* __restrict__ rec,
                                                               uint32_t* __restrict__ stat) {
  __shared__ uint64_t cols[kPrepWaves][64];
  __shared__ uint32_t pivs[kPrepWaves][64];
  const uint32_t lane = threadIdx.x & 63u, wave = uniform32(threadIdx.x >> 6);
  const uint64_t term = (uint64_t)blockIdx.x * kPrepWaves + wave;
  if (term >= count) return;  // whole waves
  const uint32_t n = T.n;
  const bool act = lane < n;
  const uint64_t off = (uint64_t)lane * T.chi + term;
  const uint64_t F = act ? T.F[off] : 0ull, G = act ? T.G[off] : 0ull, M = act ? T.M[off] : 0ull;
  const uint32_t g = act ? (uint32_t)T.gamma[off] : 0u;
  const uint64_t v = uniform64(T.v[term]), s = uniform64(T.s[term]);
  // Columns of G, and the quadratic form of the amplitude: B's strictly upper part
  // P_pq = par(F_p & M_q), p < q, symmetrised (Bs), its diagonal, gamma's low bits.
  uint64_t d = 0, P = 0;
  for (uint32_t q = 0; q < n; ++q) {
    const uint64_t cg = ballot64(((G >> q) & 1ull) != 0ull);
    if (lane == q) d = cg;
    P |= (uint64_t)par64(F & rl64(M, q)) << q;
  }
  uint64_t low = 0;
  for (uint32_t q = 0; q < n; ++q) low |= ((rl64(P, q) >> lane) & 1ull) << q;
  const uint64_t above = (lane >= 63u) ? 0ull : (~0ull << (lane + 1u));
  const uint64_t below = (1ull << lane) - 1ull;
  const uint64_t Bs = act ? ((P & above) | (low & below)) : 0ull;
  const uint64_t diag = ballot64(act && (((P >> lane) & 1ull) ^ (uint64_t)((g >> 1) & 1u) ^
                                         (uint64_t)par64(F & v & s)) != 0ull);
  const uint64_t glo = ballot64(act && (g & 1u));
  uint64_t x1 = ballot64(act && par64(G & s));
  // Reduced echelon form of the columns in v, lane = column.
  const bool inv = ((v >> lane) & 1ull) != 0ull;
  if (!inv) d = 0ull;
  uint64_t pivrows = 0;
  uint32_t mypiv = 0;
  for (uint64_t u = v; u; u &= u - 1ull) {
    const uint32_t f = (uint32_t)__builtin_ctzll(u);
    const uint64_t df = rl64(d, f);
    const uint32_t pv = df ? (uint32_t)__builtin_ctzll(df) : 0u;  // columns of an invertible G
    if (lane != f) d ^= df & bitmask64(d, pv);
    x1 ^= df & bitmask64(x1, pv);
    if (lane == f) mypiv = pv;
    pivrows |= 1ull << pv;
  }
  const uint64_t nmask = n == 64u ? ~0ull : ((1ull << n) - 1ull);
  const uint64_t N = nmask & ~pivrows;
  const uint32_t nv = (uint32_t)__popcll(v), m = (uint32_t)__popcll(N);
  // Column 0 is x1, columns 1 .. |v| the basis, lane = column.
  if (inv) {
    const uint32_t c = (uint32_t)__popcll(v & below) + 1u;
    if (c < 64u) {
      cols[wave][c] = d;
      pivs[wave][c] = mypiv;
    }
  }
  if (lane == 0u) {
    cols[wave][0] = x1;
    pivs[wave][0] = 0u;
  }
  wave_sync();
  const bool ic = lane <= nv;
  const uint64_t dc = ic ? cols[wave][lane] : 0ull;
  const uint32_t pc = ic ? pivs[wave][lane] : 0u;
  uint64_t t = 0, tu = 0;
  for (uint32_t q = 0; q < n; ++q) {
    const uint64_t Bq = rl64(Bs, q) & bitmask64(dc, q);
    t ^= Bq;
    tu ^= Bq & ((1ull << q) - 1ull);
  }
  const uint64_t y = t ^ (glo & dc);
  uint64_t K = 0;
  const uint32_t top = nv < 63u ? nv : 63u;
  for (uint32_t c = 0; c <= top; ++c) K |= (uint64_t)par64(rl64(dc, c) & y) << c;
  uint32_t kd = (uint32_t)__popcll(dc & glo) + 2u * (par64(dc & diag) ^ par64(dc & tu));
  if (lane) kd += 2u * (uint32_t)(K & 1ull);
  const uint64_t kdlo = ballot64(ic && (kd & 1u)), kdhi = ballot64(ic && (kd & 2u));
  const RecLayout L = rec_layout(n);
  uint64_t* r = rec + term * L.words;
  uint32_t* const rp = reinterpret_cast<uint32_t*>(r + L.p);
  uint32_t* const rn = reinterpret_cast<uint32_t*>(r + L.nlist);
  const uint64_t H = gather_bits(dc, N);
  if (ic) {
    rp[lane] = pc;
    uint64_t* rc = r + L.cols + 3u * lane;
    rc[0] = H;
    rc[1] = K & ~1ull;
    rc[2] = pc;
  }
  uint32_t k = 0;
  for (uint64_t u = N; u; u &= u - 1ull, ++k) {
    const uint32_t i = (uint32_t)__builtin_ctzll(u);
    const uint64_t row = ballot64(((dc >> i) & 1ull) != 0ull);
    if (lane == 0u) {
      r[L.hrow + k] = row;
      rn[k] = i;
    }
  }
  if (lane == 0u) {
    for (uint32_t e = 0; e < 2u; ++e) {
      r[L.hrow + m + e] = 0ull;
      rn[m + e] = n;
    }
    r[0] = (uint64_t)nv | ((uint64_t)m << 8) | ((uint64_t)T.omega[term] << 16);
    r[1] = kdlo;
    r[2] = kdhi;
    if (stat) {
      uint32_t* const sl = stat + quad_stat_slot(blockIdx.x);
      atomicMax(sl, nv);
      atomicMax(sl + 1, 64u - nv);
    }
  }
}

// State slices: per batch of 128 states, rows i = 0 .. n of A (row n zero) over
// ne1 = n + slots + 1 columns (constraints from column n, the last one zero), then
// the high bits of the diagonal, each entry four words of 32 states.
__host__ __device__ constexpr uint32_t slice_entries(uint32_t n, uint32_t ne1) { return (n + 2u) * ne1; }

// Ballots of 64 lanes' bits j of (x-part, constraint part), by entry of a row.
__device__ __forceinline__ void store_row(uint64_t x, uint64_t w, uint32_t n, uint32_t ne1, uint32_t lane,
                                          uint32_t half, uint32_t* __restrict__ out) {
  for (uint32_t j0 = 0; j0 < ne1; j0 += 64u) {
    uint64_t mine = 0;
    const uint32_t je = ne1 - j0 < 64u ? ne1 - j0 : 64u;
    for (uint32_t k = 0; k < je; ++k) {
      const uint32_t j = j0 + k;
      const uint64_t b = j < n ? ballot64((x >> j) & 1ull) : ballot64((w >> (j - n)) & 1ull);
      if (lane == k) mine = b;
    }
    if (lane < je) *reinterpret_cast<uint64_t*>(out + ((size_t)(j0 + lane) * 4u + 2u * half)) = mine;
  }
}

// One wave per 64 states and row: equatorial states, -A (low bits as they are,
// the diagonal's high bit flipped where its low bit is set).
__global__ __launch_bounds__(64) void k_slice_equatorial(const uint64_t* __restrict__ Aoff,
                                                         const uint8_t* __restrict__ Adiag, uint32_t n, uint32_t L,
                                                         uint32_t ne1, uint32_t* __restrict__ sl,
                                                         uint32_t* __restrict__ info) {
  const uint32_t lane = threadIdx.x, i = blockIdx.y, l = blockIdx.x * 64u + lane;
  uint64_t x = 0;
  if (l < L) {
    if (i < n) {
      x = (Aoff[(uint64_t)l * n + i] & ~(1ull << i)) | ((uint64_t)(Adiag[(uint64_t)l * n + i] & 1u) << i);
      if (n < 64u) x &= (1ull << n) - 1ull;
    } else if (i == n + 1u) {
      for (uint32_t c = 0; c < n; ++c) {
        const uint32_t dg = Adiag[(uint64_t)l * n + c];
        x |= (uint64_t)(((dg >> 1) ^ dg) & 1u) << c;
      }
    }
  }
  if (i == 0u) info[l] = n << 8;
  uint32_t* out = sl + (size_t)(blockIdx.x >> 1) * slice_entries(n, ne1) * 4u + (size_t)i * ne1 * 4u;
  store_row(x, 0ull, n, ne1, lane, blockIdx.x & 1u, out);
}

// The same for bra states (terms of Tb with Bs and the planes in their records):
// conj(<x|theta>) = 2^{-|v|/2} e^{-i pi omega/4} i^{-glo x - 2 x B x} on the
// solutions of (x F)_j = s_j, j outside v (in increasing order: slots 0, 1, ...).
// Count 2: max number of constraints.
__global__ __launch_bounds__(64) void k_slice_bras(TermsView Tb, const uint64_t* __restrict__ rec, uint32_t rec_words,
                                                   uint32_t L, uint32_t ne1, uint32_t slots,
                                                   uint32_t* __restrict__ sl, uint32_t* __restrict__ info,
                                                   uint32_t* __restrict__ stat) {
  const uint32_t lane = threadIdx.x, i = blockIdx.y, l = blockIdx.x * 64u + lane, n = Tb.n;
  const uint64_t nmask = n == 64u ? ~0ull : ((1ull << n) - 1ull);
  uint64_t x = 0, w = 0, wsrc = 0, nvm = 0;
  if (l < L) {
    const uint64_t* r = rec + (uint64_t)l * rec_words;
    const uint64_t diag = r[6u * n], glo = r[6u * n + 1u];
    nvm = nmask & ~Tb.v[l];
    if (i < n) {
      x = (r[3u * n + i] & ~(1ull << i)) | (glo & (1ull << i));
      wsrc = Tb.F[(uint64_t)i * Tb.chi + l];
    } else if (i == n + 1u) {
      x = (glo ^ diag) & nmask;
      wsrc = Tb.s[l];
    }
  }
  for (uint32_t j = 0, k = 0; j < n; ++j) {
    const uint32_t on = (uint32_t)(nvm >> j) & 1u;
    if (k < slots) w |= (uint64_t)(on & (uint32_t)(wsrc >> j)) << k;
    k += on;
  }
  if (i == 0u) {
    info[l] = l < L ? (Tb.omega[l] & 7u) | ((uint32_t)__popcll(Tb.v[l]) << 8) : 0u;
    if (l < L) atomicMax(stat + quad_stat_slot(blockIdx.x) + 2u, (uint32_t)__popcll(nvm));
  }
  uint32_t* out = sl + (size_t)(blockIdx.x >> 1) * slice_entries(n, ne1) * 4u + (size_t)i * ne1 * 4u;
  store_row(x, w, n, ne1, lane, blockIdx.x & 1u, out);
}

struct QuadArgs {
  const uint64_t* rec;
  const double2* b;
  uint64_t chi;
  const uint32_t* sl;
  const uint32_t* info;
  const uint32_t* stat;
  double2* partial;  // this launch's rows
  uint32_t n, ne1, slots, L, n_waves, n_batches;
  QuadRule rule;
  uint32_t cls;           // this launch's class
  uint32_t nc_lo, nc_hi;  // the variables (without the extra one) this launch takes
  bool many;              // there are other launches: the counts tell whether this one has any terms
};

// Columns Q per lane, at most RM rows (variables and the extra one).  Column and
// row c are at place RM - 1 - c (columns Q j + q on lane j), so that the elimination
// is straight-line code of RM steps of which a smaller form takes the last ones.
template <int Q, int RM, int NW, int OCC>
__global__ __launch_bounds__((64 * NW), OCC) void k_quad_pairs(QuadArgs A) {
  extern __shared__ __align__(16) uint32_t lds[];
  constexpr auto at = [](int c) { return RM - 1 - c; };  // place of column or row c
  constexpr int kQ0 = at(0) % Q, kJ0 = at(0) / Q;        // column 0's
  const uint32_t lane = threadIdx.x & 63u, wave = uniform32(threadIdx.x >> 6);
  const uint32_t g = lane >> 4, j = lane & 15u;
  const uint32_t n = A.n, ne1 = A.ne1;
  const uint32_t wgs = A.n_waves / NW;  // workgroups per batch
  const uint32_t batch = blockIdx.x / wgs, row0 = (blockIdx.x % wgs) * NW + wave;
  const uint32_t l0 = batch * 128u + g * 32u + 2u * j;
  uint32_t w = 0u;
  bool any_term = true;  // uniform over the grid
  if (A.slots) w = quad_stat_max(A.stat, 2u, lane);
  if (w > A.slots) w = 1u << 20;  // more constraints than columns: not for these kernels
  if (A.slots) any_term = w <= A.slots && quad_takes_class(A.rule, A.cls, w);
  if (A.many)
    any_term = any_term && quad_stat_max(A.stat, 0u, lane) + w >= A.nc_lo &&
               64u - quad_stat_max(A.stat, 1u, lane) + w <= A.nc_hi;
  double ar[2] = {0.0, 0.0}, ai[2] = {0.0, 0.0};
  if (any_term) {
    const uint4* src = reinterpret_cast<const uint4*>(A.sl) + (size_t)batch * slice_entries(n, ne1);
    for (uint32_t e = threadIdx.x; e < slice_entries(n, ne1); e += 64u * NW) reinterpret_cast<uint4*>(lds)[e] = src[e];
    __syncthreads();
    const uint32_t stride = ne1 * 16u, g4 = 4u * g;
    auto ld = [&](uint32_t byte) { return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(lds) + byte); };
    const uint32_t dhi0 = (n + 1u) * stride;
    const uint32_t inf0 = A.info[l0], inf1 = A.info[l0 + 1u];
    const RecLayout RL = rec_layout(n);
    const uint32_t nl0 = j == (uint32_t)kJ0 ? 0u : ~0u;
    for (uint64_t term = row0; term < A.chi; term += A.n_waves) {
      const uint64_t* __restrict__ r = A.rec + term * RL.words;
      const uint64_t hdr = r[0];
      const uint32_t nv = uniform32((uint32_t)hdr & 0xFFu), m = uniform32((uint32_t)(hdr >> 8) & 0xFFu);
      const uint32_t om = uniform32((uint32_t)(hdr >> 16) & 7u);
      const uint32_t nc = nv + w;
      if (nc < A.nc_lo || nc > A.nc_hi) continue;
      const uint64_t kdlo = r[1], kdhi = r[2];
      const uint64_t* __restrict__ hrow = r + RL.hrow;
      const uint32_t* __restrict__ rp = reinterpret_cast<const uint32_t*>(r + RL.p);
      const uint32_t* __restrict__ rn = reinterpret_cast<const uint32_t*>(r + RL.nlist);
      // The lane's columns.
      uint32_t Hl[Q], Hh[Q], Kl[Q], Kh[Q], B1[Q], B2[Q], D0[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t dcol = (uint32_t)RM - 1u - ((uint32_t)Q * j + (uint32_t)q);
        const uint64_t* rc = r + RL.cols + 3u * (dcol <= nv ? dcol : 0u);
        const bool on = dcol <= nv, xt = on && dcol != 0u;
        const uint64_t h = on ? rc[0] : 0ull, k = xt ? rc[1] : 0ull;
        const uint32_t p = (uint32_t)rc[2];
        Hl[q] = (uint32_t)h;
        Hh[q] = (uint32_t)(h >> 32);
        Kl[q] = (uint32_t)k;
        Kh[q] = (uint32_t)(k >> 32);
        const bool wt = dcol > nv && dcol <= nc;
        B1[q] = (xt ? p : wt ? n + (dcol - nv - 1u) : ne1 - 1u) * 16u + g4;
        B2[q] = (xt ? p : n) * stride + g4;
        D0[q] = B2[q] + (xt ? p * 16u : 0u);
      }
      // A between the columns' own rows, and the term's form.
      uint32_t S[RM][Q];
      sfor<RM>([&](auto ic) {
        constexpr int c = ic;
#pragma unroll
        for (int q = 0; q < Q; ++q) S[at(c)][q] = 0u;
        if constexpr (c > 0) {
          if ((uint32_t)c <= nv) {
            const uint32_t base = rp[c] * stride;
#pragma unroll
            for (int q = 0; q < Q; ++q)
              S[at(c)][q] = ld(base + B1[q]) ^ bit_mask(c < 32 ? Kl[q] : Kh[q], (uint32_t)c & 31u);
          } else if ((uint32_t)c <= nc) {
            const uint32_t base = (n + (uint32_t)c - nv - 1u) * 16u;
#pragma unroll
            for (int q = 0; q < Q; ++q) S[at(c)][q] = ld(base + B2[q]);
          }
        }
      });
      uint32_t lo[Q], hi[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) lo[q] = hi[q] = 0u;
      // Rows i of N, two at a time (a zero row after the last of an odd count).
      for (uint32_t i = 0; i < m; i += 2u) {
        const uint32_t n0 = rn[i], n1 = rn[i + 1u];
        const uint32_t r0 = n0 * stride, r1 = n1 * stride, r0g = r0 + g4, r1g = r1 + g4;
        uint32_t a0[Q], a1[Q], y0[Q], y1[Q], h0[Q], h1[Q], c0[Q], c1[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          a0[q] = ld(r0 + B1[q]);
          a1[q] = ld(r1 + B1[q]);
          y0[q] = a0[q];
          y1[q] = a1[q];
          h0[q] = bit_mask(i < 32u ? Hl[q] : Hh[q], i & 31u);
          h1[q] = bit_mask(i + 1u < 32u ? Hl[q] : Hh[q], (i + 1u) & 31u);
        }
        auto span = [&](uint32_t jb, uint32_t je, const uint32_t (&Hw)[Q]) {
#pragma unroll 4
          for (uint32_t jj = jb; jj < je; ++jj) {
            const uint32_t o = rn[jj] * 16u;
            const uint32_t w0 = ld(r0g + o), w1 = ld(r1g + o);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
              const uint32_t hm = bit_mask(Hw[q], jj & 31u);
              y0[q] = and_xor(w0, hm, y0[q]);
              y1[q] = and_xor(w1, hm, y1[q]);
            }
          }
        };
        span(0u, min(i, 32u), Hl);
        span(32u, max(i, 32u), Hh);
        const uint32_t w00 = ld(r0 + n0 * 16u + g4), w01 = ld(r0 + n1 * 16u + g4), w11 = ld(r1 + n1 * 16u + g4);
        const uint32_t e0 = ld(dhi0 + n0 * 16u + g4), e1 = ld(dhi0 + n1 * 16u + g4);
        // (n1 = n in the zero row: column n of row n0 meets h1 = 0 only.)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          c0[q] = y0[q];
          y0[q] = and_xor(w00, h0[q], y0[q]);
          y0[q] = and_xor(w01, h1[q], y0[q]);
          y1[q] = and_xor(w01, h0[q], y1[q]);
          c1[q] = y1[q];
          y1[q] = and_xor(w11, h1[q], y1[q]);
        }
        span(min(i + 2u, 32u), min(m, 32u), Hl);
        span(max(i + 2u, 32u), max(m, 32u), Hh);
        // Diagonal: the column's bits in rows i, i + 1.
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const uint32_t t0 = w00 & h0[q];
          hi[q] = and_xor(lo[q], t0, hi[q]);
          lo[q] ^= t0;
          hi[q] = and_xor(h0[q], e0 ^ c0[q], hi[q]);
          const uint32_t t1 = w11 & h1[q];
          hi[q] = and_xor(lo[q], t1, hi[q]);
          lo[q] ^= t1;
          hi[q] = and_xor(h1[q], e1 ^ c1[q], hi[q]);
        }
        const uint64_t hr0 = hrow[i], hr1 = hrow[i + 1u];
        sfor<RM>([&](auto ic) {
          constexpr int c = ic;
          if ((uint32_t)(c & ~3) <= nc) {
            const uint32_t m0 = (uint32_t)((int32_t)((c < 32 ? (uint32_t)hr0 : (uint32_t)(hr0 >> 32)) << (31 - (c & 31))) >> 31);
            const uint32_t m1 = (uint32_t)((int32_t)((c < 32 ? (uint32_t)hr1 : (uint32_t)(hr1 >> 32)) << (31 - (c & 31))) >> 31);
            const uint32_t b0 = row_bcast<at(c) / Q>(a0[at(c) % Q]), b1 = row_bcast<at(c) / Q>(a1[at(c) % Q]);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
              S[at(c)][q] = and_xor(m0, y0[q], S[at(c)][q]);
              S[at(c)][q] = and_xor(m1, y1[q], S[at(c)][q]);
              S[at(c)][q] = and_xor(b0, h0[q], S[at(c)][q]);
              S[at(c)][q] = and_xor(b1, h1[q], S[at(c)][q]);
            }
          }
        });
      }
      // Diagonal mod 4 of the whole form: the columns' own rows, twice the product
      // with x1 (row 0), the term's part.  Column 0's is the constant.
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t dcol = (uint32_t)RM - 1u - ((uint32_t)Q * j + (uint32_t)q);
        const uint32_t plo = ld(D0[q]), phi = ld(dhi0 + B1[q]);
        hi[q] = and_xor(lo[q], plo, hi[q] ^ phi);
        lo[q] ^= plo;
        hi[q] ^= q == kQ0 ? S[at(0)][q] & nl0 : S[at(0)][q];
        const uint32_t kl = 0u - ((uint32_t)(kdlo >> (dcol & 63u)) & 1u), kh = 0u - ((uint32_t)(kdhi >> (dcol & 63u)) & 1u);
        hi[q] = and_xor(lo[q], kl, hi[q] ^ kh);
        lo[q] ^= kl;
      }
      const uint32_t cst0 = row_bcast<kJ0>(lo[kQ0]), cst1 = row_bcast<kJ0>(hi[kQ0]);
      // Lift: column 0 becomes the extra variable.
      uint32_t lr[Q], li[Q], kx[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        lr[q] = q == kQ0 ? hi[q] & nl0 : hi[q];
        li[q] = q == kQ0 ? lr[q] | ~nl0 : lr[q];
        kx[q] = q == kQ0 ? lo[q] | ~nl0 : lo[q];
        S[at(0)][q] = q == kQ0 ? lo[q] & nl0 : lo[q];
      }
      sfor<RM>([&](auto ic) {
        constexpr int c = ic;
        if constexpr (c > 0) {
          constexpr int pc = at(c);
          const uint32_t kf = row_bcast<pc / Q>(lo[pc % Q]);
          S[pc][kQ0] &= nl0;
#pragma unroll
          for (int q = 0; q < Q; ++q) S[pc][q] = and_xor(kf, kx[q], S[pc][q]);
          S[pc][pc % Q] = j == (uint32_t)(pc / Q) ? 0u : S[pc][pc % Q];
        }
      });
      // Pair elimination.
      uint32_t sr = 0, si = 0, nzr = 0, nzi = 0, cn[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) cn[k] = 0u;
      // Place k against the places after it.
      auto pivot = [&](auto kk) {
        constexpr int k = kk, kL = k / Q, q0 = k % Q;
        uint32_t fo = 0u, Sb[Q], sv[Q], Sa[Q];  // fo: states with a partner
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          Sb[q] = sv[q] = 0u;
          Sa[q] = S[k][q];
        }
        sfor<RM - k - 1>([&](auto ic) {
          constexpr int c = k + 1 + (int)ic;
          const uint32_t s1 = row_bcast<kL>(S[c][q0]), sel = bop3<kAndNot>(s1, fo, 0u);
          fo = bop3<kOr>(s1, fo, 0u);
#pragma unroll
          for (int q = 0; q < Q; ++q) Sb[q] = and_xor(sel, S[c][q], Sb[q]);
          sv[c % Q] = j == (uint32_t)(c / Q) ? sel : sv[c % Q];
        });
        const uint32_t la = row_bcast<kL>(lr[q0]), ma = row_bcast<kL>(li[q0]);
        nzr = bop3<kAndNotOr>(la, fo, nzr);
        nzi = bop3<kAndNotOr>(ma, fo, nzi);
        if constexpr (k + 1 < RM) {
          uint32_t xb = 0, yb = 0;
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            xb = and_xor(sv[q], lr[q], xb);
            yb = and_xor(sv[q], li[q], yb);
          }
          const uint32_t lb = row_xor(xb), mb = row_xor(yb);
          sr = and_xor(la, lb, sr);
          si = and_xor(ma, mb, si);
          uint32_t carry = fo;
#pragma unroll
          for (int p = 0; p < 6; ++p) {
            const uint32_t x = cn[p] & carry;
            cn[p] ^= carry;
            carry = x;
          }
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const uint32_t ab = Sa[q] & Sb[q];
            lr[q] = and_xor(lb, Sa[q], and_xor(la, Sb[q], lr[q] ^ ab));
            li[q] = and_xor(mb, Sa[q], and_xor(ma, Sb[q], li[q] ^ ab));
          }
          sfor<RM - k - 1>([&](auto ic) {
            constexpr int c = k + 1 + (int)ic;
            const uint32_t s1 = row_bcast<kL>(S[c][q0]), s2 = row_bcast<c / Q>(Sb[c % Q]);
#pragma unroll
            for (int q = 0; q < Q; ++q) S[c][q] = and_xor(s2, Sa[q], and_xor(s1, Sb[q], S[c][q]));
          });
        }
      };
      sfor<RM>([&](auto ip) {
        if ((uint32_t)(RM - 1 - (int)ip) <= nc) pivot(ip);
      });
      // The lane's two states.
      const double2 b = A.b[term];
#pragma unroll
      for (uint32_t u = 0; u < 2u; ++u) {
        const uint32_t sh = 2u * j + u, inf = u ? inf1 : inf0;
        const bool re = !((nzr >> sh) & 1u), im = !((nzi >> sh) & 1u);
        const uint32_t s0 = (sr >> sh) & 1u, s1 = (si >> sh) & 1u;
        uint32_t nel = 0;
#pragma unroll
        for (int p = 0; p < 6; ++p) nel |= ((cn[p] >> sh) & 1u) << p;
        const bool both = re && im;
        const uint32_t kz = both ? (s0 ? (s1 ? 5u : 3u) : (s1 ? 7u : 1u)) : re ? 4u * s0 : 2u + 4u * s1;
        const uint32_t cst = ((cst0 >> sh) & 1u) + 2u * ((cst1 >> sh) & 1u);
        const uint32_t k8 = (om + 8u - (inf & 7u) + 2u * cst + kz) & 7u;
        // 2^{e2 / 2}: an odd e2 multiplies by sqrt(2).
        const int e2 = 2 * ((int)nc - (int)nel) + (both ? 1 : 0) - 2 * (int)w - (int)nv - (int)(inf >> 8);
        const double mag = ldexp((e2 & 1) ? 1.41421356237309504880 : 1.0, e2 >> 1);
        const double h = 0.70710678118654752440;
        const double x = (k8 & 1u) ? (b.x - b.y) * h : b.x, yv = (k8 & 1u) ? (b.x + b.y) * h : b.y;
        const uint32_t qd = k8 >> 1;
        const double cr = (qd & 1u) ? yv : x, ci = (qd & 1u) ? x : yv;
        const bool on = re || im;
        const double sgr = (qd == 1u || qd == 2u) ? -mag : mag, sgi = (qd >= 2u) ? -mag : mag;
        ar[u] += on ? sgr * cr : 0.0;
        ai[u] += on ? sgi * ci : 0.0;
      }
    }
  }
#pragma unroll
  for (uint32_t u = 0; u < 2u; ++u)
    if (l0 + u < A.L) A.partial[(size_t)row0 * A.L + l0 + u] = make_double2(ar[u], ai[u]);
}

}  // namespace

namespace {

// The launches: Q columns per lane, RM rows (variables and the extra one).
struct QuadClass {
  uint32_t nc_lo, nc_hi, nw, waves;  // variables taken, waves per workgroup, waves that fill the chip
};
constexpr QuadClass kClasses[3] = {{0, kQuadClassMax[0], 8, 4096},
                                   {kQuadClassMax[0] + 1u, kQuadClassMax[1], 8, 2048},
                                   {kQuadClassMax[1] + 1u, kQuadClassMax[2], 4, 1024}};

uint32_t class_waves(const QuadClass& c, uint64_t chi, uint32_t n_batches) {
  const uint64_t want = std::max<uint32_t>(c.waves / n_batches, 1u);
  const uint32_t w = (uint32_t)std::min<uint64_t>(want, chi);
  return (w + c.nw - 1u) / c.nw * c.nw;
}

}  // namespace

QuadPlan quad_plan(uint32_t n, uint64_t chi, uint32_t L, uint32_t slots) {
  QuadPlan P{};
  P.chi = chi;
  P.n_batches = (L + 127u) / 128u;
  P.slots = slots;
  // Up to 23 qubits no form is of the largest class, and 8 bras pay for the others: no
  // second set of records (n = 20, chi = 20000, 8 bras 353 µs and 380).
  if (slots && (n > 23u || L < 8u)) {
    // Linear in n; from 55 qubits on a slice leaves room for one workgroup of the
    // smallest class per compute unit.  Where a call holds the largest class it mostly
    // holds other forms as well, which leaves the class's waves uneven shares: a
    // quarter more, and half from 56 qubits on, where deep sets have forms past it
    // (n = 50, 48 bras, |v| = 25: 2.80 ms with a part of the kets and 1.96 by pairs; n = 58,
    // |v| = 55..58, 24 bras 2.99 and 2.0).
    const double small = std::max(40.0, 9.5 * n - 40.0) * (n >= 55u ? 1.55 : 1.0);
    const double us[3] = {small, std::max(100.0, 20.0 * n - 300.0),
                          std::max(800.0, 35.4 * n - 70.0) * (n >= 56u ? 1.5 : 1.25)};
    for (int k = 0; k < 3; ++k) P.rule.cost[k] = (uint32_t)(us[k] * 10.0 / 32.0);
  }
  P.rule.per = std::max(1u, L / P.n_batches);
  P.ne1 = n + slots + 1u;
  for (const QuadClass& c : kClasses)
    if (c.nc_lo <= n + slots) P.rows += class_waves(c, chi, P.n_batches);
  P.rec_words = ((size_t)chi * rec_layout(n).words + 1u) & ~(size_t)1;  // the slices are read 16 bytes at a time
  P.slice_words = (size_t)P.n_batches * slice_entries(n, P.ne1) * 2u;
  P.many = n + slots > kClasses[0].nc_hi;
  P.words = P.rec_words + P.slice_words + (size_t)P.n_batches * 64u + kQuadStatWords / 2u;
  return P;
}

uint32_t* quad_stat(const QuadPlan& P, uint64_t* work) {
  return reinterpret_cast<uint32_t*>(work + P.rec_words + P.slice_words + (size_t)P.n_batches * 64u);
}

hipError_t launch_quad_prep(const TermsView& T, uint64_t count, const QuadPlan& P, uint64_t* work, hipStream_t st) {
  const bool counts = P.many || P.slots;
  if (counts) {
    const hipError_t e = hipMemsetAsync(quad_stat(P, work), 0, kQuadStatWords * sizeof(uint32_t), st);
    if (e != hipSuccess) return e;
  }
  for (uint64_t first = 0; first < count; first += kWaveTerms) {
    const uint64_t c = std::min(kWaveTerms, count - first);
    hipLaunchKernelGGL(k_quad_prep, dim3((uint32_t)((c + kPrepWaves - 1) / kPrepWaves)), dim3(64 * kPrepWaves), 0, st,
                       terms_from(T, first), c, work + first * rec_layout(T.n).words,
                       counts ? quad_stat(P, work) : nullptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_quad_equatorial(const uint64_t* Aoff, const uint8_t* Adiag, uint32_t n, uint32_t L,
                                  const QuadPlan& P, uint64_t* work, hipStream_t st) {
  uint32_t* sl = reinterpret_cast<uint32_t*>(work + P.rec_words);
  uint32_t* info = reinterpret_cast<uint32_t*>(work + P.rec_words + P.slice_words);
  hipLaunchKernelGGL(k_slice_equatorial, dim3(2u * P.n_batches, n + 2u), dim3(64), 0, st, Aoff, Adiag, n, L, P.ne1, sl,
                     info);
  return hipGetLastError();
}

hipError_t launch_quad_bras(const TermsView& Tb, const uint64_t* chrec, uint32_t chrec_words, uint32_t L,
                            const QuadPlan& P, uint64_t* work, hipStream_t st) {
  uint32_t* sl = reinterpret_cast<uint32_t*>(work + P.rec_words);
  uint32_t* info = reinterpret_cast<uint32_t*>(work + P.rec_words + P.slice_words);
  hipLaunchKernelGGL(k_slice_bras, dim3(2u * P.n_batches, Tb.n + 2u), dim3(64), 0, st, Tb, chrec, chrec_words, L, P.ne1,
                     P.slots, sl, info, quad_stat(P, work));
  return hipGetLastError();
}

hipError_t launch_quad_pairs(const TermsView& T, uint64_t count, uint32_t L, const QuadPlan& P, uint64_t* work,
                             double2* partial, hipStream_t st) {
  QuadArgs A{};
  A.rec = work;
  A.b = T.b;
  A.chi = count;
  A.sl = reinterpret_cast<const uint32_t*>(work + P.rec_words);
  A.info = reinterpret_cast<const uint32_t*>(work + P.rec_words + P.slice_words);
  A.stat = quad_stat(P, work);
  A.n = T.n;
  A.ne1 = P.ne1;
  A.slots = P.slots;
  A.rule = P.rule;
  A.L = L;
  A.n_batches = P.n_batches;
  A.many = P.many;
  A.partial = partial;
  const uint32_t sm = slice_entries(T.n, P.ne1) * 16u;
  for (int k = 0; k < 3; ++k) {
    const QuadClass& c = kClasses[k];
    if (c.nc_lo > T.n + P.slots) break;
    A.cls = (uint32_t)k;
    A.nc_lo = c.nc_lo;
    A.nc_hi = c.nc_hi;
    A.n_waves = class_waves(c, P.chi, P.n_batches);
    const dim3 grid(P.n_batches * (A.n_waves / c.nw)), block(64u * c.nw);
    void (*const fn)(QuadArgs) = k == 0   ? k_quad_pairs<2, 28, 8, 4>
                                 : k == 1 ? k_quad_pairs<3, 48, 8, 2>
                                          : k_quad_pairs<4, 60, 4, 1>;
    if (sm > 64u * 1024u) {
      const hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn, grid, block, sm, st, A);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    A.partial += (size_t)A.n_waves * L;
  }
  return hipSuccess;
}

}  // namespace chsim
