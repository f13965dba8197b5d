// Metropolis chain over n-bit outputs (Sec. "Heuristic Metropolis simulator").
//
// Each chain c keeps, per term alpha, the Pauli Q_x = i^mu Z(t) X(u) of its
// current string x, stored as the word u | mu << 62 (t is not needed for the
// amplitude, and the product with U_C^{-1} X_j U_C is taken on the right:
// the two factors commute, so Q_x P_j = P_j Q_x).  A step proposes y = x ^ e_j:
//   u' = u ^ F_j,  mu' = mu + gamma_j + 2 par(u' & M_j),
// and <y|phi_alpha> follows from (u', mu') as in Eq. (amplitude1), O(1) words
// per term and chain.
//
// Kernels: (1) k_propose_pair (single flips; two steps per launch, the second
// for either outcome of the first, the cache brought up to date once per
// window of kMetroWin steps) or k_propose (flip masks: the tile's rows staged in
// LDS; the cache is brought up to date with an accepted mask at the next step,
// in place): lanes over terms, sums of b_alpha <y|phi_alpha> over the 256-term
// tile in FP64; (2) one workgroup per chain: add the tiles' partials in a fixed
// order, r = |A(y)|^2 / |A(x)|^2 in FP64, accept iff U < r.
#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "internal.hpp"

namespace chsim {

namespace {

struct TermAmpConst {
  uint64_t v, s;
  uint32_t w;
  double w0r, w0i;  // b_alpha 2^{-|v|/2}
};

__device__ __forceinline__ TermAmpConst load_const(const TermsView& T, uint64_t a) {
  TermAmpConst c;
  c.v = T.v[a];
  c.s = T.s[a];
  c.w = T.omega[a];
  const double2 b = T.b[a];
  const int vc = __popcll(c.v);
  const double h = 0.70710678118654752440;
  const double mag = ldexp(1.0, -(vc >> 1)) * ((vc & 1) ? h : 1.0);
  c.w0r = b.x * mag;
  c.w0i = b.y * mag;
  return c;
}

// b <x|phi> from the cached (u, mu), without branches: the rotation by
// e^{i pi k / 4} (an odd k first multiplies by e^{i pi / 4}, then i^{k >> 1}
// swaps and negates), and zero when x is outside the term's support.
__device__ __forceinline__ double2 term_value(const TermAmpConst& c, uint64_t u, uint32_t mu) {
  // u and s have no bits at or above n, so outside supp(v) is ~v.
  const bool off = ((u ^ c.s) & ~c.v) != 0ull;
  const uint32_t k = (c.w + 2u * mu + 4u * __popcll(u & c.v & c.s)) & 7u;
  const double h = 0.70710678118654752440;
  const double a = (k & 1u) ? (c.w0r - c.w0i) * h : c.w0r;
  const double b = (k & 1u) ? (c.w0r + c.w0i) * h : c.w0i;
  const uint32_t m = k >> 1;
  double re = (m & 1u) ? b : a, im = (m & 1u) ? a : b;
  re = __longlong_as_double(__double_as_longlong(re) ^ ((long long)((m ^ (m >> 1)) & 1u) << 63));
  im = __longlong_as_double(__double_as_longlong(im) ^ ((long long)(m >> 1) << 63));
  return make_double2(off ? 0.0 : re, off ? 0.0 : im);
}

constexpr uint64_t kUMask = (1ull << 62) - 1ull;

// A double moved between lanes by DPP (two 32-bit moves on the VALU).
template <int kCtrl>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, kCtrl, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), kCtrl, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum of x over the wave's 64 lanes, valid in lane 0, in a fixed order:
// within quads (lane ^ 1, lane ^ 2) and rows of 16 (half-row and row
// mirrors) by DPP moves, across the two rows of each half by one swizzle,
// and the halves by a read of lane 32.
__device__ __forceinline__ double wave_sum0(double x) {
  x += dpp_f64<0xB1>(x);   // quad_perm [1, 0, 3, 2]
  x += dpp_f64<0x4E>(x);   // quad_perm [2, 3, 0, 1]
  x += dpp_f64<0x141>(x);  // row_half_mirror
  x += dpp_f64<0x140>(x);  // row_mirror
  x += __shfl_xor(x, 16);
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 32);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 32);
  return x + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum of a double2 over the 256-thread block (fixed order); result in thread 0.
__device__ __forceinline__ double2 block_sum(double2 v, double2* scratch) {
  for (int m = 32; m >= 1; m >>= 1) {
    v.x += __shfl_down(v.x, m);
    v.y += __shfl_down(v.y, m);
  }
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  double2 r = make_double2(0.0, 0.0);
  if (threadIdx.x == 0) {
    for (int w = 0; w < 4; ++w) {
      r.x += scratch[w].x;
      r.y += scratch[w].y;
    }
  }
  return r;
}

// Few chains: the initial Q_x of every chain (the O(k n^2) start-up cost) and the tile sums of
// <x_c|psi>.
__global__ __launch_bounds__(256) void k_metro_init(TermsView T, MetroView Mv) {
  __shared__ double2 scratch[4];
  const uint64_t a = (uint64_t)blockIdx.x * kMetroTile + threadIdx.x;
  const bool live = a < T.chi;
  const uint64_t chi = T.chi;
  TermAmpConst c;
  if (live) c = load_const(T, a);
  for (uint32_t ch = 0; ch < Mv.n_chain; ++ch) {
    const uint32_t n = T.n;
    const uint64_t x = Mv.x[ch] & ((n == 64) ? ~0ull : ((1ull << n) - 1ull));
    double2 val = make_double2(0.0, 0.0);
    if (live) {
      uint64_t u = 0, xm = x;
      uint32_t mu = 0;
      while (xm) {
        const uint32_t p = (uint32_t)__builtin_ctzll(xm);
        xm &= xm - 1ull;
        u ^= T.F[(uint64_t)p * chi + a];
        mu += T.gamma[(uint64_t)p * chi + a] + 2u * par64(u & T.M[(uint64_t)p * chi + a]);
      }
      mu &= 3u;
      Mv.state[(uint64_t)ch * chi + a] = (u & kUMask) | ((uint64_t)mu << 62);
      val = term_value(c, u, mu);
    }
    const double2 tot = block_sum(val, scratch);
    if (threadIdx.x == 0) Mv.partial[(uint64_t)ch * Mv.n_tiles + blockIdx.x] = tot;
  }
}

__global__ __launch_bounds__(256) void k_chain_amp(MetroView Mv) {
  __shared__ double2 scratch[4];
  const uint32_t ch = blockIdx.x;
  double2 acc = make_double2(0.0, 0.0);
  for (uint32_t t = threadIdx.x; t < Mv.n_tiles; t += 256u) {
    const double2 v = Mv.partial[(uint64_t)ch * Mv.n_tiles + t];
    acc.x += v.x;
    acc.y += v.y;
  }
  const double2 tot = block_sum(acc, scratch);
  if (threadIdx.x == 0) Mv.amp[ch] = tot;
}


// Flip-mask proposal step y = x ^ m for every chain, per term: the chain's
// cache is first brought up to date with the mask it accepted at the
// previous step (pmask, when the mode says so; written back in place, so a
// cache word is written only after an accepted move), then Q_y = Q_x
// prod_{j in m} P_j (right products; the factors commute) and
// sum_a b_a <y|phi_a> per chain over the block's 256 terms.  The block walks
// its tile in sub-tiles of 64 terms: the rows F_p, M_p, gamma_p of the
// sub-tile are staged in LDS once ([p][term], so a wave reading row j for
// its 64 terms is conflict-free), and wave w of 8 takes the chains c = w,
// w + 8, ...; a chain's masks are wave-uniform, so the loops over their set
// bits do not diverge and each term's rows leave HBM once per step for all
// chains.
//
// With kInit it is the chains' start: Q_x = prod_{j in x} P_j from the
// identity (no cache word is read), the cache words are written, and the sums are
// those of <x|psi>.  Reading the rows once for all chains instead of once per
// chain: n = 50, chi = 2^20, 64 chains 880 µs (3944 with the term store's
// rows read by each chain); n = 12, chi = 2^16: 41 and 105.
constexpr uint32_t kSub = 64;
constexpr int kCW = 8;           // chains per wave in one pass
constexpr uint32_t kPWaves = 8;  // waves per block: kPWaves * kCW = 64 chains per pass
constexpr uint32_t kPThreads = 64 * kPWaves;
constexpr int kStage = (int)((64 * kSub + kPThreads - 1) / kPThreads);  // staging loads per thread
static_assert(kStage % 2 == 0, "staged in two halves");

template <bool kInit>
__global__ __launch_bounds__(kPThreads) void k_propose(TermsView T, MetroView Mv,
                                                       const uint64_t* __restrict__ mask,
                                                       uint32_t mode) {
  extern __shared__ __align__(16) uint8_t smem[];
  const uint32_t n = T.n;
  uint64_t* sF = reinterpret_cast<uint64_t*>(smem);  // [n][64]
  uint64_t* sM = sF + (size_t)n * kSub;               // [n][64]
  uint8_t* sG = reinterpret_cast<uint8_t*>(sM + (size_t)n * kSub);  // [n][64]
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform32(tid >> 6);
  const uint64_t chi = T.chi;
  const bool pend = !kInit && (mode & kProposeApplyPending), prop = kInit || (mode & kProposeMasks);
  const uint64_t nmask = (1ull << n) - 1ull;  // n <= 62
  // Right product by P_j for every set bit j of mm.
  auto apply = [&](uint64_t& u, uint32_t& mu, uint64_t mm) {
    while (mm) {
      const uint32_t j = (uint32_t)__builtin_ctzll(mm);
      mm &= mm - 1ull;
      u ^= sF[j * kSub + lane];
      mu += (uint32_t)sG[j * kSub + lane] + 2u * par64(u & sM[j * kSub + lane]);
    }
  };
  for (uint32_t cg = 0; cg < Mv.n_chain; cg += kPWaves * kCW) {
    // This wave's chains in the pass: cg + wave + kPWaves k, k < kCW (wave-uniform).
    uint64_t m[kCW], pm[kCW];
    double accr[kCW], acci[kCW];
#pragma unroll
    for (int k = 0; k < kCW; ++k) {
      const uint32_t ch = cg + wave + kPWaves * (uint32_t)k;
      const bool on = ch < Mv.n_chain;
      m[k] = on && prop ? uniform64(kInit ? Mv.x[ch] & nmask : mask[ch]) : 0ull;
      pm[k] = on && pend ? uniform64(Mv.pmask[ch]) : 0ull;
      accr[k] = 0.0;
      acci[k] = 0.0;
    }
    // At the start only the rows of some chain's bits are read (one chain has half of them).
    uint64_t rows = ~0ull;
    if (kInit) {
      rows = cg + lane < Mv.n_chain ? Mv.x[cg + lane] : 0ull;  // the pass's 64 chains, one per lane
      for (int k = 32; k >= 1; k >>= 1) rows |= __shfl_xor(rows, k);
    }
    for (uint32_t sub = 0; sub < kMetroTile / kSub; ++sub) {
      const uint64_t base = (uint64_t)blockIdx.x * kMetroTile + (uint64_t)sub * kSub;
      if (base >= chi) break;  // block-uniform
      __syncthreads();         // the previous sub-tile's readers are done
      // The thread's share of the sub-tile is staged in two halves; within a
      // half every load is issued before the first store to LDS.
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        uint64_t rf[kStage / 2], rm[kStage / 2];
        uint32_t rg[kStage / 2];
#pragma unroll
        for (int r = 0; r < kStage / 2; ++r) {
          const uint32_t i = tid + (uint32_t)(half * (kStage / 2) + r) * kPThreads;
          const uint32_t p = i / kSub, t = i % kSub;
          const uint64_t at = base + t;
          const bool in = i < n * kSub && at < chi && ((rows >> p) & 1ull);
          rf[r] = in ? T.F[(uint64_t)p * chi + at] : 0ull;
          rm[r] = in ? T.M[(uint64_t)p * chi + at] : 0ull;
          rg[r] = in ? T.gamma[(uint64_t)p * chi + at] : 0u;
        }
#pragma unroll
        for (int r = 0; r < kStage / 2; ++r) {
          const uint32_t i = tid + (uint32_t)(half * (kStage / 2) + r) * kPThreads;
          if (i < n * kSub) {
            sF[i] = rf[r];
            sM[i] = rm[r];
            sG[i] = (uint8_t)rg[r];
          }
        }
      }
      const uint64_t a = base + lane;
      const bool live = a < chi;
      // Every cache word of this wave's chains is requested before any is used.
      uint64_t st[kCW];
#pragma unroll
      for (int k = 0; k < kCW; ++k) {
        const uint32_t ch = cg + wave + kPWaves * (uint32_t)k;
        st[k] = (!kInit && live && (m[k] | pm[k]) != 0ull) ? Mv.state[(uint64_t)ch * chi + a] : 0ull;
      }
      TermAmpConst c{};
      if (live && prop) c = load_const(T, a);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kCW; ++k) {
        const uint32_t ch = cg + wave + kPWaves * (uint32_t)k;
        // Nothing to do, no such chain, or past chi.
        if (((m[k] | pm[k]) == 0ull && !(kInit && ch < Mv.n_chain)) || !live) continue;
        uint64_t u = st[k] & kUMask;
        uint32_t mu = (uint32_t)(st[k] >> 62);
        if (pm[k]) {
          apply(u, mu, pm[k]);
          mu &= 3u;
          Mv.state[(uint64_t)ch * chi + a] = u | ((uint64_t)mu << 62);
        }
        if (m[k] == 0ull && !kInit) continue;  // y = x: no proposal
        apply(u, mu, m[k]);
        if (kInit) Mv.state[(uint64_t)ch * chi + a] = u | ((uint64_t)(mu & 3u) << 62);
        const double2 val = term_value(c, u, mu & 3u);
        accr[k] += val.x;
        acci[k] += val.y;
      }
    }
    // One reduction over the lanes (terms) per chain.
#pragma unroll
    for (int k = 0; k < kCW; ++k) {
      const uint32_t ch = cg + wave + kPWaves * (uint32_t)k;
      if (ch >= Mv.n_chain || !prop) continue;  // wave-uniform
      double re = accr[k], im = acci[k];
      re = wave_sum0(re);
      im = wave_sum0(im);
      if (lane == 0) Mv.partial[(uint64_t)ch * Mv.n_tiles + blockIdx.x] = make_double2(re, im);
    }
  }
}

// Two single-flip steps per launch, with deferred cache updates.  Lanes over
// terms (each lane takes four terms of the 256-term tile), waves over chains.
//
// Speculation.  Steps t and t + 1 propose bits j1 and j2 that are known before
// either is decided, so one reading of a chain's cached words serves both: the
// sums for y = x + e_j1 (step t) and, for step t + 1, for x + e_j2 (step t
// rejected) and x + e_j1 + e_j2 (accepted).  The accept kernel takes both
// decisions.  That is three values per two steps instead of two, for half the
// reads of the cache and half the launches.
//
// Deferred updates.  A chain's cached (u, mu) is brought up to date only once
// per window of kMetroWin steps: a pair of steps in the window that starts at t0
// reads the cache as of t0, applies the flips the chain accepted since (right
// products by their P_j in step order: the same arithmetic as updating after
// every accepted step), then the proposals' P_j.  The first pair of the next
// window (and a final pass without a proposal at the end of a call) writes the
// brought-up-to-date cache back in place.
//
// Rows.  kSlots64, kSlots32 (n <= 30: one 32-bit half): the tile's rows of chain
// 0's bits at the pending and proposed steps are staged in LDS and serve every
// chain whose bit at that step is the same (every chain, when the chains share
// the flip bit of a step); a chain with another bit reads its row from the term
// store.  kPacked (n <= 15): every row of the tile is staged, F, M and gamma of a
// row and term in one word, so any chain's bits cost one LDS read.
//
// Values.  With gamma_j + 2 par(F_j & v & s) in place of gamma_j, mu carries
// 2 par(u & v & s) along (added once when a cached word is read), and a term's
// value is one of four, b 2^{-|v|/2} e^{i pi omega/4} i^mu, read from LDS ([mu][term]:
// no bank conflicts), or zero outside the support.  The 12 sums of two chains
// (three values, re and im) are reduced over the wave together: the halves of
// the wave exchange two sums at a time (v_permlane32_swap, then 16), so 12
// become 3 before the 16 lanes of a row are added by DPP moves: 63 instructions
// against about 240 for twelve trees.
//
// VALU issue bounds it: 102 instructions per 64 terms, chain and pair of steps at
// n = 50 (about 190 of the 279 µs per launch at chi = 2^20 and 64 chains with one
// flip bit; 537 MB read, and as much written by every second launch).  Before, one
// step per launch with the values computed per proposal: 196 µs per step, now 140;
// n = 12, chi = 2^16, 64 chains with their own bits (kPacked): 29 and 10.7.  Few chains
// (whole calls, 40 steps with own bits, n = 50, chi = 200000, in µs, one step per launch
// and now): 1 chain 469 and 440, 2 chains 533 and 528, 5 chains 711 and 644, 12 chains
// 1025 and 974.
constexpr uint32_t kGWaves = 4;
constexpr uint32_t kGSub = kMetroTile / 64;  // terms per lane
constexpr uint32_t kModeWrite = 1u;
enum { kSlots64 = 0, kSlots32 = 1, kPacked = 2 };
constexpr uint32_t kSlots = kMetroWin + 2;  // pending steps, then the two proposals
constexpr uint32_t kPackedMaxN = 15, kSlots32MaxN = 30;

// a + b over the halves of the wave: lanes 0-31 hold a's sum, lanes 32-63 b's.
__device__ __forceinline__ double swap_add32(double a, double b) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
// The same over the 16-lane rows of each half: rows 0, 2 keep a, rows 1, 3 take b.
__device__ __forceinline__ double swap_add16(double a, double b) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double row_sum(double x) {
  x += dpp_f64<0xB1>(x);   // quad_perm [1, 0, 3, 2]
  x += dpp_f64<0x4E>(x);   // quad_perm [2, 3, 0, 1]
  x += dpp_f64<0x141>(x);  // row_half_mirror
  x += dpp_f64<0x140>(x);  // row_mirror
  return x;
}

template <int kMode>
__global__ __launch_bounds__(64 * kGWaves) void k_propose_pair(TermsView T, MetroView Mv, uint32_t step,
                                                               uint32_t nprop, uint32_t pbase, uint32_t npend,
                                                               uint32_t mode) {
  constexpr bool k64 = kMode == kSlots64, kAll = kMode == kPacked;
  using Word = typename std::conditional<k64, uint64_t, uint32_t>::type;
  extern __shared__ __align__(16) uint8_t smem[];
  // Values [5][256] (the fifth row zero), then the rows.
  double2* const val = reinterpret_cast<double2*>(smem);
  uint8_t* const rows = smem + 5u * kMetroTile * sizeof(double2);
  Word* const sF = reinterpret_cast<Word*>(rows);                                 // [kSlots][256]
  Word* const sM = sF + kSlots * kMetroTile;                                      // [kSlots][256]
  uint8_t* const sG = reinterpret_cast<uint8_t*>(sM + kSlots * kMetroTile);       // [kSlots][256]
  uint32_t* const sP = reinterpret_cast<uint32_t*>(rows);                         // [n][256], kPacked
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform32(tid >> 6);
  const uint32_t n = T.n, nc = Mv.n_chain;
  const uint64_t chi = T.chi;
  const uint64_t tile0 = (uint64_t)blockIdx.x * kMetroTile;
  const bool full = tile0 + kMetroTile <= chi;  // block-uniform
  const bool write = mode & kModeWrite;
  // Term offsets within the tile, clamped to the last term in a partial tile:
  // past chi a lane reads that term's words, contributes zero (its values are
  // zero) and writes nothing.
  const uint32_t last = (uint32_t)(chi - 1ull - tile0);
  {
    // The thread's own term: values and rows.
    const uint32_t mine = min(tid, last);
    const uint64_t a = tile0 + mine;
    const uint64_t v = T.v[a], s = T.s[a], vs = v & s;
    if (nprop) {
      const TermAmpConst c = load_const(T, a);
      const double h = 0.70710678118654752440;
      const bool in = tid <= last;
      double wr = (c.w & 1u) ? (c.w0r - c.w0i) * h : c.w0r, wi = (c.w & 1u) ? (c.w0r + c.w0i) * h : c.w0i;
      for (uint32_t m = 0; m < 4u; ++m) {  // times i^m: exact
        val[((m + 4u - (c.w >> 1)) & 3u) * kMetroTile + tid] = in ? make_double2(wr, wi) : make_double2(0.0, 0.0);
        const double t = wr;
        wr = -wi;
        wi = t;
      }
      val[4u * kMetroTile + tid] = make_double2(0.0, 0.0);
    }
    if (kAll) {
      for (uint32_t p = 0; p < n; ++p) {
        const uint64_t at = (uint64_t)p * chi + a;
        const uint32_t f = (uint32_t)T.F[at];
        const uint32_t g = ((uint32_t)T.gamma[at] + 2u * (uint32_t)__popc(f & (uint32_t)vs)) & 3u;
        sP[p * kMetroTile + tid] = f | ((uint32_t)T.M[at] << 15) | (g << 30);
      }
    } else {
#pragma unroll
      for (uint32_t q = 0; q < kSlots; ++q) {
        const bool use = q < kMetroWin ? q < npend : q - kMetroWin < nprop;
        if (!use) continue;
        const uint32_t j = uniform32(Mv.jstream[q < kMetroWin ? pbase + q : step + (q - kMetroWin)]) % n;
        const uint64_t at = (uint64_t)j * chi + a, f = T.F[at];
        sF[q * kMetroTile + tid] = (Word)f;
        sM[q * kMetroTile + tid] = (Word)T.M[at];
        sG[q * kMetroTile + tid] = (uint8_t)((T.gamma[at] + 2u * (uint32_t)__popcll(f & vs)) & 3u);
      }
    }
  }
  uint32_t Wj[kSlots];
#pragma unroll
  for (uint32_t q = 0; q < kSlots; ++q) {
    const bool use = q < kMetroWin ? q < npend : q - kMetroWin < nprop;
    Wj[q] = !kAll && use ? uniform32(Mv.jstream[q < kMetroWin ? pbase + q : step + (q - kMetroWin)]) % n : ~0u;
  }
  uint32_t ao[kGSub];
  Word nv[kGSub], snv[kGSub], vs[kGSub];
#pragma unroll
  for (uint32_t sb = 0; sb < kGSub; ++sb) {
    ao[sb] = min(sb * 64u + lane, last);
    const uint64_t v = T.v[tile0 + ao[sb]], s = T.s[tile0 + ao[sb]];
    nv[sb] = (Word)~v;  // u and s have no bits at or above n
    snv[sb] = (Word)(s & ~v);
    vs[sb] = (Word)(v & s);
  }
  __syncthreads();
  auto popc = [](Word x) { return (uint32_t)(k64 ? __popcll((uint64_t)x) : __popc((uint32_t)x)); };
  // Right product by P_j (step slot q) for the lane's terms.
  auto flip = [&](Word (&u)[kGSub], uint32_t (&mu)[kGSub], uint32_t q, uint32_t j) {
    if constexpr (kAll) {
#pragma unroll
      for (uint32_t sb = 0; sb < kGSub; ++sb) {
        const uint32_t w = sP[j * kMetroTile + sb * 64u + lane];
        u[sb] ^= (Word)(w & 0x7FFFu);
        mu[sb] += (w >> 30) + 2u * popc(u[sb] & (Word)(w >> 15));  // u has 15 bits
      }
    } else if (j == Wj[q]) {  // wave-uniform
#pragma unroll
      for (uint32_t sb = 0; sb < kGSub; ++sb) {
        const uint32_t at = q * kMetroTile + sb * 64u + lane;
        u[sb] ^= sF[at];
        mu[sb] += (uint32_t)sG[at] + 2u * popc(u[sb] & sM[at]);
      }
    } else {
      const uint64_t* F = T.F + ((uint64_t)j * chi + tile0);
      const uint64_t* M = T.M + ((uint64_t)j * chi + tile0);
      const uint8_t* g = T.gamma + ((uint64_t)j * chi + tile0);
#pragma unroll
      for (uint32_t sb = 0; sb < kGSub; ++sb) {
        const Word f = (Word)F[ao[sb]];
        u[sb] ^= f;
        mu[sb] += (uint32_t)g[ao[sb]] + 2u * popc(f & vs[sb]) + 2u * popc(u[sb] & (Word)M[ao[sb]]);
      }
    }
  };
  // Sum of the lane's four terms' values.
  auto value = [&](const Word (&u)[kGSub], const uint32_t (&mu)[kGSub], double& re, double& im) {
#pragma unroll
    for (uint32_t sb = 0; sb < kGSub; ++sb) {
      const bool off = ((u[sb] & nv[sb]) ^ snv[sb]) != (Word)0;
      const uint32_t m = off ? 4u : mu[sb] & 3u;
      const double2 x = val[m * kMetroTile + sb * 64u + lane];
      re = sb ? re + x.x : x.x;
      im = sb ? im + x.y : x.y;
    }
  };
  // The wave's chains are ch = w0 + n_waves i.  Their per-chain words (the
  // pending mask and the bits of the pending and proposed steps) are read for 64
  // chains at once, chain i % 64 in lane i % 64, and taken from there by lane
  // reads, so that no wait for them also waits for the cache words in flight.
  const uint32_t w0 = blockIdx.y * kGWaves + wave, n_waves = gridDim.y * kGWaves;
  const uint32_t n_mine = nc > w0 ? (nc - w0 + n_waves - 1u) / n_waves : 0u;
  const uint32_t pmask = (1u << npend) - 1u;  // npend <= kMetroWin < 32
  const size_t plane = (size_t)nc * Mv.n_tiles;
  for (uint32_t i0 = 0; i0 < n_mine; i0 += 64u) {
    uint32_t m_pm, m_js[kSlots];
    {
      const uint32_t i = i0 + lane;
      const uint32_t ch = i < n_mine ? w0 + n_waves * i : w0;
      const uint64_t jrow = (uint64_t)ch * Mv.n_steps;
      m_pm = npend ? Mv.pend[ch] & pmask : 0u;
#pragma unroll
      for (uint32_t q = 0; q < kSlots; ++q) {
        const bool use = q < kMetroWin ? q < npend : q - kMetroWin < nprop;
        m_js[q] = use ? Mv.jstream[jrow + (q < kMetroWin ? pbase + q : step + (q - kMetroWin))] % n : 0u;
      }
    }
    const uint32_t i_end = min(n_mine - i0, 64u);
    // Chains k0 .. k0 + CP - 1: all their cache words are requested before any is
    // combined.
    auto pass = [&](auto cp, uint32_t k0) {
      constexpr uint32_t CP = decltype(cp)::value;
      uint64_t st[CP][kGSub];
#pragma unroll
      for (uint32_t h = 0; h < CP; ++h) {
        const uint32_t k = k0 + h;
        const uint64_t* sp = Mv.state + ((uint64_t)(w0 + n_waves * (i0 + k)) * chi + tile0);
#pragma unroll
        for (uint32_t sb = 0; sb < kGSub; ++sb) st[h][sb] = sp[ao[sb]];
      }
      double sum[12];  // [chain][value][re, im]
#pragma unroll
      for (uint32_t q = 6u * CP; q < 12u; ++q) sum[q] = 0.0;
#pragma unroll
      for (uint32_t h = 0; h < CP; ++h) {
        const uint32_t k = k0 + h;
        Word u[kGSub];
        uint32_t mu[kGSub];
#pragma unroll
        for (uint32_t sb = 0; sb < kGSub; ++sb) {
          u[sb] = (Word)(st[h][sb] & kUMask);
          mu[sb] = (uint32_t)(st[h][sb] >> 62) + 2u * popc(u[sb] & vs[sb]);
        }
        const uint32_t pm = (uint32_t)__builtin_amdgcn_readlane((int)m_pm, (int)k);
#pragma unroll
        for (uint32_t q = 0; q < kMetroWin; ++q)
          if ((pm >> q) & 1u) flip(u, mu, q, (uint32_t)__builtin_amdgcn_readlane((int)m_js[q], (int)k));
        if (write) {
          uint64_t* sp = Mv.state + ((uint64_t)(w0 + n_waves * (i0 + k)) * chi + tile0);
#pragma unroll
          for (uint32_t sb = 0; sb < kGSub; ++sb) {
            const uint32_t m = (mu[sb] + 2u * popc(u[sb] & vs[sb])) & 3u;
            if (full || sb * 64u + lane <= last) sp[sb * 64u + lane] = (uint64_t)u[sb] | ((uint64_t)m << 62);
          }
        }
        if (nprop == 0u) continue;
        const uint32_t j1 = (uint32_t)__builtin_amdgcn_readlane((int)m_js[kMetroWin], (int)k);
        const uint32_t j2 = (uint32_t)__builtin_amdgcn_readlane((int)m_js[kMetroWin + 1], (int)k);
        Word u1[kGSub];
        uint32_t mu1[kGSub];
#pragma unroll
        for (uint32_t sb = 0; sb < kGSub; ++sb) {
          u1[sb] = u[sb];
          mu1[sb] = mu[sb];
        }
        double* const sm = sum + 6 * h;
        flip(u1, mu1, kMetroWin, j1);
        value(u1, mu1, sm[0], sm[1]);
        if (nprop == 2u) {
          flip(u1, mu1, kMetroWin + 1u, j2);
          value(u1, mu1, sm[2], sm[3]);
          flip(u, mu, kMetroWin + 1u, j2);
          value(u, mu, sm[4], sm[5]);
        } else {
          sm[2] = sm[3] = sm[4] = sm[5] = 0.0;
        }
      }
      if (nprop == 0u) return;
      // 12 sums over 64 lanes: r[k] holds sums 4 k, 4 k + 2, 4 k + 1, 4 k + 3 in its rows.
      double r[3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        r[k] = row_sum(swap_add16(swap_add32(sum[4 * k], sum[4 * k + 1]), swap_add32(sum[4 * k + 2], sum[4 * k + 3])));
      const uint32_t rr = lane >> 4, kk = lane & 15u;
      const double x = kk == 0u ? r[0] : kk == 1u ? r[1] : r[2];
      const uint32_t f = 4u * kk + ((rr & 1u) << 1 | rr >> 1);  // [chain][value][re, im]
      const uint32_t h = f >= 6u ? 1u : 0u, g = f - 6u * h;
      if (kk < 3u && h < CP && (g < 2u || nprop == 2u)) {
        const uint32_t ch = w0 + n_waves * (i0 + k0 + h);
        double* const out = reinterpret_cast<double*>(Mv.partial + (g >> 1) * plane + (size_t)ch * Mv.n_tiles + blockIdx.x);
        out[g & 1u] = x;
      }
    };
    // Two chains per pass, an odd last one alone.
    uint32_t k0 = 0;
    for (; k0 + 1u < i_end; k0 += 2u) pass(std::integral_constant<uint32_t, 2>{}, k0);
    if (k0 < i_end) pass(std::integral_constant<uint32_t, 1>{}, k0);
  }
}

// The rows' form: 32-bit halves up to n = 30 (M and F in one register each),
// 64-bit words above; packed where n bits of F and M and two of gamma fit a word
// and reading every row of a tile costs less than the bits' rows.  It does while
// there are no more rows than slots; while the rows (17 bytes each) stay in the
// L2s, 4 MB per XCD; and past them from a number of chains with bits of their own
// that grows with n.  Whole calls of 40 steps, own bits, in µs, packed and not:
// n = 12, chi = 2^16: 2 chains 289 and 317, 12 chains 347 and 413 (one bit for all
// chains: 287 and 310, 341 and 359); chi = 2^20: n = 8, 1 chain 1230 and 1069, 2
// chains 1089 and 1222; n = 12, 3 chains 1510 and 1376, 4 chains 1566 and 1627, 12
// chains 2243 and 3604; n = 15, 5 chains 1957 and 1674, 6 chains 2062 and 2037, 8
// chains 2223 and 2425.  (One bit for all of them is not known here: n = 15, 6
// chains 2055 and 1281, 12 chains 2542 and 1666.)
constexpr uint64_t kPackedBytes = 28ull << 20;
bool packs_rows(uint32_t n, uint64_t chi, uint32_t n_chain) {
  if (n > kPackedMaxN) return false;
  return n <= kSlots || chi <= kPackedBytes / (17u * n) || n_chain >= std::max(2u, n * n / 32u);
}

// Workgroups along the chains: with few tiles the chains are split over more
// workgroups (the tile's rows staged by each), up to about four per compute
// unit; a wave keeps at least two chains, the pair of one pass.
uint32_t chain_splits(uint32_t n_tiles, uint32_t n_chain) {
  const uint32_t want = (1024u + n_tiles - 1u) / n_tiles, most = (n_chain + 2u * kGWaves - 1u) / (2u * kGWaves);
  return std::max(1u, std::min(want, most));
}

hipError_t launch_pair(const TermsView& T, MetroView& Mv, uint32_t step, uint32_t nprop, uint32_t pbase,
                       uint32_t npend, uint32_t mode, hipStream_t st) {
  const dim3 grid(Mv.n_tiles, chain_splits(Mv.n_tiles, Mv.n_chain));
  const size_t vals = 5u * kMetroTile * sizeof(double2);
  if (packs_rows(T.n, T.chi, Mv.n_chain))
    hipLaunchKernelGGL(k_propose_pair<kPacked>, grid, dim3(64 * kGWaves), vals + (size_t)T.n * kMetroTile * 4u, st, T,
                       Mv, step, nprop, pbase, npend, mode);
  else if (T.n <= kSlots32MaxN)
    hipLaunchKernelGGL(k_propose_pair<kSlots32>, grid, dim3(64 * kGWaves), vals + kSlots * kMetroTile * 9u, st, T, Mv,
                       step, nprop, pbase, npend, mode);
  else
    hipLaunchKernelGGL(k_propose_pair<kSlots64>, grid, dim3(64 * kGWaves), vals + kSlots * kMetroTile * 17u, st, T, Mv,
                       step, nprop, pbase, npend, mode);
  return hipGetLastError();
}

template <bool kInit>
hipError_t launch_masks(const TermsView& T, MetroView& Mv, const uint64_t* mask, uint32_t mode,
                        hipStream_t st) {
  const size_t sm = (size_t)T.n * kSub * 17;
  if (sm > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)k_propose<kInit>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_propose<kInit>, dim3(Mv.n_tiles), dim3(kPThreads), sm, st, T, Mv, mask, mode);
  return hipGetLastError();
}

// Steps `step` and, with nprop = 2, step + 1 of a chain: the sums of the tiles'
// partials (plane 0: the first proposal; planes 1 and 2: the second after the
// first was accepted, rejected) and the decisions.
__global__ __launch_bounds__(256) void k_metro_accept(MetroView Mv, uint32_t step, uint32_t nprop) {
  __shared__ double2 scratch[4];
  const uint32_t ch = blockIdx.x;
  const size_t plane = (size_t)Mv.n_chain * Mv.n_tiles;
  double2 acc[3];
  const double2* p = Mv.partial + (size_t)ch * Mv.n_tiles;
#pragma unroll
  for (int q = 0; q < 3; ++q) acc[q] = make_double2(0.0, 0.0);
  if (nprop == 2u) {
    for (uint32_t t = threadIdx.x; t < Mv.n_tiles; t += 256u) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const double2 v = p[q * plane + t];
        acc[q].x += v.x;
        acc[q].y += v.y;
      }
    }
  } else {
    for (uint32_t t = threadIdx.x; t < Mv.n_tiles; t += 256u) {
      const double2 v = p[t];
      acc[0].x += v.x;
      acc[0].y += v.y;
    }
  }
  double2 a[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    a[q] = make_double2(0.0, 0.0);
    if (q == 0 || nprop == 2u) a[q] = block_sum(acc[q], scratch);
  }
  if (threadIdx.x != 0) return;
  uint64_t x = Mv.x[ch];
  double2 ax = Mv.amp[ch];
  // The steps' bits in the chain's window of deferred cache updates.
  const uint32_t w = step % kMetroWin;
  uint32_t pend = w ? Mv.pend[ch] : 0u;
  uint32_t took = 0u;
  for (uint32_t k = 0; k < nprop; ++k) {
    const uint64_t idx = (uint64_t)ch * Mv.n_steps + step + k;
    const double2 ay = k == 0u ? a[0] : took ? a[1] : a[2];
    const double px = ax.x * ax.x + ax.y * ax.y;
    const double py = ay.x * ay.x + ay.y * ay.y;
    const double r = py / px;
    const double U = Mv.ustream[idx];
    took = (px > 0.0) && (r >= 1.0 || U < r);
    if (took) {
      x ^= 1ull << (Mv.jstream[idx] % Mv.n_qubits);
      ax = ay;
      pend |= 1u << (w + k);
    }
    if (Mv.trace) Mv.trace[idx] = x;
    if (Mv.accepted) Mv.accepted[idx] = (uint8_t)took;
  }
  Mv.x[ch] = x;
  Mv.amp[ch] = ax;
  Mv.pend[ch] = pend;
}

}  // namespace

hipError_t launch_metro_init(const TermsView& T, MetroView& Mv, hipStream_t st) {
  // From 8 chains on the tile's rows are staged once for all of them; below, each
  // chain reads its own bits' rows (n = 50, chi = 2^18, host time of the call:
  // 1 chain 43 µs and 63 staged, 8 chains 75 and 71, 64 chains 328 and 140).
  hipError_t e;
  if (Mv.n_chain >= 8u) {
    e = launch_masks<true>(T, Mv, nullptr, 0u, st);
  } else {
    hipLaunchKernelGGL(k_metro_init, dim3(Mv.n_tiles), dim3(kMetroTile), 0, st, T, Mv);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_chain_amp, dim3(Mv.n_chain), dim3(256), 0, st, Mv);
  return hipGetLastError();
}

hipError_t launch_metro_steps(const TermsView& T, MetroView& Mv, uint32_t n_steps, hipStream_t st) {
  static_assert(kMetroWin % 2 == 0, "a pair of steps lies in one window");
  if (n_steps == 0) return hipSuccess;
  for (uint32_t t = 0; t < n_steps; t += 2u) {
    // Steps t, t + 1 apply the accepted flips of their window's earlier steps;
    // the first pair of a window (t > 0) applies the whole previous window and
    // writes the caches back.
    const uint32_t nprop = std::min(2u, n_steps - t);
    const uint32_t w = t % kMetroWin;
    const bool close = w == 0 && t > 0;
    const uint32_t pbase = close ? t - kMetroWin : t - w, npend = close ? kMetroWin : w;
    hipError_t e = launch_pair(T, Mv, t, nprop, pbase, npend, close ? kModeWrite : 0u, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_metro_accept, dim3(Mv.n_chain), dim3(256), 0, st, Mv, t, nprop);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // The last window's accepted flips, so that every chain's current cache is
  // up to date when the call returns.
  const uint32_t t0 = (n_steps - 1u) / kMetroWin * kMetroWin;
  return launch_pair(T, Mv, 0, 0, t0, n_steps - t0, kModeWrite, st);
}

hipError_t launch_propose(const TermsView& T, MetroView& Mv, const uint64_t* mask, uint32_t mode,
                          hipStream_t st) {
  return launch_masks<false>(T, Mv, mask, mode, st);
}

}  // namespace chsim
