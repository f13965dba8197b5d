// Amplitudes <x|psi> on the matrix cores (step (b) of the hot path, n <= 60).
//
// With the quadratic form of amplitude.hip, a pair (term, x) contributes
// b 2^{-|v|/2} e^{i pi (omega mod 2)/4} i^m with
//   m = (omega >> 1) + popc(x & gamma_lo) + 2 x^T B x   (mod 4),
// or zero where one of the n - |v| conditions u_j = s_j (j outside v) fails.
// m is linear in the products x_p x_q (p < q), the bits x_p and a constant:
// a dot product of n (n - 1) / 2 + n + 1 small whole numbers, the term's
// weights (2 B_pq; gamma_lo,p + 2 B_pp; omega >> 1) in {0, 1, 2, 3} with the
// string's features in {0, 1}.  So all m of 32 terms and 32 strings are one
// chain of v_mfma_scale_f32_32x32x64_f8f6f4 on FP4 (E2M1 holds 0, 1, 2, 3
// exactly, the FP32 accumulator holds the sums, below 2^13, exactly): integer
// arithmetic, no rounding anywhere.  A condition is the parity of another
// such product with the n bits of x and a constant (one instruction).
//
// What bounds it: for n = 50, 20 instructions of 32 cycles per 32 x 32 pairs,
// 0.63 cycles of a SIMD per pair, against ceil(n / 4) + 1 LDS reads of 8 bytes
// per pair for the table kernel of amplitude.hip (0.98 of the LDS rate).  A
// VALU instruction costs 4 cycles per 64 pairs, so a pair's value is one LDS
// read: the four values b 2^{-|v|/2} ... i^m of every term sit in LDS, the sum
// comes scaled by the entry size, and its two low bits are the offset.
//
// Mapping.  A wave keeps the feature operands of 32 NB strings in registers
// (4 S registers per 32 strings, S = number of 64-feature steps) and walks
// tiles of 32 terms; the four waves of a workgroup hold different strings and
// share each tile's weights through LDS (double buffered, filled by loads
// that go straight to LDS), so a 1 KB weight operand feeds 2 NB x 4
// instructions.  With few strings and 128 tiles or more the waves take different
// tiles instead and read the weights from memory, each used once.  A lane holds one string
// (column) and 16 of a tile's 32 terms; the terms are assigned to rows so that
// a lane's registers are two groups of 8 consecutive terms in order: the FP32
// sum adds the 8 terms of a group plainly and joins the group sums with a
// two-sum, as the table kernel does.
//
// Measured (MI355X): n = 50, chi = 2^16, 4096 strings in FP32C 223 us (table
// kernel 543 us; of the 223, 79 us of matrix core time and 108 us of VALU
// issue, at 2 waves per SIMD); n = 40, chi = 110610, 4096 strings in FP64 with
// 30 conditions per term 0.97 ms (1.10 ms); n = 57, chi = 200003, 33 strings
// 46 us (269 us), bound by reading 190 MB of records; nine circuits of n = 20
// to 60, 1000 strings each, in FP64 0.28 ms under the profiler (0.51 ms).
#include <algorithm>

#include "device_common.hpp"
#include "internal.hpp"

namespace chsim {

namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr uint32_t kMT = kAmpMfmaTile;  // terms per tile
constexpr uint32_t kWaves = 4;
static_assert(kMT == 32, "one MFMA row block");

// Tile record, (S + 4) KB: S weight operands of 1 KB (lane l: row l % 32,
// features 32 (l / 32) .. + 31 of the step, 16 bytes); a head of 1 KB with the
// condition words of the first three levels ([level][half][row], 32 bits) and,
// at 768, the number of levels; 1 KB of values as floats and 2 KB as doubles
// ([register][m][half]).  Levels from the fourth on: [n][32 rows] 64-bit words
// per tile in an array of their own.
constexpr uint32_t kRecExtra = 4u, kHeadLevels = 768u;

// Term of a tile that sits in row r of the MFMA: lane half h = (r >> 2) & 1
// holds row r in register i = 4 (r >> 3) + (r & 3), and registers 8 g .. 8 g + 7
// of half h are terms 16 g + 8 h .. + 7.
__device__ __forceinline__ uint32_t row_of_term(uint32_t t) {
  const uint32_t h = (t >> 3) & 1u, i = ((t >> 4) << 3) | (t & 7u);
  return ((i >> 2) << 3) | (h << 2) | (i & 3u);
}

// Operand registers of 32 features given as bits: register k holds the bits
// k, k + 4, k + 8, ... (strings and weights use the same order), bit 0 of a
// nibble moved up to `kShift`.
template <int kShift>
__device__ __forceinline__ i32x4 spread32(uint32_t w) {
  i32x4 r;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    r[k] = (int)((k >= kShift ? w >> (k - kShift) : w << (kShift - k)) & (0x11111111u << kShift));
  return r;
}

// D = A B + C on FP4 operands (format 4), the products scaled by 2^kExp
// (block scale 2^(byte - 127) on A).
template <int kExp>
__device__ __forceinline__ f32x16 mfma_fp4(i32x4 a, i32x4 b, f32x16 c) {
  const i32x8 a8 = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
  const i32x8 b8 = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 4, 4, 0, (int)((127u + kExp) * 0x01010101u), 0, 0x7F7F7F7F);
}

// Operand with FP4 code c1, c2, c3 at the features n + 1, n + 2, n + 3 of a
// condition step (lane half holds features 32 half ..).
__device__ __forceinline__ i32x4 spare_codes(uint32_t n, uint32_t half, uint32_t c1, uint32_t c2, uint32_t c3) {
  i32x4 r = {0, 0, 0, 0};
  const uint32_t c[3] = {c1, c2, c3};
#pragma unroll
  for (uint32_t k = 0; k < 3u; ++k) {
    const uint32_t f = n + 1u + k, e = f & 31u;
#pragma unroll
    for (uint32_t g = 0; g < 4u; ++g)
      if ((f >> 5) == half && (e & 3u) == g) r[g] |= (int)(c[k] << (4u * (e >> 2)));
  }
  return r;
}

// ---------------------------------------------------------------------------
// Prologue: tile records and condition words of 32 terms per workgroup, 16
// threads per term.  Bound by the parities of B (about n^2 / 2 per term).
// ---------------------------------------------------------------------------
constexpr uint32_t kPParts = 16;

__global__ __launch_bounds__(512) void k_amp_mfma_prep(TermsView T, uint32_t S, uint8_t* __restrict__ rec,
                                                       uint64_t* __restrict__ cond) {
  extern __shared__ __align__(16) uint8_t smem[];
  const uint32_t n = T.n;
  uint64_t* const Fs = reinterpret_cast<uint64_t*>(smem);  // [n][32] rows of F
  uint64_t* const Cs = Fs + (size_t)n * kMT;               // [n][32] rows c_q of B, bits p <= q
  uint64_t* const Gp = Cs + (size_t)n * kMT;               // [16][32] parts of gamma_lo
  uint64_t* const Dp = Gp + kPParts * kMT;                 // [16][32] parts of diag(B)
  uint32_t* const most = reinterpret_cast<uint32_t*>(Dp + kPParts * kMT);
  const uint32_t t = threadIdx.x % kMT, part = threadIdx.x / kMT;
  const uint64_t chi = T.chi, a = (uint64_t)blockIdx.x * kMT + t;
  const bool on = a < chi;
  if (threadIdx.x == 0) *most = 0u;
  uint64_t glo = 0;
  // A thread's rows part, part + 16, ... (at most four), all loads at once.
  uint64_t rF[4], rM[4];
  uint32_t rg[4];
#pragma unroll
  for (uint32_t k = 0; k < 4u; ++k) {
    const uint32_t p = part + k * kPParts;
    const bool in = on && p < n;
    rF[k] = in ? T.F[(uint64_t)p * chi + a] : 0ull;
    rM[k] = in ? T.M[(uint64_t)p * chi + a] : 0ull;
    rg[k] = in ? T.gamma[(uint64_t)p * chi + a] : 0u;
  }
#pragma unroll
  for (uint32_t k = 0; k < 4u; ++k) {
    const uint32_t p = part + k * kPParts;
    if (p < n) Fs[p * kMT + t] = rF[k];
    glo |= (uint64_t)(rg[k] & 1u) << (p & 63u);
  }
  Gp[part * kMT + t] = glo;
  __syncthreads();
  const uint64_t xm = (1ull << n) - 1ull;  // n <= 60
  const uint64_t v = on ? T.v[a] : xm, s = on ? T.s[a] : 0ull;
  const uint64_t nv = ~v & xm;
  uint64_t diag = 0;
#pragma unroll
  for (uint32_t k = 0; k < 4u; ++k) {
    const uint32_t q = part + k * kPParts;
    if (q >= n) break;
    uint64_t col = 0;
    for (uint32_t p = 0; p <= q; ++p) col |= (uint64_t)par64(Fs[p * kMT + t] & rM[k]) << p;
    Cs[q * kMT + t] = col;
    diag |= (uint64_t)((((uint32_t)(col >> q)) ^ (rg[k] >> 1) ^ par64(rF[k] & v & s)) & 1u) << q;
  }
  Dp[part * kMT + t] = diag;
  const uint32_t nc = (uint32_t)__popcll(nv);
  if (part == 0) atomicMax(most, nc);
  __syncthreads();
  glo = 0;
  diag = 0;
  for (uint32_t k = 0; k < kPParts; ++k) {
    glo |= Gp[k * kMT + t];
    diag |= Dp[k * kMT + t];
  }
  const uint32_t om = on ? T.omega[a] : 0u;
  uint8_t* const tile = rec + (size_t)blockIdx.x * (S + kRecExtra) * 1024u;
  const uint32_t row = row_of_term(t);
  const uint32_t nq = n * (n - 1u) / 2u;
  // Weights: feature f < nq is the pair (p, q) with f = q (q - 1) / 2 + p, then
  // the n bits, then the constant.  FP4 codes of 0, 1, 2, 3: 0, 2, 4, 5.
  for (uint32_t wi = part; wi < 2u * S; wi += kPParts) {
    uint32_t hi = 0, mid = 0, low = 0, pos = 0, f = 32u * wi;
    uint32_t q = (uint32_t)((1.0f + sqrtf(1.0f + 8.0f * (float)f)) * 0.5f);
    while (q * (q - 1u) / 2u > f) --q;
    while ((q + 1u) * q / 2u <= f) ++q;
    while (pos < 32u && f < nq) {
      const uint32_t p = f - q * (q - 1u) / 2u, take = min(32u - pos, q - p);
      const uint32_t bits = (uint32_t)((Cs[q * kMT + t] >> p) & ((1ull << take) - 1ull));
      hi |= bits << pos;
      pos += take;
      f += take;
      ++q;
    }
    if (pos < 32u && f < nq + n) {
      const uint32_t p = f - nq, take = min(32u - pos, n - p);
      const uint64_t m = (1ull << take) - 1ull;
      const uint32_t d = (uint32_t)((diag >> p) & m), g = (uint32_t)((glo >> p) & m);
      hi |= d << pos;
      mid |= (g & ~d) << pos;
      low |= (g & d) << pos;
      pos += take;
      f += take;
    }
    if (pos < 32u && f == nq + n) {
      const uint32_t w = (om >> 1) & 3u;
      hi |= (w >> 1) << pos;
      mid |= (uint32_t)(w == 1u) << pos;
      low |= (uint32_t)(w == 3u) << pos;
    }
    i32x4 r = spread32<2>(hi);
    if (mid | low) r |= spread32<1>(mid) | spread32<0>(low);
    *reinterpret_cast<i32x4*>(tile + ((size_t)(wi >> 1) * 64u + (wi & 1u) * 32u + row) * 16u) = r;
  }
  if (part == 0) {
    // b 2^{-|v|/2}, times e^{i pi/4} for odd omega; zero past chi.
    double2 w = make_double2(0.0, 0.0);
    if (on) {
      const double2 b = T.b[a];
      const int vc = __popcll(v);
      const double h = 0.70710678118654752440;
      const double mag = ldexp(1.0, -(vc >> 1)) * ((vc & 1) ? h : 1.0);
      const double w0r = b.x * mag, w0i = b.y * mag;
      w = (om & 1u) ? make_double2((w0r - w0i) * h, (w0r + w0i) * h) : make_double2(w0r, w0i);
    }
    const uint32_t h = (t >> 3) & 1u, i = ((t >> 4) << 3) + (t & 7u);  // half, register
    float2* const v32 = reinterpret_cast<float2*>(tile + (size_t)(S + 1u) * 1024u) + i * 8u + h;
    double2* const v64 = reinterpret_cast<double2*>(tile + (size_t)(S + 2u) * 1024u) + i * 8u + h;
    for (uint32_t m = 0; m < 4u; ++m) {  // times i^m: exact
      v32[m * 2u] = make_float2((float)w.x, (float)w.y);
      v64[m * 2u] = w;
      w = make_double2(-w.y, w.x);
    }
  }
  // Condition words of level c: bit p = bit j of F_p (j the c-th position
  // outside v), bit n = s_j; zero for a term with fewer conditions.
  uint64_t* const cw = cond + (size_t)blockIdx.x * n * kMT;
  uint8_t* const head = tile + (size_t)S * 1024u;
  const uint32_t levels = *most;
  if (threadIdx.x == 0) *reinterpret_cast<uint32_t*>(head + kHeadLevels) = levels;
  // A thread takes the levels part, part + 16, part + 32, part + 48 in one pass
  // over F.
  uint32_t j[4];
  uint64_t w[4], m = nv;
#pragma unroll
  for (uint32_t k = 0; k < 4u; ++k) {
    const uint32_t c = part + k * kPParts;
    for (uint32_t i = k ? kPParts : part; i && m; --i) m &= m - 1ull;
    j[k] = c < nc ? (uint32_t)__builtin_ctzll(m) : 64u;
    w[k] = j[k] < 64u ? ((s >> j[k]) & 1ull) << n : 0ull;
  }
  if (part < levels)
    for (uint32_t p = 0; p < n; ++p) {
      const uint64_t f = Fs[p * kMT + t];
#pragma unroll
      for (uint32_t k = 0; k < 4u; ++k) {
        if (part + k * kPParts >= levels) break;
        w[k] |= (j[k] < 64u ? (f >> j[k]) & 1ull : 0ull) << p;
      }
    }
#pragma unroll
  for (uint32_t k = 0; k < 4u; ++k) {
    const uint32_t c = part + k * kPParts;
    if (c < 3u) {
      reinterpret_cast<uint32_t*>(head)[c * 64u + row] = (uint32_t)w[k];
      reinterpret_cast<uint32_t*>(head)[c * 64u + 32u + row] = (uint32_t)(w[k] >> 32);
    } else if (c < levels) {
      cw[(size_t)(c - 3u) * kMT + row] = w[k];
    }
  }
}

// ---------------------------------------------------------------------------
// Sums of a lane's string: FP32 plainly over a group of 8 terms and with a
// two-sum across groups, or FP64 (the group sums added to a running sum: the
// rounding error grows with the groups, not with the terms).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
  s = a + b;
  const float bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

template <typename T>
struct Sum;
template <>
struct Sum<float> {
  float sr = 0.f, er = 0.f, si = 0.f, ei = 0.f, br = 0.f, bi = 0.f;
  __device__ __forceinline__ void flush() {
    float s, e;
    two_sum(sr, br, s, e);
    sr = s;
    er += e;
    two_sum(si, bi, s, e);
    si = s;
    ei += e;
    br = bi = 0.f;
  }
  __device__ __forceinline__ double2 value() const {
    return make_double2((double)sr + (double)er, (double)si + (double)ei);
  }
};
template <>
struct Sum<double> {
  double sr = 0.0, si = 0.0, br = 0.0, bi = 0.0;
  __device__ __forceinline__ void flush() {
    sr += br;
    si += bi;
    br = bi = 0.0;
  }
  __device__ __forceinline__ double2 value() const { return make_double2(sr, si); }
};

using glb_ptr = const __attribute__((address_space(1))) void*;
using lds_ptr = __attribute__((address_space(3))) void*;

template <typename T>
struct Val;
template <>
struct Val<float> {
  using type = float2;
};
template <>
struct Val<double> {
  using type = double2;
};

// One work item: the strings [x0, x1) of the item against the tiles of its
// range.  kShared: the workgroup's waves hold 32 NB strings each and share the
// tiles through LDS; else every wave holds the item's (at most 32 NB) strings
// and takes every fourth tile.
template <typename T, int SMAX, int NB, bool kShared>
__device__ __forceinline__ void run_item(const AmpMfmaInst& I, const AmpItem& item, uint8_t* lds) {
  constexpr uint32_t kStr = 32u * NB;  // strings per wave
  const uint32_t lane = threadIdx.x & 63u, wave = uniform32(threadIdx.x >> 6);
  const uint32_t col = lane & 31u, half = lane >> 5;
  const uint32_t n = I.n, S = I.steps;
  const uint64_t xmask = (1ull << n) - 1ull;
  const uint32_t xbase = item.x0 + (kShared ? wave * kStr : 0u);
  // Feature words of the wave's strings (32 features each) by way of LDS: lane
  // l writes string l's words in feature order.
  uint32_t* const words = reinterpret_cast<uint32_t*>(lds) + (size_t)wave * 2u * S * kStr;
  {
    const uint32_t st = lane % kStr;
    const uint32_t xi = xbase + st;
    const uint64_t x = xi < item.x1 ? I.x[xi] & xmask : 0ull;
    uint64_t buf = 0;
    uint32_t fill = 0, at = 0;
    auto push = [&](uint32_t bits, uint32_t len) {  // len <= 32, wave-uniform
      buf |= (uint64_t)bits << fill;
      fill += len;
      if (fill >= 32u) {
        words[at * kStr + st] = (uint32_t)buf;
        buf >>= 32;
        fill -= 32u;
        ++at;
      }
    };
    for (uint32_t q = 1; q < n; ++q) {
      const uint64_t on = 0ull - ((x >> q) & 1ull);
      const uint64_t rowb = x & ((1ull << q) - 1ull) & on;
      push((uint32_t)rowb, q < 32u ? q : 32u);
      if (q > 32u) push((uint32_t)(rowb >> 32), q - 32u);
    }
    push((uint32_t)x, n < 32u ? n : 32u);
    if (n > 32u) push((uint32_t)(x >> 32), n - 32u);
    push(1u, 1u);
    while (at < 2u * S) push(0u, 32u);
  }
  __syncthreads();
  i32x4 Bq[NB][SMAX];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
    for (int s = 0; s < SMAX; ++s)
      Bq[nb][s] = (uint32_t)s < S ? spread32<1>(words[(2u * s + half) * kStr + nb * 32u + col]) : (i32x4)(0);
  }
  __syncthreads();

  constexpr uint32_t kValKB = sizeof(T) / 4u;               // KB of values of this type
  constexpr uint32_t kEntry = sizeof(T) * 2u;               // one value
  constexpr int kScale = sizeof(T) == 8 ? 5 : 4;            // m times two entries
  constexpr uint32_t kMMask = 3u << kScale;
  using V = typename Val<T>::type;
  const uint32_t recb = (S + kRecExtra) * 1024u;
  const uint32_t own = kShared ? S : 0u;                    // KB of weights staged
  const uint32_t bufb = (own + 1u + kValKB) * 1024u;        // a staged tile
  const uint32_t mine = kShared ? 0u : wave * 2u * bufb;    // this wave's buffers
  const uint32_t zero = (kShared ? 2u : 2u * kWaves) * bufb;  // 16 entries of zeros, laid out like values
  // Condition operands of the wave's strings (the bits of x and the constant at
  // feature n), and the weights of the spare features n + 1 .. n + 3: they
  // carry 6 x 6 + 6 x 4 + 2 x 2 = 64 in the third level of a group, so that the
  // group's sum lies in [2^18, 2^19) and its integer bits sit at fixed places
  // of the accumulator, the parities of the three levels at bits 5, 11 and 17.
  // They are read from LDS where they are used, to keep 12 registers free.
  uint8_t* const fixed = lds + zero + kValKB * 1024u + wave * (NB + 1u) * 1024u + lane * 16u;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const uint32_t xi = xbase + (uint32_t)nb * 32u + col;
    const uint64_t x = (xi < item.x1 ? I.x[xi] & xmask : 0ull) | (1ull << n);
    *reinterpret_cast<i32x4*>(fixed + nb * 1024) =
        spread32<1>(half ? (uint32_t)(x >> 32) : (uint32_t)x) | spare_codes(n, half, 7u, 7u, 4u);
  }
  *reinterpret_cast<i32x4*>(fixed + NB * 1024) = spare_codes(n, half, 7u, 6u, 4u);
  auto strings = [&](int nb) { return *reinterpret_cast<const i32x4*>(fixed + nb * 1024); };
  constexpr uint32_t kParities = (1u << 5) | (1u << 11) | (1u << 17);
  for (uint32_t k = threadIdx.x; k < kValKB * 256u; k += 256u) reinterpret_cast<uint32_t*>(lds + zero)[k] = 0u;
  __syncthreads();
  const uint32_t t0 = item.range * I.tiles_per_range + (kShared ? 0u : wave);
  const uint32_t t1 = min(I.tiles, (item.range + 1u) * I.tiles_per_range);
  constexpr uint32_t kStep = kShared ? 1u : kWaves;
  Sum<T> A[NB];

  // A tile's weights, head and values straight into LDS, 1 KB per instruction,
  // dealt to the waves; a wave with its own tile stages only head and values.
  auto fetch = [&](uint32_t t, uint32_t b) {
    const uint8_t* src = I.rec + (size_t)t * recb;
    const uint32_t skip = sizeof(T) == 8 ? 1u : 0u;  // doubles: past the KB of floats
    uint8_t* dst = lds + mine + (size_t)b * bufb;
    for (uint32_t k = kShared ? wave : S; k < S + 1u + kValKB; k += kShared ? kWaves : 1u)
      __builtin_amdgcn_global_load_lds((glb_ptr)(src + (k <= S ? k : k + skip) * 1024u + lane * 16u),
                                       (lds_ptr)(dst + (size_t)(kShared ? k : k - S) * 1024u), 16, 0, 0);
  };
  if (t0 < t1) fetch(t0, 0u);
  uint32_t buf = 0;
  for (uint32_t t = t0; t < t1; t += kStep) {
    const uint8_t* tile = I.rec + (size_t)t * recb;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (kShared) __syncthreads();  // the tile is in; the other buffer's readers are done
    if (t + kStep < t1) fetch(t + kStep, buf ^ 1u);
    const uint32_t at = mine + buf * bufb;
    if (kShared) tile = lds + at;
    const uint8_t* head = lds + at + own * 1024u;
    // LDS offset of this lane's values: register i at + 8 i entries, m at + 2 m entries.
    uint32_t vbase = at + (own + 1u) * 1024u + half * kEntry;
    asm("" : "+v"(vbase));  // one register: the offset is then a single and-or
    buf ^= 1u;
    const uint32_t nc = uniform32(*reinterpret_cast<const uint32_t*>(head + kHeadLevels));
    f32x16 acc[NB];
    auto weights = [&]() {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb] = (f32x16)(0.0f);
      const i32x4* ap = reinterpret_cast<const i32x4*>(tile) + lane;
      // Operands three steps ahead (past step S - 1: the head, not used).
      i32x4 a[4];
#pragma unroll
      for (uint32_t s = 0; s < 3u; ++s) a[s] = ap[min(s, S) * 64u];
#pragma unroll
      for (int s = 0; s < SMAX; s += 2) {
        if ((uint32_t)s < S) {
          a[(s + 3) & 3] = ap[min((uint32_t)s + 3u, S) * 64u];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc[nb] = mfma_fp4<kScale>(a[s & 3], Bq[nb][s], acc[nb]);
          a[s & 3] = ap[min((uint32_t)s + 4u, S) * 64u];
          if ((uint32_t)s + 1u < S) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb] = mfma_fp4<kScale>(a[(s + 1) & 3], Bq[nb][s + 1], acc[nb]);
          }
        }
      }
    };
    // Value of register i at LDS offset off.
    auto add = [&](Sum<T>& R, int i, uint32_t off) {
      const V v = *reinterpret_cast<const V*>(lds + (off + (uint32_t)i * 8u * kEntry));
      R.br += v.x;
      R.bi += v.y;
      if ((i & 7) == 7) R.flush();
    };
    // The sum, below 2^23, is in the low bits after 2^23 is added.
    auto offset = [&](float sum) { return (__float_as_uint(sum + 8388608.0f) & kMMask) | vbase; };
    auto first = [&](uint32_t k) {
      return k < nc ? reinterpret_cast<const uint32_t*>(head)[k * 64u + half * 32u + col] : 0u;
    };
    auto group = [&](uint32_t w0, uint32_t w1, uint32_t w2, int nb) {
      const i32x4 bias = *reinterpret_cast<const i32x4*>(fixed + NB * 1024);
      const i32x4 x = strings(nb);
      f32x16 r = mfma_fp4<0>(spread32<1>(w0), x, (f32x16)(0.0f));
      r = mfma_fp4<6>(spread32<1>(w1), x, r);
      return mfma_fp4<12>(spread32<1>(w2) | bias, x, r);
    };
    if (nc == 0u) {
      weights();
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) add(A[nb], i, offset(acc[nb][i]));
      continue;
    }
    if (nc <= 3u) {
      const uint32_t w0 = first(0u), w1 = first(1u), w2 = first(2u);
      weights();
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const f32x16 r = group(w0, w1, w2, nb);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const uint32_t off = offset(acc[nb][i]);
          add(A[nb], i, (__float_as_uint(r[i]) & kParities) ? zero : off);
        }
      }
      continue;
    }
    // More levels: all conditions first (most pairs of such a tile fail one),
    // bit i of dead[nb] for register i.
    const uint64_t* cw = I.cond + (size_t)t * n * kMT + col;
    uint32_t dead[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) dead[nb] = 0u;
    // Blocks of strings together where the registers allow, else in turn.
    constexpr int kTogether = SMAX <= 14 ? NB : 1;
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += kTogether) {
      uint32_t bad[kTogether][16];
#pragma unroll
      for (int k = 0; k < kTogether; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) bad[k][i] = 0u;
      uint32_t w[3];
#pragma unroll
      for (uint32_t k = 0; k < 3u; ++k) w[k] = first(k);
      for (uint32_t c = 0; c < nc; c += 3u) {
        uint32_t u[3];
#pragma unroll
        for (uint32_t k = 0; k < 3u; ++k) {
          u[k] = w[k];
          const uint32_t l = c + k;  // level l + 3
          w[k] = l + 3u < nc ? reinterpret_cast<const uint32_t*>(cw + (size_t)l * kMT)[half] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kTogether; ++k) {
          const f32x16 r = group(u[0], u[1], u[2], b0 + k);
#pragma unroll
          for (int i = 0; i < 16; ++i) bad[k][i] |= __float_as_uint(r[i]);
        }
        // Every fourth group: is any pair left?
        if (c % 12u == 9u && c + 3u < nc) {
          bool some = false;
#pragma unroll
          for (int k = 0; k < kTogether; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) some = some || (bad[k][i] & kParities) == 0u;
          if (__ballot(some) == 0ull) break;
        }
      }
#pragma unroll
      for (int k = 0; k < kTogether; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) dead[b0 + k] |= (bad[k][i] & kParities) ? 1u << i : 0u;
    }
    bool some = false;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) some = some || dead[nb] != 0xFFFFu;
    if (__ballot(some) == 0ull) continue;
    weights();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t off = offset(acc[nb][i]);
        add(A[nb], i, (dead[nb] & (1u << i)) ? zero : off);
      }
  }
  // The waves of a split item add their sums in wave order.
  double2* const sums = reinterpret_cast<double2*>(lds);
  if (!kShared) __syncthreads();
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    double2 r = A[nb].value();
    r.x += __shfl_xor(r.x, 32);
    r.y += __shfl_xor(r.y, 32);
    const uint32_t xi = xbase + (uint32_t)nb * 32u + col;
    if (!kShared) {
      if (half == 0u) sums[wave * kStr + (uint32_t)nb * 32u + col] = r;
    } else if (half == 0u && xi < item.x1) {
      I.partial[(size_t)item.range * I.n_x + xi] = r;
    }
  }
  if (!kShared) {
    __syncthreads();
    const uint32_t xi = item.x0 + threadIdx.x;
    if (threadIdx.x < kStr && xi < item.x1) {
      double2 r = sums[threadIdx.x];
      for (uint32_t w = 1; w < kWaves; ++w) {
        r.x += sums[w * kStr + threadIdx.x].x;
        r.y += sums[w * kStr + threadIdx.x].y;
      }
      I.partial[(size_t)item.range * I.n_x + xi] = r;
    }
  }
}

// Register classes by the number of steps S: the strings a wave can hold.
// 8 S + 60 registers (two blocks of strings) fit 256 up to S = 20 (n <= 50).
template <typename T, bool kShared>
__global__ __launch_bounds__(256, 2) void k_amp_mfma(const AmpMfmaInst* __restrict__ insts,
                                                     const AmpItem* __restrict__ items) {
  extern __shared__ __align__(16) uint8_t lds[];
  const AmpItem item = items[blockIdx.x];
  if (item.x1 <= item.x0) return;  // padding of the block order
  const AmpMfmaInst& I = insts[item.inst];
  if (I.steps <= 4u) run_item<T, 4, 2, kShared>(I, item, lds);
  else if (I.steps <= 8u) run_item<T, 8, 2, kShared>(I, item, lds);
  else if (I.steps <= 14u) run_item<T, 14, 2, kShared>(I, item, lds);
  else if (I.steps <= 20u) run_item<T, 20, 2, kShared>(I, item, lds);
  else run_item<T, 32, 1, kShared>(I, item, lds);
}

// out[i] = the sum of the partial rows of string i in row order (FP64): a
// 256-thread block takes 8 strings (over all requests) at a time and 32 slices of
// their rows; the slice sums are added in slice order.
constexpr uint32_t kRedX = 8, kRedSlices = 32;
// Blocks of a launch.  A grid of 2^32 threads (2^27 strings) or more is cut short
// without an error, so past 2^26 strings the blocks go round.
constexpr uint32_t kRedBlocks = 1u << 23;
__global__ __launch_bounds__(256) void k_amp_mfma_reduce(const AmpMfmaInst* __restrict__ insts,
                                                         const uint64_t* __restrict__ prefix, uint32_t n_inst) {
  __shared__ double2 part[kRedSlices][kRedX];
  const uint32_t xl = threadIdx.x % kRedX, sl = threadIdx.x / kRedX;
  const uint64_t total = prefix[n_inst];
  for (uint64_t g0 = (uint64_t)blockIdx.x * kRedX;;) {
    const uint64_t g = g0 + xl;
    const bool on = g < total;
    uint32_t lo = 0;
    uint64_t i = 0;
    double re = 0.0, im = 0.0;
    if (on) {
      uint32_t hi = n_inst;
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid;
      }
      const AmpMfmaInst& I = insts[lo];
      i = g - prefix[lo];
      const uint32_t r0 = (uint32_t)((uint64_t)I.rows * sl / kRedSlices);
      const uint32_t r1 = (uint32_t)((uint64_t)I.rows * (sl + 1) / kRedSlices);
      for (uint32_t t = r0; t < r1; ++t) {
        const double2 v = I.partial[(uint64_t)t * I.n_x + i];
        re += v.x;
        im += v.y;
      }
    }
    part[sl][xl] = make_double2(re, im);
    __syncthreads();
    if (sl == 0 && on) {
      double sr = 0.0, si = 0.0;
      for (uint32_t k = 0; k < kRedSlices; ++k) {
        sr += part[k][xl].x;
        si += part[k][xl].y;
      }
      insts[lo].out[i] = make_double2(sr, si);
    }
    g0 += (uint64_t)gridDim.x * kRedX;
    if (g0 >= total) break;  // uniform; a block's first strings are always there
    __syncthreads();  // the slices are read before the next strings' are written
  }
}

}  // namespace

uint32_t amp_mfma_steps(uint32_t n) { return (n * (n + 1u) / 2u + 1u + 63u) / 64u; }
uint32_t amp_mfma_strings(uint32_t n) { return amp_mfma_steps(n) <= 20u ? 64u : 32u; }

uint32_t amp_mfma_tile_bytes(uint32_t n) { return (amp_mfma_steps(n) + kRecExtra) * 1024u; }

hipError_t launch_amp_mfma_prep(const TermsView& T, uint8_t* rec, uint64_t* cond, hipStream_t st) {
  const uint32_t tiles = (uint32_t)((T.chi + kMT - 1) / kMT);
  const size_t sm = ((size_t)2 * T.n + 2 * kPParts) * kMT * sizeof(uint64_t) + 16;
  hipLaunchKernelGGL(k_amp_mfma_prep, dim3(tiles), dim3(kMT * kPParts), sm, st, T, amp_mfma_steps(T.n), rec, cond);
  return hipGetLastError();
}

hipError_t launch_amp_mfma_sums(const AmpMfmaInst* insts_d, const AmpItem* items_d, uint32_t n_items,
                                uint32_t n_split, uint32_t max_steps, bool fp32c, hipStream_t st) {
  // Two staged tiles (split items: head and values alone, two buffers per
  // wave), a table of zeros and the fixed condition operands; at the start the
  // same memory holds the four waves' feature words (8 S x strings x 4 bytes <=
  // 2 S KB).
  const uint32_t n_shared = n_items - n_split;
  const uint32_t kv = fp32c ? 1u : 2u;
  const size_t sm = std::max<size_t>(2u * (max_steps + 1u + kv), 2u * kWaves * (1u + kv)) * 1024u + kv * 1024u + kWaves * 3u * 1024u;
  hipError_t e = hipSuccess;
  if (sm > 65536)
    for (const void* f : {(const void*)k_amp_mfma<float, true>, (const void*)k_amp_mfma<float, false>,
                          (const void*)k_amp_mfma<double, true>, (const void*)k_amp_mfma<double, false>})
      if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm)) != hipSuccess) return e;
  if (n_shared) {
    if (fp32c) hipLaunchKernelGGL((k_amp_mfma<float, true>), dim3(n_shared), dim3(256), sm, st, insts_d, items_d);
    else hipLaunchKernelGGL((k_amp_mfma<double, true>), dim3(n_shared), dim3(256), sm, st, insts_d, items_d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (n_split) {
    const AmpItem* it = items_d + n_shared;
    if (fp32c) hipLaunchKernelGGL((k_amp_mfma<float, false>), dim3(n_split), dim3(256), sm, st, insts_d, it);
    else hipLaunchKernelGGL((k_amp_mfma<double, false>), dim3(n_split), dim3(256), sm, st, insts_d, it);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_amp_mfma(const AmpMfmaInst* insts_d, const AmpItem* items_d, uint32_t n_items, uint32_t n_split,
                           uint32_t max_steps, bool fp32c, const uint64_t* prefix_d, uint32_t n_inst,
                           uint64_t total_x, hipStream_t st) {
  const hipError_t e = launch_amp_mfma_sums(insts_d, items_d, n_items, n_split, max_steps, fp32c, st);
  if (e != hipSuccess) return e;
  const uint32_t blocks = (uint32_t)std::min<uint64_t>((total_x + kRedX - 1) / kRedX, kRedBlocks);
  hipLaunchKernelGGL(k_amp_mfma_reduce, dim3(blocks), dim3(256), 0, st, insts_d, prefix_d, n_inst);
  return hipGetLastError();
}

void amp_mfma_plan(const std::vector<AmpRequestPlan>& reqs, std::vector<AmpItem>& items, uint32_t* n_split,
                   std::vector<uint32_t>& tiles_per_range, std::vector<uint32_t>& rows) {
  // A tile against one workgroup's strings costs its MFMA steps plus about
  // half as much as 14 steps for the sums; an item also builds its feature
  // operands, worth about 6 tiles.
  constexpr uint64_t kSplitTiles = 128;
  const size_t R = reqs.size();
  std::vector<uint64_t> tiles(R), chunks(R);
  std::vector<uint32_t> per_wg(R);
  std::vector<bool> split(R);
  std::vector<double> tcost(R);
  double total = 0.0;
  for (size_t q = 0; q < R; ++q) {
    const uint32_t str = amp_mfma_strings(reqs[q].n);
    tiles[q] = (reqs[q].chi + kMT - 1) / kMT;
    // Up to two waves' worth of strings: the waves split the tiles, since a
    // workgroup that shares them would leave half of its waves idle (calls at
    // n = 50, chi = 2^18: 64 strings 45 µs split and 65 shared, 128 strings 57 and
    // 65; n = 20, chi = 10^5: 17 and 28, 19 and 28; n = 57: equal, bound by the records).
    // With few tiles a call is latency alone, and staged weights arrive sooner than
    // those a wave reads for itself (33 strings, calls in µs, split and shared: chi = 300
    // n = 24 41.7 and 40.6, n = 60 46.9 and 43.5; chi = 3000 42.9 and 41.5, 46.7 and 44.3; chi =
    // 10000 43.2 and 44.5, 47.7 and 48.4).
    split[q] = reqs[q].n_x <= 2u * str && tiles[q] >= kSplitTiles;
    per_wg[q] = split[q] ? str : str * kWaves;
    chunks[q] = (reqs[q].n_x + per_wg[q] - 1) / per_wg[q];
    tcost[q] = (amp_mfma_steps(reqs[q].n) + 8.0) * (str == 64u ? 2.0 : 1.0);
    if (split[q]) tcost[q] /= kWaves;
    total += (double)tiles[q] * (double)chunks[q] * tcost[q];
  }
  // 512 workgroups are resident (two per compute unit, 256 registers per
  // lane): one request takes one round of them, several requests items of
  // about half a round's share, dealt longest first.
  const double slots = 512.0;
  tiles_per_range.assign(R, 1);
  rows.assign(R, 1);
  struct Run {  // the items of one (request, range): its chunks
    uint32_t q, rg;
    double cost;
  };
  std::vector<Run> runs[2];
  for (size_t q = 0; q < R; ++q) {
    uint64_t ranges;
    if (R == 1) ranges = std::max<uint64_t>(1, (uint64_t)slots / chunks[q]);
    else ranges = (uint64_t)std::max(1.0, (double)tiles[q] * tcost[q] / std::max(total / (2.0 * slots), 1e-9));
    const uint64_t least = split[q] ? kWaves : 1;  // tiles per range
    ranges = std::min<uint64_t>(ranges, std::max<uint64_t>(1, tiles[q] / least));
    const uint64_t per = (tiles[q] + ranges - 1) / ranges;
    ranges = (tiles[q] + per - 1) / per;
    tiles_per_range[q] = (uint32_t)per;
    rows[q] = (uint32_t)ranges;
    for (uint64_t rg = 0; rg < ranges; ++rg) {
      const uint64_t nt = std::min<uint64_t>(tiles[q], (rg + 1) * per) - rg * per;
      runs[split[q]].push_back(Run{(uint32_t)q, (uint32_t)rg, (double)nt * tcost[q]});
    }
  }
  items.clear();
  *n_split = 0;
  for (int sp = 0; sp < 2; ++sp) {
    std::stable_sort(runs[sp].begin(), runs[sp].end(), [](const Run& a, const Run& b) { return a.cost > b.cost; });
    // Workgroups are dealt to the 8 XCDs in turn: a range's chunks go to one
    // XCD, whose L2 then holds the range's tiles; short queues are padded.
    std::vector<AmpItem> queue[8];
    for (size_t k = 0; k < runs[sp].size(); ++k) {
      auto* best = &queue[0];
      for (auto& c : queue)
        if (c.size() < best->size()) best = &c;
      const Run& r = runs[sp][k];
      for (uint32_t x0 = 0; x0 < reqs[r.q].n_x; x0 += per_wg[r.q])
        best->push_back(AmpItem{r.q, r.rg, x0, std::min<uint32_t>(reqs[r.q].n_x, x0 + per_wg[r.q])});
    }
    size_t longest = 0;
    for (auto& c : queue) longest = std::max(longest, c.size());
    const size_t before = items.size();
    for (size_t k = 0; k < longest; ++k)
      for (auto& c : queue) items.push_back(k < c.size() ? c[k] : AmpItem{0u, 0u, 0u, 0u});
    while (items.size() > before && items.back().x1 == 0u) items.pop_back();
    if (sp) *n_split = (uint32_t)(items.size() - before);
  }
}

}  // namespace chsim
