// Term generation and CH-form evolution (step (a) of the hot path).
//
// Branch choice: exact enumeration (Eq. (Vphi)) or the i.i.d. draws of the
// Sparsification Lemma.  Evolution: the CH-form update rules of the
// Clifford-simulator section (L[S], L[CZ], L[CX]; the Hadamard update of
// Eqs. (H1)-(H7) with Prop. H, whose C-layer V_C acts through the right rules
// R[CX], R[CZ], R[S]).
//
// Mapping: a term is a group of LPT lanes (a sub-wave; 64 / LPT terms per
// wave) and each lane holds RPL tableau rows (F_p, G_p, M_p as uint64,
// gamma_p).  A left rule touches one or two rows: it costs a few in-group
// broadcasts (ds_bpermute, readlane for a whole-wave group) and a masked XOR,
// shared by all the terms of the wave.  The Hadamard update broadcasts row p,
// computes t, u, alpha, beta once per lane, and applies V_C to every row at
// once: each batch of commuting right rules (CX_{q,i} for i in a set W,
// CZ_{q,i} for i in V_1) collapses to a parity and a masked XOR per row.
#include "device_common.hpp"
#include "internal.hpp"

namespace chsim {

// ---------------------------------------------------------------------------
// Branch choice and coefficients, one thread per term.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_choose(TermsView T, const SlotTable* __restrict__ slots,
                                                uint32_t mode, uint64_t seed, double scale) {
  const uint64_t a = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= T.chi) return;
  double br = 1.0, bi = 0.0;
  if (mode == CHSIM_EXACT) {
    uint64_t rem = a;
    for (uint32_t p = 0; p < T.n_slot; ++p) {
      const uint32_t nb = slots[p].n_branch;
      const uint32_t j = (uint32_t)(rem % nb);
      rem /= nb;
      T.branch[(uint64_t)p * T.chi + a] = (uint8_t)j;
      const double cr = slots[p].coef_re[j], ci = slots[p].coef_im[j];
      const double nr = br * cr - bi * ci;
      bi = br * ci + bi * cr;
      br = nr;
    }
  } else {
    for (uint32_t p = 0; p < T.n_slot; ++p) {
      const SlotTable& st = slots[p];
      const double u = philox_uniform53(seed, a, p, kStreamSparsify);
      const double uw = u * st.total;
      uint32_t j = st.n_branch - 1;
      for (uint32_t i = 0; i + 1 < st.n_branch; ++i)
        if (uw < st.cum[i]) {
          j = i;
          break;
        }
      T.branch[(uint64_t)p * T.chi + a] = (uint8_t)j;
      const double cr = st.unit_re[j], ci = st.unit_im[j];
      const double nr = br * cr - bi * ci;
      bi = br * ci + bi * cr;
      br = nr;
    }
    br *= scale;
    bi *= scale;
  }
  T.b[a] = make_double2(br, bi);
}

hipError_t launch_choose(const TermsView& T, const SlotTable* slots, uint32_t mode, uint64_t seed,
                         double scale, hipStream_t st) {
  const uint32_t blocks = (uint32_t)((T.chi + 255) / 256);
  hipLaunchKernelGGL(k_choose, dim3(blocks), dim3(256), 0, st, T, slots, mode, seed, scale);
  return hipGetLastError();
}

EvolveShape evolve_shape_for(uint32_t n, int lanes) {
  EvolveShape s;
  s.lanes = lanes;
  s.rows = lanes > 0 ? (int)((n + (uint32_t)lanes - 1) / (uint32_t)lanes) : 0;
  if (s.rows < 1) s.rows = 1;
  return s;
}

// Default: columns in registers, 4 lanes per term.  A single qubit has its row in a
// register: there is nothing to transpose (65536 terms: 48 µs and 52 by columns).
EvolveShape evolve_default_shape(uint32_t n) {
  EvolveShape s = evolve_shape_for(n, 4);
  s.cols = n > 1u;
  return s;
}

uint64_t evolve_capacity(EvolveShape s, uint32_t n, uint32_t cus) {
  if (!s.cols) return 0u;
  return (uint64_t)cus * 4u * (uint64_t)evolve_cols_waves(s.lanes, evolve_shape_for(n, s.lanes).rows) * 64u /
         (uint64_t)s.lanes;
}

// Instantiated shapes: lanes in {4, 8, 16, 32, 64} with rows = ceil(n / lanes)
// and lanes * rows <= 64; columns in registers: lanes in {4, 8, 16}.
bool evolve_shape_supported(EvolveShape s, uint32_t n) {
  if (s.cols)
    return (s.lanes == 4 || s.lanes == 8 || s.lanes == 16) && n >= 1 && n <= 64 &&
           (uint32_t)s.lanes * 16u >= n;
  const bool lanes_ok = s.lanes == 4 || s.lanes == 8 || s.lanes == 16 || s.lanes == 32 || s.lanes == 64;
  return lanes_ok && s.rows >= 1 && (uint32_t)(s.lanes * s.rows) >= n && s.lanes * s.rows <= 64;
}

hipError_t launch_evolve_job(const EvolveJob& J, const DGate* gates, uint32_t n_gates, bool from_zero,
                             uint32_t* err, EvolveShape shape, hipStream_t st) {
  const uint32_t n = J.dst.n;
  if (shape.lanes == 0) shape = evolve_default_shape(n);
  if (!evolve_shape_supported(shape, n)) return hipErrorInvalidValue;
  if (shape.cols) {
    const int cols = evolve_shape_for(n, shape.lanes).rows;
    if (shape.lanes == 16) return launch_evolve_c16(cols, J, gates, n_gates, from_zero, err, st);
    if (shape.lanes == 8) return launch_evolve_c8(cols, J, gates, n_gates, from_zero, err, st);
    return cols <= 10 ? launch_evolve_c4a(cols, J, gates, n_gates, from_zero, err, st)
                      : launch_evolve_c4b(cols, J, gates, n_gates, from_zero, err, st);
  }
  if (shape.lanes == 4) return launch_evolve_l4(shape.rows, J, gates, n_gates, from_zero, err, st);
  if (shape.lanes == 8) return launch_evolve_l8(shape.rows, J, gates, n_gates, from_zero, err, st);
  if (shape.lanes == 64) return launch_evolve_w64(J, gates, n_gates, from_zero, err, st);
  return launch_evolve_wide(shape.lanes, shape.rows, J, gates, n_gates, from_zero, err, st);
}

hipError_t launch_evolve(const TermsView& T, const DGate* gates, uint32_t n_gates,
                         const uint32_t* slot_seq, uint32_t n_occ, bool from_zero, uint32_t* err,
                         EvolveShape shape, hipStream_t st) {
  EvolveJob J;
  J.src = T;
  J.dst = T;
  J.src_rs = J.dst_rs = T.chi;
  J.src_is = J.dst_is = 1;
  J.src_idx = nullptr;
  J.br_idx = nullptr;
  J.branch = T.branch;
  J.chi_br = T.chi;
  J.count_dev = nullptr;
  J.count = T.chi;
  J.slot_seq = slot_seq;
  J.n_occ = n_occ;
  return launch_evolve_job(J, gates, n_gates, from_zero, err, shape, st);
}

// Materialise |0^n> for every term (used when terms are read before any gate).
__global__ __launch_bounds__(256) void k_set_zero(TermsView T) {
  const uint64_t a = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= T.chi) return;
  for (uint32_t p = 0; p < T.n; ++p) {
    const uint64_t off = (uint64_t)p * T.chi + a;
    T.F[off] = 1ull << p;
    T.G[off] = 1ull << p;
    T.M[off] = 0ull;
    T.gamma[off] = 0;
  }
  T.v[a] = 0ull;
  T.s[a] = 0ull;
  T.omega[a] = 0;
}

namespace {

// One launch for the nine arrays of a term store: a 256-thread workgroup copies
// R x 4 KB of one of them, 16 bytes per thread and load (arrays start on 16 bytes; one
// load per thread while that leaves few workgroups, four above 32 MB).  The arrays of a
// small instance are too short to fill the chip, and a copy each cost a launch and
// its gap: n = 20, chi = 3001, eight copies of the terms in a call of 1.69 ms, 1.34
// with one launch each.
constexpr uint32_t kCopyArrays = 9;
struct CopyList {
  const uint8_t* src[kCopyArrays];
  uint8_t* dst[kCopyArrays];
  uint64_t bytes[kCopyArrays];
  uint32_t first[kCopyArrays + 1];  // workgroups before each array
};

template <uint32_t R>
__global__ __launch_bounds__(256) void k_terms_copy(CopyList c) {
  constexpr uint32_t kChunk = 4096u * R;
  uint32_t k = 0;
  while (blockIdx.x >= c.first[k + 1]) ++k;
  const uint64_t at = (uint64_t)(blockIdx.x - c.first[k]) * kChunk;
  const uint64_t end = min(c.bytes[k], at + kChunk);
  const uint8_t* src = c.src[k];
  uint8_t* dst = c.dst[k];
  uint4 v[R];
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint64_t o = at + r * 4096u + threadIdx.x * 16u;
    if (o + 16u <= end) v[r] = *reinterpret_cast<const uint4*>(src + o);
  }
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint64_t o = at + r * 4096u + threadIdx.x * 16u;
    if (o + 16u <= end) *reinterpret_cast<uint4*>(dst + o) = v[r];
    else
      for (uint64_t b = o; b < end; ++b) dst[b] = src[b];
  }
}

}  // namespace

hipError_t launch_terms_copy(const TermsView& a, const TermsView& d, bool branches, hipStream_t st) {
  const uint64_t rows = (uint64_t)a.n * a.chi;
  const void* const src[kCopyArrays] = {a.F, a.G, a.M, a.gamma, a.v, a.s, a.omega, a.b, a.branch};
  void* const dst[kCopyArrays] = {d.F, d.G, d.M, d.gamma, d.v, d.s, d.omega, d.b, d.branch};
  const uint64_t bytes[kCopyArrays] = {rows * 8, rows * 8, rows * 8, rows,  a.chi * 8,
                                       a.chi * 8, a.chi, a.chi * sizeof(double2), branches ? (uint64_t)a.n_slot * a.chi : 0};
  CopyList c{};
  uint64_t blocks = 0, total = 0;
  for (uint64_t b : bytes) total += b;
  const uint64_t chunk = total > (32u << 20) ? 16384u : 4096u;
  for (uint32_t k = 0; k < kCopyArrays; ++k) {
    c.src[k] = static_cast<const uint8_t*>(src[k]);
    c.dst[k] = static_cast<uint8_t*>(dst[k]);
    c.bytes[k] = bytes[k];
    c.first[k] = (uint32_t)blocks;
    blocks += (bytes[k] + chunk - 1) / chunk;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  }
  c.first[kCopyArrays] = (uint32_t)blocks;
  if (chunk == 4096u) hipLaunchKernelGGL(k_terms_copy<1>, dim3((uint32_t)blocks), dim3(256), 0, st, c);
  else hipLaunchKernelGGL(k_terms_copy<4>, dim3((uint32_t)blocks), dim3(256), 0, st, c);
  return hipGetLastError();
}

hipError_t launch_set_zero(const TermsView& T, hipStream_t st) {
  const uint32_t blocks = (uint32_t)((T.chi + 255) / 256);
  hipLaunchKernelGGL(k_set_zero, dim3(blocks), dim3(256), 0, st, T);
  return hipGetLastError();
}

// Three-step sampler: w = s with bits flipped where v and flips agree; x = w G^T.
__global__ __launch_bounds__(256) void k_sample(TermsView T, const uint64_t* __restrict__ alpha,
                                                const uint64_t* __restrict__ flips,
                                                uint64_t* __restrict__ x_out, uint32_t count) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint64_t a = alpha[i];
  const uint64_t w = T.s[a] ^ (T.v[a] & flips[i]);
  uint64_t x = 0;
  for (uint32_t r = 0; r < T.n; ++r) x |= (uint64_t)par64(w & T.G[(uint64_t)r * T.chi + a]) << r;
  x_out[i] = x;
}

hipError_t launch_sample(const TermsView& T, const uint64_t* alpha, const uint64_t* flips,
                         uint64_t* x_out, uint32_t count, hipStream_t st) {
  hipLaunchKernelGGL(k_sample, dim3((count + 255) / 256), dim3(256), 0, st, T, alpha, flips, x_out,
                     count);
  return hipGetLastError();
}

}  // namespace chsim
