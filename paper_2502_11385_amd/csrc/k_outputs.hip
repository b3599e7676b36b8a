// Further outputs of a state: the k most probable outcomes, and expectation
// values of Pauli strings.
//
// Top-k decides on the key p = re*re + im*im computed in FP64 with every
// product and the sum rounded separately (no fused multiply-add), so the
// decision is the same as any plain FP64 evaluation of that expression.
// p >= 0, so the key's bit pattern orders like its value.  One histogram
// pass over the state, by the key's top 16 bits (its exponent and four bits
// of its fraction), finds the bin of the k-th key; a second pass gathers the
// keys from that bin's lower bound up, and the host sorts them: two reads of
// the state at HBM's rate where 12-bit digits took three or more (27 qubits,
// k = 64: 0.70 -> 0.48 ms complex64, 1.17 -> 0.84 ms complex128).  Where those
// are too many (states of many equal magnitudes), a radix select on 12-bit
// digits below the bin's (one histogram pass per digit, integer counts) fixes
// the threshold key; the elements above it are gathered, and the remaining
// places go to the elements equal to it in index order.
#include <algorithm>
#include <mutex>

#include "reduce_core.h"

namespace qsv {

constexpr int kTopkBins = 4096;  // 12-bit digits

template <typename C>
__device__ __forceinline__ uint64_t topk_key(C v) {
  // no contraction into a fused multiply-add: each operation rounds
#pragma clang fp contract(off)
  const double x = double(v.x), y = double(v.y);
  const double xx = x * x, yy = y * y;
  const double p = xx + yy;
  return uint64_t(__double_as_longlong(p));
}

// Histogram by the keys' top 16 bits, in LDS: 32768 bins for keys without
// the sign bit and one for those with it (a NaN may carry it), whose order
// among themselves the first pass does not need.  Bound by HBM with one
// work-group of 1024 threads and eight loads in flight per thread on a CU;
// finer bins than the 12 top bits save the pass that refines them, and
// spread the LDS additions.  A work-group's counts fit 32 bits (at most 2^26
// keys each), the state's do not: 2^32 equal amplitudes share a bin on 32
// qubits.
constexpr int kTopkWide = (1 << 15) + 1;

__device__ __forceinline__ uint32_t topk_wide_bin(uint64_t key) {
  const uint32_t d = uint32_t(key >> 48);
  return d < (1u << 15) ? d : (1u << 15);
}

// A wave whose keys share a bin (states of few amplitudes that are not 0)
// adds their number once: additions to one address go one after the other.
__device__ __forceinline__ void topk_wide_add(unsigned int* wide,
                                              uint64_t key) {
  const uint32_t bin = topk_wide_bin(key);
  const uint32_t first = __builtin_amdgcn_readfirstlane(bin);
  const uint64_t lanes = __ballot(1);
  if (__ballot(bin == first) != lanes)
    atomicAdd(&wide[bin], 1u);
  else if ((threadIdx.x & 63u) == uint32_t(__builtin_ctzll(lanes)))
    atomicAdd(&wide[first], uint32_t(__popcll(lanes)));
}

template <typename C>
__global__ void __launch_bounds__(1024)
    topk_wide_kernel(const C* __restrict__ a, uint64_t count,
                     unsigned long long* __restrict__ hist) {
  extern __shared__ unsigned int wide[];
  for (int b = threadIdx.x; b < kTopkWide; b += 1024) wide[b] = 0;
  __syncthreads();
  const uint64_t stride = uint64_t(gridDim.x) * 1024;
  uint64_t i = uint64_t(blockIdx.x) * 1024 + threadIdx.x;
  for (; i + 7 * stride < count; i += 8 * stride) {
    C v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = a[i + j * stride];
#pragma unroll
    for (int j = 0; j < 8; ++j) topk_wide_add(wide, topk_key(v[j]));
  }
  for (; i < count; i += stride) topk_wide_add(wide, topk_key(a[i]));
  __syncthreads();
  for (int b = threadIdx.x; b < kTopkWide; b += 1024)
    if (wide[b]) atomicAdd(&hist[b], (unsigned long long)wide[b]);
}

// The bin of the k-th largest key into *found.
__global__ void __launch_bounds__(1024)
    topk_find_kernel(const unsigned long long* __restrict__ hist, uint64_t k,
                     TopkFound* __restrict__ found) {
  __shared__ unsigned long long sum[1024];
  // thread t owns bins from the top: kTopkWide - 1 - t * 33 downwards
  constexpr int kPer = (kTopkWide + 1023) / 1024;
  const int top = kTopkWide - 1 - int(threadIdx.x) * kPer;
  unsigned long long mine = 0;
  for (int j = 0; j < kPer; ++j)
    if (top - j >= 0) mine += hist[top - j];
  sum[threadIdx.x] = mine;
  __syncthreads();
  for (int w = 1; w < 1024; w <<= 1) {
    const unsigned long long add =
        threadIdx.x >= unsigned(w) ? sum[threadIdx.x - w] : 0;
    __syncthreads();
    sum[threadIdx.x] += add;
    __syncthreads();
  }
  unsigned long long cum = sum[threadIdx.x] - mine;
  if (cum < k && cum + mine >= k) {  // one thread: count >= k
    for (int j = 0; j < kPer; ++j) {
      const unsigned long long h = hist[top - j];
      if (cum + h >= k) {
        found->bin = uint64_t(top - j);
        found->above = cum;
        found->in_bin = h;
        break;
      }
      cum += h;
    }
  }
}

// Gather (key, index) of every element from the found bin up, unless they
// are more than cap.
template <typename C>
__global__ void __launch_bounds__(256)
    topk_gather_kernel(const C* __restrict__ a, uint64_t count,
                       TopkFound* __restrict__ found, uint64_t cap,
                       KeyIndex* __restrict__ out) {
  if (found->above + found->in_bin > cap) return;
  const uint32_t bin = uint32_t(found->bin);
  const uint64_t stride = uint64_t(gridDim.x) * 256;
  auto put = [&](uint64_t key, uint64_t i) {
    if (topk_wide_bin(key) < bin) return;
    const unsigned long long slot = atomicAdd(&found->gathered, 1ull);
    if (slot < cap) out[slot] = KeyIndex{key, i};
  };
  uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x;
  for (; i + 7 * stride < count; i += 8 * stride) {
    C v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = a[i + j * stride];
#pragma unroll
    for (int j = 0; j < 8; ++j) put(topk_key(v[j]), i + j * stride);
  }
  for (; i < count; i += stride) put(topk_key(a[i]), i);
}

// Histogram of digit (key >> shift) & (bins - 1) over the keys whose bits
// under `mask` equal `prefix`.
template <typename C>
__global__ void __launch_bounds__(256)
    topk_hist_kernel(const C* __restrict__ a, uint64_t count, uint64_t mask,
                     uint64_t prefix, int shift, int bins,
                     unsigned long long* __restrict__ hist) {
  __shared__ unsigned int h[kTopkBins];
  for (int b = threadIdx.x; b < kTopkBins; b += 256) h[b] = 0;
  __syncthreads();
  const uint64_t stride = uint64_t(gridDim.x) * 256;
  for (uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x; i < count;
       i += stride) {
    const uint64_t k = topk_key(a[i]);
    if ((k & mask) == prefix)
      atomicAdd(&h[(k >> shift) & uint64_t(bins - 1)], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < bins; b += 256)
    if (h[b]) atomicAdd(&hist[b], (unsigned long long)h[b]);
}

// Gather (key, index) of every element with (key & mask) > prefix, or >=
// prefix when `ge`; positions come from an integer counter (order is fixed
// afterwards by sorting on (key, index)).
template <typename C>
__global__ void __launch_bounds__(256)
    topk_collect_kernel(const C* __restrict__ a, uint64_t count,
                        uint64_t mask, uint64_t prefix, int ge,
                        unsigned long long* __restrict__ counter, uint64_t cap,
                        KeyIndex* __restrict__ out) {
  const uint64_t stride = uint64_t(gridDim.x) * 256;
  for (uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x; i < count;
       i += stride) {
    const uint64_t k = topk_key(a[i]);
    const uint64_t m = k & mask;
    if (ge ? m >= prefix : m > prefix) {
      const unsigned long long slot = atomicAdd(counter, 1ull);
      if (slot < cap) out[slot] = KeyIndex{k, i};
    }
  }
}

// Elements equal to the threshold key in each block's contiguous range.
template <typename C>
__global__ void __launch_bounds__(256)
    topk_tie_count_kernel(const C* __restrict__ a, uint64_t count,
                          uint64_t chunk, uint64_t key,
                          unsigned long long* __restrict__ counts) {
  __shared__ unsigned int tot;
  if (threadIdx.x == 0) tot = 0;
  __syncthreads();
  const uint64_t lo = uint64_t(blockIdx.x) * chunk;
  const uint64_t hi = lo + chunk < count ? lo + chunk : count;
  unsigned int c = 0;
  for (uint64_t i = lo + threadIdx.x; i < hi; i += 256)
    c += topk_key(a[i]) == key ? 1u : 0u;
  atomicAdd(&tot, c);
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = tot;
}

// The first `need` elements equal to the threshold key, in index order:
// block b starts at rank offsets[b] and ranks its own equal elements in
// index order (wave ballots, then waves in order).
template <typename C>
__global__ void __launch_bounds__(256)
    topk_tie_collect_kernel(const C* __restrict__ a, uint64_t count,
                            uint64_t chunk, uint64_t key,
                            const unsigned long long* __restrict__ offsets,
                            uint64_t need, KeyIndex* __restrict__ out) {
  __shared__ unsigned int wave_cnt[4];
  const uint64_t base = offsets[blockIdx.x];
  if (base >= need) return;  // uniform over the block
  const uint64_t lo = uint64_t(blockIdx.x) * chunk;
  const uint64_t hi = lo + chunk < count ? lo + chunk : count;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint64_t run = base;
  for (uint64_t s = lo; s < hi && run < need; s += 256) {
    const uint64_t i = s + threadIdx.x;
    const bool eq = i < hi && topk_key(a[i]) == key;
    const uint64_t bal = __ballot(eq);
    if (lane == 0) wave_cnt[wv] = __popcll(bal);
    __syncthreads();
    uint64_t before = 0;
    for (int w = 0; w < wv; ++w) before += wave_cnt[w];
    const uint64_t mine = __popcll(bal & ((uint64_t(1) << lane) - 1));
    const uint64_t rank = run + before + mine;
    if (eq && rank < need) out[rank] = KeyIndex{key, i};
    uint64_t total = 0;
    for (int w = 0; w < 4; ++w) total += wave_cnt[w];
    __syncthreads();
    run += total;
  }
}

template <typename C>
static const C* as(const void* p) {
  return static_cast<const C*>(p);
}

unsigned topk_grid(uint64_t count) {
  const uint64_t g = (count + 255) / 256;
  return unsigned(g < 4096 ? g : 4096);
}

__global__ void __launch_bounds__(256)
    topk_clear_kernel(unsigned long long* __restrict__ hist,
                      TopkFound* __restrict__ found) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b < kTopkWide) hist[b] = 0;
  if (b == 0) *found = TopkFound{};
}

size_t topk_hist_bytes() {
  return size_t(kTopkWide) * sizeof(unsigned long long);
}

template <typename C>
static hipError_t topk_select(const C* a, uint64_t count, uint64_t k,
                              unsigned long long* hist, TopkFound* found,
                              uint64_t cap, KeyIndex* out,
                              hipStream_t stream) {
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [] {
    attr_err = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&topk_wide_kernel<C>),
        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  });
  if (attr_err != hipSuccess) return attr_err;
  // one work-group per CU, a state of fewer amplitudes one per 2048; the
  // gather, whose pairs the host sorts, in fewer pieces
  const uint64_t g = (count + 2047) / 2048, gg = (count + 8191) / 8192;
  topk_clear_kernel<<<(kTopkWide + 255) / 256, 256, 0, stream>>>(hist, found);
  topk_wide_kernel<C><<<unsigned(g < 256 ? g : 256), 1024,
                        kTopkWide * sizeof(unsigned int), stream>>>(a, count,
                                                                    hist);
  topk_find_kernel<<<1, 1024, 0, stream>>>(hist, k, found);
  topk_gather_kernel<C><<<unsigned(gg < 2048 ? gg : 2048), 256, 0, stream>>>(
      a, count, found, cap, out);
  return hipGetLastError();
}

hipError_t launch_topk_select(int prec, const void* amp, uint64_t count,
                              uint64_t k, unsigned long long* hist,
                              TopkFound* found, uint64_t cap, KeyIndex* out,
                              hipStream_t stream) {
  if (prec == 1)
    return topk_select(as<float2>(amp), count, k, hist, found, cap, out,
                       stream);
  return topk_select(as<double2>(amp), count, k, hist, found, cap, out, stream);
}

hipError_t launch_topk_hist(int prec, const void* amp, uint64_t count,
                            uint64_t mask, uint64_t prefix, int shift,
                            int bins, unsigned long long* hist,
                            hipStream_t stream) {
  const unsigned g = topk_grid(count);
  if (prec == 1)
    topk_hist_kernel<float2><<<g, 256, 0, stream>>>(
        as<float2>(amp), count, mask, prefix, shift, bins, hist);
  else
    topk_hist_kernel<double2><<<g, 256, 0, stream>>>(
        as<double2>(amp), count, mask, prefix, shift, bins, hist);
  return hipGetLastError();
}

hipError_t launch_topk_collect(int prec, const void* amp, uint64_t count,
                               uint64_t mask, uint64_t prefix, int ge,
                               unsigned long long* counter, uint64_t cap,
                               KeyIndex* out, hipStream_t stream) {
  const unsigned g = topk_grid(count);
  if (prec == 1)
    topk_collect_kernel<float2><<<g, 256, 0, stream>>>(
        as<float2>(amp), count, mask, prefix, ge, counter, cap, out);
  else
    topk_collect_kernel<double2><<<g, 256, 0, stream>>>(
        as<double2>(amp), count, mask, prefix, ge, counter, cap, out);
  return hipGetLastError();
}

hipError_t launch_topk_ties(int prec, const void* amp, uint64_t count,
                            uint64_t key, unsigned blocks, uint64_t chunk,
                            unsigned long long* counts,
                            const unsigned long long* offsets, uint64_t need,
                            KeyIndex* out, hipStream_t stream) {
  if (!offsets) {
    if (prec == 1)
      topk_tie_count_kernel<float2><<<blocks, 256, 0, stream>>>(
          as<float2>(amp), count, chunk, key, counts);
    else
      topk_tie_count_kernel<double2><<<blocks, 256, 0, stream>>>(
          as<double2>(amp), count, chunk, key, counts);
  } else {
    if (prec == 1)
      topk_tie_collect_kernel<float2><<<blocks, 256, 0, stream>>>(
          as<float2>(amp), count, chunk, key, offsets, need, out);
    else
      topk_tie_collect_kernel<double2><<<blocks, 256, 0, stream>>>(
          as<double2>(amp), count, chunk, key, offsets, need, out);
  }
  return hipGetLastError();
}

// ------------------------------------------------------ Pauli expectations
//
// For P = i^{|x & z|} X^x Z^z (x: qubits with X or Y, z: qubits with Z or
// Y), P|i> = i^{|x & z|} (-1)^{|i & z|} |i ^ x>, so
// <psi|P|psi> = Re(i^{|x & z|} S), S = sum_i conj(a_{i^x}) a_i (-1)^{|i & z|}.
// With x != 0 the terms of i and i ^ x are t and (-1)^{|x & z|} conj(t): S is
// twice the real part (|x & z| even) or i times twice the imaginary part
// (odd) of the sum over the i with the highest bit of x clear.  So a term
// reads every amplitude once and sums one real number per pair; with x = 0
// it sums one per amplitude.  Each block sums consecutive pairs in FP64 with
// Neumaier compensation, in a fixed order; one block per term then sums the
// blocks.
//
// Bound by HBM, one read of the state per term.  All terms of a call go in
// one launch, neighbouring blocks taking the same part of the state for
// different terms, so that terms share what the caches still hold.  Four
// terms on 27 qubits: 1.32 -> 0.62 ms complex64, 2.02 -> 1.24 ms complex128
// (one term 0.33 -> 0.21 and 0.46 -> 0.37 ms), against summing both parts of
// every amplitude's term, a launch and a final sum of 32768 blocks per term.

// At most 2^11 blocks per term: eight per CU with a single term.
constexpr int kPauliBlocksLog = 11;
constexpr int kPauliMinChunkLog = 8;

static int pauli_chunk_log(int pairs_log) {
  return pairs_log - kPauliBlocksLog > kPauliMinChunkLog
             ? pairs_log - kPauliBlocksLog
             : kPauliMinChunkLog;
}

template <typename C>
__device__ __forceinline__ double pauli_value(C y, C x, bool imag) {
  // conj(x) y: real part xr yr + xi yi, imaginary part xr yi - xi yr
  const double xr = double(x.x), xi = double(x.y);
  const double u = double(imag ? y.y : y.x);
  const double v = double(imag ? -y.x : y.y);
  return __builtin_fma(xr, u, xi * v);
}

template <typename C, bool DIAG>
__device__ __forceinline__ void pauli_block(const C* __restrict__ a,
                                            uint64_t count, int chunk_log,
                                            uint64_t chunk, uint64_t xm,
                                            uint64_t zm, double* s,
                                            double* c) {
  const int hb = DIAG ? 0 : 63 - __clzll((long long)xm);
  const bool imag = !DIAG && (__popcll(xm & zm) & 1);
  const uint64_t start = chunk << chunk_log;
  const uint64_t full = start + (uint64_t(1) << chunk_log);
  const uint64_t end = full < count ? full : count;
#pragma unroll 4
  for (uint64_t k = start + threadIdx.x; k < end; k += 256) {
    const uint64_t i = DIAG ? k : insert_zero64(k, hb);
    double v = DIAG ? prob_of(a[i]) : pauli_value(a[i], a[i ^ xm], imag);
    if (__popcll(i & zm) & 1) v = -v;
    nadd(*s, *c, v);
  }
}

template <typename C>
__global__ void __launch_bounds__(256)
    pauli_partial_kernel(const C* __restrict__ a, int n, PauliTerms terms,
                         uint32_t n_terms, double* __restrict__ partial) {
  __shared__ double sh[512];
  const uint32_t t = blockIdx.x % n_terms;
  const uint64_t chunk = blockIdx.x / n_terms;
  const uint64_t xm = terms.x[t], zm = terms.z[t];
  const int pairs_log = xm ? n - 1 : n;
  const uint64_t count = uint64_t(1) << pairs_log;
  int cl = pairs_log - kPauliBlocksLog;
  if (cl < kPauliMinChunkLog) cl = kPauliMinChunkLog;
  double s = 0, c = 0;
  if (chunk << cl >= count) return;  // a term with x needs half the blocks
  if (xm) pauli_block<C, false>(a, count, cl, chunk, xm, zm, &s, &c);
  else pauli_block<C, true>(a, count, cl, chunk, xm, zm, &s, &c);
  block_reduce_pair(s, c, sh);
  if (threadIdx.x == 0) {
    double* p = partial + (uint64_t(t) * (1u << kPauliBlocksLog) + chunk) * 2;
    p[0] = s;
    p[1] = c;
  }
}

// out[2 t], out[2 t + 1]: real and imaginary part of term t's S.
__global__ void __launch_bounds__(256)
    pauli_final_kernel(const double* __restrict__ partial, int n,
                       PauliTerms terms, double* __restrict__ out) {
  __shared__ double sh[512];
  const uint32_t t = blockIdx.x;
  const uint64_t xm = terms.x[t], zm = terms.z[t];
  const int pairs_log = xm ? n - 1 : n;
  int cl = pairs_log - kPauliBlocksLog;
  if (cl < kPauliMinChunkLog) cl = kPauliMinChunkLog;
  const uint32_t blocks =
      pairs_log > cl ? 1u << (pairs_log - cl) : 1u;
  const double* p = partial + uint64_t(t) * (2u << kPauliBlocksLog);
  double s = 0, c = 0;
#pragma unroll 8
  for (uint32_t b = threadIdx.x; b < blocks; b += 256) {
    nadd(s, c, p[2 * b]);
    c += p[2 * b + 1];
  }
  block_reduce_pair(s, c, sh);
  if (threadIdx.x == 0) {
    const double v = (s + c) * (xm ? 2.0 : 1.0);
    const bool imag = __popcll(xm & zm) & 1;
    out[2 * t] = imag ? 0.0 : v;
    out[2 * t + 1] = imag ? v : 0.0;
  }
}

size_t pauli_scratch_bytes(int n_terms) {
  return size_t(std::min(n_terms, kPauliBatch)) * (2u << kPauliBlocksLog) *
         sizeof(double);
}

hipError_t launch_pauli(int prec, const void* amp, int n, int n_terms,
                        const uint64_t* x_masks, const uint64_t* z_masks,
                        double* scratch, double* out_dev,
                        hipStream_t stream) {
  for (int t0 = 0; t0 < n_terms; t0 += kPauliBatch) {
    const int nt = std::min(kPauliBatch, n_terms - t0);
    PauliTerms terms = {};
    bool diag = false;
    for (int t = 0; t < nt; ++t) {
      terms.x[t] = x_masks[t0 + t];
      terms.z[t] = z_masks[t0 + t];
      diag = diag || !terms.x[t];
    }
    // blocks of the term with the most pairs
    const int pl = diag || n == 0 ? n : n - 1;
    const int cl = pauli_chunk_log(pl);
    const unsigned blocks = (pl > cl ? 1u << (pl - cl) : 1u) * unsigned(nt);
    if (prec == 1)
      pauli_partial_kernel<float2><<<blocks, 256, 0, stream>>>(
          as<float2>(amp), n, terms, uint32_t(nt), scratch);
    else
      pauli_partial_kernel<double2><<<blocks, 256, 0, stream>>>(
          as<double2>(amp), n, terms, uint32_t(nt), scratch);
    pauli_final_kernel<<<nt, 256, 0, stream>>>(scratch, n, terms,
                                               out_dev + 2 * t0);
  }
  return hipGetLastError();
}

}  // namespace qsv
