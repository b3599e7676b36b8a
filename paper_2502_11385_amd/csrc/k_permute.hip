// Qubit relabelling pass: qubit q of the state becomes qubit perm[q].
//
// This is the data movement of the paper's swap insertion (Section III.B):
// one pass moves busy high qubits to low positions, where later tiles and
// coalesced runs cover them.  A work-group takes tiles of source indices
// spanned by the lowest source qubits and the qubits that land on the lowest
// destination qubits, as many of both as a tile of 32 KiB holds (8 KiB for
// small states, see qsv_permute_qubits): its reads and its writes are
// contiguous runs (512 bytes or more where the two sets are disjoint, 256 in
// small tiles), with the tile transposed through LDS in between.
//
// Bound by HBM (2^n amplitudes read and written), given enough bytes in
// flight: each thread loads 8 (complex128) or 16 (complex64) amplitudes
// of a 32 KiB tile before it stores any, and five such tiles share a CU.  Random permutation
// of 27 qubits, complex128: 1.60 -> 0.82 ms (5.25 TB/s); the tiles of at most
// 4 KiB before had one load in flight per thread and a work-group each.
//
// The file also holds the other kernels that only move data: the state's copy
// and the upload of programs.
#include "device_common.h"

namespace qsv {

// Copy of a state (16-byte elements, 8 in flight per thread).
template <bool NT>
__global__ void __launch_bounds__(256)
    copy_kernel(const double2* __restrict__ src, double2* __restrict__ dst,
                uint64_t count) {
  for (uint64_t b = uint64_t(blockIdx.x) * 2048; b < count;
       b += uint64_t(gridDim.x) * 2048) {
    const uint64_t i = b + threadIdx.x;
    if (b + 2048 <= count) {
      double2 v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = stream_load<NT>(src + i + e * 256);
#pragma unroll
      for (int e = 0; e < 8; ++e) stream_store<NT>(dst + i + e * 256, v[e]);
    } else {
      for (uint64_t k = i; k < count; k += 256) dst[k] = src[k];
    }
  }
}

hipError_t launch_copy(const void* src, void* dst, uint64_t bytes,
                       hipStream_t stream) {
  if (bytes % sizeof(double2)) return hipErrorInvalidValue;
  const uint64_t count = bytes / sizeof(double2);
  const uint64_t rows = (count + 2047) / 2048;
  const unsigned grid = unsigned(rows < 2048 ? rows : 2048);
  const double2* s = static_cast<const double2*>(src);
  double2* d = static_cast<double2*>(dst);
  if (bytes > kStreamBytes) copy_kernel<true><<<grid, 256, 0, stream>>>(s, d, count);
  else copy_kernel<false><<<grid, 256, 0, stream>>>(s, d, count);
  return hipGetLastError();
}

// Upload of a program: the device reads the pinned staging buffer itself.  A
// copy by the runtime goes to a DMA engine, and the kernels before and after
// it wait for each other through signals: 20 us between a 12-qubit circuit's
// basis fill and its tile pass (circuit 98 -> 85 us without).  Long programs
// stay with the engine, whose rate then counts for more than the signals.
constexpr uint64_t kUploadKernelBytes = uint64_t(1) << 20;

__global__ void __launch_bounds__(256)
    upload_kernel(const double2* __restrict__ host, double2* __restrict__ dev,
                  uint64_t count) {
  const uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < count) dev[i] = host[i];
}

hipError_t launch_upload(const void* host, void* dev, uint64_t bytes,
                         hipStream_t stream) {
  if (bytes > kUploadKernelBytes)
    return hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, stream);
  const uint64_t count = (bytes + sizeof(double2) - 1) / sizeof(double2);
  upload_kernel<<<unsigned((count + 255) / 256), 256, 0, stream>>>(
      static_cast<const double2*>(host), static_cast<double2*>(dev), count);
  return hipGetLastError();
}

// Work-group g takes tiles g, g + gridDim.x, ...  A tile-local source index
// r = tid + e * blockDim.x sits in LDS slot slot(r), which XORs r's bits into
// its lowest ones so that both the stores (r consecutive) and the loads (r
// varying in the bits that land on the lowest destination qubits) spread
// over the banks.  Every map used here (slot, the spreading of r over the
// source qubits and of the destination index over its qubits, the
// destination-to-source map) is linear over XOR, so each splits into a
// per-thread part and a per-step part e, which the host gives.
template <typename C, int NE, bool NT>
__global__ void __launch_bounds__(256)
    permute_kernel(const C* __restrict__ src, C* __restrict__ dst,
                   PermArgs p, uint64_t tiles) {
  extern __shared__ double lds_raw[];
  C* lds = reinterpret_cast<C*>(lds_raw);
  const uint32_t tid = threadIdx.x;
  uint64_t s_thr = 0, d_thr = 0;
  uint32_t w_thr = 0, g_thr = 0;
  for (int j = 0; j < p.s; ++j) {
    const uint32_t bit = (tid >> j) & 1u;
    s_thr |= uint64_t(bit) << p.s_bits[j];
    d_thr |= uint64_t(bit) << p.d_bits[j];
    w_thr ^= bit ? p.w_slot[j] : 0u;
    g_thr ^= bit ? p.g_slot[j] : 0u;
  }
  for (uint64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    // tile index -> source base (outer source bits) and its destination
    uint64_t sb = 0, db = 0;
    for (int j = 0; j < p.n_outer; ++j) {
      const uint64_t bit = (t >> j) & 1;
      sb |= bit << p.outer_src[j];
      db |= bit << p.outer_dst[j];
    }
    C v[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) v[e] = stream_load<NT>(src + (sb | s_thr | p.se[e]));
#pragma unroll
    for (int e = 0; e < NE; ++e) lds[w_thr ^ p.we[e]] = v[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < NE; ++e)
      stream_store<NT>(dst + (db | d_thr | p.de[e]), lds[g_thr ^ p.ge[e]]);
    __syncthreads();  // the next tile reuses the LDS
  }
}

template <typename C>
static hipError_t permute_launch(const void* src, void* dst, int n,
                                 const PermArgs& p, hipStream_t stream) {
  const uint64_t tiles = uint64_t(1) << (n - p.s);
  const unsigned threads = (1u << p.s) < 256u ? (1u << p.s) : 256u;
  // a few rounds per resident work-group (five on each of 256 CUs)
  const unsigned grid = unsigned(tiles < 8192 ? tiles : 8192);
  const size_t lds = sizeof(C) << p.s;
  const bool nt = (sizeof(C) << n) > kStreamBytes;
#define QSV_P(NE)                                                  \
  if (nt)                                                          \
    permute_kernel<C, NE, true><<<grid, threads, lds, stream>>>(   \
        static_cast<const C*>(src), static_cast<C*>(dst), p, tiles); \
  else                                                             \
    permute_kernel<C, NE, false><<<grid, threads, lds, stream>>>(  \
        static_cast<const C*>(src), static_cast<C*>(dst), p, tiles)
  switch (p.ne) {
    case 1: QSV_P(1); break;
    case 2: QSV_P(2); break;
    case 4: QSV_P(4); break;
    case 8: QSV_P(8); break;
    case 16: QSV_P(16); break;
    default: return hipErrorInvalidValue;
  }
#undef QSV_P
  return hipGetLastError();
}

hipError_t launch_permute(int prec, const void* src, void* dst, int n,
                          const PermArgs& p, hipStream_t stream) {
  if (p.s < 0 || p.s > kPermMaxTileBits || p.s > n || p.ne < 1 || p.ne > 16 ||
      uint64_t(p.ne) * ((1u << p.s) < 256u ? (1u << p.s) : 256u) != (1ull << p.s))
    return hipErrorInvalidValue;
  if (p.n_outer != n - p.s) return hipErrorInvalidValue;
  if (prec == 1) return permute_launch<float2>(src, dst, n, p, stream);
  return permute_launch<double2>(src, dst, n, p, stream);
}

}  // namespace qsv
