// Cut reconstruction kernels (Section III.A).
//
// Step 1 builds, for every subcircuit, the term vectors of the one-cut
// identity applied to each of its cut ends: a downstream end contributes
// p(|0>), p(|1>), 2p(|+>) - p(|0>) - p(|1>) or 2p(|+i>) - p(|0>) - p(|1>)
// (eqs 3.3-3.6); an upstream end contributes, by shot attribution (eq 3.7),
// I + Z and I - Z from the I-basis readout (2 p(0) and 2 p(1)), or the
// signed X or Y readout p(0) - p(1).  Step 2 forms, for every outcome x of
// the uncut circuit, (1/2)^K times the sum over all 4^K joint term choices
// of the product of the subcircuits' term vectors at x's bits.
#include <cstring>

#include "cut_internal.h"
#include "device_common.h"

namespace qsv {

__device__ __forceinline__ double cut_prob(const CutArgs& a, uint64_t i) {
  return a.probs_fp64 ? static_cast<const double*>(a.probs)[i]
                      : double(static_cast<const float*>(a.probs)[i]);
}

__global__ void __launch_bounds__(256)
    cut_terms_kernel(CutArgs a) {
  const uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (g >= a.total_entries) return;
  int s = 0;
  while (s + 1 < a.n_sub && a.subs[s + 1].entry_begin <= g) ++s;
  const CutSubDev& sd = a.subs[s];
  const uint64_t local = g - sd.entry_begin;
  const uint32_t t = uint32_t(local >> sd.eff);
  const uint64_t y = local & ((uint64_t(1) << sd.eff) - 1);
  uint64_t idx0 = 0;
  for (int i = 0; i < sd.eff; ++i) idx0 |= ((y >> i) & 1) << sd.out_pos[i];
  // choices per end: downstream ends with term 0/1 read one variant, with
  // term 2/3 three; upstream ends with term 0/1 read one outcome, with
  // term 2/3 both
  int nch[kCutMaxEnds];
  uint32_t total = 1;
  for (int e = 0; e < sd.n_ends; ++e) {
    const int d = (t >> (2 * e)) & 3;
    nch[e] = d < 2 ? 1 : (sd.end_kind[e] == 0 ? 3 : 2);
    total *= uint32_t(nch[e]);
  }
  const uint64_t* vo = a.voff + sd.v_offset;
  double acc = 0.0;
  for (uint32_t c = 0; c < total; ++c) {
    uint32_t r = c;
    uint64_t v = 0, idx = idx0;
    double coef = 1.0;
    for (int e = 0; e < sd.n_ends; ++e) {
      const int d = (t >> (2 * e)) & 3;
      const int k = int(r % uint32_t(nch[e]));
      r /= uint32_t(nch[e]);
      if (sd.end_kind[e] == 0) {
        // initial state label and its coefficient
        int label = d;
        if (d >= 2) {
          label = k == 0 ? d : k - 1;
          coef *= k == 0 ? 2.0 : -1.0;
        }
        v += uint64_t(label) * uint64_t(sd.end_mult[e]);
      } else {
        // readout basis I (terms 0, 1), X (2) or Y (3), and the outcome
        const int basis = d < 2 ? 0 : d - 1;
        v += uint64_t(basis) * uint64_t(sd.end_mult[e]);
        int m;
        if (d < 2) {
          m = d;
          coef *= 2.0;
        } else {
          m = k;
          coef *= k ? -1.0 : 1.0;
        }
        idx |= uint64_t(m) << sd.end_pos[e];
      }
    }
    acc += coef * cut_prob(a, vo[v] + idx);
  }
  a.T[sd.t_offset + local] = acc;
}

// The subcircuit's output index of outcome x (bit i = its i-th output).
__device__ __forceinline__ uint64_t cut_gather(const CutSubDev& sd,
                                               uint64_t x) {
  uint64_t v = 0;
  for (int r = 0; r < sd.n_runs; ++r)
    v |= ((x >> sd.run_src[r]) & ((uint64_t(1) << sd.run_len[r]) - 1))
         << sd.run_dst[r];
  return v;
}

// One thread per outcome x: the sum over all 4^K term choices of the
// product of the subcircuits' entries.
__global__ void __launch_bounds__(256)
    cut_kron_simple_kernel(CutArgs a, const double* __restrict__ T,
                           double* __restrict__ out) {
  const uint64_t x = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (x >= (uint64_t(1) << a.n_qubits)) return;
  uint64_t y[kCutMaxSub];
  for (int s = 0; s < a.n_sub; ++s) y[s] = cut_gather(a.subs[s], x);
  double acc = 0.0;
  for (uint64_t t = 0; t < a.n_terms; ++t) {
    const uint64_t* row = a.tt + t * uint64_t(a.n_sub);
    double prod = 1.0;
    for (int s = 0; s < a.n_sub; ++s) prod *= T[row[s] + y[s]];
    acc += prod;
  }
  out[x] = acc * ldexp(1.0, -a.n_cuts);
}


// One wave per nb blocks of 64 consecutive outcomes (n_qubits >= 6).
// Within a block the uniform subcircuits' entries are the same for every
// lane, so the sum factors: p(x) = (1/2)^K sum_c W[c] prod_{varying s}
// T_s(c)[y_s(x)], with W[c] = sum_u prod_{uniform s} T_s(c, u)[y_s].  The
// wave first forms every block's products over the uniform subcircuits for
// all (c, u) in parallel, then W[c] by summing over u in increasing order,
// then each lane sums over c in increasing order for its outcomes.
constexpr int kCutWaveLds = 512;  // doubles of LDS per wave

__global__ void __launch_bounds__(256)
    cut_kron_wave_kernel(CutArgs a, const double* __restrict__ T,
                         double* __restrict__ out, int nb) {
  __shared__ double lds[4][kCutWaveLds];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint64_t nx = uint64_t(1) << a.n_qubits;
  const uint64_t x0 = (uint64_t(blockIdx.x) * 4 + wv) * 64 * uint64_t(nb);
  if (x0 >= nx) return;  // whole waves exit
  double* P = lds[wv];                               // [nb][n_c][n_u]
  double* W = P + uint64_t(nb) * a.n_c * a.n_u;      // [nb][n_c]
  const uint64_t ncu = a.n_c * a.n_u;
  for (uint64_t i = lane; i < uint64_t(nb) * ncu; i += 64) {
    const uint64_t blk = i / ncu, cu = i - blk * ncu;
    const uint64_t xb = x0 + blk * 64;
    const uint64_t* row = a.ttu + cu * uint64_t(a.n_uni);
    double prod = 1.0;
    for (int k = 0; k < a.n_uni; ++k)
      prod *= T[row[k] + cut_gather(a.subs[a.uni_sub[k]], xb)];
    P[i] = prod;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (uint64_t i = lane; i < uint64_t(nb) * a.n_c; i += 64) {
    double sum = 0.0;
    for (uint64_t u = 0; u < a.n_u; ++u) sum += P[i * a.n_u + u];
    W[i] = sum;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const double scale = ldexp(1.0, -a.n_cuts);
  for (int blk = 0; blk < nb; ++blk) {
    const uint64_t x = x0 + uint64_t(blk) * 64 + uint64_t(lane);
    uint64_t yv[kCutMaxVary];
#pragma unroll
    for (int k = 0; k < kCutMaxVary; ++k)
      yv[k] = k < a.n_vary ? cut_gather(a.subs[a.vary_sub[k]], x) : 0;
    double acc = 0.0;
    for (uint64_t c = 0; c < a.n_c; ++c) {
      const uint64_t* row = a.ttv + c * uint64_t(a.n_vary);
      double prod = W[uint64_t(blk) * a.n_c + c];
#pragma unroll
      for (int k = 0; k < kCutMaxVary; ++k)
        if (k < a.n_vary) prod *= T[row[k] + yv[k]];
      acc += prod;
    }
    out[x] = acc * scale;
  }
}

// One work-group per 2^F rows of 256 consecutive outcomes (uncut qubits
// 0..7 are the threads).  The varying subcircuits' outputs reach into the
// rows and maybe above them (vary_pos, fixed per work-group); the qubits of
// free_pos belong to uniform subcircuits alone and number the rows.  With
// V[c] = prod_{varying s} T_s(c)[y_s], fixed per thread, and
// W[f][c] = sum_u prod_{uniform s} T_s(c, u)[y_s], the same for a whole row,
// p(f, x) = (1/2)^K sum_c W[f][c] V[c].
//
// Bound by the HBM write of the outcomes (8 bytes each, n_c multiply-adds):
// V stays in registers over all rows and W is formed once per row, where a
// wave per 64 outcomes formed both again for each block and waited for their
// loads.  2^28 outcomes, 2 cuts, n_c = 4: 0.88 -> 0.39 ms a call, 5.5 TB/s.
// ALL: the terms of the sums over u are formed by all the threads, a round at a
// time, and added in increasing u as one thread would: a thread per W alone made
// few outcomes with many cuts wait for a chain of 4^cuts loads (12 qubits, 4
// cuts, n_u = 64: 95 -> 40 us a call).
template <int NC, bool ALL>
__global__ void __launch_bounds__(256)
    cut_kron_tile_kernel(CutArgs a, const double* __restrict__ T,
                         double* __restrict__ out, int rows_log) {
  __shared__ double W[(1 << kCutRowsLog) * NC];
  const uint32_t tid = threadIdx.x;
  const int chunk_log = a.n_free - rows_log;
  const uint64_t chunk = blockIdx.x & ((uint64_t(1) << chunk_log) - 1);
  const uint64_t vary = blockIdx.x >> chunk_log;
  uint64_t xv = 0, x0 = 0, mask = 0;
  for (int i = 0; i < a.n_vary_hi; ++i)
    xv |= ((vary >> i) & 1) << a.vary_pos[i];
  for (int i = 0; i < rows_log; ++i) mask |= uint64_t(1) << a.free_pos[i];
  for (int i = 0; i < chunk_log; ++i)
    x0 |= ((chunk >> i) & 1) << a.free_pos[rows_log + i];
  const int rows = 1 << rows_log;
  const uint64_t n_u = a.n_u;
  const int n_w = rows * NC;
  auto row_x = [&](int f) {
    uint64_t x = x0;
    for (int b = 0; b < rows_log; ++b)
      x |= uint64_t((f >> b) & 1) << a.free_pos[b];
    return x;
  };
  if constexpr (!ALL) {
    for (int i = tid; i < n_w; i += 256) {
      const int f = i / NC, c = i % NC;
      const uint64_t x = row_x(f);
      double sum = 0.0;
      for (uint64_t u = 0; u < n_u; ++u) {
        const uint64_t* row = a.ttu + (uint64_t(c) * n_u + u) * uint64_t(a.n_uni);
        double prod = 1.0;
        for (int k = 0; k < a.n_uni; ++k)
          prod *= T[row[k] + cut_gather(a.subs[a.uni_sub[k]], x)];
        sum += prod;
      }
      W[i] = sum;
    }
  } else {
    __shared__ double P[2 * 256];  // a round's terms, two rounds in turn
    __shared__ uint32_t Y[kCutMaxSub << kCutRowsLog];
    // output index of each uniform subcircuit in each row
    for (int i = tid; i < rows * a.n_uni; i += 256)
      Y[i] = uint32_t(cut_gather(a.subs[a.uni_sub[i >> rows_log]],
                                 row_x(i & (rows - 1))));
    __syncthreads();
    const uint32_t per = 256 / n_w;  // threads per W: a power of two, as n_u is
    const uint32_t step = per < n_u ? per : uint32_t(n_u);
    const uint32_t i = tid & (n_w - 1), g = tid / n_w;
    const int f = i / NC, c = i % NC;
    double sum = 0.0;
    int buf = 0;
    for (uint64_t u = 0; u < n_u; u += step, buf ^= 256) {
      if (g < step) {
        const uint64_t* row =
            a.ttu + (uint64_t(c) * n_u + u + g) * uint64_t(a.n_uni);
        double prod = 1.0;
        for (int k = 0; k < a.n_uni; ++k)
          prod *= T[row[k] + Y[(k << rows_log) + f]];
        P[buf + g * n_w + i] = prod;
      }
      __syncthreads();
      if (g == 0)
        for (uint32_t j = 0; j < step; ++j) sum += P[buf + j * n_w + i];
    }
    if (g == 0) W[i] = sum;
  }
  const uint64_t xt = xv | tid;
  double V[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) V[c] = 1.0;
  for (int k = 0; k < a.n_vary; ++k) {
    const uint64_t y = cut_gather(a.subs[a.vary_sub[k]], xt);
#pragma unroll
    for (int c = 0; c < NC; ++c) V[c] *= T[a.ttv[c * a.n_vary + k] + y];
  }
  __syncthreads();
  const double scale = ldexp(1.0, -a.n_cuts);
  double* o = out + (xt | x0);
  uint64_t x = 0;
#pragma unroll 4
  for (int f = 0; f < rows; ++f) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) acc += W[f * NC + c] * V[c];
    o[x] = acc * scale;
    x = ((x | ~mask) + 1) & mask;  // the next subset of the rows' qubits
  }
}

__global__ void __launch_bounds__(256)
    cut_tables_kernel(CutTables t, uint64_t* __restrict__ dst, int words) {
  for (int i = threadIdx.x; i < words; i += 256) dst[i] = t.w[i];
}

hipError_t launch_cut_tables(char* dst, const char* host, size_t bytes,
                             hipStream_t stream) {
  CutTables t;
  for (size_t at = 0; at < bytes; at += sizeof t) {
    const size_t part = bytes - at < sizeof t ? bytes - at : sizeof t;
    std::memcpy(t.w, host + at, part);
    cut_tables_kernel<<<1, 256, 0, stream>>>(
        t, reinterpret_cast<uint64_t*>(dst + at), int((part + 7) / 8));
  }
  return hipGetLastError();
}

template <int NC>
static void launch_cut_tile(const CutArgs& a, double* out,
                            hipStream_t stream) {
  // rows per work-group: as many as W holds, fewer while that would leave
  // less than four work-groups per CU
  int rows_log = a.n_free < kCutRowsLog ? a.n_free : kCutRowsLog;
  while (rows_log > 2 && a.n_vary_hi + a.n_free - rows_log < 10) --rows_log;
  const unsigned blocks = 1u << (a.n_vary_hi + a.n_free - rows_log);
  // All the threads form the terms where they outnumber W and its sums are long:
  // 20 qubits with NC = 16 and n_u = 1 take 20.4 us without and 23.6 with, n_u =
  // 4 23.8 and 26.8, n_u = 16 52 and 49; NC = 4 with n_u = 16 34 and 21.
  if ((NC << rows_log) <= 128 && a.n_u >= (NC > 4 ? NC : 4))
    cut_kron_tile_kernel<NC, true><<<blocks, 256, 0, stream>>>(a, a.T, out,
                                                               rows_log);
  else
    cut_kron_tile_kernel<NC, false><<<blocks, 256, 0, stream>>>(a, a.T, out,
                                                                rows_log);
}

hipError_t launch_cut(const CutArgs& a, double* out, hipStream_t stream) {
  if (a.total_entries) {
    const uint64_t blocks = (a.total_entries + 255) / 256;
    cut_terms_kernel<<<unsigned(blocks), 256, 0, stream>>>(a);
  }
  if (a.n_low) {
    if (a.n_c == 1) launch_cut_tile<1>(a, out, stream);
    else if (a.n_c == 4) launch_cut_tile<4>(a, out, stream);
    else if (a.n_c == 16) launch_cut_tile<16>(a, out, stream);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  const uint64_t nx = uint64_t(1) << a.n_qubits;
  // blocks of 64 outcomes per wave: up to 16, within the wave's LDS share
  // (nb * n_c * (n_u + 1) doubles) and the number of blocks
  int nb = 16;
  while (nb > 1 && (uint64_t(nb) * a.n_c * (a.n_u + 1) > uint64_t(kCutWaveLds) ||
                    uint64_t(nb) * 64 > nx))
    nb >>= 1;
  if (a.n_qubits >= 6 && a.n_vary <= kCutMaxVary &&
      a.n_c * (a.n_u + 1) <= uint64_t(kCutWaveLds)) {
    const uint64_t waves = nx / (64 * uint64_t(nb));
    cut_kron_wave_kernel<<<unsigned((waves + 3) / 4), 256, 0, stream>>>(
        a, a.T, out, nb);
  } else
    cut_kron_simple_kernel<<<unsigned((nx + 255) / 256), 256, 0, stream>>>(
        a, a.T, out);
  return hipGetLastError();
}

}  // namespace qsv
