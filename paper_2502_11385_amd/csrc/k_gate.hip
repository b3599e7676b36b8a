// Plain per-gate kernels: basis-state initialisation, dense k-target gates
// with controls (strided pair/quad/... updates), diagonal gates.
//
// A dense gate visits only the 2^(n-k-c) cosets whose control bits are 1:
// thread g expands g by inserting zero bits at the sorted target and control
// positions, sets the control bits, and updates the 2^k amplitudes at
// base + sum_j bit_j(r) 2^targets[j].  Consecutive threads take consecutive
// g, so for targets above the lowest few qubits both halves of every pair are
// contiguous HBM streams 2^t amplitudes apart.
#include "device_common.h"

namespace qsv {

// ---------------------------------------------------------------- init

template <typename T>
__global__ void __launch_bounds__(256)
    fill_basis_kernel(typename CxT<T>::type* __restrict__ a, uint64_t count,
                      uint64_t index) {
  using C = typename CxT<T>::type;
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
       i < count; i += stride) {
    C v;
    v.x = (i == index) ? T(1) : T(0);
    v.y = T(0);
    a[i] = v;
  }
}

hipError_t launch_fill_basis(int prec, void* amp, int n, uint64_t index,
                             hipStream_t stream) {
  const uint64_t count = uint64_t(1) << n;
  const unsigned blocks = grid_blocks(count, 256, 1u << 18);
  if (prec == 1)
    fill_basis_kernel<float><<<blocks, 256, 0, stream>>>(
        static_cast<float2*>(amp), count, index);
  else
    fill_basis_kernel<double><<<blocks, 256, 0, stream>>>(
        static_cast<double2*>(amp), count, index);
  return hipGetLastError();
}

// ---------------------------------------------------------------- dense

struct DenseArgs {
  uint64_t n_groups;
  uint64_t cmask;
  uint64_t lowmask;  // controls the lanes test themselves (LowMode)
  int32_t npos;
  int32_t pad;
  int32_t pos[40];   // sorted positions of targets and controls
  int32_t tq[8];     // targets, targets[0] = least significant matrix bit
  double m[32];      // matrix for k <= 2 (row-major, interleaved)
  const double* mptr;  // matrix for k >= 3
};

// Low fixed bits.  A pass that visits only the amplitudes whose fixed bits
// (controls, or the bits a diagonal pass needs set) are 1 walks runs of 2^p
// amplitudes, p the lowest such bit; where the runs are short every line is
// fetched anyway and each wave covers its lines in part.  For the lowest bits
// the lanes walk whole runs and test the bits themselves, and where one is 0
// they either store the amplitudes back unchanged (keep: whole lines are
// written) or leave them alone (skip).  Chosen by measurement on 30-qubit
// passes (ms, before and after):
//   keep, runs under 64 bytes: complex64 control on qubit 0, 1 or 2,
//     3.46 -> 2.81; complex64 CZ on qubit 0, 1 or 2, 1.57 -> 1.40;
//     complex128 CZ on qubit 0 or 1, 3.27 -> 2.90;
//   skip: complex64 control on qubit 3, 2.75-3.00 -> 2.47-2.90 over
//     targets 0 to 29; CZ on qubit 3 complex64, 1.21 -> 1.17; CZ on qubit 2
//     or 3 complex128, 3.00 -> 2.62 and 1.55 -> 1.42.
// Not taken: skip for a complex64 control on qubit 4 (target 29: 1.73 ->
// 1.51, but targets 0, 8, 15: 1.46-1.58 -> 1.54-1.63) or 5, 6 (likewise
// mixed), for a complex64 CZ on qubit 4 (0.77 -> 1.10), and testing higher
// bits beside keep ones (complex128 CZ on qubits 1, 2: 6.26 -> 6.53), so a
// gate with bits of both kinds has only its keep bits tested.  The
// complex128 dense kernel keeps the plain walk: neither form gained there
// (storing back made the compiler wait on each 16-byte store).
struct LowBits {
  uint64_t keep, skip;
};
constexpr LowBits kDenseLowC64 = {0x7, 0x8};
constexpr LowBits kDenseLowC128 = {0, 0};
constexpr LowBits kDiagLowC64 = {0x7, 0x8};
constexpr LowBits kDiagLowC128 = {0x3, 0xc};

// The fixed bits the lanes test: the keep bits among `fixed` if any, else
// its skip bits.
static uint64_t lane_tested(uint64_t fixed, LowBits lb) {
  return (fixed & lb.keep) ? fixed & lb.keep : fixed & lb.skip;
}

// How a dense pass treats the controls in args.lowmask: kLowNone has none;
// otherwise the lanes test them and, where one is 0, store the amplitudes
// back unchanged (kLowKeep: whole lines are written) or store nothing
// (kLowSkip).
enum LowMode { kLowNone, kLowKeep, kLowSkip };

// PTR: the matrix comes from device memory (FP64, rounded once to T while
// staged in LDS); otherwise from the kernel arguments (k <= 2).
template <typename T, int K, bool PTR, int LOW, bool NT>
__global__ void __launch_bounds__(256)
    dense_kernel(typename CxT<T>::type* __restrict__ a, DenseArgs args) {
  using C = typename CxT<T>::type;
  constexpr int D = 1 << K;
  __shared__ C smat[PTR ? D * D : 1];
  if constexpr (PTR) {
    for (int e = threadIdx.x; e < D * D; e += blockDim.x) {
      C v;
      v.x = T(args.mptr[2 * e]);
      v.y = T(args.mptr[2 * e + 1]);
      smat[e] = v;
    }
    __syncthreads();
  }
  uint64_t off[D];
#pragma unroll
  for (int r = 0; r < D; ++r) {
    uint64_t o = 0;
#pragma unroll
    for (int j = 0; j < K; ++j)
      if (r >> j & 1) o |= uint64_t(1) << args.tq[j];
    off[r] = o;
  }
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
       g < args.n_groups; g += stride) {
    uint64_t base = g;
    for (int p = 0; p < args.npos; ++p) base = insert_zero64(base, args.pos[p]);
    base |= args.cmask;
    const bool on =
        LOW == kLowNone || (base & args.lowmask) == args.lowmask;
    C v[D];
#pragma unroll
    for (int r = 0; r < D; ++r) v[r] = stream_load<NT>(a + base + off[r]);
    // All inputs are in registers, so each output can be stored at once.
#pragma unroll
    for (int r = 0; r < D; ++r) {
      T re = 0, im = 0;
#pragma unroll
      for (int s = 0; s < D; ++s) {
        T mr, mi;
        if constexpr (PTR) {
          mr = smat[r * D + s].x;
          mi = smat[r * D + s].y;
        } else {
          mr = T(args.m[2 * (r * D + s)]);
          mi = T(args.m[2 * (r * D + s) + 1]);
        }
        re += mr * v[s].x - mi * v[s].y;
        im += mr * v[s].y + mi * v[s].x;
      }
      C w;
      w.x = re;
      w.y = im;
      if constexpr (LOW == kLowKeep)
        stream_store<NT>(a + base + off[r], on ? w : v[r]);
      else if (on)
        stream_store<NT>(a + base + off[r], w);
    }
  }
}

template <typename T, int LOW, bool NT>
static void dense_dispatch_t(void* amp, int k, unsigned blocks,
                             const DenseArgs& args, hipStream_t stream) {
  using C = typename CxT<T>::type;
  C* a = static_cast<C*>(amp);
  const bool ptr = args.mptr != nullptr;
  switch (k) {
    case 1:
      if (ptr)
        dense_kernel<T, 1, true, LOW, NT><<<blocks, 256, 0, stream>>>(a, args);
      else
        dense_kernel<T, 1, false, LOW, NT><<<blocks, 256, 0, stream>>>(a, args);
      break;
    case 2:
      if (ptr)
        dense_kernel<T, 2, true, LOW, NT><<<blocks, 256, 0, stream>>>(a, args);
      else
        dense_kernel<T, 2, false, LOW, NT><<<blocks, 256, 0, stream>>>(a, args);
      break;
    case 3:
      dense_kernel<T, 3, true, LOW, NT><<<blocks, 256, 0, stream>>>(a, args);
      break;
  }
}

template <typename T, bool NT>
static void dense_dispatch_nt(void* amp, int k, unsigned blocks,
                              const DenseArgs& args, hipStream_t stream) {
  constexpr LowBits lb = sizeof(T) == 4 ? kDenseLowC64 : kDenseLowC128;
  if constexpr (lb.keep | lb.skip) {
    if (args.lowmask & lb.keep) {
      dense_dispatch_t<T, kLowKeep, NT>(amp, k, blocks, args, stream);
      return;
    }
    if (args.lowmask) {
      dense_dispatch_t<T, kLowSkip, NT>(amp, k, blocks, args, stream);
      return;
    }
  }
  dense_dispatch_t<T, kLowNone, NT>(amp, k, blocks, args, stream);
}

// Whether a pass over `bytes` of a state streams past the cache: the bytes are
// more than it holds, and a wave's accesses, in runs of 2^low amplitudes
// (`low`: the lowest bit inserted into its indexes), cover whole 128-byte
// lines.  Where they cover a line in parts, it has to stay cached between
// them: 30 qubits complex64, targets 0, 7 and 22, 4.63 ms streamed and 3.2
// cached.
// Where they do, one-target gates on 29 qubits complex64 gain 6 to 12 %, on 28
// qubits complex128 5 to 7 %.  `bytes` are those between the pass's fixed bits:
// half of a 512 MiB state stays cached from one gate to the next (26 qubits
// complex64, control on qubit 25: 66 us cached, 81 streamed).
template <typename T>
static bool streamed(uint64_t bytes, int low) {
  return bytes > kStreamBytes && (2 * sizeof(T) << low) >= 128;
}

template <typename T>
static void dense_dispatch(void* amp, int k, unsigned blocks,
                           const DenseArgs& args, hipStream_t stream) {
  // (a control 2 KiB up, above the lowest target: 28 qubits complex64, control 8,
  // target 4, 451 us cached and 468 streamed)
  constexpr int kBit2K = sizeof(T) == 4 ? 8 : 7;
  if (streamed<T>((2 * sizeof(T) * args.n_groups) << k, args.pos[0]) &&
      !((args.cmask >> kBit2K & 1) && args.pos[0] < kBit2K))
    dense_dispatch_nt<T, true>(amp, k, blocks, args, stream);
  else
    dense_dispatch_nt<T, false>(amp, k, blocks, args, stream);
}

static void sorted_positions(uint64_t mask, int32_t* pos, int32_t* npos) {
  int j = 0;
  for (int q = 0; q < 64; ++q)
    if (mask >> q & 1) pos[j++] = q;
  *npos = j;
}

hipError_t launch_dense(int prec, void* amp, int n, const HostGate& g,
                        const double* dev_matrix, hipStream_t stream) {
  // 4-5 targets run on the matrix cores (launch_fused_apply)
  if (g.k > 3) return hipErrorInvalidValue;
  DenseArgs args = {};
  args.lowmask =
      lane_tested(g.cmask, prec == 1 ? kDenseLowC64 : kDenseLowC128);
  args.cmask = g.cmask & ~args.lowmask;
  sorted_positions(g.tmask | args.cmask, args.pos, &args.npos);
  args.n_groups = uint64_t(1) << (n - args.npos);
  for (int j = 0; j < g.k; ++j) args.tq[j] = g.t[j];
  if (g.k <= 2) {
    for (size_t e = 0; e < g.m.size(); ++e) args.m[e] = g.m[e];
  } else {
    if (!dev_matrix) return hipErrorInvalidValue;
    args.mptr = dev_matrix;
  }
  const unsigned blocks = grid_blocks(args.n_groups, 256);
  if (prec == 1)
    dense_dispatch<float>(amp, g.k, blocks, args, stream);
  else
    dense_dispatch<double>(amp, g.k, blocks, args, stream);
  return hipGetLastError();
}

// Dense k-qubit matrix from device memory on qubits q (no controls); used
// for fused blocks with k <= 3.
hipError_t launch_dense_dev(int prec, void* amp, int n, int k,
                            const int32_t* q, const double* dev_matrix,
                            hipStream_t stream) {
  if (!dev_matrix || k < 1 || k > 3) return hipErrorInvalidValue;
  DenseArgs args = {};
  args.n_groups = uint64_t(1) << (n - k);
  uint64_t mask = 0;
  for (int j = 0; j < k; ++j) {
    args.tq[j] = q[j];
    mask |= uint64_t(1) << q[j];
  }
  sorted_positions(mask, args.pos, &args.npos);
  args.mptr = dev_matrix;
  const unsigned blocks = grid_blocks(args.n_groups, 256);
  if (prec == 1)
    dense_dispatch<float>(amp, k, blocks, args, stream);
  else
    dense_dispatch<double>(amp, k, blocks, args, stream);
  return hipGetLastError();
}

// ---------------------------------------------------------------- diagonal

struct DiagArgs {
  uint64_t n_items;
  uint64_t fixed_mask;  // bits forced to 1 (controls; + targets if masked)
  uint64_t lowmask;     // fixed bits the lanes test themselves
  int32_t npos;
  int32_t k;
  int32_t pos[40];      // sorted positions of the fixed bits
  int32_t tq[8];
  double d[64];         // diagonal entries (re, im); masked: d[0..1] = phase
};

// Multiply amplitudes by a diagonal's factor where the controls (fixed_mask
// and lowmask) are satisfied: by one phase (kPhase: the targets are in the
// masks as well), or by d[r(i)], r the target bits: read from LDS (kTable), or
// chosen in registers where there are one or two targets (kTable1, kTable2).
// Lanes whose lowmask bits are not all 1 store their amplitude back unchanged
// (kKeep) or leave it alone (kSkip; kSkipLine: do not load it either).
// Bound by the amplitudes' bytes: each thread has U loads in flight.
//
// A lane-dependent index into the kernel arguments was one more dependent load
// per amplitude (27 qubits complex64, one target, four loads in flight: 440 ->
// 330 us).  With one load in flight the wait for the LDS table counts: choosing
// in registers (complex64), and under a control on qubit 3, half of whose
// lines need not be read, not loading those and filling the table under the
// first loads (27 qubits, one target, control 3: index 401, LDS 432, registers
// 325 us complex64; 454, 540, 362 complex128; five targets 432, 440, 422 and
// 484, 543, 479).  The other complex128 tables stay with LDS: 695 us where
// registers take 725.
enum DiagFactor { kPhase, kTable1, kTable2, kTable };
enum DiagLow { kKeep, kSkip, kSkipLine };

template <typename T, DiagFactor F, DiagLow LOW, int U, bool NT>
__global__ void __launch_bounds__(256)
    diag_kernel(typename CxT<T>::type* __restrict__ a, DiagArgs args) {
  using C = typename CxT<T>::type;
  __shared__ C tab[F == kTable ? 1 << kMaxK : 1];
  auto entry = [&](int r) {
    C f;
    f.x = T(args.d[2 * r]);
    f.y = T(args.d[2 * r + 1]);
    return f;
  };
  auto fill = [&] {
    if (threadIdx.x < 1u << args.k) tab[threadIdx.x] = entry(threadIdx.x);
    __syncthreads();
  };
  constexpr int n_e = F == kTable2 ? 4 : F == kTable1 ? 2 : 1;
  C e[n_e];
#pragma unroll
  for (int r = 0; r < n_e; ++r) e[r] = entry(r);
  bool filled = F != kTable;
  if constexpr (LOW != kSkipLine) {
    if (!filled) fill();
    filled = true;
  }
  const uint64_t stride = uint64_t(gridDim.x) * (256 * U);
  for (uint64_t g = uint64_t(blockIdx.x) * (256 * U) + threadIdx.x;
       g < args.n_items; g += stride) {
    uint64_t i[U];
    C v[U];
    bool on[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      i[u] = g + 256 * u;
      for (int p = 0; p < args.npos; ++p)
        i[u] = insert_zero64(i[u], args.pos[p]);
      i[u] |= args.fixed_mask;
      on[u] = (i[u] & args.lowmask) == args.lowmask;
      if (LOW != kSkipLine || on[u]) v[u] = stream_load<NT>(a + i[u]);
    }
    if (!filled) {  // the work-group's threads take the same rounds
      fill();
      filled = true;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      C f = e[0];
      if constexpr (F == kTable) {
        int r = 0;
        for (int j = 0; j < args.k; ++j)
          r |= int((i[u] >> args.tq[j]) & 1) << j;
        f = tab[r];
      } else if constexpr (F != kPhase) {
        f = csel((i[u] >> args.tq[0]) & 1, e[1], f);
        if constexpr (F == kTable2)
          f = csel((i[u] >> args.tq[1]) & 1,
                   csel((i[u] >> args.tq[0]) & 1, e[3], e[2]), f);
      }
      if constexpr (LOW != kKeep) {
        if (on[u]) stream_store<NT>(a + i[u], cmul(v[u], f));
      } else {
        stream_store<NT>(a + i[u], on[u] ? cmul(v[u], f) : v[u]);
      }
    }
  }
}

hipError_t launch_diag(int prec, void* amp, int n, const HostGate& g,
                       hipStream_t stream) {
  DiagArgs args = {};
  args.k = g.k;
  for (int j = 0; j < g.k; ++j) args.tq[j] = g.t[j];
  const int d = 1 << g.k;
  if (g.masked_phase) {
    args.fixed_mask = g.tmask | g.cmask;
    args.d[0] = g.m[2 * ((d - 1) * d + (d - 1))];
    args.d[1] = g.m[2 * ((d - 1) * d + (d - 1)) + 1];
  } else {
    args.fixed_mask = g.cmask;
    for (int r = 0; r < d; ++r) {
      args.d[2 * r] = g.m[2 * (r * d + r)];
      args.d[2 * r + 1] = g.m[2 * (r * d + r) + 1];
    }
  }
  const LowBits lb = prec == 1 ? kDiagLowC64 : kDiagLowC128;
  args.lowmask = lane_tested(args.fixed_mask, lb);
  const bool skip = args.lowmask && !(args.lowmask & lb.keep);
  args.fixed_mask &= ~args.lowmask;
  sorted_positions(args.fixed_mask, args.pos, &args.npos);
  args.n_items = uint64_t(1) << (n - args.npos);
  // complex64: four amplitudes per thread once that leaves every CU a
  // work-group (n_items is a power of two, so that the chunks of 1024 are
  // full), and streamed where `streamed` says so.  complex128 gained nothing
  // from either (28 qubits, one-target table 1.44 and 1.43 ms) and lost under
  // low bits (CZ(3, 27) 0.37 -> 0.54), complex64 lost where lanes skip
  // (CZ(3, 4) on 29 qubits 0.67 -> 0.76), where the runs between the fixed
  // bits do not cover whole lines (CZ(2, 3) 1.22 -> 1.50; with lane-tested bits
  // below, runs of one line neither gained nor lost) and, beyond half of the
  // cache, where bit 8 is fixed, so that a thread's loads are 4 KiB apart and a
  // work-group's miss every other 2 KiB (phase on qubit 8 of 27, 186 us with one
  // load and 260 with four, of 24 19.8 and 18.3; qubits 7 and 9 of 27, 178 and
  // 180 with one, 166 with four): those take one.  So do phases on 2^29
  // amplitudes and more (31 qubits, CZ(4, 15) 1.40 and 1.58 ms, a phase on
  // qubit 30 2.72 and 2.85), where a thread's rounds are 2 GiB apart.
  const int low = args.npos ? args.pos[0] : n;
  const uint64_t bytes = sizeof(float2) * args.n_items;
  const bool wide = prec == 1 && !skip && low >= (args.lowmask ? 5 : 4) &&
                    !((args.fixed_mask >> 8 & 1) && bytes > kStreamBytes / 2) &&
                    !(g.masked_phase && args.n_items >= uint64_t(1) << 29) &&
                    args.n_items >= uint64_t(1) << 18;
  const bool nt = wide && streamed<float>(bytes, low);
  // (n_items a multiple of 256: whole work-groups at the table's barrier; beyond
  // 2^29 complex64 gains less from the lines left out than from full rows: one
  // target on 30 qubits 2.71 and 2.35 ms, 2.50 with the index)
  const bool skip_line =
      skip && (args.lowmask >> 3 & 1) && args.n_items >= 256 && !g.masked_phase &&
      (prec == 2 || args.n_items < uint64_t(1) << 29);
  // Several rounds, a grid of 2^20 work-groups, are worth more than one up to
  // 2^31 amplitudes where complex64 has one load in flight (phase on qubit 3 of
  // 30: 2.36 and 2.48 ms) and where a table is filled under the loads (complex128
  // with three targets, control 3, 30 qubits: 3.31 and 3.59; 3.04 with the
  // index).  The others: complex64 one-target table on 31 qubits 6.11 and 5.58,
  // complex128 phase on qubit 0 of 30 6.5 and 5.8.
  const bool rounds = (prec == 1 && !wide) || (skip_line && g.k > 2);
  const unsigned blocks = grid_blocks(args.n_items, wide ? 1024 : 256,
                                      rounds ? 1u << 20 : 1u << 23);
#define QSV_DIAG(T, F, LOW, U, NT)                                \
  diag_kernel<T, F, LOW, U, NT><<<blocks, 256, 0, stream>>>(      \
      static_cast<CxT<T>::type*>(amp), args)
#define QSV_DIAG_LINE(T)                                          \
  (g.k == 1   ? QSV_DIAG(T, kTable1, kSkipLine, 1, false)         \
   : g.k == 2 ? QSV_DIAG(T, kTable2, kSkipLine, 1, false)         \
              : QSV_DIAG(T, kTable, kSkipLine, 1, false))
#define QSV_DIAG_LOW(T, F)                                        \
  (skip ? QSV_DIAG(T, F, kSkip, 1, false) : QSV_DIAG(T, F, kKeep, 1, false))
#define QSV_DIAG_WIDE(F)                                          \
  (nt ? QSV_DIAG(float, F, kKeep, 4, true) : QSV_DIAG(float, F, kKeep, 4, false))
  if (prec == 1) {
    if (skip_line) QSV_DIAG_LINE(float);
    else if (g.masked_phase)
      wide ? QSV_DIAG_WIDE(kPhase) : QSV_DIAG_LOW(float, kPhase);
    else if (wide) QSV_DIAG_WIDE(kTable);
    else if (g.k == 1) QSV_DIAG_LOW(float, kTable1);
    else if (g.k == 2) QSV_DIAG_LOW(float, kTable2);
    else QSV_DIAG_LOW(float, kTable);
  } else {
    if (skip_line) QSV_DIAG_LINE(double);
    else if (g.masked_phase) QSV_DIAG_LOW(double, kPhase);
    else QSV_DIAG_LOW(double, kTable);
  }
#undef QSV_DIAG_WIDE
#undef QSV_DIAG_LOW
#undef QSV_DIAG_LINE
#undef QSV_DIAG
  return hipGetLastError();
}

}  // namespace qsv
