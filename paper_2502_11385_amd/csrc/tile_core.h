// Register-tile core shared by the tile-pass kernel and the batch kernel.
//
// A tile of 2^L amplitudes lives in registers, 2^RB per thread.  A register
// layout names the RB tile-local bits that select a thread's register; the
// other tile bits come from the thread index.  Every dense gate of a
// segment targets a register bit, so its 2x2 update stays in the thread;
// between segments the tile is re-laid out through LDS.
#pragma once
#include "device_common.h"

namespace qsv {

// Pair update (x0, x1) <- M (x0, x1) for a 2x2 complex M = m[0..7]
// (row-major, interleaved), in place: x0 = (a, b), x1 = (c, d).  Each
// output first sums the three terms that do not read its own input (in
// t0..t3, the four chains interleaved), then adds its own term into its own
// register.  Written as one asm block per pair so that the amplitudes stay
// in their registers through every switch arm of an op: compiled code
// computed the new values into fresh registers and copied all sixteen
// amplitudes back at the arms' join (32 moves per op, a fifth of its
// instructions).  The FP64 form's matrix is in scalar registers where it is
// uniform (SM; each instruction reads one of them, at the same rate).
#define QSV_PAIR_F32(MC)                                                      \
  asm volatile(                                                               \
      "v_mul_f32 %[t0], -%[m1], %[b]\n\t"                                     \
      "v_mul_f32 %[t1], %[m1], %[a]\n\t"                                      \
      "v_mul_f32 %[t2], %[m4], %[a]\n\t"                                      \
      "v_mul_f32 %[t3], %[m4], %[b]\n\t"                                      \
      "v_fmac_f32 %[t0], %[m2], %[c]\n\t"                                     \
      "v_fmac_f32 %[t1], %[m2], %[d]\n\t"                                     \
      "v_fma_f32 %[t2], -%[m5], %[b], %[t2]\n\t"                              \
      "v_fmac_f32 %[t3], %[m5], %[a]\n\t"                                     \
      "v_fma_f32 %[t0], -%[m3], %[d], %[t0]\n\t"                              \
      "v_fmac_f32 %[t1], %[m3], %[c]\n\t"                                     \
      "v_fma_f32 %[t2], -%[m7], %[d], %[t2]\n\t"                              \
      "v_fmac_f32 %[t3], %[m7], %[c]\n\t"                                     \
      "v_fma_f32 %[a], %[m0], %[a], %[t0]\n\t"                                \
      "v_fma_f32 %[b], %[m0], %[b], %[t1]\n\t"                                \
      "v_fma_f32 %[c], %[m6], %[c], %[t2]\n\t"                                \
      "v_fma_f32 %[d], %[m6], %[d], %[t3]"                                     \
      : [a] "+v"(x0.x), [b] "+v"(x0.y), [c] "+v"(x1.x), [d] "+v"(x1.y),     \
        [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)        \
      : [m0] MC(m0r), [m1] MC(m0i), [m2] MC(m1r), [m3] MC(m1i),             \
        [m4] MC(m2r), [m5] MC(m2i), [m6] MC(m3r), [m7] MC(m3i))
#define QSV_PAIR_F64(MC)                                                      \
  asm volatile(                                                               \
      "v_mul_f64 %[t0], -%[m1], %[b]\n\t"                                     \
      "v_mul_f64 %[t1], %[m1], %[a]\n\t"                                      \
      "v_mul_f64 %[t2], %[m4], %[a]\n\t"                                      \
      "v_mul_f64 %[t3], %[m4], %[b]\n\t"                                      \
      "v_fma_f64 %[t0], %[m2], %[c], %[t0]\n\t"                               \
      "v_fma_f64 %[t1], %[m2], %[d], %[t1]\n\t"                               \
      "v_fma_f64 %[t2], -%[m5], %[b], %[t2]\n\t"                              \
      "v_fma_f64 %[t3], %[m5], %[a], %[t3]\n\t"                               \
      "v_fma_f64 %[t0], -%[m3], %[d], %[t0]\n\t"                              \
      "v_fma_f64 %[t1], %[m3], %[c], %[t1]\n\t"                               \
      "v_fma_f64 %[t2], -%[m7], %[d], %[t2]\n\t"                              \
      "v_fma_f64 %[t3], %[m7], %[c], %[t3]\n\t"                               \
      "v_fma_f64 %[a], %[m0], %[a], %[t0]\n\t"                                \
      "v_fma_f64 %[b], %[m0], %[b], %[t1]\n\t"                                \
      "v_fma_f64 %[c], %[m6], %[c], %[t2]\n\t"                                \
      "v_fma_f64 %[d], %[m6], %[d], %[t3]"                                     \
      : [a] "+v"(x0.x), [b] "+v"(x0.y), [c] "+v"(x1.x), [d] "+v"(x1.y),     \
        [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)        \
      : [m0] MC(m0r), [m1] MC(m0i), [m2] MC(m1r), [m3] MC(m1i),             \
        [m4] MC(m2r), [m5] MC(m2i), [m6] MC(m3r), [m7] MC(m3i))
#define QSV_SREG(x) "s"(x)
#define QSV_VREG(x) "v"(x)

// A 2x2 matrix in vector registers, and an FP64 one in scalar registers
// (m as the pair update's m0r..m3i).  Every FP32 multiply and FMA, in the
// two- and the three-operand encoding, with or without a negation, issues at
// twice the rate of the same instruction reading a scalar register on this
// chip (1.0 to 1.2 ns against 1.8 to 1.9 ns a wave with six waves a SIMD),
// so complex64 ops copy their uniform matrix to vector registers once, four
// 64-bit moves.  FP64 instructions take 1.8 to 1.9 ns either way.
template <typename T>
struct VecMat {
  T m[8];
};
struct ScalarMat64 {
  double m[8];
};

#define QSV_PAIR_ARGS(v)                                                      \
  const auto m0r = v.m[0], m0i = v.m[1], m1r = v.m[2], m1i = v.m[3],          \
             m2r = v.m[4], m2i = v.m[5], m3r = v.m[6], m3i = v.m[7];          \
  decltype(x0.x) t0, t1, t2, t3
template <typename C>
__device__ __forceinline__ void pair2x2(C& x0, C& x1, const VecMat<float>& v) {
  QSV_PAIR_ARGS(v);
  QSV_PAIR_F32(QSV_VREG);
}
template <typename C>
__device__ __forceinline__ void pair2x2(C& x0, C& x1, const VecMat<double>& v) {
  QSV_PAIR_ARGS(v);
  QSV_PAIR_F64(QSV_VREG);
}
template <typename C>
__device__ __forceinline__ void pair2x2(C& x0, C& x1, const ScalarMat64& v) {
  QSV_PAIR_ARGS(v);
  QSV_PAIR_F64(QSV_SREG);
}

// A matrix as an op's fields hold it: 64-bit words in scalar registers, two
// FP32 entries (real part first) or one FP64 entry each.
template <typename T>
constexpr int kMatWords = sizeof(T);

template <typename T>
__device__ __forceinline__ T mat_entry(const uint64_t* q, int e) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(float, uint32_t(q[e >> 1] >> (32 * (e & 1))));
  else
    return __builtin_bit_cast(double, q[e]);
}

template <typename T>
__device__ __forceinline__ auto uniform_mat(const uint64_t* q) {
  if constexpr (sizeof(T) == 4) {
    VecMat<float> v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint64_t d;
      asm volatile("v_mov_b64 %0, %1" : "=v"(d) : "s"(q[e]));
      v.m[2 * e] = __builtin_bit_cast(float, uint32_t(d));
      v.m[2 * e + 1] = __builtin_bit_cast(float, uint32_t(d >> 32));
    }
    return v;
  } else {
    ScalarMat64 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v.m[e] = mat_entry<double>(q, e);
    return v;
  }
}

// The matrix of each thread: q1 where `sel`, else q0.  Both are uniform: q0
// is moved to every lane, then q1 to the selected ones, one 64-bit move a
// word each.  (A select takes at most one scalar operand, its mask, so
// compiled code moved every entry of both matrices to vector registers and
// then selected: six issues a word instead of two.)
template <typename T>
__device__ __forceinline__ VecMat<T> thread_mat(const uint64_t* q0,
                                                const uint64_t* q1, bool sel) {
  const uint64_t mask = __builtin_amdgcn_ballot_w64(sel);
  VecMat<T> v;
  uint64_t d[kMatWords<T>], all;
  if constexpr (sizeof(T) == 4) {
    asm volatile(
        "s_mov_b64 %[all], exec\n\t"
        "v_mov_b64 %[d0], %[a0]\n\t"
        "v_mov_b64 %[d1], %[a1]\n\t"
        "v_mov_b64 %[d2], %[a2]\n\t"
        "v_mov_b64 %[d3], %[a3]\n\t"
        "s_mov_b64 exec, %[mask]\n\t"
        "v_mov_b64 %[d0], %[b0]\n\t"
        "v_mov_b64 %[d1], %[b1]\n\t"
        "v_mov_b64 %[d2], %[b2]\n\t"
        "v_mov_b64 %[d3], %[b3]\n\t"
        "s_mov_b64 exec, %[all]"
        : [all] "=&s"(all), [d0] "=&v"(d[0]), [d1] "=&v"(d[1]),
          [d2] "=&v"(d[2]), [d3] "=&v"(d[3])
        : [mask] "s"(mask), [a0] "s"(q0[0]), [a1] "s"(q0[1]), [a2] "s"(q0[2]),
          [a3] "s"(q0[3]), [b0] "s"(q1[0]), [b1] "s"(q1[1]), [b2] "s"(q1[2]),
          [b3] "s"(q1[3]));
#pragma unroll
    for (int e = 0; e < 8; ++e)
      v.m[e] = __builtin_bit_cast(float, uint32_t(d[e >> 1] >> (32 * (e & 1))));
  } else {
    asm volatile(
        "s_mov_b64 %[all], exec\n\t"
        "v_mov_b64 %[d0], %[a0]\n\t"
        "v_mov_b64 %[d1], %[a1]\n\t"
        "v_mov_b64 %[d2], %[a2]\n\t"
        "v_mov_b64 %[d3], %[a3]\n\t"
        "v_mov_b64 %[d4], %[a4]\n\t"
        "v_mov_b64 %[d5], %[a5]\n\t"
        "v_mov_b64 %[d6], %[a6]\n\t"
        "v_mov_b64 %[d7], %[a7]\n\t"
        "s_mov_b64 exec, %[mask]\n\t"
        "v_mov_b64 %[d0], %[b0]\n\t"
        "v_mov_b64 %[d1], %[b1]\n\t"
        "v_mov_b64 %[d2], %[b2]\n\t"
        "v_mov_b64 %[d3], %[b3]\n\t"
        "v_mov_b64 %[d4], %[b4]\n\t"
        "v_mov_b64 %[d5], %[b5]\n\t"
        "v_mov_b64 %[d6], %[b6]\n\t"
        "v_mov_b64 %[d7], %[b7]\n\t"
        "s_mov_b64 exec, %[all]"
        : [all] "=&s"(all), [d0] "=&v"(d[0]), [d1] "=&v"(d[1]),
          [d2] "=&v"(d[2]), [d3] "=&v"(d[3]), [d4] "=&v"(d[4]),
          [d5] "=&v"(d[5]), [d6] "=&v"(d[6]), [d7] "=&v"(d[7])
        : [mask] "s"(mask), [a0] "s"(q0[0]), [a1] "s"(q0[1]), [a2] "s"(q0[2]),
          [a3] "s"(q0[3]), [a4] "s"(q0[4]), [a5] "s"(q0[5]), [a6] "s"(q0[6]),
          [a7] "s"(q0[7]), [b0] "s"(q1[0]), [b1] "s"(q1[1]), [b2] "s"(q1[2]),
          [b3] "s"(q1[3]), [b4] "s"(q1[4]), [b5] "s"(q1[5]), [b6] "s"(q1[6]),
          [b7] "s"(q1[7]));
#pragma unroll
    for (int e = 0; e < 8; ++e) v.m[e] = __builtin_bit_cast(double, d[e]);
  }
  return v;
}

// The controls of an op inside the tile: an amplitude is under all of them
// where its thread's bits and its register's are.  The registers' part is
// uniform, so that one comparison per op is made in vector registers (one
// per register kept up to eight of them beside the tile).
struct Controls {
  bool thread;         // this thread's bits
  uint32_t mask, reg;  // the mask, and its register bits

  // rt: the thread's part of the index; all: all the register bits
  __device__ __forceinline__ Controls(uint32_t lctrl, uint32_t rt,
                                      uint32_t all)
      : thread((rt & lctrl) == (lctrl & ~all)),
        mask(lctrl),
        reg(lctrl & all) {}
  // register of index offset lr
  __device__ __forceinline__ bool on(uint32_t lr) const {
    return thread && (lr & mask) == reg;
  }
};

template <int I, int R, typename C, typename M>
__device__ __forceinline__ void dense1_regs(C* a, const M& m) {
#pragma unroll
  for (int j = 0; j < R; ++j)
    if (!(j & (1 << I))) pair2x2(a[j], a[j | (1 << I)], m);
}

// The same update, applied only where every tile-local bit of lctrl is 1.
template <int I, int R, typename T, typename C>
__device__ __forceinline__ void dense1_ctrl_regs(C* a, const uint64_t* q,
                                                 const Controls& ctl,
                                                 const uint32_t* lr) {
  const auto m = uniform_mat<T>(q);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if (j & (1 << I)) continue;
    const int j1 = j | (1 << I);
    C y0 = a[j], y1 = a[j1];
    pair2x2(y0, y1, m);
    const bool on = ctl.on(lr[j]);
    a[j] = csel(on, y0, a[j]);
    a[j1] = csel(on, y1, a[j1]);
  }
}

// And with the matrix chosen per pair by tile-local bit mbit: q0 where the
// bit is 0, q1 where it is 1 (mbit differs from the target).  Every pair
// under q0 (kept where selected), then under q1: twice the FMAs of a plain
// op, but one uniform matrix at a time (selecting one per pair set the
// register peak of the whole kernel, for an op class that circuits rarely
// produce).
template <int I, int R, typename T, typename C>
__device__ __forceinline__ void dense1_mux_regs(C* a, const uint64_t* q0,
                                                const uint64_t* q1,
                                                const Controls& ctl,
                                                uint32_t rt,
                                                const uint32_t* lr, int mbit) {
  const bool tsel = ((rt >> mbit) & 1u) != 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto m = uniform_mat<T>(h ? q1 : q0);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j & (1 << I)) continue;
      const int j1 = j | (1 << I);
      const bool sel = tsel || ((lr[j] >> mbit) & 1u) != 0;
      C y0 = a[j], y1 = a[j1];
      pair2x2(y0, y1, m);
      const bool keep = ctl.on(lr[j]) && (h ? sel : !sel);
      a[j] = csel(keep, y0, a[j]);
      a[j1] = csel(keep, y1, a[j1]);
    }
  }
}

// Both by target register.
template <int R, bool MUX, typename T, typename C>
__device__ __forceinline__ void dense1_dispatch(int reg, C* a,
                                                const uint64_t* q0,
                                                const uint64_t* q1,
                                                const Controls& ctl,
                                                uint32_t rt, const uint32_t* lr,
                                                int mbit) {
#define QSV_D1(I)                                                          \
  case I:                                                                  \
    if constexpr ((1 << I) < R) {                                          \
      if constexpr (MUX)                                                   \
        dense1_mux_regs<I, R, T>(a, q0, q1, ctl, rt, lr, mbit);            \
      else                                                                 \
        dense1_ctrl_regs<I, R, T>(a, q0, ctl, lr);                         \
      break;                                                               \
    } else {                                                               \
      __builtin_unreachable();                                             \
    }
  switch (reg) {
    QSV_D1(0)
    QSV_D1(1)
    QSV_D1(2)
    QSV_D1(3)
    QSV_D1(4)
    default:
      __builtin_unreachable();  // the planner emits reg < RB only
  }
#undef QSV_D1
}

// The mux update when the mux bit is register bit K of the segment: which
// matrix a pair takes is known at compile time.  The pairs of q0, then those
// of q1, one matrix at a time.
template <int I, int K, int R, typename T, typename C>
__device__ __forceinline__ void dense1_muxreg_regs(C* a, const uint64_t* q0,
                                                   const uint64_t* q1) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto m = uniform_mat<T>(h ? q1 : q0);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j & (1 << I)) continue;
      if ((j >> K & 1) != h) continue;
      pair2x2(a[j], a[j | (1 << I)], m);
    }
  }
}

// Register layout: reg_bits[i] (ascending) is the tile-local bit selecting
// register i; the remaining bits, ascending, come from the thread index.
template <int RB>
struct Layout {
  int rb[RB];
};

template <int RB>
__device__ __forceinline__ uint32_t thread_local_base(const Layout<RB>& lay,
                                                      uint32_t tid) {
  // inserting a zero bit at p doubles the bits from p up
  uint32_t rt = tid;
#pragma unroll
  for (int i = 0; i < RB; ++i) rt += rt & (0xFFFFFFFFu << lay.rb[i]);
  return rt;
}

template <int RB>
__device__ __forceinline__ uint32_t reg_offset(const Layout<RB>& lay, int j) {
  uint32_t o = 0;
#pragma unroll
  for (int i = 0; i < RB; ++i)
    if (j >> i & 1) o |= 1u << lay.rb[i];
  return o;
}

// Work-group barrier for an exchange through LDS.  It waits for this wave's
// LDS (and scalar) accesses only, not for its outstanding global memory
// operations: a streaming tile pass keeps the next tile's prefetch and this
// tile's stores in flight across the exchanges.  The asm is also a compiler
// barrier, so no LDS access moves across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Store and load one complex amplitude at LDS byte address `at` (as a
// two-element vector of its component type).
template <typename C>
__device__ __forceinline__ void lds_store(uint32_t at, const C& v) {
  using E = decltype(v.x);
  typedef E V __attribute__((ext_vector_type(2)));
  V w;
  w.x = v.x;
  w.y = v.y;
  *(__attribute__((address_space(3))) V*)(size_t(at)) = w;
}
template <typename C>
__device__ __forceinline__ void lds_load(uint32_t at, C& v) {
  using E = decltype(v.x);
  typedef E V __attribute__((ext_vector_type(2)));
  const V w = *(const __attribute__((address_space(3))) V*)(size_t(at));
  v.x = w.x;
  v.y = w.y;
}

// LDS map of a tile's re-layouts (the host filled the register offsets of
// the same one: tile_lds_map, finalize_program).
template <typename T, bool HALVES>
constexpr LdsMap lds_map() {
  return sizeof(T) == 4 ? (HALVES ? kLds4 : kLds8) : (HALVES ? kLds8 : kLds16);
}

// Move the tile to another layout through LDS: register j of a thread goes
// to byte rf ^ sf[j], then comes from byte rt ^ st[j] (rf, rt: the thread's
// part in either layout; sf, st: the registers' parts, uniform).  The
// kernels place no other shared variable before the tile, so it starts at
// LDS address 0.  HALVES: the real parts, then the imaginary parts, each
// through a copy of the tile with one component per amplitude: half the
// LDS, so that more work-groups fit on a CU, for two more barriers and
// twice the LDS instructions.  Threads with active == false (beyond the
// tile) only join the barriers.
template <bool HALVES, int R, typename C>
__device__ __forceinline__ void relayout(C* a, const uint32_t* sf,
                                         const uint32_t* st, uint32_t rf,
                                         uint32_t rt, bool active) {
  if constexpr (!HALVES) {
    if (active) {
#pragma unroll
      for (int j = 0; j < R; ++j) lds_store(rf ^ sf[j], a[j]);
    }
    lds_barrier();
    if (active) {
#pragma unroll
      for (int j = 0; j < R; ++j) lds_load(rt ^ st[j], a[j]);
    }
    lds_barrier();
  } else {
    using E = decltype(a[0].x);
    typedef __attribute__((address_space(3))) E lds_t;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (active) {
#pragma unroll
        for (int j = 0; j < R; ++j)
          *(lds_t*)(size_t(rf ^ sf[j])) = h ? a[j].y : a[j].x;
      }
      lds_barrier();
      if (active) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const E v = *(const lds_t*)(size_t(rt ^ st[j]));
          if (h) a[j].y = v; else a[j].x = v;
        }
      }
      lds_barrier();
    }
  }
}

// e^{2 pi i t / 2^32} for a fixed-point fraction of a turn, from the
// angle's octant and a Taylor polynomial on [0, pi/4].  The top three bits
// of t give the octant o; the rest, f < 2^29, the angle inside it.  In odd
// octants the polynomial takes the complementary angle pi/4 - x (from
// 2^29 - f), so that its argument stays in [0, pi/4]; then cos and sin of
// the whole angle are those of the octant's reflection:
//   o:   0    1    2    3    4    5    6    7
//   cos  c    s   -s   -c   -c   -s    s    c
//   sin  s    c    c    s   -s   -c   -c   -s
// Truncating sin after x^9 / 9! and cos after x^10 / 10! leaves below 2e-9
// on [0, pi/4], under FP32 rounding.  Few registers: it runs while the
// whole tile is live.
__device__ __forceinline__ float2 turn_phase32(uint32_t t) {
  const uint32_t o = t >> 29;
  const uint32_t f = t & 0x1FFFFFFFu;
  const uint32_t g = (o & 1u) ? 0x20000000u - f : f;
  const float x = float(g) * (6.28318530717958648f * 0x1p-32f);
  const float x2 = x * x;
  float s = __builtin_fmaf(x2, 1.0f / 362880.0f, -1.0f / 5040.0f);
  s = __builtin_fmaf(x2, s, 1.0f / 120.0f);
  s = __builtin_fmaf(x2, s, -1.0f / 6.0f);
  s = __builtin_fmaf(x2 * x, s, x);
  float c = __builtin_fmaf(x2, -1.0f / 3628800.0f, 1.0f / 40320.0f);
  c = __builtin_fmaf(x2, c, -1.0f / 720.0f);
  c = __builtin_fmaf(x2, c, 1.0f / 24.0f);
  c = __builtin_fmaf(x2, c, -0.5f);
  c = __builtin_fmaf(x2, c, 1.0f);
  const bool swap = ((o + 1u) >> 1) & 1u;  // octants 1, 2, 5, 6
  const float cv = swap ? s : c, sv = swap ? c : s;
  const bool neg_c = ((o + 2u) >> 2) & 1u;  // octants 2..5
  const bool neg_s = (o >> 2) & 1u;         // octants 4..7
  return make_float2(neg_c ? -cv : cv, neg_s ? -sv : sv);
}

// e^{2 pi i t / 2^64} in FP64 (the int64 -> double rounding is 2^-53 of a
// half turn at most).
__device__ __forceinline__ double2 turn_phase64(uint64_t t) {
  const double y = double(int64_t(t)) * 0x1p-63;
  double sn, cs;
  sincospi(y, &sn, &cs);
  return make_double2(cs, sn);
}

// Multiply the register tile by a PhaseBlock's factor.  Per thread, each
// accumulator sums the angles of its terms whose thread and outer bits are
// all 1 (terms without thread bits are uniform over the tile); then one
// phase per accumulator multiplies the registers that carry its register
// bit, and the register table (terms on register bits only) the rest.
template <typename T, int RB>
__device__ __forceinline__ void phase_block(typename CxT<T>::type* a,
                                            const PhaseBlock* pb_gen,
                                            uint32_t rt, uint64_t base) {
  using C = typename CxT<T>::type;
  using U = typename std::conditional<sizeof(T) == 4, uint32_t, uint64_t>::type;
  constexpr int R = 1 << RB;
  const cptr<PhaseBlock> pb = as_const(pb_gen);
  cptr<PhaseTerm> t = as_const(reinterpret_cast<const PhaseTerm*>(pb_gen + 1));
  // A term's first 16 bytes (outer mask, thread mask, 32-bit turns) are
  // read as one vector, so that each term costs one scalar load round trip.
  auto head = [](cptr<PhaseTerm> p, uint64_t* gm, uint32_t* tm, U* w) {
    const u32x4 h = *(cptr<u32x4>)(p);
    *gm = uint64_t(h.x) | (uint64_t(h.y) << 32);
    *tm = h.z;
    if constexpr (sizeof(T) == 4) *w = U(h.w);
    else *w = U(p->turns);
  };
  // one accumulator at a time: only its sum and its phase are live beside
  // the tile
#pragma unroll
  for (int k = 0; k <= RB; ++k) {
    U au = 0;
    const int nu = pb->n_uni[k];
#pragma unroll 4
    for (int i = 0; i < nu; ++i, ++t) {
      uint64_t gm;
      uint32_t tm;
      U w;
      head(t, &gm, &tm, &w);
      au += (base & gm) == gm ? w : U(0);
    }
    U av = 0;
    const int nv = pb->n_thr[k];
#pragma unroll 4
    for (int i = 0; i < nv; ++i, ++t) {
      uint64_t gm;
      uint32_t tm;
      U w;
      head(t, &gm, &tm, &w);
      const bool on = ((base & gm) == gm) & ((rt & tm) == tm);
      av += on ? w : U(0);
    }
    const bool any = nu + nv > 0;
    C f;
    if (any) {
      if constexpr (sizeof(T) == 4) f = turn_phase32(au + av);
      else f = turn_phase64(au + av);
    }
    if (k > 0) {
      if (!any) continue;
#pragma unroll
      for (int j = 0; j < R; ++j)
        if (j >> (k - 1) & 1) a[j] = cmul(a[j], f);
    } else if (any && pb->has_table) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        C u;
        if constexpr (sizeof(T) == 4) u = make_float2(pb->tf[2 * j], pb->tf[2 * j + 1]);
        else u = make_double2(pb->td[2 * j], pb->td[2 * j + 1]);
        a[j] = cmul(a[j], cmul(f, u));
      }
    } else if (any) {
#pragma unroll
      for (int j = 0; j < R; ++j) a[j] = cmul(a[j], f);
    } else if (pb->has_table) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        C u;
        if constexpr (sizeof(T) == 4) u = make_float2(pb->tf[2 * j], pb->tf[2 * j + 1]);
        else u = make_double2(pb->td[2 * j], pb->td[2 * j + 1]);
        a[j] = cmul(a[j], u);
      }
    }
  }
}

// The fields of one tile op that the kernels read: its 32-byte header and
// both matrices (FP32 for complex64 states, FP64 for complex128), loaded in
// one batch of scalar loads.
template <typename T>
struct OpFields {
  int32_t code, arg;
  uint32_t lctrl;
  int32_t blob;
  uint64_t gctrl;
  int32_t dbit0, dbit1;
  uint64_t m0[kMatWords<T>], m1[kMatWords<T>];
};

template <typename T>
__device__ __forceinline__ OpFields<T> load_op(const TileOp* op) {
  OpFields<T> f;
  const cptr<u32x4> h = as_const(reinterpret_cast<const u32x4*>(op));
  const u32x4 h0 = h[0], h1 = h[1];
  f.code = int32_t(h0.x);
  f.arg = int32_t(h0.y);
  f.lctrl = h0.z;
  f.blob = int32_t(h0.w);
  f.gctrl = uint64_t(h1.x) | (uint64_t(h1.y) << 32);
  f.dbit0 = int32_t(h1.z);
  f.dbit1 = int32_t(h1.w);
  constexpr int W = kMatWords<T>;
  const cptr<u32x4> mv = as_const(reinterpret_cast<const u32x4*>(
      sizeof(T) == 4 ? static_cast<const void*>(op->mf)
                     : static_cast<const void*>(op->m)));
#pragma unroll
  for (int i = 0; i < W / 2; ++i) {
    const u32x4 u = mv[i], v = mv[W / 2 + i];
    f.m0[2 * i] = uint64_t(u.x) | (uint64_t(u.y) << 32);
    f.m0[2 * i + 1] = uint64_t(u.z) | (uint64_t(u.w) << 32);
    f.m1[2 * i] = uint64_t(v.x) | (uint64_t(v.y) << 32);
    f.m1[2 * i + 1] = uint64_t(v.z) | (uint64_t(v.w) << 32);
  }
  return f;
}

// Every field of an op is live in scalar registers from here on: without
// this the compiler sinks each load to its first use, and the op waits for
// several dependent rounds of scalar loads instead of one.
template <typename T>
__device__ __forceinline__ void pin_op_fields(OpFields<T>& f) {
  asm volatile("" : "+s"(f.code), "+s"(f.arg), "+s"(f.lctrl), "+s"(f.blob),
                    "+s"(f.gctrl), "+s"(f.dbit0), "+s"(f.dbit1));
#pragma unroll
  for (int e = 0; e < kMatWords<T>; ++e)
    asm volatile("" : "+s"(f.m0[e]), "+s"(f.m1[e]));
}

// Read one word of each 64-byte line of a pass's program that its kernel
// will use, sixteen reads in flight at a time, the waves of the work-group
// sharing the lines.  An op's fields are one batch of scalar loads that the
// op waits for; on a program just uploaded each batch missed every cache
// (about 500 ns an op where one work-group runs on a CU, more than the op's
// arithmetic), and these reads take all the misses at once, under the
// tile's own loads.  Measured (kernel time, no reads -> reads): 12 qubits,
// 144 ops in one tile 133 -> 88 us; 20 qubits, 446 ops in 13 passes
// 600 -> 478 us.  Later work-groups of a large grid find the lines cached
// and must not spend the reads again (30 qubits, every tile reading: 1.2 %
// slower; a batch reading for every tile: 3 %), so the tile kernel calls
// this from a pass's first kWarmTiles work-groups only, and the batch kernel
// once per variant that a work-group comes to (192 variants: 4.54 ->
// 4.42 ms).
constexpr uint32_t kWarmTiles = 1024;
template <typename T>
__device__ __forceinline__ void warm_program(const TilePass* pass,
                                             const TileSeg* segs,
                                             const TileOp* ops, uint32_t tid) {
  static_assert(sizeof(TileOp) == 256, "four lines per slot");
  static_assert(sizeof(TileSeg) == 160, "five half lines per segment");
  // lines of an op that load_op reads: its header and mf, mf2, or its
  // header and m, m2
  constexpr int LN = sizeof(T) == 4 ? 2 : 4;
  const cptr<TilePass> cp = as_const(pass);
  const cptr<uint32_t> p =
      as_const(reinterpret_cast<const uint32_t*>(ops + cp->op_begin));
  // the last wave reads the segments while the others read ops
  const cptr<uint32_t> ps =
      as_const(reinterpret_cast<const uint32_t*>(segs + cp->seg_begin));
  const int n_seg = (cp->nseg * int(sizeof(TileSeg)) + 63) / 64;
  const int n_op_lines = cp->n_ops * LN;
  const int n_lines = n_op_lines + cp->n_blob * 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int waves = (int(blockDim.x) + 63) >> 6;
  for (int i = (waves - 1 - wave) * 8; i < n_seg; i += waves * 8) {
    uint32_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = ps[(i + j < n_seg ? i + j : n_seg - 1) * 16];
    asm volatile("" ::"s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]),
                 "s"(v[5]), "s"(v[6]), "s"(v[7]));
  }
  for (int i = wave * 16; i < n_lines; i += waves * 16) {
    uint32_t v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int l = i + j < n_lines ? i + j : n_lines - 1;
      const int line = l < n_op_lines
                           ? (l / LN) * 4 + l % LN
                           : cp->n_ops * 4 + (l - n_op_lines);
      v[j] = p[line * 16];
    }
    asm volatile("" ::"s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]),
                 "s"(v[5]), "s"(v[6]), "s"(v[7]), "s"(v[8]), "s"(v[9]),
                 "s"(v[10]), "s"(v[11]), "s"(v[12]), "s"(v[13]), "s"(v[14]),
                 "s"(v[15]));
  }
}

// The registers' LDS offsets of a layout, scalar loads issued together.
template <int RB>
__device__ __forceinline__ void load_lds_offsets(const uint32_t* p,
                                                 uint32_t* so) {
  if constexpr (RB <= 4) {
    const cptr<u32x4> v = as_const(reinterpret_cast<const u32x4*>(p));
#pragma unroll
    for (int i = 0; i < (1 << RB) / 4; ++i) {
      const u32x4 u = v[i];
      so[4 * i] = u.x;
      so[4 * i + 1] = u.y;
      so[4 * i + 2] = u.z;
      so[4 * i + 3] = u.w;
    }
  } else {
    // 32 offsets per layout do not fit the scalar registers beside an op's
    // fields: those of the register bits, and their combinations
    const cptr<uint32_t> v = as_const(p);
    so[0] = 0;
#pragma unroll
    for (int i = 0; i < RB; ++i) so[1 << i] = v[1 << i];
#pragma unroll
    for (int j = 1; j < (1 << RB); ++j)
      so[j] = so[j & (j - 1)] ^ so[j & -j];
  }
}

// One hot op: kCodeUniform, kCodeRegMux or kCodeThreadMux on target register
// bit I (mux register bit K).  f holds its fields and leaves with the next
// op's.  These are read while the op computes, once its own matrix has left
// f; a register mux, whose two matrices stay live, reads them afterwards.
// Tried instead, both no faster where few work-groups run and slower where
// many do: a second set of fields for every class, copied over afterwards
// (24 moves an op), or with the loop unrolled over the two sets (twice the
// code: 24 qubits 2.10 against 1.95 ms).
template <int CLS, int I, int K, int RB, typename T, typename C>
__device__ __forceinline__ void hot_op(C* a, OpFields<T>& f, uint64_t base,
                                       uint32_t rt, const TileOp* next) {
  constexpr int R = 1 << RB, W = kMatWords<T>;
  // the barriers keep the compiler from moving the loads below the update,
  // and their first use above its end
  if constexpr (CLS == kCodeUniform) {
    // one matrix for the whole tile, chosen by one bit of its base index (an
    // outer mux qubit, or bit 63, which no index has); the choice is made on
    // the bit patterns, so it stays scalar
    const bool second = ((base >> (f.arg & 63)) & 1) != 0;
    uint64_t q[W];
#pragma unroll
    for (int e = 0; e < W; ++e) {
      q[e] = second ? f.m1[e] : f.m0[e];
      asm volatile("" : "+s"(q[e]));
    }
    const auto m = uniform_mat<T>(q);
    f = load_op<T>(next);
    __builtin_amdgcn_sched_barrier(0);
    dense1_regs<I, R>(a, m);
    __builtin_amdgcn_sched_barrier(0);
  } else if constexpr (CLS == kCodeThreadMux) {
    // mux bit in the thread index: one matrix per thread
    const VecMat<T> m =
        thread_mat<T>(f.m0, f.m1, ((rt >> f.arg) & 1u) != 0);
    f = load_op<T>(next);
    __builtin_amdgcn_sched_barrier(0);
    dense1_regs<I, R>(a, m);
    __builtin_amdgcn_sched_barrier(0);
  } else {
    __builtin_amdgcn_sched_barrier(0);
    dense1_muxreg_regs<I, K, R, T>(a, f.m0, f.m1);
    __builtin_amdgcn_sched_barrier(0);
    f = load_op<T>(next);
  }
  pin_op_fields(f);
}

// The hot op whose code f holds (op.code < kCodeCtrl << 6).
template <int RB, typename T, typename C>
__device__ __forceinline__ void hot_dispatch(C* a, OpFields<T>& f,
                                             uint64_t base, uint32_t rt,
                                             const TileOp* next) {
#define QSV_HOT(CLS, I, K)                                                \
  case (CLS << 6) | (K << 3) | I:                                         \
    if constexpr (I < RB && K < RB && (CLS != kCodeRegMux || I != K)) {   \
      hot_op<CLS, I, K, RB, T>(a, f, base, rt, next);                     \
      break;                                                              \
    } else {                                                              \
      __builtin_unreachable(); /* the planner emits reg bits below RB */  \
    }
#define QSV_HOT_K(I)                                                      \
  QSV_HOT(kCodeRegMux, I, 0) QSV_HOT(kCodeRegMux, I, 1)                   \
  QSV_HOT(kCodeRegMux, I, 2) QSV_HOT(kCodeRegMux, I, 3)                   \
  QSV_HOT(kCodeRegMux, I, 4)
#define QSV_HOT_I(CLS)                                                    \
  QSV_HOT(CLS, 0, 0) QSV_HOT(CLS, 1, 0) QSV_HOT(CLS, 2, 0)                \
  QSV_HOT(CLS, 3, 0) QSV_HOT(CLS, 4, 0)
  switch (f.code) {
    QSV_HOT_I(kCodeUniform)
    QSV_HOT_I(kCodeThreadMux)
    QSV_HOT_K(0)
    QSV_HOT_K(1)
    QSV_HOT_K(2)
    QSV_HOT_K(3)
    QSV_HOT_K(4)
    default:
      __builtin_unreachable();
  }
#undef QSV_HOT
#undef QSV_HOT_K
#undef QSV_HOT_I
}

// Apply every segment of one tile pass to the register tile `a`, which is
// in the I/O layout on entry and is left in the I/O layout on exit.  `base`
// is the tile's global index with all tile bits zero (outer controls and
// diagonal bits outside the tile are read from it).
//
// Where few work-groups run (small states), each wave's own chain of
// latencies bounds the pass: the scalar loads of an op, the branches to its
// code, the address arithmetic of a re-layout.  So an op's fields are read
// while the op before it computes, the hot ops are reached through one
// switch on the planner's code, and a re-layout takes its LDS offsets from
// the segment record. 
template <typename T, int RB, bool HALVES>
__device__ __forceinline__ void tile_apply(typename CxT<T>::type* a,
                                           const TilePass* pass,
                                           const TileSeg* segs,
                                           const TileOp* ops, uint64_t base,
                                           uint32_t tid, bool active) {
  using C = typename CxT<T>::type;
  constexpr int R = 1 << RB;
  constexpr LdsMap kMap = lds_map<T, HALVES>();
  const cptr<TilePass> cp = as_const(pass);
  const int nseg = cp->nseg;
  const TileSeg* sg = segs + cp->seg_begin;
  const uint32_t* lds_from = pass->lds;
  // thread tid's part of a tile index in the current layout (the I/O layout
  // takes the low bits)
  uint32_t rt = tid;
  uint32_t at = lds_place(kMap, tid);  // its place in LDS
  int o = cp->op_begin;
  OpFields<T> f = load_op<T>(ops + o);
  pin_op_fields(f);
  for (int s = 0; s < nseg; ++s, ++sg) {
    const cptr<u32x4> head = as_const(reinterpret_cast<const u32x4*>(sg));
    const u32x4 h0 = head[0], h1 = head[1];
    uint32_t sf[R], st[R];
    load_lds_offsets<RB>(lds_from, sf);
    load_lds_offsets<RB>(sg->lds, st);
    const int32_t bits[5] = {int32_t(h0.x), int32_t(h0.y), int32_t(h0.z),
                             int32_t(h0.w), int32_t(h1.x)};
    const int o_end = int32_t(h1.w);
    Layout<RB> lay;
#pragma unroll
    for (int i = 0; i < RB; ++i) lay.rb[i] = bits[i];
    const uint32_t to = thread_local_base(lay, tid);
    if (h1.y) {
      const uint32_t at_to = lds_place(kMap, to);
      relayout<HALVES, R>(a, sf, st, at, at_to, active);
      at = at_to;
    }
    rt = to;
    lds_from = sg->lds;
    while (o < o_end) {
      const TileOp* op = ops + o;
      if (f.code < (kCodeCtrl << 6)) {
        hot_dispatch<RB, T>(a, f, base, rt, op + 1);
        ++o;
        continue;
      }
      // controlled, phase and diagonal ops
      const int cls = f.code >> 6;
      if ((base & f.gctrl) == f.gctrl) {  // else an outer control is 0
      const int reg = f.code & 7;
      uint32_t lr[R];
#pragma unroll
      for (int j = 0; j < R; ++j) lr[j] = reg_offset(lay, j);
      const Controls ctl(f.lctrl, rt, lr[R - 1]);
      if (cls == kCodeCtrl) {
        const bool second = ((base >> (f.arg & 63)) & 1) != 0;
        uint64_t q[kMatWords<T>];
#pragma unroll
        for (int e = 0; e < kMatWords<T>; ++e) {
          q[e] = second ? f.m1[e] : f.m0[e];
          asm volatile("" : "+s"(q[e]));
        }
        dense1_dispatch<R, false, T>(reg, a, q, nullptr, ctl, rt, lr, 0);
      } else if (cls == kCodeCtrlMux) {
        dense1_dispatch<R, true, T>(reg, a, f.m0, f.m1, ctl, rt, lr, f.arg);
      } else if (cls == kCodePhaseBlock) {
        phase_block<T, RB>(
            a,
            reinterpret_cast<const PhaseBlock*>(
                reinterpret_cast<const char*>(op) + f.blob),
            rt, base);
      } else if (cls == kCodePhase) {
        C ph;
        ph.x = mat_entry<T>(f.m0, 0);
        ph.y = mat_entry<T>(f.m0, 1);
        if constexpr (sizeof(T) == 4)  // see VecMat
          asm volatile("" : "+v"(ph.x), "+v"(ph.y));
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const bool on = ctl.on(lr[j]);
          const C y = cmul(a[j], ph);
          a[j] = csel(on, y, a[j]);
        }
      } else {  // kCodeDiag
        const int dk = f.arg;
        const int d0 = f.dbit0, d1 = f.dbit1;
        const uint32_t g0 =
            d0 < 0 ? uint32_t((base >> ((-1 - d0) & 63)) & 1) : 0u;
        const uint32_t g1 =
            (dk > 1 && d1 < 0) ? uint32_t((base >> ((-1 - d1) & 63)) & 1) : 0u;
        C t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          t[e].x = mat_entry<T>(f.m0, 2 * e);
          t[e].y = mat_entry<T>(f.m0, 2 * e + 1);
        }
        // thread parts of the two index bits, once per op
        const bool t0 = d0 >= 0 ? ((rt >> (d0 & 31)) & 1u) != 0 : g0 != 0;
        const bool t1 =
            dk > 1 && (d1 >= 0 ? ((rt >> (d1 & 31)) & 1u) != 0 : g1 != 0);
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const bool b0 = t0 || (d0 >= 0 && ((lr[j] >> (d0 & 31)) & 1u) != 0);
          const bool b1 =
              t1 || (dk > 1 && d1 >= 0 && ((lr[j] >> (d1 & 31)) & 1u) != 0);
          const C f01 = csel(b0, t[1], t[0]);
          const C f23 = csel(b0, t[3], t[2]);
          const C fv = csel(b1, f23, f01);
          const bool on = ctl.on(lr[j]);
          const C y = cmul(a[j], fv);
          a[j] = csel(on, y, a[j]);
        }
      }
      }
      ++o;
      f = load_op<T>(ops + o);
      pin_op_fields(f);
    }
  }
  if (cp->moved) {
    uint32_t sf[R], st[R];
    load_lds_offsets<RB>(lds_from, sf);
    load_lds_offsets<RB>(pass->lds, st);
    relayout<HALVES, R>(a, sf, st, at, lds_place(kMap, tid), active);
  }
}

// Tile index -> global index of the tile's first amplitude: the index's
// bits spread over the non-tile qubits, run by run (four cover every tile
// of up to four groups of consecutive qubits, so that the usual tile needs
// one batch of loads).
__device__ __forceinline__ uint64_t tile_base(const TilePass* pass,
                                              uint32_t tile) {
  const cptr<TilePass> cp = as_const(pass);
  uint64_t base = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)  // unused runs have mask 0
    base |= uint64_t(tile & cp->out_mask[i]) << cp->out_shift[i];
  for (int i = 4; i < cp->n_out; ++i)
    base |= uint64_t(tile & cp->out_mask[i]) << cp->out_shift[i];
  return base;
}

template <typename C>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void* p) {
  // stride 0 (raw), the full 32-bit byte range, gfx9 word-3 layout with a
  // 32-bit data format; offsets used here stay below 2^31
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), short(0),
                                           int(0xffffffffu), 0x00020000);
}

// Element index of a thread's part of the I/O layout (its tile-local
// thread bits spread over the tile qubits).
template <int RB>
__device__ __forceinline__ uint32_t io_thread_index(const TilePass* pass,
                                                    uint32_t tid) {
  const int W = pass->L - RB;
  uint32_t o = 0;
  for (int b = 0; b < W; ++b)
    if (tid >> b & 1) o |= 1u << pass->q[b];
  return o;
}

// Raw buffer loads and stores at a 32-bit byte offset and a uniform one from
// a uniform buffer resource (no per-access address arithmetic).
__device__ __forceinline__ float2 load_at(const float2*,
                                          __amdgpu_buffer_rsrc_t r,
                                          uint32_t boff, uint32_t soff) {
  return __builtin_bit_cast(
      float2, __builtin_amdgcn_raw_buffer_load_b64(r, boff, soff, 0));
}
__device__ __forceinline__ double2 load_at(const double2*,
                                           __amdgpu_buffer_rsrc_t r,
                                           uint32_t boff, uint32_t soff) {
  return __builtin_bit_cast(
      double2, __builtin_amdgcn_raw_buffer_load_b128(r, boff, soff, 0));
}
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t r,
                                         uint32_t boff, uint32_t soff,
                                         float2 v) {
  using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, boff,
                                        soff, 0);
}
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t r,
                                         uint32_t boff, uint32_t soff,
                                         float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r,
                                        boff, soff, 0);
}
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t r,
                                         uint32_t boff, uint32_t soff,
                                         double v) {
  using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, boff,
                                        soff, 0);
}
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t r,
                                         uint32_t boff, uint32_t soff,
                                         double2 v) {
  using V = decltype(__builtin_amdgcn_raw_buffer_load_b128(r, 0, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(V, v), r, boff,
                                         soff, 0);
}

}  // namespace qsv
