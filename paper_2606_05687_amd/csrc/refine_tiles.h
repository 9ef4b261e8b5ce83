// Building blocks of the FP64 refinement kernels (refine.hip: two contacts,
// refine_wide.hip: four): hand-offs and reductions within a wave, 16 x 16 tiles
// on the FP64 matrix cores, the elimination of 12-input systems, products of
// horizon chains, and range-checked access to the stage arrays.
#pragma once

#include "pinmpc_internal.h"

namespace pinmpc {

namespace {

constexpr int W64 = 64;

// Pointers with their address space spelled out: the context lives in LDS,
// so the compiler cannot infer where its pointers point, and generic (flat)
// accesses would make every wait on one load a wait on all memory in flight.
#define GMEM __attribute__((address_space(1)))
#define LMEM __attribute__((address_space(3)))
typedef const GMEM float* gcf;
typedef const GMEM double* gcd;
typedef GMEM double* gd;

// A phase of the refinement runs in one 64-lane wave.  LDS operations of a
// wave execute in issue order, so handing data between the lanes of the wave
// through LDS needs only a point the compiler does not move memory accesses
// across (wsync).  gsync is used where one phase's global outputs feed the next
// phase, not inside the stage loops.
__device__ inline void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// Global memory written by one lane and read by another: the fence at workgroup
// scope.  It orders the accesses; it does not wait for the stores, nor need it to: the
// waves of a workgroup share a CU, whose vector memory path and L1 take their accesses
// in the order of issue.  No barrier: where a problem's workgroup holds several waves
// (a pair's second wave, one per chunk of the associative scan), the others join the
// first only at the recursion's own meetings, after which they read what it stored.
__device__ inline void gsync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
}
// A condition that is the same in every lane, for a scalar branch.
__device__ inline bool scalar(bool c) { return __builtin_amdgcn_readfirstlane((int)c) != 0; }
// lane within the wave (the workgroup may hold several waves)
__device__ inline int lane_id() { return (int)(threadIdx.x & 63); }
// The lane in a register of its own.  What a phase derives from it (offsets,
// masks) stays with the phase: found equal to another phase's and kept in
// registers across the whole kernel it is spilled, and its reload between the
// loads of a stage waits for them.
__device__ inline int fresh_lane() {
  int l = lane_id();
  asm volatile("" : "+v"(l));
  return l;
}

// Reductions over the wave without LDS: the DPP permutations (quads, half rows,
// rows) and the row and half-wave swaps, every lane ending with the result.
// A step through ds_bpermute instead waits for an LDS round trip.
template <int CTRL>
__device__ inline uint32_t dpp32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ inline double dpp64(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(double, ((uint64_t)dpp32<CTRL>((uint32_t)(b >> 32)) << 32) |
                                        dpp32<CTRL>((uint32_t)b));
}
// a and b become the two operands of a reduction across 16-lane rows
// (HALF: across the wave's halves).
template <bool HALF>
__device__ inline void swap_rows(uint32_t v, uint32_t& a, uint32_t& b) {
  if constexpr (HALF) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    a = r[0];
    b = r[1];
  }
}
template <bool HALF>
__device__ inline void swap_rows(double v, double& a, double& b) {
  const uint64_t w = __builtin_bit_cast(uint64_t, v);
  uint32_t al, bl, ah, bh;
  swap_rows<HALF>((uint32_t)w, al, bl);
  swap_rows<HALF>((uint32_t)(w >> 32), ah, bh);
  a = __builtin_bit_cast(double, ((uint64_t)ah << 32) | al);
  b = __builtin_bit_cast(double, ((uint64_t)bh << 32) | bl);
}
template <class F>
__device__ inline double wave_reduce(double v, F op) {
  v = op(v, dpp64<0xB1>(v));    // quad_perm 1 0 3 2
  v = op(v, dpp64<0x4E>(v));    // quad_perm 2 3 0 1
  v = op(v, dpp64<0x141>(v));   // row_half_mirror
  v = op(v, dpp64<0x140>(v));   // row_mirror
  double a, b;
  swap_rows<false>(v, a, b);
  v = op(a, b);
  swap_rows<true>(v, a, b);
  return op(a, b);
}
// v, or infinity if it is not a number: fmax drops a NaN, and a residual of NaNs
// would pass for zero.
__device__ inline double no_nan(double v) { return v == v ? v : __builtin_inf(); }
__device__ inline double wave_max(double v) {
  return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}
__device__ inline double wave_min(double v) {
  return wave_reduce(v, [](double a, double b) { return fmin(a, b); });
}
__device__ inline double wave_sum(double v) {
  return wave_reduce(v, [](double a, double b) { return a + b; });
}
template <class F>
__device__ inline uint32_t wave_reduce32(uint32_t v, F op) {
  v = op(v, dpp32<0xB1>(v));
  v = op(v, dpp32<0x4E>(v));
  v = op(v, dpp32<0x141>(v));
  v = op(v, dpp32<0x140>(v));
  uint32_t a, b;
  swap_rows<false>(v, a, b);
  v = op(a, b);
  swap_rows<true>(v, a, b);
  return op(a, b);
}
__device__ inline int wave_max_int(int v) {
  return (int)wave_reduce32((uint32_t)v, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
__device__ inline uint64_t wave_xor(uint64_t v) {
  const auto x = [](uint32_t a, uint32_t b) { return a ^ b; };
  return ((uint64_t)wave_reduce32((uint32_t)(v >> 32), x) << 32) | wave_reduce32((uint32_t)v, x);
}

// ------------------------------------------------------------ 16 x 16 tiles
//
// The stage recursion works on 16 x 16 FP64 tiles (13 states, 12 inputs, zero
// padded) held in registers in the result layout of the FP64 matrix-core
// product (16 x 16 x 4 per instruction): lane l = 16 g + j holds items
// q = 0..3, item q being entry (4 q + g, j).  The same layout is the right
// operand of the product chunk by chunk, and read as the left operand it is
// the transposed tile.  So for tiles U, V in registers mmT(U, V) = U^T V takes
// four instructions and leaves a tile again: products chain with no data
// movement.  Vectors ride in column VC of a tile (lanes 13, 29, 45, 61).

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int VC = 13;

__device__ inline d4 zero4() {
  d4 z = {0.0, 0.0, 0.0, 0.0};
  return z;
}
__device__ inline int tg() { return lane_id() >> 4; }
__device__ inline int tj() { return lane_id() & 15; }

// U^T V + acc, contracting over the first 4 NQ rows (NQ = 3: the input rows).
template <int NQ>
__device__ inline d4 mmT(d4 u, d4 v, d4 acc) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(u[q], v[q], acc, 0, 0, 0);
  return acc;
}

__device__ inline d4 sel(bool c, d4 a) { return c ? a : zero4(); }

typedef unsigned int u2 __attribute__((ext_vector_type(2)));

typedef double d2 __attribute__((ext_vector_type(2)));

// One contact's block: m the 3 x 3 force block, d the moment diagonals, v the
// vector.
struct InputBlock {
  double m[3][3], d[3], v[6];
};
__device__ inline void store_block(gd base, const InputBlock& t) {
  GMEM d2* p = (GMEM d2*)base;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    p[2 * a] = d2{t.m[a][0], t.m[a][1]};
    p[2 * a + 1] = d2{t.m[a][2], t.v[a]};
    p[6 + a] = d2{t.d[a], t.v[3 + a]};
  }
}

// Raw stage data.  The stage loops fetch the next stage's data a whole stage
// ahead.  All stage arrays are read and written through buffer instructions:
// each lane's offset within a stage is fixed for the whole loop, the stage is a
// scalar offset, and an entry that a tile does not hold has an offset past the
// end, so it reads as zero (and its store is dropped) without masks or branches.
__device__ inline int clampi(int v, int hi) { return v < hi ? v : hi; }
__device__ inline void pin(const d4& t) {
  asm volatile("" ::"v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]));
}
__device__ inline void pin(double t) { asm volatile("" ::"v"(t)); }
__device__ inline void pin_memory() { asm volatile("" ::: "memory"); }
// A pointer read from the LDS context, made wave-uniform (scalar registers):
// the stage loops then neither re-read the context after their LDS stores
// nor hold its pointers in vector registers.
template <class T>
__device__ inline T uni(T p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (T)(((uint64_t)hi << 32) | lo);
}

__device__ inline double uni(double d) {
  const uint64_t v = __builtin_bit_cast(uint64_t, d);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

typedef unsigned int u3 __attribute__((ext_vector_type(3)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
constexpr int OOB = 0x40000000;   // an offset past the end of every array
template <class P>
__device__ inline __amdgpu_buffer_rsrc_t rsrc(P base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
}
__device__ inline float ldf(__amdgpu_buffer_rsrc_t r, int off, int soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
__device__ inline double ldd(__amdgpu_buffer_rsrc_t r, int off, int soff) {
  const u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0);
  double v;
  __builtin_memcpy(&v, &w, 8);
  return v;
}
__device__ inline void ldf3(__amdgpu_buffer_rsrc_t r, int off, int soff, float v[3]) {
  const u3 w = __builtin_amdgcn_raw_buffer_load_b96(r, off, soff, 0);
  __builtin_memcpy(v, &w, 12);
}
__device__ inline void ldf4(__amdgpu_buffer_rsrc_t r, int off, int soff, float v[4]) {
  const u4 w = __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0);
  __builtin_memcpy(v, &w, 16);
}
__device__ inline void ldd2(__amdgpu_buffer_rsrc_t r, int off, int soff, double v[2]) {
  const u4 w = __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0);
  __builtin_memcpy(v, &w, 16);
}
__device__ inline void std1(__amdgpu_buffer_rsrc_t r, int off, int soff, double v) {
  u2 w;
  __builtin_memcpy(&w, &v, 8);
  __builtin_amdgcn_raw_buffer_store_b64(w, r, off, soff, 0);
}
__device__ inline void std2(__amdgpu_buffer_rsrc_t r, int off, int soff, double a, double b) {
  u4 w;
  __builtin_memcpy(&w, &a, 8);
  __builtin_memcpy((char*)&w + 8, &b, 8);
  __builtin_amdgcn_raw_buffer_store_b128(w, r, off, soff, 0);
}

// Byte offset of tile entry (r, c) in an input block T, or OOB.
__device__ inline int t_offset(int r, int c) {
  const int i = r / 6, a = r % 6, b = c % 6;
  int o = -1;
  if (r < NU && c < NU && c / 6 == i) {
    if (a < 3 && b < 3) o = 4 * a + b;
    else if (a >= 3 && a == b) o = 12 + 2 * (a - 3);
  } else if (r < NU && c == VC) {
    o = a < 3 ? 4 * a + 3 : 13 + 2 * (a - 3);
  }
  return o < 0 ? OOB : (i * 18 + o) * 8;
}

// Weights that make a homogeneous tile exactly symmetric from itself and its
// transpose: the average on the 13 x 13 block, column VC as it is, row VC its
// transpose, zero elsewhere.
struct SymWeights {
  d4 own, other;
};
__device__ inline SymWeights sym_weights(int lane = lane_id()) {
  SymWeights w;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * q + (lane >> 4), c = lane & 15;
    w.own[q] = (r < NX && c < NX) ? 0.5 : ((c == VC && r < NX) ? 1.0 : 0.0);
    w.other[q] = (r < NX && c < NX) ? 0.5 : ((r == VC && c < NX) ? 1.0 : 0.0);
  }
  return w;
}
// S so symmetrised (its rounding is not symmetric, and an asymmetric part is
// carried back through the open-loop A and grows along the horizon).
__device__ inline d4 symmetrize(d4 S, const SymWeights& w, double* buf, int lane = lane_id()) {
  const int g = lane >> 4, j = lane & 15;
#pragma unroll
  for (int q = 0; q < 4; ++q) buf[(4 * q + g) * 17 + j] = S[q];
  wsync();
#pragma unroll
  for (int q = 0; q < 4; ++q) S[q] = fma(w.other[q], buf[j * 17 + 4 * q + g], w.own[q] * S[q]);
  wsync();
  return S;
}

// c[r] += (c[r] of lane P of this 16-lane row) * s for r in [LO, HI), the
// leading wait states as in fmac_row_bcast12.
template <int P, int LO, int HI>
__device__ inline void fmac_rows(double (&c)[12], double s) {
  if constexpr (LO < HI) asm volatile("s_nop 1");
#pragma unroll
  for (int r = LO; r < HI; ++r)
    asm volatile(
        "v_fmac_f64_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "+v"(c[r])
        : "v"(s), "i"(P));
  // the next pivot is broadcast from row P + 1: no closer than two wait states
  if constexpr (LO == P + 1 && HI - LO <= 2) asm volatile("s_nop 1");
}

// The same with the system's factors kept: forward elimination only
// (H = U^T D U, U unit upper), lane c < 12 ending with column c of U above
// 1 / d_c; the right-hand sides hold D^-1 U^-T b.
template <int p = 0>
__device__ inline void factor(double (&col)[12], int hc, uint32_t unit) {
  if constexpr (p < 12) {
    if (!((unit >> p) & 1u)) {
      const double rd = recip(row_bcast<p>(col[p]));
      const double t = col[p] * rd;
      fmac_rows<p, p + 1, 12>(col, -t);
      col[p] = hc == p ? rd : t;
    }
    factor<p + 1>(col, hc, unit);
  }
}
// ... and back substitution of the right-hand sides by U (the factor's lanes
// take a zero factor and keep their entries).
template <int p = 11>
__device__ inline void back_substitute(double (&col)[12], bool is_h, uint32_t unit) {
  if constexpr (p > 0) {
    if (!((unit >> p) & 1u)) fmac_rows<p, 0, p>(col, is_h ? 0.0 : -col[p]);
    back_substitute<p - 1>(col, is_h, unit);
  }
}

// Row g's lanes turned by 3 g: lane i takes lane i + 3 g of its row.
__device__ inline double turn_rows(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  uint32_t w[2] = {(uint32_t)b, (uint32_t)(b >> 32)};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int x = (int)w[h];
    int r = __builtin_amdgcn_update_dpp(x, x, 0x103, 0x2, 0xF, false);   // row_shl:3, row 1
    r = __builtin_amdgcn_update_dpp(r, x, 0x106, 0x4, 0xF, false);       // row_shl:6, row 2
    r = __builtin_amdgcn_update_dpp(r, x, 0x109, 0x8, 0xF, false);       // row_shl:9, row 3
    w[h] = (uint32_t)r;
  }
  return __builtin_bit_cast(double, ((uint64_t)w[1] << 32) | w[0]);
}
// s + sum_q (turned vector's lane q of the row) * m[q], q = 0..3 (0..2).  The
// leading wait states separate the DPP reads from the vector write of t.
__device__ inline double dot4(double t, const double (&m)[4], double s) {
  asm volatile("s_nop 1\n"
               "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               : "+v"(s)
               : "v"(t), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]));
  return s;
}
__device__ inline double dot3(double t, const double (&m)[3], double s) {
  asm volatile("s_nop 1\n"
               "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               : "+v"(s)
               : "v"(t), "v"(m[0]), "v"(m[1]), "v"(m[2]));
  return s;
}
// The four rows' partial sums, added in every lane.
__device__ inline double row_total(double s) {
  double a, b;
  swap_rows<false>(s, a, b);
  s = a + b;
  swap_rows<true>(s, a, b);
  return a + b;
}
// s + sum_r (v of lane r of this 16-lane row) * a[r], r = 0..12, over four
// interleaved accumulators: the DPP row broadcast of v rides in each fused
// multiply-add.  The leading two wait states separate the block's DPP reads
// of v from a vector write of v just before it.
__device__ inline double dot_row_bcast13(double v, const double (&a)[13], double s) {
  double s1 = 0.0, s2 = 0.0, s3 = 0.0;
#define PINMPC_DOT(acc, r, ai) \
  "v_fmac_f64_dpp %" #acc ", %4, %" #ai " row_newbcast:" #r " row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
  asm volatile("s_nop 1\n"
               PINMPC_DOT(0, 0, 5) PINMPC_DOT(1, 1, 6) PINMPC_DOT(2, 2, 7) PINMPC_DOT(3, 3, 8)
               PINMPC_DOT(0, 4, 9) PINMPC_DOT(1, 5, 10) PINMPC_DOT(2, 6, 11) PINMPC_DOT(3, 7, 12)
               PINMPC_DOT(0, 8, 13) PINMPC_DOT(1, 9, 14) PINMPC_DOT(2, 10, 15)
               PINMPC_DOT(3, 11, 16) PINMPC_DOT(0, 12, 17)
               : "+v"(s), "+v"(s1), "+v"(s2), "+v"(s3)
               : "v"(v), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]),
                 "v"(a[6]), "v"(a[7]), "v"(a[8]), "v"(a[9]), "v"(a[10]), "v"(a[11]),
                 "v"(a[12]));
#undef PINMPC_DOT
  return (s + s1) + (s2 + s3);
}

// Whether any of `count` floats is not finite (this lane's share).  Eight loads
// are in flight at a time: one at a time, each iteration waits for memory.
__device__ inline int any_nonfinite(gcf v, int count) {
  int nf = 0;
  for (int e0 = lane_id(); e0 < count; e0 += 8 * W64) {
    float x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = e0 + t * W64;
      x[t] = v[e < count ? e : e0];
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) nf |= !isfinite(x[t]);
  }
  return nf;
}

}  // namespace

}  // namespace pinmpc
