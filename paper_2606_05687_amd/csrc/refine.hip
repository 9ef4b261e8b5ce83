// FP64 refinement and certification of the ADMM result, one workgroup per problem:
// one 64-lane wave, two for the recursions (Waves::PAIR), or one per chunk of the
// horizon (Waves::SCAN).
//
// The ADMM of Sec. III reaches the QP optimum only in the limit; its last
// projection fixes a guess of the active faces of every contact's wrench set.
// From that guess the kernel runs, all in FP64:
//  A. active-set passes: solve the equality-constrained LQ problem with each
//     contact's input restricted to the affine hull of its face (Riccati
//     recursion over the horizon with u_k = c_k + P_k w_k), evaluate the KKT
//     residuals with costates from the adjoint recursion and row multipliers
//     from the face, and update the faces by the primal-dual active-set rule
//     (row active iff mu_i s_i + (G_i u - h_i) > 0); stop when certified, when
//     the face set repeats, or after refine_passes passes;
//  B. if not certified: a primal-dual interior point with Mehrotra's
//     predictor-corrector on the same QP (each Newton step a Riccati recursion
//     with input Hessian R + G^T diag(z/s) G), then faces from z > s and
//  C. active-set passes again from those faces (polish_passes).
// The returned u is the last equality-constrained solution, x its rollout in
// FP64, and res the normalised residuals (r_dyn, r_ineq, r_stat, r_comp,
// r_sign) of that point.
#include "refine_tiles.h"

namespace pinmpc {

namespace {

// Every function is part of its kernel: with a call, a recursion that takes all
// 256 registers saves and restores up to a hundred of the caller's through scratch
// memory (about a tenth of an equality pass at full occupancy).
#define INLINE __attribute__((always_inline)) inline

// One problem's view: its inputs and its FP64 scratch block, all as
// pointers to the problem's own first stage, so stage k is plain k.
struct Scalars {
  double mu, fz, tm, mg;
  double i1, i2;          // 1 / (1 + mu^2), 1 / (1 + 2 mu^2): the pyramid's Gram inverses
  double img, itm;        // 1 / mg, 1 / tm: the interior point's row scales
};
struct Ctx : Scalars {
  int b, N, n;
  const LMEM double* Q;   // LDS copies of the diagonal weights
  const LMEM double* R;
  gcf A, B, e, x_ref, u_ref, x0;
  const GMEM uint8_t* contact;
  gd rT, rT2, rK, rF, rS;    // per-stage compact blocks (TS_T, TS_K, ... doubles)
  gd rM;   // closed loops of a Newton step, over T2 and the padding
  gd ru, rx, rq, rs, rz, rds, rdz, rrc, rdu, rdx;
  gd rPV, rGV;   // long horizons: the stage buffers of the rollout and costates
  GMEM int32_t* faces;
};

// ------------------------------------------------------------ small helpers

// A copy of the scalars in scalar registers.
__device__ inline Scalars scalars(const Ctx& C) {
  return {uni(C.mu), uni(C.fz), uni(C.tm), uni(C.mg), uni(C.i1), uni(C.i2), uni(C.img), uni(C.itm)};
}

// The 11 rows of one stance contact's wrench constraints G (f, tau) <= h: the
// pyramid's sides f_x - mu f_z, -f_x - mu f_z, f_y - mu f_z, -f_y - mu f_z <= 0,
// f_z <= fz_max, then tau_a <= tau_max and -tau_a <= tau_max.  The products skip
// G's zeros (a dense row is six multiply-adds, and the compiler keeps those with
// a zero).  G u:
__device__ inline void rows_of(const Scalars& C, const double u[6], double gu[NROW]) {
  gu[0] = fma(-C.mu, u[2], u[0]);
  gu[1] = fma(-C.mu, u[2], -u[0]);
  gu[2] = fma(-C.mu, u[2], u[1]);
  gu[3] = fma(-C.mu, u[2], -u[1]);
  gu[4] = u[2];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    gu[5 + a] = u[3 + a];
    gu[8 + a] = -u[3 + a];
  }
}
// o + G^T v
__device__ inline void rows_T(const Scalars& C, const double v[NROW], double o[6]) {
  o[0] += v[0] - v[1];
  o[1] += v[2] - v[3];
  o[2] += fma(-C.mu, (v[0] + v[1]) + (v[2] + v[3]), v[4]);
#pragma unroll
  for (int a = 0; a < 3; ++a) o[3 + a] += v[5 + a] - v[8 + a];
}
// h_r, the row's scale and the interior point's inverse scale (r a constant)
__device__ inline double row_h(const Scalars& C, int r) { return r < 4 ? 0.0 : (r == 4 ? C.fz : C.tm); }
__device__ inline double row_scale(const Scalars& C, int r) { return r < 5 ? C.mg : C.tm; }
__device__ inline double row_isc(const Scalars& C, int r) { return r < 5 ? C.img : C.itm; }
// face bit of row r
__device__ inline int row_bit(int r) { return r < 5 ? (1 << r) : (1 << (8 + (r - 5))); }

__device__ inline bool face_apex(int code) {
  const int f = code & 31;
  return ((f & 3) == 3) || ((f & 12) == 12);
}

// The face of a set of active rows: all of an apex's force rows, and only the
// upper of two opposite moment rows.
__device__ inline int settle_face(int code) {
  if (face_apex(code)) code = (code & ~31) | FACE_APEX;
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if ((code >> (8 + a) & 1) && (code >> (11 + a) & 1)) code &= ~(1 << (11 + a));
  return code;
}

// The force part of a face that is not the apex: the active side rows along x
// and y (sign of the row, 0 if neither is active; both of a pair would be the
// apex) and whether the normal-force bound is active.
struct ForceFace {
  double sx, sy;
  bool top;
};
__device__ inline ForceFace force_face(int code) {
  ForceFace f;
  f.sx = (code & 1) ? 1.0 : ((code & 2) ? -1.0 : 0.0);
  f.sy = (code & 4) ? 1.0 : ((code & 8) ? -1.0 : 0.0);
  f.top = (code >> 4) & 1;
  return f;
}

// Affine hull of a contact's face: projector P (6x6, block diagonal) and a
// point c with u = c + P w spanning the face,
//   P = I - G_A^T (G_A G_A^T)^{-1} G_A,   c = G_A^T (G_A G_A^T)^{-1} h_A
// for the force block with active rows A.  Its eight cases in closed form
// (the side rows are [s_x, 0, -mu], [0, s_y, -mu]): at the normal-force bound
// f_z and every component with an active side row are fixed; otherwise one
// side row leaves its plane, two the line along [s_x mu, s_y mu, 1].
__device__ inline void face_affine(int code, const Scalars& C, double P[6][6], double c[6]) {
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    c[a] = 0.0;
#pragma unroll
    for (int b = 0; b < 6; ++b) P[a][b] = 0.0;
  }
  if (!face_apex(code)) {
    const ForceFace f = force_face(code);
    const double mu = C.mu;
    if (f.top) {
      c[0] = f.sx * mu * C.fz;
      c[1] = f.sy * mu * C.fz;
      c[2] = C.fz;
      P[0][0] = f.sx == 0.0 ? 1.0 : 0.0;
      P[1][1] = f.sy == 0.0 ? 1.0 : 0.0;
    } else {
      const bool two = f.sx != 0.0 && f.sy != 0.0, any = f.sx != 0.0 || f.sy != 0.0;
      const double d[3] = {two ? f.sx * mu : f.sx, two ? f.sy * mu : f.sy, two ? 1.0 : -mu};
      const double w = two ? C.i2 : (any ? -C.i1 : 0.0);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) P[a][b] = w * (d[a] * d[b]) + ((a == b && !two) ? 1.0 : 0.0);
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (code >> (8 + a) & 1) c[3 + a] = C.tm;
    else if (code >> (11 + a) & 1) c[3 + a] = -C.tm;
    else P[3 + a][3 + a] = 1.0;
  }
}

// ------------------------------------------------- a contact-stage's data
//
// The passes over the rows run one lane per contact-stage.  With a few waves per
// SIMD each trip to memory costs 2000 to 4000 cycles and the arithmetic of a pass
// about as much, so a pass loads all it needs at once, before any branch on it
// (a load under `if (u_ref)` or `if (contact)` is one more trip: six of them,
// one per component of u_ref, made a pass over 20 stages 30 to 50 thousand
// cycles), through buffer instructions: scalar bases, one offset per lane.

typedef __amdgpu_buffer_rsrc_t Buf;
// inputs of contact-stage e (6 of 12 per stage: 48 bytes each)
__device__ inline void ld6(Buf r, int e, double v[6]) {
#pragma unroll
  for (int t = 0; t < 6; t += 2) ldd2(r, e * 48 + t * 8, 0, v + t);
}
__device__ inline void st6(Buf r, int e, const double v[6]) {
#pragma unroll
  for (int t = 0; t < 6; t += 2) std2(r, e * 48 + t * 8, 0, v[t], v[t + 1]);
}
// the reference inputs (an empty buffer where there are none: zeros)
__device__ inline Buf uref_buf(const Ctx& C) {
  const gcf p = uni(C.u_ref);
  return rsrc(p ? p : uni(C.A), p ? C.N * NU * 4 : 0);
}
__device__ inline void ldu6(Buf r, int e, float v[6]) {
  ldf3(r, e * 24, 0, v);
  ldf3(r, e * 24 + 12, 0, v + 3);
}
// A row's entries for consecutive contact-stages e are consecutive in memory,
// `step` bytes apart per row: the lanes of a pass load and store whole lines.
__device__ inline Buf row_buf(const Ctx& C, gd p) { return rsrc(uni(p), 2 * C.n * NROW * 8); }
__device__ inline void load_r(Buf r, int step, int e, double x[NROW]) {
#pragma unroll
  for (int q = 0; q < NROW; ++q) x[q] = ldd(r, e * 8, q * step);
}
__device__ inline void store_r(Buf r, int step, int e, const double x[NROW]) {
#pragma unroll
  for (int q = 0; q < NROW; ++q) std1(r, e * 8, q * step, x[q]);
}
template <int M, class T>
__device__ inline void pin_all(const T (&v)[M]) {
#pragma unroll
  for (int t = 0; t < M; ++t) asm volatile("" ::"v"(v[t]));
}
__device__ inline void copy_doubles(gd dst, gd src, int count) {
  const Buf r = rsrc(uni(src), count * 8);
  for (int e0 = fresh_lane(); e0 < count; e0 += 8 * W64) {
    double v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = ldd(r, (e0 + t * W64) * 8, 0);
    pin_memory();
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (e0 + t * W64 < count) dst[e0 + t * W64] = v[t];
  }
}

// --------------------------------------------------------------- LDS state

// Hand-off buffers of the stage recursion; everything else of a stage lives
// in registers as 16 x 16 tiles.
constexpr int GC = 14;            // column stride of the elimination's hand-off
struct ShR {
  // [H | Hwx | hw | 0] of the stage by column, 12 + 16 columns: a lane moves its
  // column as 16-byte pairs, and the stride spreads both that and the tile
  // accesses over all banks
  alignas(16) double G[(NU + 16) * GC];
  double ST[16 * 17];             // a tile for its transpose
  // the right-hand sides by column between the two triangular solves (Z; the last
  // column takes what the lanes of H write), or H^{-1} by column (chunk summaries)
  alignas(16) double Z[17 * GC];
};
struct Sh {
  // the Riccati recursion's hand-off buffers and the stage vectors of the
  // rollout and the costates share storage: they are never in use together
  union {
    struct {
      ShR r;
      alignas(16) double G1[(NU + 16) * GC];   // a pair's second system (odd stages)
    } p;
    struct {
      double PV[PINMPC_NMAX * 16];   // x_{k+1}, Q (x_{k+1} - r_k), p_{k+1}
      double GV[PINMPC_NMAX * 16];   // u_k, R (u_k - u_ref_k), g_k
    } c;
  };
  double Qd[NX], Rd[NU]; // diagonal weights of the problem
  // inputs of each contact-stage whose pivot is a unit vector (see build_eq)
  uint8_t unit[2 * PINMPC_NMAX_LONG];
};

// The per-stage 16-wide vectors of the rollout and the costate chain: in LDS
// up to PINMPC_NMAX stages; for longer horizons (LONG) in the problem's scratch
// block, where a hand-off between lanes needs the barrier with its memory fence
// instead of the wave's LDS ordering.
template <bool LONG>
struct StageBufs;
template <>
struct StageBufs<false> {
  double* PV;
  double* GV;
  __device__ StageBufs(Sh& sh, const Ctx&) : PV(sh.c.PV), GV(sh.c.GV) {}
};
template <>
struct StageBufs<true> {
  gd PV;
  gd GV;
  __device__ StageBufs(Sh&, const Ctx& C) : PV(C.rPV), GV(C.rGV) {}
};
template <bool LONG>
__device__ inline void bufsync() {
  if constexpr (LONG) gsync();
  else wsync();
}

// Stage blocks in memory hold only the entries a tile can have nonzero (the
// layouts are listed with refine_block_doubles).  For the value function a map packs, for each of a
// lane's four tile items, the item's offset in the block (in doubles, 8 bits
// per item) or 255 for an item the block does not hold.  Blocks are read and
// written with buffer instructions whose range is the block: an item mapped
// to 255 lies past the end (255 doubles exceed every block), so its load
// returns zero and its store is dropped by the hardware's range check.  A
// fetch issued a stage ahead thus needs no masking and stores need no
// branches.
constexpr uint32_t NOT_HELD = 255;
static_assert(TS_S < 255, "the block must end before the out-of-range offset");
__device__ inline uint32_t pack_map(const int o[4]) {
  uint32_t m = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) m |= (uint32_t)o[q] << (8 * q);
  return m;
}
// value function: S symmetric (13 x 13, lower triangle) and s; `store` selects
// the lower triangle and column VC, a load fills both triangles, column VC and
// row VC
__device__ inline uint32_t map_S(bool store) {
  const int lane = fresh_lane();
  int o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * q + (lane >> 4), c = lane & 15;
    const int hi = r > c ? r : c, lo = r > c ? c : r;
    const bool sym = r < NX && c < NX && (!store || c <= r);
    const bool vec = hi == VC && lo < NX && (!store || c == VC);
    o[q] = sym ? hi * (hi + 1) / 2 + lo : (vec ? NX * (NX + 1) / 2 + lo : (int)NOT_HELD);
  }
  return pack_map(o);
}
// buffer resource over one stage block of `doubles` entries (raw buffer:
// stride 0, 32-bit data format, range checked against the block's bytes)
__device__ inline __amdgpu_buffer_rsrc_t block_rsrc(gcd base, int doubles) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, doubles * 8, 0x00020000);
}
// Item q's byte offset, kept in a vector register: an offset the compiler
// could prove constant would otherwise move into the instruction's immediate
// field, and the range check is meant to see every offset the same way.
__device__ inline int map_offset(uint32_t map, int q) {
  int off = (int)(((map >> (8 * q)) & 255) * 8);
  asm volatile("" : "+v"(off));
  return off;
}
// (Element values move through memcpy: a bit cast applied directly to a
// vector element has been seen to read element 0 for every element.)
__device__ inline d4 ld_map(gcd base, int doubles, uint32_t map) {
  const __amdgpu_buffer_rsrc_t r = block_rsrc(base, doubles);
  d4 t;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, map_offset(map, q), 0, 0);
    double v;
    __builtin_memcpy(&v, &w, 8);
    t[q] = v;
  }
  return t;
}
__device__ inline void st_map(gd base, int doubles, uint32_t map, d4 t) {
  const __amdgpu_buffer_rsrc_t r = block_rsrc(base, doubles);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double v = t[q];
    u2 w;
    __builtin_memcpy(&w, &v, 8);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, map_offset(map, q), 0, 0);
  }
}

// ------------------------------------------------------------ stage inputs
//
// Written in parallel over (stage, contact) before a recursion: each lane forms
// its contact's force block, moment diagonals and vector in registers and stores
// them whole (18 doubles, as 16-byte pairs).

enum class Mode { EQ, NEWTON };

// Inputs of a stage that the projector removes exactly (a zero column): every
// input of a swing contact; on an equality pass also the force of an apex face,
// the components that the normal-force bound fixes and each moment at its bound.
// For those, the stage system [H | Hwx | hw] has exactly e_j as row and column j,
// and its elimination skips them (bitwise the same result).  One byte per
// contact-stage, in LDS.
__device__ inline uint32_t unit_bits(int code) {
  uint32_t m = 0;
  if ((code & 31) == FACE_APEX) m = 7;
  else if (code & 16) m = 4u | ((code & 3) ? 1u : 0u) | ((code & 12) ? 2u : 0u);
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if (((code >> (8 + a)) & 1) || ((code >> (11 + a)) & 1)) m |= 8u << a;
  return m;
}

// Equality passes, stages 0..kn-1: T the face projector P and point c of each
// contact, T2 the terms P R P + I - P and P R (c - u_ref) of the stage's
// quadratic that need no value function.
__device__ inline void build_eq(const Ctx& C, const double* Rd, uint8_t* unit, int kn) {
  const Scalars sc = scalars(C);
  const Buf rR = uref_buf(C);
  const auto ct = uni(C.contact);
  const auto fc = uni(C.faces);
  const gd pT = uni(C.rT), pT2 = uni(C.rT2);
  for (int e = fresh_lane(); e < kn * 2; e += W64) {
    const int i = e & 1;
    float ur[6];
    const int code = fc[e];
    const bool on = ct[e];
    ldu6(rR, e, ur);
    pin_all(ur);
    pin_memory();
    InputBlock t, t2;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      t.d[a] = 0.0;
      t2.d[a] = 1.0;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        t.m[a][b] = 0.0;
        t2.m[a][b] = a == b ? 1.0 : 0.0;
      }
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) t.v[a] = t2.v[a] = 0.0;
    uint32_t u = 0x3F;
    if (on) {
      u = unit_bits(code);
      double P[6][6], c[6], R[6], rho[6];
      face_affine(code, sc, P, c);
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        R[a] = Rd[6 * i + a];
        rho[a] = R[a] * (c[a] - (double)ur[a]);
        t.v[a] = c[a];
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        double v = 0.0;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          t.m[a][b] = P[a][b];
          double x = (a == b ? 1.0 : 0.0) - P[a][b];
#pragma unroll
          for (int l = 0; l < 3; ++l) x += P[a][l] * R[l] * P[l][b];
          t2.m[a][b] = x;
          v += P[a][b] * rho[b];
        }
        t2.v[a] = v;
        const double p = P[3 + a][3 + a];
        t.d[a] = p;
        t2.d[a] = p * R[3 + a] * p + 1.0 - p;
        t2.v[3 + a] = p * rho[3 + a];
      }
    }
    unit[e] = (uint8_t)u;
    store_block(pT + (size_t)e * 18, t);
    store_block(pT2 + (size_t)e * 18, t2);
  }
}

// Newton steps: the input block of stance contact-stage e at (u, s, z), the
// input Hessian R + G^T diag(z/s) G and the linear term R (u - u_ref) +
// G^T c_rows at the affine target s z (rows scaled by sc: weight z / (s sc^2),
// coefficient (z + (-s z + z rp) / s) / sc = z rp / (s sc), rp = (g u - h) / sc
// + s).
__device__ inline void newton_block(const Scalars& C, const double* R, gd T, int e,
                                    const double u[6], const float ur[6], const double sv[NROW],
                                    const double zv[NROW]) {
  double gu[NROW], d[NROW], c[NROW];
  InputBlock t;
  rows_of(C, u, gu);
#pragma unroll
  for (int r = 0; r < NROW; ++r) {
    const double isc = row_isc(C, r);
    const double rp = fma(gu[r] - row_h(C, r), isc, sv[r]), zs = zv[r] * recip(sv[r]);
    d[r] = zs * (isc * isc);
    c[r] = zs * rp * isc;
  }
#pragma unroll
  for (int a = 0; a < 6; ++a) t.v[a] = R[a] * (u[a] - (double)ur[a]);
  rows_T(C, c, t.v);
  t.m[0][0] = R[0] + (d[0] + d[1]);
  t.m[1][1] = R[1] + (d[2] + d[3]);
  t.m[2][2] = R[2] + fma(C.mu * C.mu, (d[0] + d[1]) + (d[2] + d[3]), d[4]);
  t.m[0][1] = t.m[1][0] = 0.0;
  t.m[0][2] = t.m[2][0] = -C.mu * (d[0] - d[1]);
  t.m[1][2] = t.m[2][1] = -C.mu * (d[2] - d[3]);
#pragma unroll
  for (int a = 0; a < 3; ++a) t.d[a] = R[3 + a] + (d[5 + a] + d[8 + a]);
  store_block(T + (size_t)e * 18, t);
}

// The stage inputs of a recursion over stages 0..kn-1, visible to every lane
// (a Newton step's are written by the interior point as it moves its iterate).
template <Mode mode>
__device__ inline void build(const Ctx& C, Sh& sh, int kn) {
  gsync();
  if constexpr (mode == Mode::EQ) {
    build_eq(C, sh.Rd, sh.unit, kn);
    gsync();
  }
}

// ------------------------------------------------------ Riccati recursion
//
// Solves   min sum_k 1/2 x_{k+1}^T Q x_{k+1} + q_k^T x_{k+1}
//                    + 1/2 u_k^T R'_k u_k + rho_k^T u_k
//          s.t. x_{k+1} = A_k x_k + B_k u_k + e_k,  u_k = c_k + P_k w_k
// (P_k an orthogonal projector) by the backward recursion on the value
// function V(x) = 1/2 x^T S x + s^T x and the forward rollout.
//   EQ:     the equality-constrained tracking problem of the faces
//           (q = -Q r, rho = -R u_ref, R' = R, e from the data);
//   NEWTON: the interior-point Newton step, x_0 = 0, e = 0,
//           q = Q (x_{k+1} - r), R' = R + G^T diag(z/s) G, P the stance mask,
//           c = 0.
// Per stage, with W = S + Q, Bp = B P and d = B c + e:
//   H = P R' P + Bp^T W Bp + (I - P),  Hwx = Bp^T W A,
//   hw = P (R' c + rho) + Bp^T (W d + q + s),
//   K = -H^{-1} Hwx, kap = -H^{-1} hw,
//   S <- A^T W A + Hwx^T K,  s <- A^T (W d + q + s) + Hwx^T kap.
// EQ keeps each stage's value function [S_k | s_k] (symmetrised, as used);
// stage k's factors depend on the faces of stages k..N-1 only, so a pass
// whose faces differ from the previous pass's only before stage ktop
// rebuilds the inputs and reruns the backward recursion for stages
// 0..ktop-1 only, starting from the kept [S_ktop | s_ktop]; the result is
// bitwise that of the whole recursion.
//
// The tiles are homogeneous: row and column VC carry the linear terms, so that
// the matrix products carry the vectors along.  With
//   Wt = [[W, q + s], [(q + s)^T, 0]]   and   D1 = [Bp | 0 | d], 1 at (VC, VC)
// D3 = Wt^T D1 holds W Bp, in row VC Bp^T (q + s) and in column VC W d + q + s;
// then D3^T D1 + T2 = [H | 0 | hw] with nothing left to add.  With [A | d] in the
// same form (1 at (VC, VC)) D2 = Wt^T [A | d] holds W A and, in column VC, W d + q
// + s; D1^T D2 is Hwx and A^T D2 the value function without the gains' part.
// FP64 vector instructions and FP64 matrix instructions do not overlap on this
// chip (a group of one matrix product of 64 cycles and 12 multiply-adds takes
// 134 cycles in one wave), so a stage costs the sum of both and is made of as
// few of either as possible: 26 (NEWTON: 23) matrix instructions.

template <Mode mode>
struct BackRaw;
template <>
struct BackRaw<Mode::EQ> {
  float a[4], b[3], xr[4], ev[4];
  double T[3], T2[3];
};
template <>
struct BackRaw<Mode::NEWTON> {
  float a[4], b[4], bt[3];
  double q[4], T[3];
};

// Gauss-Jordan elimination without pivoting of a 12-row system whose leading
// 12 x 12 block sits in lanes 0..11 of every 16-lane row (column c in lane c of
// each row, the rows identical) and whose right-hand sides occupy the other
// lanes.  Bit p of the wave-uniform `unit` marks a pivot whose row and column are
// exactly the unit vector e_p: its step changes nothing and is skipped.
template <int p = 0>
__device__ inline void eliminate(double (&col)[12], uint32_t unit) {
  if constexpr (p < 12) {
    if (!((unit >> p) & 1u)) {
      const double t = col[p] * recip(row_bcast<p>(col[p]));
      fmac_rows<p, 0, p>(col, -t);
      fmac_rows<p, p + 1, 12>(col, -t);
      col[p] = t;
    }
    eliminate<p + 1>(col, unit);
  }
}
// Newton steps, which keep the factors of H for the corrector: forward elimination
// only (lanes as above; see `factor` for the factors).  z (LDS) takes the right-hand
// sides between the two triangular solves, z = U^-T b, and col D^-1 z: the value
// function needs only these two, Hwx^T H^-1 Hwx = z^T D^-1 z, and the back
// substitution to [K | kap] = U^-1 D^-1 z follows beside it.
template <int p = 0>
__device__ inline void forward_eliminate(double (&col)[12], double* z, int hc, uint32_t unit) {
  if constexpr (p < 12) {
    z[p] = col[p];
    if (!((unit >> p) & 1u)) {
      const double rd = recip(row_bcast<p>(col[p]));
      const double t = col[p] * rd;
      fmac_rows<p, p + 1, 12>(col, -t);
      col[p] = hc == p ? rd : t;
    }
    forward_eliminate<p + 1>(col, z, hc, unit);
  }
}
// Backward recursion over stages k_hi - 1 down to k_lo from the value
// function Ss of x_{k_hi} (S in rows and columns 0..12, s in row and column
// VC); returns the value function of x_{k_lo}.  It stores each stage's gains
// and feedforward (and, for equality passes, its value function; for Newton
// steps the factors of H).
// ELEM: the chunk summary of the associative scan instead (see below): the
// recursion starts from a zero value at x_{k_hi}, stores nothing and also
// composes the closed-loop affine map TE (transposed, offset in row 13,
// (13, 13) = 1) and the reachability term CE of the chunk.
template <Mode mode, bool ELEM>
__device__ INLINE d4 backward(const Ctx& C, ShR& sr,
                                                             const uint8_t* unit, int k_lo,
                                                             int k_hi, d4 Ss, d4* TEo, d4* CEo) {
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  constexpr bool newton = (mode == Mode::NEWTON);
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const gcf pe = uni(C.e), pA = uni(C.A);
  const auto rA = rsrc(pA, N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * NU * 4);
  const auto rX = rsrc(uni(C.x_ref), N * NX * 4);
  const auto rE = rsrc(pe ? pe : pA, pe ? N * NX * 4 : 0);
  const auto rQ = rsrc(uni(C.rq), N * NX * 8);
  const auto rT = rsrc(uni(C.rT), N * TS_T * 8), rT2 = rsrc(uni(C.rT2), N * TS_T * 8);
  const auto rK = rsrc(uni(C.rK), N * TS_K * 8), rF = rsrc(uni(C.rF), N * TS_F * 8);
  const gd prS = uni(C.rS);
  const auto rM = rsrc(uni(C.rM), N * TS_M * 8);
  // this lane's offsets within a stage: rows 4q + g of A and B^T (EQ) or B,
  // of column VC (and, as item 3 of group 1, row VC) of the vectors, of T, K, F
  const int oA = j < NX ? (g * NX + j) * 4 : OOB;
  const int oA3 = (g == 0 && j < NX) ? (12 * NX + j) * 4 : OOB;
  const int oBt = j < NX ? (j * NU + g) * 4 : OOB;
  const int oB = newton ? (j < NU ? (g * NU + j) * 4 : OOB) : oBt;
  const int oB3 = (newton && g == 0 && j < NU) ? (12 * NU + j) * 4 : OOB;
  const int oV = j == VC ? g : OOB / 8;
  const int oV3 = (g == 0 && j == VC) ? 12 : ((g == 1 && j < NX) ? j : OOB / 8);
  const int oE3 = (g == 0 && j == VC) ? 48 : OOB;
  int oT[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) oT[q] = t_offset(4 * q + g, j);
  const int oK = j <= VC ? (g * (NX + 1) + j) * 8 : OOB;
  const int oF = j < NU ? (g * NU + j) * 8 : OOB;
  const int oM = j <= VC ? (g * (NX + 1) + j) * 8 : OOB;
  const int oM3 = (g == 0 && j <= VC) ? (12 * (NX + 1) + j) * 8 : OOB;
  const uint32_t mS = map_S(true);
  // Q on the diagonal, and where q = -Q r lies (column and row VC)
  d4 Qd, Qv;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * q + g;
    Qd[q] = (r == j && j < NX) ? C.Q[clampi(j, NX - 1)] : 0.0;
    Qv[q] = (j == VC && r < NX) ? C.Q[clampi(r, NX - 1)]
                                : ((r == VC && j < NX) ? C.Q[clampi(j, NX - 1)] : 0.0);
  }
  const SymWeights sw = sym_weights(lane);
  const double one = (g == 1 && j == VC) ? 1.0 : 0.0;   // (VC, VC) as item 3
  auto fetch = [&](int k, BackRaw<mode>& s) {
#pragma unroll
    for (int q = 0; q < 3; ++q) s.a[q] = ldf(rA, oA + q * 4 * NX * 4, k * (NX * NX * 4));
    s.a[3] = ldf(rA, oA3, k * (NX * NX * 4));
#pragma unroll
    for (int q = 0; q < 3; ++q)
      s.b[q] = ldf(rB, oB + q * (newton ? 4 * NU * 4 : 16), k * (NX * NU * 4));
    if constexpr (newton) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
        if constexpr (!ELEM) s.bt[q] = ldf(rB, oBt + q * 16, k * (NX * NU * 4));
      s.b[3] = ldf(rB, oB3, k * (NX * NU * 4));
#pragma unroll
      for (int q = 0; q < 3; ++q) s.q[q] = ldd(rQ, oV * 8 + q * 32, k * (NX * 8));
      s.q[3] = ldd(rQ, oV3 * 8, k * (NX * 8));
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        s.xr[q] = ldf(rX, oV * 4 + q * 16, k * (NX * 4));
        s.ev[q] = ldf(rE, oV * 4 + q * 16, k * (NX * 4));
        s.T2[q] = ldd(rT2, oT[q], k * (TS_T * 8));
      }
      s.xr[3] = ldf(rX, oV3 * 4, k * (NX * 4));
      s.ev[3] = ldf(rE, oE3, k * (NX * 4));
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) s.T[q] = ldd(rT, oT[q], k * (TS_T * 8));
  };

  BackRaw<mode> raw;
  fetch(k_hi > k_lo ? k_hi - 1 : k_lo, raw);
  d4 TE = zero4(), CE = zero4();
  if constexpr (ELEM) {
#pragma unroll
    for (int q = 0; q < 4; ++q) TE[q] = (4 * q + g == j && j <= VC) ? 1.0 : 0.0;
  }
  for (int k = k_hi - 1; k >= k_lo; --k) {
    // this stage's data
    d4 At, D1, Wt, H0 = zero4();   // H0: the part of [H | hw] without W
    d4 Bt = zero4();               // B^T
#pragma unroll
    for (int q = 0; q < 4; ++q) At[q] = (double)raw.a[q];
    uint32_t ub;
    {
      const uint32_t u0 = unit[2 * k], u1 = unit[2 * k + 1];
      ub = (uint32_t)__builtin_amdgcn_readfirstlane((int)(u0 | (u1 << 6)));
    }
    if constexpr (newton) {
      // B with the swing contacts' columns zero
      const bool keep = j < NU && !((ub >> j) & 1u);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        D1[q] = keep ? (double)raw.b[q] : 0.0;
        Wt[q] = Ss[q] + (Qd[q] + raw.q[q]);
      }
      D1[3] += one;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        H0[q] = raw.T[q];
        if constexpr (!ELEM) Bt[q] = (double)raw.bt[q];
      }
      pin(Bt);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        D1[q] = (double)raw.ev[q];
        Wt[q] = Ss[q] + fma(-Qv[q], (double)raw.xr[q], Qd[q]);
      }
      D1[3] += one;
      // [B P | 0 | B c + e]
#pragma unroll
      for (int q = 0; q < 3; ++q)
        D1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)raw.b[q], raw.T[q], D1, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 3; ++q) H0[q] = raw.T2[q];
    }
    if constexpr (ELEM) {
      if (k == k_hi - 1) Wt = zero4();   // a zero value at x_{k_hi}
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) At[q] = j == VC ? D1[q] : At[q];   // [A | d], 1 at (VC, VC)
    pin(At); pin(D1); pin(Wt); pin(H0);
    pin_memory();
    if (k > k_lo) fetch(k - 1, raw);

    const d4 D3 = mmT<4>(Wt, D1, zero4());   // [W Bp | 0 | W d + q + s], row VC Bp^T (q + s)
    // H0 added once: where R dominates, each product added to it would round u
    const d4 D4 = mmT<4>(D3, D1, zero4()) + H0;   // [H | 0 | hw]
    const d4 D2 = mmT<4>(Wt, At, zero4());   // [W A | W d + q + s]
    const d4 D5 = mmT<4>(D1, D2, zero4());   // Hwx
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int r = 4 * q + g;
      if (j < NU) sr.G[j * GC + r] = D4[q];
      sr.G[(NU + j) * GC + r] = -(j == VC ? D4[q] : D5[q]);
    }
    // A^T [W A | W d + q + s], the part of the value function without gains
    const d4 SA = mmT<4>(At, D2, zero4());
    wsync();
    static_assert(NU == 12, "row elimination is written for 12 inputs");
    const int hc = lane & 15, rhs = 4 * (lane >> 4) + hc - NU;
    const bool is_h = hc < NU;
    double col[NU];
    double* gc = sr.G + (is_h ? hc : NU + rhs) * GC;
#pragma unroll
    for (int r = 0; r < NU; ++r) col[r] = gc[r];
    wsync();
    d4 ZT = zero4(), YT = zero4();
    if constexpr (ELEM) {
      double icol[NU];
#pragma unroll
      for (int r = 0; r < NU; ++r) icol[r] = is_h ? col[r] : ((r == rhs) ? 1.0 : 0.0);
      gj_rows2(col, icol, ub);
      if (!is_h && rhs < NU) {
#pragma unroll
        for (int r = 0; r < NU; ++r) sr.Z[rhs * GC + r] = icol[r];
      }
    } else if constexpr (!newton) {
      eliminate(col, ub);
    } else {
      forward_eliminate(col, sr.Z + (is_h ? 16 : rhs) * GC, hc, ub);
      if (!is_h) {
#pragma unroll
        for (int r = 0; r < NU; ++r) gc[r] = col[r];
      }
      wsync();
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        ZT[q] = -sr.Z[j * GC + 4 * q + g];
        YT[q] = sr.G[(NU + j) * GC + 4 * q + g];
      }
      wsync();
      back_substitute(col, is_h, ub);
    }
    if (newton ? (!is_h || lane < NU) : !is_h) {
#pragma unroll
      for (int r = 0; r < NU; ++r) gc[r] = col[r];
    }
    wsync();
    d4 KK = zero4();
#pragma unroll
    for (int q = 0; q < 3; ++q) KK[q] = sr.G[(NU + j) * GC + 4 * q + g];   // [K | kap]
    if constexpr (!ELEM) {
#pragma unroll
      for (int q = 0; q < 3; ++q) std1(rK, oK + q * 4 * (NX + 1) * 8, k * (TS_K * 8), KK[q]);
      if constexpr (newton) {
        // U above and below the diagonal, 1 / d on it
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const int r = 4 * q + g, c = clampi(j, NU - 1);
          const int hi = r > c ? r : c, lo = r > c ? c : r;
          std1(rF, oF + q * 4 * NU * 8, k * (TS_F * 8), sr.G[hi * GC + lo]);
        }
      }
    } else {
      d4 HI = zero4(), BpT = zero4(), Ah;
#pragma unroll
      for (int q = 0; q < 4; ++q) sr.ST[(4 * q + g) * 17 + j] = D1[q];
      wsync();
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int r = 4 * q + g;
        HI[q] = (j < NU) ? sr.Z[clampi(j, NU - 1) * GC + r] : 0.0;
        BpT[q] = sr.ST[j * 17 + r];
      }
      wsync();
      // the stage's closed-loop map [A + Bp K | d + Bp kap] with a 1 at
      // (13, 13), composed after the chunk's map; the reachability term
      // grows by A_E Bp H^-1 Bp^T A_E^T (A_E before the composition)
      const d4 LK = mmT<3>(BpT, KK, zero4());    // [Bp K | Bp kap]
#pragma unroll
      for (int q = 0; q < 4; ++q)
        Ah[q] = (j < NX) ? At[q] + LK[q] : ((j == VC) ? LK[q] + D1[q] : 0.0);
      const d4 RT = mmT<4>(D1, TE, zero4());     // (A_E Bp)^T in rows 0..11
      const d4 Y = mmT<3>(HI, RT, zero4());      // H^-1 (A_E Bp)^T
      CE = mmT<3>(RT, Y, CE);
      TE = mmT<4>(Ah, TE, zero4());
    }
    // S = A^T W A - Hwx^T H^-1 Hwx, s = A^T (W d + q + s) - Hwx^T H^-1 hw
    constexpr bool zy = newton && !ELEM;
    Ss = symmetrize(zy ? mmT<3>(ZT, YT, SA) : mmT<3>(D5, KK, SA), sw, sr.ST, lane);
    if constexpr (newton && !ELEM) {
      // the closed loop [A + B K | B kap] for the chains
      const d4 M = mmT<3>(Bt, KK, At);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        std1(rM, q < 3 ? oM + q * 4 * (NX + 1) * 8 : oM3, k * (TS_M * 8), M[q]);
    }
    if constexpr (mode == Mode::EQ && !ELEM) st_map(prS + (size_t)k * TS_S, TS_S, mS, Ss);
  }
  if constexpr (ELEM) {
    *TEo = TE;
    *CEo = CE;
  }
  return Ss;
}

// --------------------------------------------------- chains over the horizon
//
// The rollout, the costates and the corrector's vector recursion are chains of
// 13-vector products y = M x, one stage after the other.  Every 16-lane row g
// holds the whole vector (entry j in lane j, the rows identical) and takes the
// entries 3g .. 3g + 3 of the contraction (3g + 1 .. 3g + 3 for g > 0): lane j
// of row g holds those of M's row j, so a stage loads each matrix entry once
// into the wave, as one wide load where they are consecutive (a matrix row held
// by every lane was 13 loads, each served four times over: the loads, about 15
// cycles each in the one address unit of 8 waves, then bound the chains).  The
// row's vector entries reach its lanes by DPP broadcast from a copy of x turned
// by 3g lanes, and the partial sums of the four rows meet through the row and
// half-wave swaps.

// s + sum_a (w of lane a of this 16-lane row) * m[a] over the force components,
// lanes 0..2 and 6..8.
__device__ inline double dot_forces(double w, const double (&m)[6], double s) {
  asm volatile("s_nop 1\n"
               "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %5 row_newbcast:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %6 row_newbcast:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               "v_fmac_f64_dpp %0, %1, %7 row_newbcast:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
               : "+v"(s)
               : "v"(w), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]));
  return s;
}

// Forward rollout of an equality pass after its recursion (all N stages): u = P
// (K x + kap) + c, x' = A x + B u + e, with u_k in GV and x_{k+1} in PV.  The
// gains lie in the range of the projector only up to the elimination's rounding,
// which is relative to H's largest entries, while outside that range H is the
// identity: with inputs in units in which H is large the part outside is far above
// the tolerance, and without P the states were not those of the inputs on their
// faces (inputs in units of 10 kN: one problem in ten was not certified).  Stage
// data is fetched a ring of six stages ahead, about 3000 cycles, as a trip to
// memory takes (unconditionally, so every path back to the loop head has issued
// the same loads).
template <bool LONG>
__device__ INLINE void forward(const Ctx& C, Sh& sh) {
  gsync();
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const gcf pe = uni(C.e), pA = uni(C.A);
  const auto rA = rsrc(pA, N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * NU * 4);
  const auto rE = rsrc(pe ? pe : pA, pe ? N * NX * 4 : 0);
  const auto rK = rsrc(uni(C.rK), N * TS_K * 8), rT = rsrc(uni(C.rT), N * TS_T * 8);
  const StageBufs<LONG> sb(sh, C);
  const int oA = j < NX ? (j * NX + 3 * g) * 4 : OOB, oB = j < NX ? (j * NU + 3 * g) * 4 : OOB;
  const int oK = j < NU ? (j * (NX + 1) + 3 * g) * 8 : OOB;
  const int oKap = (g == 0 && j < NU) ? (j * (NX + 1) + NX) * 8 : OOB;
  const int oE = (g == 0 && j < NX) ? j * 4 : OOB;
  // row j of [P | c]: three entries and c (forces), or the diagonal and c (moments)
  const bool force = j % 6 < 3;
  const int oP = j < NU ? ((j / 6) * 18 + (force ? 4 * (j % 6) : 12 + 2 * (j % 6 - 3))) * 8 : OOB;
  const int oP2 = force ? oP + 16 : OOB;
  struct FwdRaw {
    double k[4], kap, p[4];
    float a[4], b[3], e;
  };
  auto ffetch = [&](int k, FwdRaw& s) {
    ldd2(rK, oK, k * (TS_K * 8), s.k);
    ldd2(rK, oK + 16, k * (TS_K * 8), s.k + 2);
    s.kap = ldd(rK, oKap, k * (TS_K * 8));
    ldd2(rT, oP, k * (TS_T * 8), s.p);
    ldd2(rT, oP2, k * (TS_T * 8), s.p + 2);
    ldf4(rA, oA, k * (NX * NX * 4), s.a);
    ldf3(rB, oB, k * (NX * NU * 4), s.b);
    s.e = ldf(rE, oE, k * (NX * 4));
  };
  constexpr int FD = 6;
  FwdRaw ring[FD];
#pragma unroll
  for (int d = 0; d < FD; ++d) {
    ffetch(d < N ? d : N - 1, ring[d]);
    pin_memory();
  }
  double xv = j < NX ? (double)uni(C.x0)[clampi(j, NX - 1)] : 0.0;   // x_k, entry j
  auto step = [&](int k, FwdRaw& r) __attribute__((always_inline)) {
    double km[4], a[4], b[3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      km[q] = (q == 0 && g) ? 0.0 : r.k[q];
      a[q] = (q == 0 && g) ? 0.0 : (double)r.a[q];
      pin(km[q]);
      pin(a[q]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      b[q] = (double)r.b[q];
      pin(b[q]);
    }
    double pm[6];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      pm[q] = j < 3 ? r.p[q] : 0.0;
      pm[3 + q] = (j >= 6 && j < 9) ? r.p[q] : 0.0;
      pin(pm[q]);
      pin(pm[3 + q]);
    }
    const double kap = r.kap, pd = force ? 0.0 : r.p[0], cc = force ? r.p[3] : r.p[1],
                 ee = (double)r.e;
    pin(kap); pin(pd); pin(cc); pin(ee);
    pin_memory();
    ffetch(k + FD < N ? k + FD : N - 1, r);
    const double xt = turn_rows(xv);
    const double w = row_total(dot4(xt, km, kap));
    const double ax = dot4(xt, a, ee);
    const double u = dot_forces(w, pm, fma(pd, w, cc));
    xv = row_total(dot3(turn_rows(u), b, ax));
    if (lane < NU) sb.GV[k * 16 + j] = u;
    if (lane < NX) sb.PV[k * 16 + j] = xv;
  };
  static_assert(FD == 6, "one line below per ring slot");
  for (int k = 0;; k += FD) {
    if (!(k < N)) break;
    step(k, ring[0]);
    if (!(k + 1 < N)) break;
    step(k + 1, ring[1]);
    if (!(k + 2 < N)) break;
    step(k + 2, ring[2]);
    if (!(k + 3 < N)) break;
    step(k + 3, ring[3]);
    if (!(k + 4 < N)) break;
    step(k + 4, ring[4]);
    if (!(k + 5 < N)) break;
    step(k + 5, ring[5]);
  }
  bufsync<LONG>();
}

// The rollout of a Newton step (from x = 0), by the closed loops [M | m] that its
// recursion leaves: x' = M x + m is the chain, w = K x + kap follows for four
// stages at a time, one per 16-lane row.  The chain has one dependent product per
// stage instead of two and issues half the instructions (its one wave is bound by
// their number).  VECK: kap_k comes in GV and m_k = B kap_k in PV (a corrector's)
// instead of the stored ones.
template <bool LONG, bool VECK>
__device__ INLINE void forward_map(const Ctx& C, Sh& sh) {
  gsync();
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const auto rK = rsrc(uni(C.rK), N * TS_K * 8);
  const auto rM = rsrc(uni(C.rM), N * TS_M * 8);
  const StageBufs<LONG> sb(sh, C);
  const int oM = j < NX ? (j * (NX + 1) + 3 * g) * 8 : OOB;
  const int oV = (g == 0 && j < NX) ? (j * (NX + 1) + NX) * 8 : OOB;
  struct FwdRaw {
    double m[4], v;
  };
  auto ffetch = [&](int k, FwdRaw& s) {
    ldd2(rM, oM, k * (TS_M * 8), s.m);
    ldd2(rM, oM + 16, k * (TS_M * 8), s.m + 2);
    if constexpr (VECK) s.v = lane < NX ? sb.PV[k * 16 + j] : 0.0;
    else s.v = ldd(rM, oV, k * (TS_M * 8));
  };
  constexpr int FD = 12;
  FwdRaw ring[FD];
#pragma unroll
  for (int d = 0; d < FD; ++d) {
    ffetch(d < N ? d : N - 1, ring[d]);
    pin_memory();
  }
  double xv = 0.0;   // x_k, entry j
  auto step = [&](int k, FwdRaw& r) __attribute__((always_inline)) {
    double m[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      m[q] = (q == 0 && g) ? 0.0 : r.m[q];
      pin(m[q]);
    }
    const double v = r.v;
    pin(v);
    pin_memory();
    ffetch(k + FD < N ? k + FD : N - 1, r);
    xv = row_total(dot4(turn_rows(xv), m, v));
    if (lane < NX) sb.PV[k * 16 + j] = xv;
  };
  static_assert(FD == 12, "one line below per ring slot");
  for (int k = 0;; k += FD) {
    if (!(k < N)) break;
    step(k, ring[0]);
    if (!(k + 1 < N)) break;
    step(k + 1, ring[1]);
    if (!(k + 2 < N)) break;
    step(k + 2, ring[2]);
    if (!(k + 3 < N)) break;
    step(k + 3, ring[3]);
    if (!(k + 4 < N)) break;
    step(k + 4, ring[4]);
    if (!(k + 5 < N)) break;
    step(k + 5, ring[5]);
    if (!(k + 6 < N)) break;
    step(k + 6, ring[6]);
    if (!(k + 7 < N)) break;
    step(k + 7, ring[7]);
    if (!(k + 8 < N)) break;
    step(k + 8, ring[8]);
    if (!(k + 9 < N)) break;
    step(k + 9, ring[9]);
    if (!(k + 10 < N)) break;
    step(k + 10, ring[10]);
    if (!(k + 11 < N)) break;
    step(k + 11, ring[11]);
  }
  bufsync<LONG>();
  const int oK = j < NU ? (g * TS_K + j * (NX + 1)) * 8 : OOB;
  auto kfetch = [&](int k0, double (&s)[NX + 1]) {
#pragma unroll
    for (int l = 0; l <= NX; l += 2) ldd2(rK, oK + l * 8, k0 * (TS_K * 8), s + l);
  };
  constexpr int KD = 3;
  double kn[KD][NX + 1];
#pragma unroll
  for (int d = 0; d < KD; ++d) {
    kfetch(4 * d < N ? 4 * d : 0, kn[d]);
    pin_memory();
  }
  auto gain = [&](int k0, double (&r)[NX + 1]) __attribute__((always_inline)) {
    const int k = k0 + g;
    double km[NX], kap = r[NX];
#pragma unroll
    for (int l = 0; l < NX; ++l) {
      km[l] = r[l];
      pin(km[l]);
    }
    pin(kap);
    pin_memory();
    kfetch(k0 + 4 * KD < N ? k0 + 4 * KD : k0, r);
    const bool on = j < NU && k < N;
    if constexpr (VECK) kap = on ? sb.GV[k * 16 + j] : 0.0;
    const double x = (k > 0 && j < NX && k < N) ? sb.PV[(k - 1) * 16 + j] : 0.0;
    const double w = dot_row_bcast13(x, km, kap);
    if (on) sb.GV[k * 16 + j] = w;
  };
  static_assert(KD == 3, "one line below per ring slot");
  for (int k0 = 0;; k0 += 4 * KD) {
    if (!(k0 < N)) break;
    gain(k0, kn[0]);
    if (!(k0 + 4 < N)) break;
    gain(k0 + 4, kn[1]);
    if (!(k0 + 8 < N)) break;
    gain(k0 + 8, kn[2]);
  }
  bufsync<LONG>();
}

// The sequential recursion over the whole horizon (one wave), then the rollout.
template <Mode mode, bool LONG>
__device__ INLINE void rollout(const Ctx& C, Sh& sh) {
  if constexpr (mode == Mode::EQ) forward<LONG>(C, sh);
  else forward_map<LONG, false>(C, sh);
}
template <Mode mode, bool LONG>
__device__ INLINE void riccati_t(const Ctx& C, Sh& sh, int ktop) {
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  ktop = (mode == Mode::EQ) ? __builtin_amdgcn_readfirstlane(ktop < N ? ktop : N) : N;
  build<mode>(C, sh, ktop);
  const d4 Vk =
      (ktop < N) ? ld_map(uni(C.rS) + (size_t)ktop * TS_S, TS_S, map_S(false)) : zero4();
  backward<mode, false>(C, sh.p.r, sh.unit, 0, ktop, Vk, nullptr, nullptr);
  rollout<mode, LONG>(C, sh);
}

// Second right-hand side of a Newton step with the stored factors.  In: its
// linear term rho_k = GV + smu PV; out: kap_k in GV and m_k = B kap_k in PV, as
// the rollout takes them.  With wv = q + s and hw = Bp^T wv + rho the recursion of
// the linear part is s <- A^T wv + K^T hw (Hwx^T kap = K^T hw) = M^T wv + K^T rho
// with the closed loop M = A + Bp K: one product per stage in the chain.  K^T rho
// comes before it and kap = -H^{-1} hw, by the two triangular solves, after it,
// for four stages at a time (one per 16-lane row).
template <bool LONG>
__device__ INLINE void newton_vector(const Ctx& C, Sh& sh, double smu) {
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const StageBufs<LONG> sb(sh, C);
  const auto rB = rsrc(uni(C.B), N * NX * NU * 4), rM = rsrc(uni(C.rM), N * TS_M * 8);
  const auto rK = rsrc(uni(C.rK), N * TS_K * 8), rQ = rsrc(uni(C.rq), N * NX * 8);
  const auto rF = rsrc(uni(C.rF), N * TS_F * 8);
  {
    const int oK = j < NX ? (g * TS_K + j) * 8 : OOB;
    auto kfetch = [&](int k0, double (&s)[NU]) {
#pragma unroll
      for (int r = 0; r < NU; ++r) s[r] = ldd(rK, oK + r * (NX + 1) * 8, k0 * (TS_K * 8));
    };
    constexpr int KD = 3;
    double kn[KD][NU];
#pragma unroll
    for (int d = 0; d < KD; ++d) {
      kfetch(4 * d < N ? 4 * d : 0, kn[d]);
      pin_memory();
    }
    auto term = [&](int k0, double (&r)[NU]) __attribute__((always_inline)) {
      const int k = k0 + g;
      double kc[NX];
#pragma unroll
      for (int l = 0; l < NU; ++l) {
        kc[l] = r[l];
        pin(kc[l]);
      }
      kc[NU] = 0.0;
      pin_memory();
      kfetch(k0 + 4 * KD < N ? k0 + 4 * KD : k0, r);
      const bool on = j < NU && k < N;
      const double rho = on ? fma(smu, sb.PV[k * 16 + j], sb.GV[k * 16 + j]) : 0.0;
      const double v = dot_row_bcast13(rho, kc, 0.0);
      if (on) sb.GV[k * 16 + j] = rho;
      if (j < NX && k < N) sb.PV[k * 16 + j] = v;
    };
    static_assert(KD == 3, "one line below per ring slot");
    for (int k0 = 0;; k0 += 4 * KD) {
      if (!(k0 < N)) break;
      term(k0, kn[0]);
      if (!(k0 + 4 < N)) break;
      term(k0 + 4, kn[1]);
      if (!(k0 + 8 < N)) break;
      term(k0 + 8, kn[2]);
    }
  }
  bufsync<LONG>();
  const int oM = j < NX ? (3 * g * (NX + 1) + j) * 8 : OOB, oM0 = (g == 0 && j < NX) ? j * 8 : OOB;
  const int oQ = j < NX ? j * 8 : OOB;
  struct VecRaw {
    double m[4], q, v;
  };
  auto vfetch = [&](int k, VecRaw& s) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      s.m[q] = ldd(rM, q == 0 ? oM0 : oM + q * (NX + 1) * 8, k * (TS_M * 8));
    s.q = ldd(rQ, oQ, k * (NX * 8));
    s.v = lane < NX ? sb.PV[k * 16 + j] : 0.0;
  };
  constexpr int VD = 12;
  VecRaw ring[VD];
#pragma unroll
  for (int d = 0; d < VD; ++d) {
    vfetch(N - 1 - d >= 0 ? N - 1 - d : 0, ring[d]);
    pin_memory();
  }
  double s = 0.0;   // value function's linear part, entry j
  auto step = [&](int k, VecRaw& r) __attribute__((always_inline)) {
    double m[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      m[q] = r.m[q];
      pin(m[q]);
    }
    const double qk = r.q, v = r.v;
    pin(qk);
    pin(v);
    pin_memory();
    vfetch(k - VD >= 0 ? k - VD : 0, r);
    const double wv = qk + s;
    if (lane < NX) sb.PV[k * 16 + j] = wv;
    s = row_total(dot4(turn_rows(wv), m, v));
  };
  static_assert(VD == 12, "one line below per ring slot");
  for (int k = N - 1;; k -= VD) {
    if (!(k >= 0)) break;
    step(k, ring[0]);
    if (!(k - 1 >= 0)) break;
    step(k - 1, ring[1]);
    if (!(k - 2 >= 0)) break;
    step(k - 2, ring[2]);
    if (!(k - 3 >= 0)) break;
    step(k - 3, ring[3]);
    if (!(k - 4 >= 0)) break;
    step(k - 4, ring[4]);
    if (!(k - 5 >= 0)) break;
    step(k - 5, ring[5]);
    if (!(k - 6 >= 0)) break;
    step(k - 6, ring[6]);
    if (!(k - 7 >= 0)) break;
    step(k - 7, ring[7]);
    if (!(k - 8 >= 0)) break;
    step(k - 8, ring[8]);
    if (!(k - 9 >= 0)) break;
    step(k - 9, ring[9]);
    if (!(k - 10 >= 0)) break;
    step(k - 10, ring[10]);
    if (!(k - 11 >= 0)) break;
    step(k - 11, ring[11]);
  }
  bufsync<LONG>();
  const int oF = j < NU ? (g * TS_F + j * NU) * 8 : OOB;
  const int oBt = j < NU ? (g * NX * NU + j) * 4 : OOB;      // B^T's row j
  const int oB = j < NX ? (g * NX + j) * NU * 4 : OOB;       // B's row j
  struct TriRaw {
    double f[NU], rd;
    float bt[NX], b[NU];
  };
  auto tfetch = [&](int k0, TriRaw& s) {
#pragma unroll
    for (int r = 0; r < NX; ++r) s.bt[r] = ldf(rB, oBt + r * NU * 4, k0 * (NX * NU * 4));
#pragma unroll
    for (int p = 0; p < NU; p += 2) ldd2(rF, oF + p * 8, k0 * (TS_F * 8), s.f + p);
    s.rd = ldd(rF, oF + j * 8, k0 * (TS_F * 8));
#pragma unroll
    for (int l = 0; l < NU; l += 4) ldf4(rB, oB + l * 4, k0 * (NX * NU * 4), s.b + l);
  };
  constexpr int TD = 2;
  TriRaw tri[TD];
#pragma unroll
  for (int d = 0; d < TD; ++d) {
    tfetch(4 * d < N ? 4 * d : 0, tri[d]);
    pin_memory();
  }
  auto solve = [&](int k0, TriRaw& r) __attribute__((always_inline)) {
    const int k = k0 + g;
    const bool on = j < NU && k < N;
    double f[NU], rd = r.rd, bt[NX], b[NX];
#pragma unroll
    for (int p = 0; p < NX; ++p) {
      if (p < NU) {
        f[p < NU ? p : 0] = r.f[p < NU ? p : 0];
        pin(f[p < NU ? p : 0]);
      }
      bt[p] = (double)r.bt[p];
      b[p] = p < NU ? (double)r.b[p < NU ? p : 0] : 0.0;
      pin(bt[p]);
      pin(b[p]);
    }
    pin(rd);
    pin_memory();
    tfetch(k0 + 4 * TD < N ? k0 + 4 * TD : k0, r);
    const double wv = (j < NX && k < N) ? sb.PV[k * 16 + j] : 0.0;
    const double rho = on ? sb.GV[k * 16 + j] : 0.0;
    double y = dot_row_bcast13(wv, bt, rho);
    if (!on || sh.unit[2 * k + j / 6]) y = 0.0;   // a swing contact's inputs
    // y <- U^-T y, then D^-1, then U^-1
#define PINMPC_TRI(p, use)                                                                      \
  {                                                                                             \
    const double m = (use) ? -f[p] : 0.0;                                                       \
    asm volatile(                                                                               \
        "s_nop 1\n"                                                                             \
        "v_fmac_f64_dpp %0, %0, %1 row_newbcast:" #p " row_mask:0xf bank_mask:0xf bound_ctrl:1" \
        : "+v"(y)                                                                               \
        : "v"(m));                                                                              \
  }
    PINMPC_TRI(0, j > 0) PINMPC_TRI(1, j > 1) PINMPC_TRI(2, j > 2) PINMPC_TRI(3, j > 3)
    PINMPC_TRI(4, j > 4) PINMPC_TRI(5, j > 5) PINMPC_TRI(6, j > 6) PINMPC_TRI(7, j > 7)
    PINMPC_TRI(8, j > 8) PINMPC_TRI(9, j > 9) PINMPC_TRI(10, j > 10)
    y *= rd;
    PINMPC_TRI(11, j < 11) PINMPC_TRI(10, j < 10) PINMPC_TRI(9, j < 9) PINMPC_TRI(8, j < 8)
    PINMPC_TRI(7, j < 7) PINMPC_TRI(6, j < 6) PINMPC_TRI(5, j < 5) PINMPC_TRI(4, j < 4)
    PINMPC_TRI(3, j < 3) PINMPC_TRI(2, j < 2) PINMPC_TRI(1, j < 1)
#undef PINMPC_TRI
    const double kap = on ? -y : 0.0;
    const double mk = dot_row_bcast13(kap, b, 0.0);
    if (on) sb.GV[k * 16 + j] = kap;
    if (j < NX && k < N) sb.PV[k * 16 + j] = mk;
  };
  static_assert(TD == 2, "one line below per ring slot");
  for (int k0 = 0;; k0 += 4 * TD) {
    if (!(k0 < N)) break;
    solve(k0, tri[0]);
    if (!(k0 + 4 < N)) break;
    solve(k0 + 4, tri[1]);
  }
  bufsync<LONG>();
}

// ------------------------------------------------------- two waves per problem
//
// The recursion of one problem as a pair of waves, where the chip has room for
// both (see launch_refine).  The first forms H and hw and eliminates; the second
// forms Hwx and the part of the value function without gains beside that and
// finishes the value function.  Per stage three meetings in LDS: the system is
// complete, it is eliminated, the value function is known.  While the first
// eliminates, the second also takes the stage before through the back
// substitution (Newton steps) and stores what the chains read (gains, factors,
// closed loops).  A stage's chain is then 8 + 3 matrix instructions and the
// forward elimination instead of 23 + 3 and both triangular solves; the results are bitwise those of
// one wave.  The second wave waits at a barrier while the first does all else.
enum { PAIR_EXIT = 0, PAIR_EQ = 1, PAIR_NEWTON = 2 };
struct PairCtl {
  int op, ktop;
};
__shared__ PairCtl pair_ctl;

// LDS hand-off between the waves: what this wave wrote has arrived.  The loads
// in flight from memory go on (the fence of __syncthreads would wait for them).
__device__ inline void pair_meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The symmetrised value function from the raw one in LDS.
__device__ inline d4 read_sym(const SymWeights& w, const double* buf, int lane) {
  const int g = lane >> 4, j = lane & 15;
  d4 S;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    S[q] = fma(w.other[q], buf[j * 17 + 4 * q + g], w.own[q] * buf[(4 * q + g) * 17 + j]);
  return S;
}

// One wave's side of the recursion over stages ktop - 1 .. 0 (FIRST: the wave
// that eliminates).
template <Mode mode, bool FIRST>
__device__ INLINE void pair_backward(const Ctx& C, Sh& sh, int ktop) {
  ShR& sr = sh.p.r;
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  constexpr bool newton = (mode == Mode::NEWTON);
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const gcf pe = uni(C.e), pA = uni(C.A);
  const auto rA = rsrc(pA, N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * NU * 4);
  const auto rX = rsrc(uni(C.x_ref), N * NX * 4);
  const auto rE = rsrc(pe ? pe : pA, pe ? N * NX * 4 : 0);
  const auto rQ = rsrc(uni(C.rq), N * NX * 8);
  const auto rT = rsrc(uni(C.rT), N * TS_T * 8), rT2 = rsrc(uni(C.rT2), N * TS_T * 8);
  const auto rK = rsrc(uni(C.rK), N * TS_K * 8), rF = rsrc(uni(C.rF), N * TS_F * 8);
  const auto rM = rsrc(uni(C.rM), N * TS_M * 8);
  const gd prS = uni(C.rS);
  const int oA = j < NX ? (g * NX + j) * 4 : OOB;
  const int oA3 = (g == 0 && j < NX) ? (12 * NX + j) * 4 : OOB;
  const int oBt = j < NX ? (j * NU + g) * 4 : OOB;
  const int oB = j < NU ? (g * NU + j) * 4 : OOB;
  const int oB3 = (g == 0 && j < NU) ? (12 * NU + j) * 4 : OOB;
  const int oV = j == VC ? g : OOB / 8;
  const int oV3 = (g == 0 && j == VC) ? 12 : ((g == 1 && j < NX) ? j : OOB / 8);
  const int oE3 = (g == 0 && j == VC) ? 48 : OOB;
  int oT[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) oT[q] = t_offset(4 * q + g, j);
  const int oK = j <= VC ? (g * (NX + 1) + j) * 8 : OOB;
  const int oF = j < NU ? (g * NU + j) * 8 : OOB;
  const int oK3 = (g == 0 && j <= VC) ? (12 * (NX + 1) + j) * 8 : OOB;
  const uint32_t mS = map_S(true);
  d4 Qd, Qv;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * q + g;
    Qd[q] = (r == j && j < NX) ? sh.Qd[clampi(j, NX - 1)] : 0.0;
    Qv[q] = (j == VC && r < NX) ? sh.Qd[clampi(r, NX - 1)]
                                : ((r == VC && j < NX) ? sh.Qd[clampi(j, NX - 1)] : 0.0);
  }
  const SymWeights sw = sym_weights(lane);
  const double one = (g == 1 && j == VC) ? 1.0 : 0.0;
  struct Raw {
    float a[4], b[4], bt[3], xr[4], ev[4];
    double q[4], T[3], T2[3];
  };
  auto fetch = [&](int k, Raw& s) {
    if constexpr (!FIRST) {
#pragma unroll
      for (int q = 0; q < 3; ++q) s.a[q] = ldf(rA, oA + q * 4 * NX * 4, k * (NX * NX * 4));
      s.a[3] = ldf(rA, oA3, k * (NX * NX * 4));
    }
    if constexpr (!FIRST || !newton) {
#pragma unroll
      for (int q = 0; q < 3; ++q) s.bt[q] = ldf(rB, oBt + q * 16, k * (NX * NU * 4));
    }
    if constexpr (newton) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        s.b[q] = ldf(rB, oB + q * 4 * NU * 4, k * (NX * NU * 4));
        s.q[q] = ldd(rQ, oV * 8 + q * 32, k * (NX * 8));
      }
      s.b[3] = ldf(rB, oB3, k * (NX * NU * 4));
      s.q[3] = ldd(rQ, oV3 * 8, k * (NX * 8));
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        s.xr[q] = ldf(rX, oV * 4 + q * 16, k * (NX * 4));
        s.ev[q] = ldf(rE, oV * 4 + q * 16, k * (NX * 4));
        if constexpr (FIRST) s.T2[q] = ldd(rT2, oT[q], k * (TS_T * 8));
      }
      s.xr[3] = ldf(rX, oV3 * 4, k * (NX * 4));
      s.ev[3] = ldf(rE, oE3, k * (NX * 4));
    }
    if constexpr (FIRST || !newton) {
#pragma unroll
      for (int q = 0; q < 3; ++q) s.T[q] = ldd(rT, oT[q], k * (TS_T * 8));
    }
  };
  Raw raw;
  fetch(ktop > 0 ? ktop - 1 : 0, raw);
  d4 Ss = (ktop < N) ? ld_map(prS + (size_t)ktop * TS_S, TS_S, map_S(false)) : zero4();
  const int hc = lane & 15, rhs = 4 * (lane >> 4) + hc - NU;
  const bool is_h = hc < NU;
  // the second wave's previous stage, its gains yet to be solved for and stored
  d4 Ap = zero4(), Bp = zero4(), KE = zero4();
  uint32_t up = 0;
  auto finish = [&](int k) {
    if constexpr (!newton) {
#pragma unroll
      for (int q = 0; q < 3; ++q) std1(rK, oK + q * 4 * (NX + 1) * 8, k * (TS_K * 8), KE[q]);
      return;
    }
    double* G = (k & 1) ? sh.p.G1 : sr.G;
    double col[NU];
    double* gc = G + (is_h ? hc : NU + rhs) * GC;
#pragma unroll
    for (int r = 0; r < NU; ++r) col[r] = gc[r];
    back_substitute(col, is_h, up);
    if (!is_h) {
#pragma unroll
      for (int r = 0; r < NU; ++r) gc[r] = col[r];
    }
    wsync();
    d4 KK = zero4();   // [K | kap]
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int r = 4 * q + g, c = clampi(j, NU - 1);
      KK[q] = G[(NU + j) * GC + r];
      std1(rK, oK + q * 4 * (NX + 1) * 8, k * (TS_K * 8), KK[q]);
      // U above and below the diagonal, 1 / d on it
      std1(rF, oF + q * 4 * NU * 8, k * (TS_F * 8), G[(r > c ? r : c) * GC + (r > c ? c : r)]);
    }
    wsync();
    const d4 M = mmT<3>(Bp, KK, Ap);   // [A + B K | B kap]
#pragma unroll
    for (int q = 0; q < 4; ++q)
      std1(rM, q < 3 ? oK + q * 4 * (NX + 1) * 8 : oK3, k * (TS_M * 8), M[q]);
  };
  for (int k = ktop - 1; k >= 0; --k) {
    d4 At = zero4(), D1, Wt, H0 = zero4(), Bt = zero4();
    uint32_t ub;
    {
      const uint32_t u0 = sh.unit[2 * k], u1 = sh.unit[2 * k + 1];
      ub = (uint32_t)__builtin_amdgcn_readfirstlane((int)(u0 | (u1 << 6)));
    }
    if (k < ktop - 1) Ss = read_sym(sw, sr.ST, lane);
    if constexpr (newton) {
      const bool keep = j < NU && !((ub >> j) & 1u);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        D1[q] = keep ? (double)raw.b[q] : 0.0;
        Wt[q] = Ss[q] + (Qd[q] + raw.q[q]);
      }
      D1[3] += one;
      if constexpr (FIRST) {
#pragma unroll
        for (int q = 0; q < 3; ++q) H0[q] = raw.T[q];
      } else {
#pragma unroll
        for (int q = 0; q < 3; ++q) Bt[q] = (double)raw.bt[q];
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        D1[q] = (double)raw.ev[q];
        Wt[q] = Ss[q] + fma(-Qv[q], (double)raw.xr[q], Qd[q]);
      }
      D1[3] += one;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        Bt[q] = (double)raw.bt[q];
        D1 = __builtin_amdgcn_mfma_f64_16x16x4f64(Bt[q], raw.T[q], D1, 0, 0, 0);
        if constexpr (FIRST) H0[q] = raw.T2[q];
      }
    }
    if constexpr (!FIRST) {
      // [A | d] with a 1 at (VC, VC)
#pragma unroll
      for (int q = 0; q < 4; ++q) At[q] = j == VC ? D1[q] : (double)raw.a[q];
    }
    pin(At); pin(D1); pin(Wt); pin(H0); pin(Bt);
    pin_memory();
    if (k > 0) fetch(k - 1, raw);
    double* G = (k & 1) ? sh.p.G1 : sr.G;
    if constexpr (FIRST) {
      const d4 D3 = mmT<4>(Wt, D1, zero4());
      const d4 D4 = mmT<4>(D3, D1, zero4()) + H0;   // [H | 0 | hw]
      if (j < NU || j == VC) {
        double* gc = G + (j < NU ? j : NU + VC) * GC + g;
#pragma unroll
        for (int q = 0; q < 3; ++q) gc[4 * q] = j < NU ? D4[q] : -D4[q];
      }
      pair_meet();   // the system is complete
      double col[NU];
      double* gc = G + (is_h ? hc : NU + rhs) * GC;
#pragma unroll
      for (int r = 0; r < NU; ++r) col[r] = gc[r];
      if constexpr (newton) forward_eliminate(col, sr.Z + (is_h ? 16 : rhs) * GC, hc, ub);
      else eliminate(col, ub);
      wsync();
      if (newton ? (!is_h || lane < NU) : !is_h) {
#pragma unroll
        for (int r = 0; r < NU; ++r) gc[r] = col[r];
      }
      pair_meet();   // it is eliminated
      if (k > 0) pair_meet();   // the value function is known
    } else {
      const d4 D2 = mmT<4>(Wt, At, zero4());   // [W A | W d + q + s]
      const d4 D5 = mmT<4>(D1, D2, zero4());   // Hwx
      if (j != VC) {
#pragma unroll
        for (int q = 0; q < 3; ++q) G[(NU + j) * GC + 4 * q + g] = -D5[q];
      }
      pair_meet();   // the system is complete
      const d4 SA = mmT<4>(At, D2, zero4());
      if (k < ktop - 1) {
        finish(k + 1);
        if constexpr (!newton) st_map(prS + (size_t)(k + 1) * TS_S, TS_S, mS, Ss);
      }
      Ap = At;
      Bp = Bt;
      up = ub;
      pair_meet();   // it is eliminated
      d4 ZT = zero4(), YT = zero4();   // NEWTON: -z, D^-1 z; EQ: Hwx, [K | kap]
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        ZT[q] = newton ? -sr.Z[j * GC + 4 * q + g] : D5[q];
        YT[q] = G[(NU + j) * GC + 4 * q + g];
      }
      KE = YT;
      if (k > 0) {
        const d4 S = mmT<3>(ZT, YT, SA);
#pragma unroll
        for (int q = 0; q < 4; ++q) sr.ST[(4 * q + g) * 17 + j] = S[q];
        pair_meet();   // the value function is known
      }
    }
  }
  if constexpr (!FIRST) {
    if (ktop > 0) finish(0);
    gsync();       // the stores come before the first wave's loads
  }
  pair_meet();
}

// The first wave's recursion and rollout.
template <Mode mode, bool LONG>
__device__ INLINE void riccati_pair(const Ctx& C, Sh& sh, int ktop) {
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  ktop = (mode == Mode::EQ) ? __builtin_amdgcn_readfirstlane(ktop < N ? ktop : N) : N;
  build<mode>(C, sh, ktop);
  if (lane_id() == 0) pair_ctl = {mode == Mode::EQ ? PAIR_EQ : PAIR_NEWTON, ktop};
  pair_meet();   // the command and the stage inputs
  pair_backward<mode, true>(C, sh, ktop);
  rollout<mode, LONG>(C, sh);
}
// The second wave: the first's commands until it releases it.
template <bool NEWTON>
__device__ INLINE void pair_helper(const Ctx& C, Sh& sh) {
  for (;;) {
    pair_meet();
    const int op = __builtin_amdgcn_readfirstlane(pair_ctl.op);
    const int ktop = __builtin_amdgcn_readfirstlane(pair_ctl.ktop);
    if (op == PAIR_EXIT) return;
    if (!NEWTON || op == PAIR_EQ) pair_backward<Mode::EQ, false>(C, sh, ktop);
    else pair_backward<Mode::NEWTON, false>(C, sh, ktop);
  }
}
__device__ inline void pair_release() {
  if (lane_id() == 0) pair_ctl.op = PAIR_EXIT;
  pair_meet();
}

// ---------------------------------------- associative scan over the horizon
//
// The backward recursion composes one map of the value function per stage,
// and that composition is associative.  With the horizon [0, ktop) cut into
// chunks, each chunk's composition (its summary) is formed on its own, the
// value functions at the chunk boundaries follow from the summaries alone,
// from the last chunk back to the first, and every chunk then runs the
// ordinary recursion from its boundary value, all chunks at once.  The
// summary of stages [k0, k1), from a zero value at x_{k1}, is
//   A_E, b_E  the closed-loop affine map from x_{k0} to x_{k1} (TE),
//   C_E       its reachability term, the sum of A' Bp H^-1 Bp^T A'^T (CE),
//   S_E, s_E  the value function of x_{k0} (SE),
// and the value function at x_{k0} for a value (S, s) at x_{k1} is, with
// J = S + Q and eta = -(s + q_{k1-1}) (the cost of x_{k1} included),
//   G = (J^-1 + C_E)^-1,   S_0 = A_E^T G A_E + S_E,
//   s_0 = s_E - A_E^T (I - G C_E)(eta - J b_E).
// The recursion is the paper's horizon-parallel treatment (Sec. III) applied
// to the LQ solve of the refinement: depth about 3 N / W + W stage steps for
// W chunks instead of N.  One wave per chunk: the problem's first wave runs
// the refinement; the others (helpers) take the scan's commands at the
// workgroup barrier and run the summaries and recursions of their chunks.

constexpr int SCAN_WMAX = 8;       // chunks (waves) per problem
constexpr int SCAN_MIN_CHUNK = 4;  // fewer stages per chunk: sequential
enum { SCAN_EXIT = 0, SCAN_EQ = 1, SCAN_NEWTON = 2 };
struct ScanCtl {
  int op, nch;
  int bounds[SCAN_WMAX + 1];
};
constexpr int TILE_D = 256;   // doubles of a register tile kept in LDS (lane-major)

__shared__ ScanCtl scan_ctl;
extern __shared__ __attribute__((aligned(16))) double scan_dyn[];

// Dynamic LDS of a scanning workgroup with W waves: the helpers' hand-off
// buffers, three summary tiles per chunk and a boundary value per chunk.
struct ScanLds {
  ShR* shr;
  double* exch;
  double* bnd;
};
__device__ inline ScanLds scan_lds(int W) {
  ScanLds L;
  L.shr = reinterpret_cast<ShR*>(scan_dyn);
  L.exch = scan_dyn + (size_t)(W - 1) * (sizeof(ShR) / 8);
  L.bnd = L.exch + (size_t)W * 3 * TILE_D;
  return L;
}

__device__ inline void st_tile_lds(double* base, const d4& t) {
  const int l = lane_id();
#pragma unroll
  for (int q = 0; q < 4; ++q) base[l * 4 + q] = t[q];
}
__device__ inline d4 ld_tile_lds(const double* base) {
  const int l = lane_id();
  d4 t;
#pragma unroll
  for (int q = 0; q < 4; ++q) t[q] = base[l * 4 + q];
  return t;
}

__device__ inline double readlane_d(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Inverse of the SPD 13 x 13 block of a tile by Gauss-Jordan elimination
// without pivoting: lane c < 13 holds column c of the matrix, lane 16 + c
// column c of the identity; each pivot's column reaches every lane by lane
// reads.  buf: 256 doubles of LDS.
__device__ INLINE d4 inv13(const d4& M, double* buf) {
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
#pragma unroll
  for (int q = 0; q < 4; ++q) buf[(4 * q + g) * 16 + j] = M[q];
  wsync();
  const int c = lane & 15;
  const bool mat = lane < NX, idn = lane >= 16 && lane < 16 + NX;
  double col[NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) col[r] = mat ? buf[r * 16 + c] : ((idn && r == c) ? 1.0 : 0.0);
  wsync();
#pragma unroll
  for (int pv = 0; pv < NX; ++pv) {
    double m[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) m[r] = readlane_d(col[r], pv);
    const double rp = col[pv] * recip(m[pv]);
#pragma unroll
    for (int r = 0; r < NX; ++r)
      if (r != pv) col[r] = fma(-m[r], rp, col[r]);
    col[pv] = rp;
  }
  if (idn) {
#pragma unroll
    for (int r = 0; r < NX; ++r) buf[r * 16 + c] = col[r];
  }
  wsync();
  d4 R;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * q + g;
    R[q] = (r < NX && j < NX) ? buf[r * 16 + j] : 0.0;
  }
  wsync();
  return R;
}

// Value function [S_0 | s_0] at x_{k0} of a chunk with summary (TE, CE, SE)
// for the value V = [S | s] at x_{k1}; om holds q_{k1-1} in column VC.
__device__ INLINE d4 combine_value(const d4& TE, const d4& CE, const d4& SE, const d4& V, const d4& om,
                            double Qj, double* buf) {
  const int g = tg(), j = tj();
  d4 J, eta, E13;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * q + g;
    J[q] = (j < NX) ? V[q] + ((r == j) ? Qj : 0.0) : 0.0;
    eta[q] = (j == VC && r < NX) ? -(V[q] + om[q]) : 0.0;
    E13[q] = (r == VC && j == VC) ? 1.0 : 0.0;
  }
  const d4 Ji = inv13(J, buf);
  d4 X;
#pragma unroll
  for (int q = 0; q < 4; ++q) X[q] = (j < NX) ? Ji[q] + CE[q] : 0.0;
  const d4 G = inv13(X, buf);
  // b_E (row 13 of TE) as column VC, then t = eta - J b_E, u = (I - G C_E) t
  d4 bE = mmT<4>(TE, E13, zero4());
#pragma unroll
  for (int q = 0; q < 4; ++q) bE[q] = (4 * q + g < NX) ? bE[q] : 0.0;
  const d4 t = eta - mmT<4>(J, bE, zero4());
  const d4 u = t - mmT<4>(G, mmT<4>(CE, t, zero4()), zero4());
  // A_E: the transpose of TE's 13 x 13 block
#pragma unroll
  for (int q = 0; q < 4; ++q) buf[(4 * q + g) * 16 + j] = TE[q];
  wsync();
  d4 AE;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * q + g;
    AE[q] = (r < NX && j < NX) ? buf[j * 16 + r] : 0.0;
  }
  wsync();
  const d4 GA = mmT<4>(G, AE, zero4());
  d4 S0 = mmT<4>(AE, GA, SE);                     // [A^T G A + S_E | s_E]
  S0 -= sel(j == VC, mmT<4>(AE, u, zero4()));     // s_E - A^T u
  return symmetrize(S0, sym_weights(), buf);
}

// The backward recursion as a scan over the horizon (the problem's first
// wave; the helpers run scan_helper).  Falls back to the sequential recursion
// when the horizon is too short to cut.
template <Mode mode, bool LONG>
__device__ INLINE void riccati_scan(const Ctx& C, Sh& sh, int ktop) {
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  ktop = (mode == Mode::EQ) ? __builtin_amdgcn_readfirstlane(ktop < N ? ktop : N) : N;
  build<mode>(C, sh, ktop);
  constexpr bool newton = (mode == Mode::NEWTON);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const int W = (int)(blockDim.x >> 6);
  const int nch = __builtin_amdgcn_readfirstlane(
      ktop / SCAN_MIN_CHUNK < W ? ktop / SCAN_MIN_CHUNK : W);
  const d4 Vk = (ktop < N) ? ld_map(uni(C.rS) + (size_t)ktop * TS_S, TS_S, map_S(false)) : zero4();
  if (nch < 2) {
    backward<mode, false>(C, sh.p.r, sh.unit, 0, ktop, Vk, nullptr, nullptr);
    rollout<mode, LONG>(C, sh);
    return;
  }
  const ScanLds L = scan_lds(W);
  if (lane == 0) {
    scan_ctl.op = newton ? SCAN_NEWTON : SCAN_EQ;
    scan_ctl.nch = nch;
    for (int w = 0; w <= nch; ++w) scan_ctl.bounds[w] = (int)(((long)w * ktop) / nch);
  }
  __syncthreads();   // the command reaches the helpers
  __syncthreads();   // the helpers' chunk summaries are in LDS
  // boundary values, from the last chunk back to the first (the first chunk's
  // summary is not needed: its recursion starts from the boundary value)
  const gcf pxr = uni(C.x_ref);
  const gd prq = uni(C.rq);
  const double Qj = C.Q[clampi(j, NX - 1)];
  double* buf = L.exch;   // the first chunk's summary slot, free
  d4 V = Vk;
  st_tile_lds(L.bnd + (size_t)(nch - 1) * TILE_D, V);
  for (int w = nch - 1; w >= 1; --w) {
    const int k1 = __builtin_amdgcn_readfirstlane((int)(((long)(w + 1) * ktop) / nch));
    d4 om;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 4 * q + g;
      const int rc = clampi(r, NX - 1);
      const size_t at = (size_t)(k1 - 1) * NX + rc;
      const double v = newton ? prq[at] : -C.Q[rc] * (double)pxr[at];
      om[q] = (j == VC && r < NX) ? v : 0.0;
    }
    const double* ex = L.exch + (size_t)w * 3 * TILE_D;
    V = combine_value(ld_tile_lds(ex), ld_tile_lds(ex + TILE_D), ld_tile_lds(ex + 2 * TILE_D), V,
                      om, Qj, buf);
    st_tile_lds(L.bnd + (size_t)(w - 1) * TILE_D, V);
  }
  __syncthreads();   // the boundary values reach the helpers
  backward<mode, false>(C, sh.p.r, sh.unit, 0, (int)(ktop / nch), V, nullptr, nullptr);
  __syncthreads();   // every chunk's gains and values are stored
  rollout<mode, LONG>(C, sh);
}

// A helper wave of a scanning workgroup: summary and recursion of its chunk
// for every scan command, until the first wave releases it.
__device__ INLINE void scan_helper(const Ctx& C, const uint8_t* unit) {
  const int wave = (int)(threadIdx.x >> 6), W = (int)(blockDim.x >> 6);
  const ScanLds L = scan_lds(W);
  ShR& sr = L.shr[wave - 1];
  for (;;) {
    __syncthreads();   // a command
    const int op = __builtin_amdgcn_readfirstlane(scan_ctl.op);
    if (op == SCAN_EXIT) return;
    const int nch = __builtin_amdgcn_readfirstlane(scan_ctl.nch);
    const bool mine = wave < nch;
    const int k0 = mine ? __builtin_amdgcn_readfirstlane(scan_ctl.bounds[wave]) : 0;
    const int k1 = mine ? __builtin_amdgcn_readfirstlane(scan_ctl.bounds[wave + 1]) : 0;
    if (mine) {
      d4 TE, CE, SE;
      if (op == SCAN_EQ)
        SE = backward<Mode::EQ, true>(C, sr, unit, k0, k1, zero4(), &TE, &CE);
      else
        SE = backward<Mode::NEWTON, true>(C, sr, unit, k0, k1, zero4(), &TE, &CE);
      double* ex = L.exch + (size_t)wave * 3 * TILE_D;
      st_tile_lds(ex, TE);
      st_tile_lds(ex + TILE_D, CE);
      st_tile_lds(ex + 2 * TILE_D, SE);
    }
    __syncthreads();   // summaries written
    __syncthreads();   // boundary values written
    if (mine) {
      const d4 V = ld_tile_lds(L.bnd + (size_t)wave * TILE_D);
      if (op == SCAN_EQ)
        backward<Mode::EQ, false>(C, sr, unit, k0, k1, V, nullptr, nullptr);
      else
        backward<Mode::NEWTON, false>(C, sr, unit, k0, k1, V, nullptr, nullptr);
    }
    __syncthreads();   // chunk recursions done
  }
}

// Releases the helpers of a scanning workgroup (the first wave, once).
__device__ inline void scan_release() {
  if (lane_id() == 0) scan_ctl.op = SCAN_EXIT;
  __syncthreads();
}
// How a problem's recursion runs: by one wave, by two, or as a scan over the horizon.
enum class Waves { ONE, PAIR, SCAN };
template <Mode mode, bool LONG, Waves WV>
__device__ INLINE void riccati(const Ctx& C, Sh& sh, int ktop) {
  if constexpr (WV == Waves::SCAN) riccati_scan<mode, LONG>(C, sh, ktop);
  else if constexpr (WV == Waves::PAIR) riccati_pair<mode, LONG>(C, sh, ktop);
  else riccati_t<mode, LONG>(C, sh, ktop);
}

// The equality pass's point from its rollout (u_k in GV, x_{k+1} in PV): inputs
// moved by rounding exactly onto their faces (closed form), states, and what
// the costates start from, Q (x_{k+1} - r_k) in PV and R (u_k - u_ref_k) in GV.
template <bool LONG>
__device__ INLINE void eq_point(const Ctx& C, Sh& sh) {
  const int lane = lane_id(), N = __builtin_amdgcn_readfirstlane(C.N);
  const StageBufs<LONG> sb(sh, C);
  const Scalars sc = scalars(C);
  const Buf rR = uref_buf(C), rU = rsrc(uni(C.ru), N * NU * 8);
  const auto ct = uni(C.contact);
  const auto fc = uni(C.faces);
  for (int e = fresh_lane(); e < N * 2; e += W64) {
    const int k = e >> 1, i = e & 1;
    float ur[6];
    const int code = fc[e];
    const bool on = ct[e];
    ldu6(rR, e, ur);
    double u[6];
#pragma unroll
    for (int a = 0; a < 6; ++a) u[a] = sb.GV[k * 16 + 6 * i + a];
    pin_all(ur);
    pin_all(u);
    pin_memory();
    if (on) {
      if (face_apex(code)) {
        u[0] = u[1] = u[2] = 0.0;
      } else {
        const ForceFace f = force_face(code);
        const double m = sc.mu;
        if (f.top) {
          if (f.sx != 0.0) u[0] = f.sx * m * sc.fz;
          if (f.sy != 0.0) u[1] = f.sy * m * sc.fz;
          u[2] = sc.fz;
        } else if (f.sx != 0.0 && f.sy != 0.0) {
          const double t = (m * (f.sx * u[0] + f.sy * u[1]) + u[2]) * sc.i2;
          u[0] = f.sx * m * t;
          u[1] = f.sy * m * t;
          u[2] = t;
        } else if (f.sx != 0.0 || f.sy != 0.0) {
          const double t = (f.sx * u[0] + f.sy * u[1] - m * u[2]) * sc.i1;
          u[0] -= f.sx * t;
          u[1] -= f.sy * t;
          u[2] += m * t;
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (code >> (8 + a) & 1) u[3 + a] = sc.tm;
        else if (code >> (11 + a) & 1) u[3 + a] = -sc.tm;
      }
    } else {
#pragma unroll
      for (int a = 0; a < 6; ++a) u[a] = 0.0;
    }
    st6(rU, e, u);
#pragma unroll
    for (int a = 0; a < 6; ++a)
      sb.GV[k * 16 + 6 * i + a] = sh.Rd[6 * i + a] * (u[a] - (double)ur[a]);
  }
  const Buf rX = rsrc(uni(C.x_ref), N * NX * 4);
  const gd px = uni(C.rx);
  for (int e0 = fresh_lane(); e0 < N * NX; e0 += 8 * W64) {
    double x[8], xr[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = e0 + t * W64, ec = e < N * NX ? e : e0;
      xr[t] = (double)ldf(rX, e * 4, 0);
      x[t] = sb.PV[(ec / NX) * 16 + ec % NX];
    }
    pin_memory();
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = e0 + t * W64;
      if (e < N * NX) {
        px[NX + e] = x[t];
        sb.PV[(e / NX) * 16 + e % NX] = sh.Qd[e % NX] * (x[t] - xr[t]);
      }
    }
  }
  if (lane < NX) px[lane] = (double)uni(C.x0)[lane];
  bufsync<LONG>();
}

// The same stage vectors from a point (ru, rx) in memory.
template <bool LONG>
__device__ inline void load_point(const Ctx& C, Sh& sh) {
  gsync();
  const int N = C.N;
  const StageBufs<LONG> sb(sh, C);
  for (int e = fresh_lane(); e < N * NX; e += W64)
    sb.PV[(e / NX) * 16 + e % NX] = C.Q[e % NX] * (C.rx[NX + e] - (double)C.x_ref[e]);
  for (int e = fresh_lane(); e < N * NU; e += W64) {
    const double ur = C.u_ref ? (double)C.u_ref[e] : 0.0;
    sb.GV[(e / NU) * 16 + e % NU] = C.R[e % NU] * (C.ru[e] - ur);
  }
  bufsync<LONG>();
}

// Costates p_{k+1} = Q (x_{k+1} - r_k) + A_{k+1}^T p_{k+2} (a chain, its data
// fetched CD stages ahead) and the reduced gradient g_k = R (u_k - u_ref_k) +
// B_k^T p_{k+1} (then, four stages at a time, one per 16-lane row), from and into
// the stage buffers.  Returns the state-side magnitude max |Q (x_{k+1} - r_k)|,
// |p|, |A^T p| over all stages, which the KKT scaling needs.
template <bool LONG>
__device__ INLINE double costates_grad(const Ctx& C, Sh& sh) {
  const StageBufs<LONG> sb(sh, C);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const auto rA = rsrc(uni(C.A), N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * NU * 4);
  const int oA = j < NX ? (3 * g * NX + j) * 4 : OOB, oA0 = (g == 0 && j < NX) ? j * 4 : OOB;
  // stage k needs A_{k+1}; at k = N - 1 the clamped stage multiplies p_{N+1} = 0
  struct CosRaw {
    float a[4];
    double q;
  };
  auto cfetch = [&](int k, CosRaw& s) {
    const int at = clampi(k + 1, N - 1) * (NX * NX * 4);
    s.a[0] = ldf(rA, oA0, at);
#pragma unroll
    for (int q = 1; q < 4; ++q) s.a[q] = ldf(rA, oA + q * NX * 4, at);
    s.q = j < NX ? sb.PV[k * 16 + j] : 0.0;
  };
  constexpr int CD = 12;
  CosRaw ring[CD];
#pragma unroll
  for (int d = 0; d < CD; ++d) {
    cfetch(N - 1 - d >= 0 ? N - 1 - d : 0, ring[d]);
    pin_memory();   // issued in ring order, as the loop issues them
  }
  double p = 0.0;   // p_{k+2}, entry j
  double tstate = 0.0;
  auto step = [&](int k, CosRaw& r) __attribute__((always_inline)) {
    double a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = (double)r.a[q];
      pin(a[q]);
    }
    const double qx = r.q;
    pin(qx);
    pin_memory();
    cfetch(k - CD >= 0 ? k - CD : 0, r);
    const double ap = row_total(dot4(turn_rows(p), a, 0.0));
    p = qx + ap;
    tstate = fmax(tstate, fmax(fabs(qx), fmax(fabs(p), fabs(ap))));
    if (lane < NX) sb.PV[k * 16 + j] = p;
  };
  static_assert(CD == 12, "one line below per ring slot");
  for (int k = N - 1;; k -= CD) {
    if (!(k >= 0)) break;
    step(k, ring[0]);
    if (!(k - 1 >= 0)) break;
    step(k - 1, ring[1]);
    if (!(k - 2 >= 0)) break;
    step(k - 2, ring[2]);
    if (!(k - 3 >= 0)) break;
    step(k - 3, ring[3]);
    if (!(k - 4 >= 0)) break;
    step(k - 4, ring[4]);
    if (!(k - 5 >= 0)) break;
    step(k - 5, ring[5]);
    if (!(k - 6 >= 0)) break;
    step(k - 6, ring[6]);
    if (!(k - 7 >= 0)) break;
    step(k - 7, ring[7]);
    if (!(k - 8 >= 0)) break;
    step(k - 8, ring[8]);
    if (!(k - 9 >= 0)) break;
    step(k - 9, ring[9]);
    if (!(k - 10 >= 0)) break;
    step(k - 10, ring[10]);
    if (!(k - 11 >= 0)) break;
    step(k - 11, ring[11]);
  }
  bufsync<LONG>();
  const int oB = j < NU ? (g * NX * NU + j) * 4 : OOB;
  auto bfetch = [&](int k0, float (&s)[NX]) {
#pragma unroll
    for (int r = 0; r < NX; ++r) s[r] = ldf(rB, oB + r * NU * 4, k0 * (NX * NU * 4));
  };
  constexpr int GD = 4;
  float br[GD][NX];
#pragma unroll
  for (int d = 0; d < GD; ++d) {
    bfetch(4 * d < N ? 4 * d : 0, br[d]);
    pin_memory();
  }
  auto grad = [&](int k0, float (&r)[NX]) __attribute__((always_inline)) {
    const int k = k0 + g;
    double b[NX];
#pragma unroll
    for (int l = 0; l < NX; ++l) {
      b[l] = (double)r[l];
      pin(b[l]);
    }
    pin_memory();
    bfetch(k0 + 4 * GD < N ? k0 + 4 * GD : k0, r);
    const bool on = j < NU && k < N;
    const double pk = (j < NX && k < N) ? sb.PV[k * 16 + j] : 0.0;
    const double ru = on ? sb.GV[k * 16 + j] : 0.0;
    const double gk = dot_row_bcast13(pk, b, ru);
    if (on) sb.GV[k * 16 + j] = gk;
  };
  static_assert(GD == 4, "one line below per ring slot");
  for (int k0 = 0;; k0 += 4 * GD) {
    if (!(k0 < N)) break;
    grad(k0, br[0]);
    if (!(k0 + 4 < N)) break;
    grad(k0 + 4, br[1]);
    if (!(k0 + 8 < N)) break;
    grad(k0 + 8, br[2]);
    if (!(k0 + 12 < N)) break;
    grad(k0 + 12, br[3]);
  }
  bufsync<LONG>();
  return wave_max(tstate);
}

// x = rollout of ru from x0, in FP64, into rx: the stage terms B u + e for four
// stages at a time, then the chain.
template <bool LONG>
__device__ INLINE void rollout_ru(const Ctx& C, Sh& sh) {
  gsync();
  const StageBufs<LONG> sb(sh, C);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const gcf pe = uni(C.e), pA = uni(C.A);
  const auto rA = rsrc(pA, N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * NU * 4);
  const auto rE = rsrc(pe ? pe : pA, pe ? N * NX * 4 : 0), rU = rsrc(uni(C.ru), N * NU * 8);
  const int oB = j < NX ? (g * NX + j) * NU * 4 : OOB;
  const int oE = j < NX ? (g * NX + j) * 4 : OOB, oU = j < NU ? (g * NU + j) * 8 : OOB;
  for (int k0 = 0; k0 < N; k0 += 4) {
    float b[NU];
#pragma unroll
    for (int l = 0; l < NU; l += 4) ldf4(rB, oB + l * 4, k0 * (NX * NU * 4), b + l);
    double bd[NX];
#pragma unroll
    for (int l = 0; l < NX; ++l) bd[l] = l < NU ? (double)b[l < NU ? l : 0] : 0.0;
    const double u = ldd(rU, oU, k0 * (NU * 8)), e = (double)ldf(rE, oE, k0 * (NX * 4));
    const double d = dot_row_bcast13(u, bd, e);
    if (j < NX && k0 + g < N) sb.PV[(k0 + g) * 16 + j] = d;
  }
  bufsync<LONG>();
  const int oA = j < NX ? (j * NX + 3 * g) * 4 : OOB;
  struct RollRaw {
    float a[4];
    double t;
  };
  auto rfetch = [&](int k, RollRaw& s) {
    ldf4(rA, oA, k * (NX * NX * 4), s.a);
    s.t = j < NX ? sb.PV[k * 16 + j] : 0.0;
  };
  constexpr int RD = 12;
  RollRaw ring[RD];
#pragma unroll
  for (int d = 0; d < RD; ++d) {
    rfetch(d < N ? d : N - 1, ring[d]);
    pin_memory();
  }
  double xv = j < NX ? (double)uni(C.x0)[clampi(j, NX - 1)] : 0.0;
  auto step = [&](int k, RollRaw& r) __attribute__((always_inline)) {
    double a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = (q == 0 && g) ? 0.0 : (double)r.a[q];
      pin(a[q]);
    }
    const double t = r.t;
    pin(t);
    pin_memory();
    rfetch(k + RD < N ? k + RD : N - 1, r);
    xv = row_total(dot4(turn_rows(xv), a, 0.0)) + t;
    if (lane < NX) sb.PV[k * 16 + j] = xv;
  };
  static_assert(RD == 12, "one line below per ring slot");
  for (int k = 0;; k += RD) {
    if (!(k < N)) break;
    step(k, ring[0]);
    if (!(k + 1 < N)) break;
    step(k + 1, ring[1]);
    if (!(k + 2 < N)) break;
    step(k + 2, ring[2]);
    if (!(k + 3 < N)) break;
    step(k + 3, ring[3]);
    if (!(k + 4 < N)) break;
    step(k + 4, ring[4]);
    if (!(k + 5 < N)) break;
    step(k + 5, ring[5]);
    if (!(k + 6 < N)) break;
    step(k + 6, ring[6]);
    if (!(k + 7 < N)) break;
    step(k + 7, ring[7]);
    if (!(k + 8 < N)) break;
    step(k + 8, ring[8]);
    if (!(k + 9 < N)) break;
    step(k + 9, ring[9]);
    if (!(k + 10 < N)) break;
    step(k + 10, ring[10]);
    if (!(k + 11 < N)) break;
    step(k + 11, ring[11]);
  }
  bufsync<LONG>();
  if (lane < NX) C.rx[lane] = (double)C.x0[lane];
  for (int e = fresh_lane(); e < N * NX; e += W64) C.rx[NX + e] = sb.PV[(e / NX) * 16 + e % NX];
  gsync();
}

// Order-independent hash term of contact-stage e's face code.
__device__ inline uint64_t face_hash(int code, int e) {
  uint64_t v = (uint64_t)(code + 1) * 0x9E3779B97F4A7C15ull ^ ((uint64_t)(e + 1) * 0xC2B2AE3D27D4EB4Full);
  v ^= v >> 29;
  return v * 0xBF58476D1CE4E5B9ull;
}

// A face update's outcome: the hash of the new face set and one past the last
// stage whose face changed (0: none did).
struct FaceUpdate {
  uint64_t hash;
  int ktop;
};

// Row multipliers of each stance contact from its face and the gradient, and
// the normalised KKT residuals of the current (u, x, p, mu).  Returns KKT.
// With update, also the primal-dual active-set update of the faces (row active iff
// mu_r s_r + (G_r u - h_r) > 0): the multipliers it needs are in registers here.
// The force multipliers solve G_A^T mu_A = -g_f on the face's rows (least
// squares); the Gram systems of the eight faces that are not the apex are solved
// in closed form (see face_affine).
template <bool LONG>
__device__ INLINE double multipliers_kkt(const Ctx& C, Sh& sh, double res[PINMPC_NRES],
                                 double term_state, bool update, FaceUpdate* upd) {
  const StageBufs<LONG> sb(sh, C);
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const Scalars sc = scalars(C);
  const Buf rR = uref_buf(C), rU = rsrc(uni(C.ru), N * NU * 8);
  const auto ct = uni(C.contact);
  const auto fc = uni(C.faces);
  double r_ineq = 0.0, stat = 0.0, term = term_state, comp = 0.0, mumax = 0.0, neg = 0.0;
  uint64_t hsh = 0;
  int kch = 0;
  for (int e = fresh_lane(); e < N * 2; e += W64) {
    const int k = e >> 1, i = e & 1;
    // the contact-stage's inputs, gradient and multipliers in registers
    double u[6], g[6], mu[NROW];
    float ur[6];
    const int code = fc[e];
    const bool on = ct[e];
    ld6(rU, e, u);
    ldu6(rR, e, ur);
#pragma unroll
    for (int a = 0; a < 6; ++a) g[a] = sb.GV[k * 16 + 6 * i + a];
    pin_all(u);
    pin_all(ur);
    pin_all(g);
    pin_memory();
    int fresh = 0;
    if (!on) {
      for (int a = 0; a < 6; ++a) r_ineq = fmax(r_ineq, fabs(u[a]) * sc.img);
    } else {
#pragma unroll
      for (int r = 0; r < NROW; ++r) mu[r] = 0.0;
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        const double ru = sh.Rd[6 * i + a] * (u[a] - (double)ur[a]);
        term = fmax(term, fmax(fabs(ru), fabs(g[a] - ru)));
      }
      if (face_apex(code)) {
        // at the apex the four side rows are dependent: take the three-row
        // subset whose multipliers are most nonnegative (some subset is
        // nonnegative exactly when -g_f lies in the normal cone of the apex).
        // The rows are [+-1, 0, -mu] and [0, +-1, -mu]: with b = -g_f and
        // S = -b_z / mu the three-row systems are
        //   mu0 - mu1 = b_x,  mu2 - mu3 = b_y,  mu0 + mu1 + mu2 + mu3 = S
        // with the dropped multiplier zero, solved in closed form
        const double bx = -g[0], by = -g[1], S = g[2] / sc.mu;
        double cand[4][4];
        cand[0][0] = 0.0;                    cand[0][1] = -bx;
        cand[0][2] = 0.5 * (S + bx + by);    cand[0][3] = 0.5 * (S + bx - by);
        cand[1][0] = bx;                     cand[1][1] = 0.0;
        cand[1][2] = 0.5 * (S - bx + by);    cand[1][3] = 0.5 * (S - bx - by);
        cand[2][0] = 0.5 * (S + by + bx);    cand[2][1] = 0.5 * (S + by - bx);
        cand[2][2] = 0.0;                    cand[2][3] = -by;
        cand[3][0] = 0.5 * (S - by + bx);    cand[3][1] = 0.5 * (S - by - bx);
        cand[3][2] = by;                     cand[3][3] = 0.0;
        double best = -1e300;
        int pick = 0;
#pragma unroll
        for (int drop = 0; drop < 4; ++drop) {
          double mn = 1e300;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i != drop) mn = fmin(mn, cand[drop][i]);
          if (mn > best) {
            best = mn;
            pick = drop;
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          double v = cand[0][i];
#pragma unroll
          for (int d = 1; d < 4; ++d) v = (pick == d) ? cand[d][i] : v;
          mu[i] = v;
        }
      } else {
        const ForceFace f = force_face(code);
        const double m = sc.mu;
        double mx, my, mt = 0.0;
        if (f.top) {
          // the bound fixes f_z: each side row alone holds its component
          mx = -f.sx * g[0];
          my = -f.sy * g[1];
          mt = m * (mx + my) - g[2];
        } else {
          const double rx = f.sx != 0.0 ? m * g[2] - f.sx * g[0] : 0.0;
          const double ry = f.sy != 0.0 ? m * g[2] - f.sy * g[1] : 0.0;
          const bool two = f.sx != 0.0 && f.sy != 0.0;
          const double w = two ? sc.i2 : sc.i1, d = two ? m * m * (rx - ry) : 0.0;
          mx = (rx + d) * w;
          my = (ry - d) * w;
        }
        mu[0] = f.sx > 0.0 ? mx : 0.0;
        mu[1] = f.sx < 0.0 ? mx : 0.0;
        mu[2] = f.sy > 0.0 ? my : 0.0;
        mu[3] = f.sy < 0.0 ? my : 0.0;
        mu[4] = mt;
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (code >> (8 + a) & 1) mu[5 + a] = -g[3 + a];
        else if (code >> (11 + a) & 1) mu[8 + a] = g[3 + a];
      }
      // residual pieces, and the updated face
      double gu[NROW], gm[6] = {0, 0, 0, 0, 0, 0};
      rows_of(sc, u, gu);
      rows_T(sc, mu, gm);
#pragma unroll
      for (int r = 0; r < NROW; ++r) {
        const double d = gu[r] - row_h(sc, r);
        r_ineq = fmax(r_ineq, fmax(0.0, d) * sc.img);
        comp = fmax(comp, mu[r] * fmax(0.0, -d));
        mumax = fmax(mumax, mu[r]);
        neg = fmax(neg, -mu[r]);
        if (fma(mu[r], row_scale(sc, r), d) > 0.0) fresh |= row_bit(r);
      }
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        term = fmax(term, fabs(gm[a]));
        stat = fmax(stat, no_nan(fabs(g[a] + gm[a])));
      }
      fresh = settle_face(fresh);
    }
    if (update) {
      if (code != fresh) {
        kch = k + 1;
        fc[e] = fresh;
      }
      hsh ^= face_hash(fresh, e);
    }
  }
  if (update) {
    upd->ktop = wave_max_int(kch);
    upd->hash = wave_xor(hsh);
  }
  // the state-side term norms (|Q (x - r)|, |p|, |A^T p|) come in as
  // term_state from the costate recursion, which holds them
  r_ineq = wave_max(r_ineq);
  stat = wave_max(stat);
  term = wave_max(term);
  comp = wave_max(comp);
  mumax = wave_max(mumax);
  neg = wave_max(neg);
  res[0] = 0.0;   // r_dyn: filled by the caller from the rollout
  res[1] = r_ineq;
  res[2] = term < __builtin_inf() ? stat / (1.0 + term) : term;
  res[3] = comp / (1.0 + mumax * sc.mg);
  res[4] = fmax(0.0, neg) / (1.0 + term);
  double kkt = 0.0;
  for (int i = 1; i < PINMPC_NRES; ++i) kkt = fmax(kkt, no_nan(res[i]));
  return kkt;
}

// Dynamics residual of the FP64 trajectory (rx, ru), four stages at a time (one
// per 16-lane row, state j in lane j).
__device__ INLINE double dyn_residual(const Ctx& C) {
  gsync();
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const gcf pe = uni(C.e), pA = uni(C.A);
  const auto rA = rsrc(pA, N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * NU * 4);
  const auto rE = rsrc(pe ? pe : pA, pe ? N * NX * 4 : 0);
  const auto rU = rsrc(uni(C.ru), N * NU * 8), rX = rsrc(uni(C.rx), (N + 1) * NX * 8);
  const int oA = j < NX ? (g * NX + j) * NX * 4 : OOB, oB = j < NX ? (g * NX + j) * NU * 4 : OOB;
  const int oX = j < NX ? (g * NX + j) * 8 : OOB, oU = j < NU ? (g * NU + j) * 8 : OOB;
  const int oE = j < NX ? (g * NX + j) * 4 : OOB;
  struct DynRaw {
    float a[NX], b[NU], e;
    double x, xn, u;
  };
  auto fetch = [&](int k0, DynRaw& s) {
#pragma unroll
    for (int l = 0; l < NU; l += 4) {
      ldf4(rA, oA + l * 4, k0 * (NX * NX * 4), s.a + l);
      ldf4(rB, oB + l * 4, k0 * (NX * NU * 4), s.b + l);
    }
    s.a[NU] = ldf(rA, oA + NU * 4, k0 * (NX * NX * 4));
    s.e = ldf(rE, oE, k0 * (NX * 4));
    s.x = ldd(rX, oX, k0 * (NX * 8));
    s.xn = ldd(rX, oX + NX * 8, k0 * (NX * 8));
    s.u = ldd(rU, oU, k0 * (NU * 8));
  };
  constexpr int DD = 3;
  DynRaw ring[DD];
#pragma unroll
  for (int d = 0; d < DD; ++d) {
    fetch(4 * d < N ? 4 * d : 0, ring[d]);
    pin_memory();
  }
  double res = 0.0;
  auto step = [&](int k0, DynRaw& r) __attribute__((always_inline)) {
    double a[NX], b[NX];
#pragma unroll
    for (int l = 0; l < NX; ++l) {
      a[l] = (double)r.a[l];
      b[l] = l < NU ? (double)r.b[l < NU ? l : 0] : 0.0;
      pin(a[l]);
      pin(b[l]);
    }
    const double x = r.x, xn = r.xn, u = r.u, ee = (double)r.e;
    pin(x); pin(xn); pin(u); pin(ee);
    pin_memory();
    fetch(k0 + 4 * DD < N ? k0 + 4 * DD : k0, r);
    const double ax = dot_row_bcast13(x, a, 0.0), bu = dot_row_bcast13(u, b, 0.0);
    const double d = xn - ax - bu - ee;
    const double den = 1.0 + fmax(fabs(xn), fmax(fabs(ax), fabs(bu)));
    if (j < NX && k0 + g < N) res = fmax(res, no_nan(fabs(d) / den));
  };
  static_assert(DD == 3, "one line below per ring slot");
  for (int k0 = 0;; k0 += 4 * DD) {
    if (!(k0 < N)) break;
    step(k0, ring[0]);
    if (!(k0 + 4 < N)) break;
    step(k0 + 4, ring[1]);
    if (!(k0 + 8 < N)) break;
    step(k0 + 8, ring[2]);
  }
  return wave_max(res);
}

// Faces from slack: rows whose slack is below tol * row scale.
__device__ INLINE void faces_from_u(const Ctx& C, double tol) {
  gsync();
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const Scalars sc = scalars(C);
  const Buf rU = rsrc(uni(C.ru), N * NU * 8);
  for (int e = fresh_lane(); e < N * 2; e += W64) {
    double u[6], gu[NROW];
    const bool on = uni(C.contact)[e];
    ld6(rU, e, u);
    rows_of(sc, u, gu);
    int code = 0;
#pragma unroll
    for (int r = 0; r < NROW; ++r)
      if ((row_h(sc, r) - gu[r]) / row_scale(sc, r) <= tol) code |= row_bit(r);
    if (face_apex(code)) code = (code & ~31) | FACE_APEX;
    uni(C.faces)[e] = on ? code : 0;
  }
  wsync();
}

// One active-set pass: equality-constrained solve on the current faces (`solve`;
// else the point in memory is taken as it is), costates, multipliers and
// residuals.  `ktop` < N: the faces of stages ktop..N-1 are those of the previous
// equality-constrained solve, whose tiles and factors are still in the scratch
// block.  The pass's x is the FP64 rollout of its u, so its dynamics residual is
// rounding only: it is checked once, on the final trajectory, by the caller.
template <bool LONG, Waves WV>
__device__ INLINE double eq_pass(const Ctx& C, Sh& sh, double res[PINMPC_NRES], bool solve,
                                 int ktop, bool update, FaceUpdate* upd) {
  if (solve) {
    riccati<Mode::EQ, LONG, WV>(C, sh, ktop);
    eq_point<LONG>(C, sh);
  } else {
    load_point<LONG>(C, sh);
  }
  const double ts = costates_grad<LONG>(C, sh);
  return multipliers_kkt<LONG>(C, sh, res, ts, update, upd);
}

// Faces of the interior point's iterate: row active iff z > s.
__device__ INLINE void faces_from_zs(const Ctx& C) {
  gsync();
  const int N = __builtin_amdgcn_readfirstlane(C.N), step = __builtin_amdgcn_readfirstlane(C.n) * 16;
  const Buf rS = row_buf(C, C.rs), rZ = row_buf(C, C.rz);
  for (int e = fresh_lane(); e < N * 2; e += W64) {
    double zv[NROW], sv[NROW];
    const bool on = uni(C.contact)[e];
    load_r(rZ, step, e, zv);
    load_r(rS, step, e, sv);
    int code = 0;
#pragma unroll
    for (int r = 0; r < NROW; ++r)
      if (zv[r] > sv[r]) code |= row_bit(r);
    uni(C.faces)[e] = on ? settle_face(code) : 0;
  }
  wsync();
}

// Work done by the refinement of one problem: equality-constrained passes
// (active-set, crossover and polish passes), interior-point iterations, and
// the stages whose backward recursion an equality pass factored (a pass that
// restarts at stage ktop factors ktop stages).
struct Counts {
  int eq, ipm, stf;
};

// Least centring weight of the corrector after SIGMA_FROM iterations.
// Mehrotra's (mu_aff / mu)^3 alone lets a few products run far ahead of the
// others on degenerate problems, and the steps then stay short for tens of
// iterations: 64 problems of 100 to 400 stages took up to 130.  Few problems up
// to 64 stages reach that many: of 2 x 4096 of 30 to 60 stages with a normal-force
// bound 1.15 times the weight and narrow moment bounds 25, which then take up to 49
// iterations (72 without the floor) and are all certified either way.
constexpr int SIGMA_FROM = 40;
constexpr double SIGMA_MIN = 0.05;

// The input blocks and pivot masks of every contact-stage from the iterate
// (u, s, z) in memory: the identity and zero for a swing contact.
__device__ INLINE void newton_blocks(const Ctx& C, Sh& sh) {
  gsync();
  const int N = __builtin_amdgcn_readfirstlane(C.N), step = __builtin_amdgcn_readfirstlane(C.n) * 16;
  const Scalars sc = scalars(C);
  const Buf rU = rsrc(uni(C.ru), N * NU * 8), rR = uref_buf(C);
  const Buf rS = row_buf(C, C.rs), rZ = row_buf(C, C.rz);
  const gd pT = uni(C.rT);
  for (int e = fresh_lane(); e < N * 2; e += W64) {
    double u[6], sv[NROW], zv[NROW];
    float ur[6];
    const bool on = uni(C.contact)[e];
    ld6(rU, e, u);
    ldu6(rR, e, ur);
    load_r(rS, step, e, sv);
    load_r(rZ, step, e, zv);
    pin_all(u);
    pin_all(ur);
    pin_all(sv);
    pin_all(zv);
    pin_memory();
    sh.unit[e] = on ? 0 : 0x3F;
    if (on) {
      newton_block(sc, sh.Rd + 6 * (e & 1), pT, e, u, ur, sv, zv);
    } else {
      InputBlock t;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        t.d[a] = 1.0;
        t.v[a] = t.v[3 + a] = 0.0;
#pragma unroll
        for (int b = 0; b < 3; ++b) t.m[a][b] = a == b ? 1.0 : 0.0;
      }
      store_block(pT + (size_t)e * 18, t);
    }
  }
}

// A contact-stage's iterate and step, in the registers of the lane that owns it.
struct RowState {
  double u[6], s[NROW], z[NROW], ds[NROW], dz[NROW];
  float ur[6];
};

// Interior-point fallback.  Rows scaled by mg (force rows) and tau_max
// (moment rows).  Crossover: once the face guess z > s is the same after two
// consecutive iterations, one equality-constrained pass on those faces is
// tried (the iterate is kept aside and restored if it does not certify).  ipm_run
// iterates until it wants such a pass (true: the iterate is kept aside) or is
// done (false: the faces from z > s are left for the polish passes).
//
// Besides the recursions an iteration passes three times over its rows, one lane
// per contact-stage: the predictor's steps and the corrector's linear term, the
// corrector's steps, and the move to the new iterate with its faces and its next
// input blocks.  The few problems that come here leave the chip nearly empty
// (about 430 waves on its 1024 SIMDs with 4096 problems of 20 stages), so a pass
// costs its latency: the trip to memory, the reciprocals and the reductions.
// Ratios therefore share the reciprocal of a product and are reduced as one
// maximum of step over distance, and the last two passes keep a contact-stage's
// rows in registers while every lane has only one.
struct IpmState {
  int it;
  uint64_t hprev;
  double m, smz, rpn;   // stance rows; this lane's share of s z, largest row residual
};
template <bool LONG>
__device__ INLINE void ipm_start(const Ctx& C, Sh& sh, IpmState& st) {
  gsync();
  const int N = __builtin_amdgcn_readfirstlane(C.N), step = __builtin_amdgcn_readfirstlane(C.n) * 16;
  const auto ct = uni(C.contact);
  // number of stance rows
  int mloc = 0;
  for (int e = fresh_lane(); e < N * 2; e += W64)
    if (ct[e]) mloc += NROW;
  st = {0, 0, wave_sum((double)mloc), 0.0, 0.0};
  // initial point: the current ru (the ADMM point) and its rollout in rx,
  // slacks at least 1, multipliers 1 (a start from the last active-set pass,
  // its slacks and multipliers floored at 1e-1 .. 1e-3, took as long or
  // longer: the early steps near the boundary are short); and the residuals
  // of that point
  {
    const Scalars sc = scalars(C);
    const Buf rU = rsrc(uni(C.ru), N * NU * 8), rS = row_buf(C, C.rs), rZ = row_buf(C, C.rz);
    for (int e = fresh_lane(); e < N * 2; e += W64) {
      double u[6], gu[NROW], sv[NROW], zv[NROW];
      const bool on = ct[e];
      ld6(rU, e, u);
      rows_of(sc, u, gu);
#pragma unroll
      for (int r = 0; r < NROW; ++r) {
        const double d = gu[r] - row_h(sc, r), isc = row_isc(sc, r);
        sv[r] = fmax(-d * isc, 1.0);
        zv[r] = 1.0;
        if (on) {
          st.rpn = fmax(st.rpn, fabs(fma(d, isc, sv[r])));
          st.smz += sv[r] * zv[r];
        }
      }
      store_r(rS, step, e, sv);
      store_r(rZ, step, e, zv);
    }
  }
  {
    const Buf rX = rsrc(uni(C.rx), (N + 1) * NX * 8), rXr = rsrc(uni(C.x_ref), N * NX * 4);
    const gd pq = uni(C.rq);
    for (int e0 = fresh_lane(); e0 < N * NX; e0 += 4 * W64) {
      double x[4], xr[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        x[t] = ldd(rX, (NX + e0 + t * W64) * 8, 0);
        xr[t] = (double)ldf(rXr, (e0 + t * W64) * 4, 0);
      }
      pin_memory();
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int e = e0 + t * W64;
        if (e < N * NX) pq[e] = sh.Qd[e % NX] * (x[t] - xr[t]);
      }
    }
  }
}
template <bool LONG, Waves WV>
__device__ INLINE bool ipm_run(const Ctx& C, Sh& sh, IpmState& st, int maxit) {
  if (st.m == 0.0) return false;
  const int N = __builtin_amdgcn_readfirstlane(C.N), step = __builtin_amdgcn_readfirstlane(C.n) * 16;
  const auto ct = uni(C.contact);
  const StageBufs<LONG> sb(sh, C);
  const bool one_each = 2 * N <= W64;   // every lane owns at most one contact-stage
  newton_blocks(C, sh);   // (an equality pass leaves its own blocks)
  for (; st.it < maxit; ++st.it) {
    const int it = st.it;
    const double sz = wave_sum(st.smz), muv = sz / st.m;
    if (scalar(muv <= 1e-10 && wave_max(st.rpn) <= 1e-9)) break;
    // predictor (affine target s z)
    riccati<Mode::NEWTON, LONG, WV>(C, sh, N);
    const Scalars sc = scalars(C);
    const Buf rU = rsrc(uni(C.ru), N * NU * 8), rR = uref_buf(C);
    const Buf rS = row_buf(C, C.rs), rZ = row_buf(C, C.rz);
    const Buf rC = row_buf(C, C.rrc);   // complementarity target, less sigma mu
    // its row steps; the largest step to the boundary, as 1 / max(1, step over
    // distance); the sums that give the complementarity after any step,
    // s z + a (s dz + z ds) + a^2 ds dz; and the corrector's linear term per
    // input for the target s z + ds dz - sigma mu, whose part in sigma mu goes
    // to PV and the rest to GV
    double over = 1.0, sm1 = 0.0, sm2 = 0.0;
    for (int e = fresh_lane(); e < N * 2; e += W64) {
      const int k = e >> 1, i = e & 1;
      double u[6], du[6], sv[NROW], zv[NROW];
      float ur[6];
      const bool on = ct[e];
      ld6(rU, e, u);
      ldu6(rR, e, ur);
      load_r(rS, step, e, sv);
      load_r(rZ, step, e, zv);
#pragma unroll
      for (int t = 0; t < 6; ++t) du[t] = sb.GV[k * 16 + 6 * i + t];
      pin_all(u);
      pin_all(ur);
      pin_all(sv);
      pin_all(zv);
      pin_all(du);
      pin_memory();
      double ra[6] = {0, 0, 0, 0, 0, 0}, rb[6] = {0, 0, 0, 0, 0, 0};
      if (on) {
        double gu[NROW], gdu[NROW], cv[NROW], ca[NROW], cb[NROW];
#pragma unroll
        for (int t = 0; t < 6; ++t) ra[t] = sh.Rd[6 * i + t] * (u[t] - (double)ur[t]);
        rows_of(sc, u, gu);
        rows_of(sc, du, gdu);
#pragma unroll
        for (int r = 0; r < NROW; ++r) {
          const double isc = row_isc(sc, r), is = recip(sv[r]);
          const double rp = fma(gu[r] - row_h(sc, r), isc, sv[r]);
          const double ds = -fma(gdu[r], isc, rp);
          const double t = ds * is, dz = -fma(zv[r], t, zv[r]);
          over = fmax(over, fmax(-t, 1.0 + t));
          sm1 += sv[r] * dz + zv[r] * ds;
          sm2 += ds * dz;
          cv[r] = fma(ds, dz, sv[r] * zv[r]);
          ca[r] = fma(fma(zv[r], rp, -cv[r]), is, zv[r]) * isc;
          cb[r] = is * isc;
        }
        store_r(rC, step, e, cv);
        rows_T(sc, ca, ra);
        rows_T(sc, cb, rb);
      }
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        sb.GV[k * 16 + 6 * i + t] = ra[t];
        sb.PV[k * 16 + 6 * i + t] = rb[t];
      }
    }
    const double aa = recip(wave_max(over));
    const double mu_aff = fmax(fma(aa, fma(aa, wave_sum(sm2), wave_sum(sm1)), sz), 0.0) / st.m;
    const double ratio = mu_aff / muv, cube = ratio * ratio * ratio,
                 smu = (it < SIGMA_FROM ? cube : fmax(cube, SIGMA_MIN)) * muv;
    // corrector: the recursion's vector part and the rollout with the
    // predictor's factors
    bufsync<LONG>();
    newton_vector<LONG>(C, sh, smu);
    forward_map<LONG, true>(C, sh);
    // its row steps, and the largest step over distance
    over = 1.0;
    auto row_steps = [&](int e, bool on, RowState& w) __attribute__((always_inline)) {
      const int k = e >> 1, i = e & 1;
      double du[6], gu[NROW], gdu[NROW], cv[NROW];
      ld6(rU, e, w.u);
      ldu6(rR, e, w.ur);
      load_r(rS, step, e, w.s);
      load_r(rZ, step, e, w.z);
      load_r(rC, step, e, cv);
#pragma unroll
      for (int t = 0; t < 6; ++t) du[t] = sb.GV[k * 16 + 6 * i + t];
      rows_of(sc, w.u, gu);
      rows_of(sc, du, gdu);
#pragma unroll
      for (int r = 0; r < NROW; ++r) {
        const double isc = row_isc(sc, r);
        const double rp = fma(gu[r] - row_h(sc, r), isc, w.s[r]);
        const double isz = recip(w.s[r] * w.z[r]), is = w.z[r] * isz, iz = w.s[r] * isz;
        w.ds[r] = -fma(gdu[r], isc, rp);
        w.dz[r] = -fma(w.z[r], w.ds[r], cv[r] - smu) * is;
        if (on) over = fmax(over, fmax(-w.ds[r] * is, -w.dz[r] * iz));
      }
    };
    // the step, the residuals and affine target of the new point, its face guess
    // and its input block; a lane moves its own contact-stage (swing inputs stay 0)
    uint64_t hsh = 0;
    double smz = 0.0, rpn = 0.0;
    const gd pT = uni(C.rT);
    const auto fc = uni(C.faces);
    auto advance = [&](int e, RowState& w, double a) __attribute__((always_inline)) {
      const int k = e >> 1, i = e & 1;
      double gu[NROW];
      int code = 0;
#pragma unroll
      for (int t = 0; t < 6; ++t) w.u[t] += a * sb.GV[k * 16 + 6 * i + t];
      st6(rU, e, w.u);
      rows_of(sc, w.u, gu);
#pragma unroll
      for (int r = 0; r < NROW; ++r) {
        w.s[r] += a * w.ds[r];
        w.z[r] += a * w.dz[r];
        rpn = fmax(rpn, fabs(fma(gu[r] - row_h(sc, r), row_isc(sc, r), w.s[r])));
        smz += w.s[r] * w.z[r];
        if (w.z[r] > w.s[r]) code |= row_bit(r);
      }
      store_r(rS, step, e, w.s);
      store_r(rZ, step, e, w.z);
      code = settle_face(code);
      fc[e] = code;
      hsh ^= face_hash(code, e);
      newton_block(sc, sh.Rd + 6 * i, pT, e, w.u, w.ur, w.s, w.z);
    };
    double a;
    if (one_each) {
      RowState w;
      const int lane = fresh_lane();
      const int e = lane < 2 * N ? lane : 2 * N - 1;   // surplus lanes repeat the last's loads
      const bool on = ct[e] && lane < 2 * N;
      row_steps(e, on, w);
      a = 0.99 * recip(wave_max(over));
      if (on) advance(e, w, a);
    } else {
      const Buf rDs = row_buf(C, C.rds), rDz = row_buf(C, C.rdz);
      for (int e = fresh_lane(); e < N * 2; e += W64) {
        RowState w;
        row_steps(e, ct[e], w);
        store_r(rDs, step, e, w.ds);
        store_r(rDz, step, e, w.dz);
      }
      a = 0.99 * recip(wave_max(over));
      for (int e = fresh_lane(); e < N * 2; e += W64) {
        RowState w;
        const bool on = ct[e];
        ld6(rU, e, w.u);
        ldu6(rR, e, w.ur);
        load_r(rS, step, e, w.s);
        load_r(rZ, step, e, w.z);
        load_r(rDs, step, e, w.ds);
        load_r(rDz, step, e, w.dz);
        pin_all(w.u);
        pin_all(w.ur);
        pin_all(w.s);
        pin_all(w.z);
        pin_all(w.ds);
        pin_all(w.dz);
        pin_memory();
        if (on) advance(e, w, a);
      }
    }
    // states (x_0 is fixed) and their cost gradients: loads of a group first,
    // then its stores
    {
      const Buf rX = rsrc(uni(C.rx), (N + 1) * NX * 8), rXr = rsrc(uni(C.x_ref), N * NX * 4);
      const gd px = uni(C.rx), pq = uni(C.rq);
      for (int e0 = fresh_lane(); e0 < N * NX; e0 += 8 * W64) {
        double x[8], xr[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int e = e0 + t * W64, ec = e < N * NX ? e : e0;
          x[t] = ldd(rX, (NX + e) * 8, 0);
          xr[t] = (double)ldf(rXr, e * 4, 0);
          x[t] += a * sb.PV[(ec / NX) * 16 + ec % NX];
        }
        pin_memory();
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int e = e0 + t * W64;
          if (e < N * NX) {
            px[NX + e] = x[t];
            pq[e] = sh.Qd[e % NX] * (x[t] - xr[t]);
          }
        }
      }
    }
    st.smz = smz;
    st.rpn = rpn;
    const uint64_t h = wave_xor(hsh);
    const bool cross = scalar(it >= 1 && h == st.hprev);
    st.hprev = h;
    if (cross) {
      // the step buffers are free between iterations: keep the iterate there
      ++st.it;
      gsync();
      copy_doubles(uni(C.rdu), C.ru, N * NU);
      copy_doubles(uni(C.rdx), C.rx, (N + 1) * NX);
      return true;
    }
  }
  faces_from_zs(C);
  return false;
}

// The ADMM's input iterate, unscaled, into ru (swing inputs exactly 0).
__device__ INLINE void admm_point(const Ctx& C, gcf zsrc, gcf sf, float tsc) {
  gsync();
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const auto ct = uni(C.contact);
  const gd pu = uni(C.ru);
  for (int e0 = fresh_lane(); e0 < N * NU; e0 += 4 * W64) {
    float z[4], f[4];
    int on[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = e0 + t * W64, ec = e < N * NU ? e : e0, k = ec / NU, j = ec % NU;
      z[t] = zsrc[(k * NSTATE) * NL + NX + j];
      f[t] = sf[k];
      on[t] = ct[k * 2 + j / 6];
    }
    pin_memory();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = e0 + t * W64, j = e % NU;
      const double sc = (j % 6 < 3) ? (double)f[t] : (double)tsc;
      if (e < N * NU) pu[e] = on[t] ? (double)z[t] * sc : 0.0;
    }
  }
  wsync();
}

// PHASE 1 runs every problem's active-set passes; a problem they do not
// certify (with the interior point enabled) is appended to ws.rlist and left
// to PHASE 2, which runs the interior point and the polish passes for the
// listed problems only (surplus blocks exit).  The slow problems thus start
// together instead of behind a second round of easy ones.
// The doubles of a buffer as floats, zero past its end.
__device__ inline void put_floats(float* out, Buf r, int count) {
  for (int e0 = fresh_lane(); e0 < count; e0 += 8 * W64) {
    double v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = ldd(r, (e0 + t * W64) * 8, 0);
    pin_memory();
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (e0 + t * W64 < count) out[e0 + t * W64] = (float)v[t];
  }
}

// The first wave releases a workgroup's other waves on every way out.
template <Waves WV>
struct Release {
  __device__ INLINE ~Release() {
    if constexpr (WV == Waves::SCAN) scan_release();
    if constexpr (WV == Waves::PAIR) pair_release();
  }
};

constexpr int threads_of(Waves w) {
  return w == Waves::SCAN ? W64 * SCAN_WMAX : (w == Waves::PAIR ? 2 * W64 : W64);
}
template <int PHASE, bool LONG, Waves WV>
__global__ void __launch_bounds__(threads_of(WV), 2) refine_kernel(Problem p, Workspace ws, float* out_u,
                                                    float* out_x, float* out_res,
                                                    int32_t* out_iters, int32_t* out_status,
                                                    int32_t* out_detail,
                                                    int admm_iters, int accel, int refine,
                                                    int pass_a, int ipm_max, int pass_c,
                                                    double tol, int pass_1, int pair_max) {
  __shared__ Sh sh;
  // the problem context lives in LDS: its pointers are loaded where they are
  // used instead of being held in registers across the whole kernel
  __shared__ Ctx C;
  int pb = blockIdx.x;
  if (PHASE == 2) {
    const int listed = ws.rcount[0];
    if ((int)blockIdx.x >= listed) return;
    // of the two builds launched, the one that this many problems are faster with
    if (WV != Waves::SCAN && (listed <= pair_max) != (WV == Waves::PAIR)) return;
    pb = ws.rlist[blockIdx.x];
  }
  if constexpr (WV == Waves::PAIR) {
    if (threadIdx.x >= W64) {
      pair_helper<PHASE == 2>(C, sh);
      return;
    }
  }
  if constexpr (WV == Waves::SCAN) {
    // with the horizon scan the workgroup holds one wave per chunk: all but
    // the first take the scan's commands until the first releases them
    if (threadIdx.x >= W64) {
      scan_helper(C, sh.unit);
      return;
    }
  }
  const Release<WV> release;
  const int lane = lane_id();
  if (lane == 0) {
  C.b = pb;
  C.n = p.n_max;
  C.N = horizon(p, C.b);
  const size_t s0 = (size_t)C.b * C.n;
  C.mu = p.mu[C.b];
  C.fz = p.fz_max[C.b];
  C.tm = p.tau_max[C.b];
  C.mg = weight_of(p, C.b);
  C.i1 = 1.0 / (1.0 + C.mu * C.mu);
  C.i2 = 1.0 / (1.0 + 2.0 * C.mu * C.mu);
  C.img = 1.0 / C.mg;
  C.itm = 1.0 / C.tm;
  C.Q = (const LMEM double*)sh.Qd;
  C.R = (const LMEM double*)sh.Rd;
  C.A = (gcf)(p.A + s0 * NX * NX);
  C.B = (gcf)(p.B + s0 * NX * NU);
  C.e = p.e ? (gcf)(p.e + s0 * NX) : nullptr;
  C.x_ref = (gcf)(p.x_ref + s0 * NX);
  C.u_ref = p.u_ref ? (gcf)(p.u_ref + s0 * NU) : nullptr;
  C.x0 = (gcf)(p.x0 + (size_t)C.b * NX);
  C.contact = (const GMEM uint8_t*)(p.contact + s0 * 2);
  {
    const int n = C.n;
    gd blk = (gd)(ws.rblk + (size_t)C.b * refine_block_doubles(n));
    C.rT = blk;                       blk += (size_t)n * TS_T;
    C.rT2 = C.rM = blk;               blk += (size_t)n * (TS_T + TS_PAD);
    C.rF = blk;                       blk += (size_t)n * TS_F;
    C.rK = blk;                       blk += (size_t)n * TS_K;
    C.rS = blk;                       blk += (size_t)n * TS_S;
    C.ru = blk;                       blk += (size_t)n * NU;
    C.rq = blk;                       blk += (size_t)n * NX;
    C.rs = blk;                       blk += (size_t)n * 2 * NROW;
    C.rz = blk;                       blk += (size_t)n * 2 * NROW;
    C.rds = blk;                      blk += (size_t)n * 2 * NROW;
    C.rdz = blk;                      blk += (size_t)n * 2 * NROW;
    C.rrc = blk;                      blk += (size_t)n * 2 * NROW;
    C.rdu = blk;                      blk += (size_t)n * NU;
    C.rx = blk;                       blk += (size_t)(n + 1) * NX;
    C.rdx = blk;                      blk += (size_t)(n + 1) * NX;
    C.rPV = blk;                      blk += (size_t)n * 16;
    C.rGV = blk;   // inside the block only for n > PINMPC_NMAX (LONG)
    C.faces = (GMEM int32_t*)(ws.faces + s0 * 2);
  }
  }
  if (lane < NX) sh.Qd[lane] = p.Q[(size_t)pb * NX + lane];
  if (lane < NU) sh.Rd[lane] = p.R[(size_t)pb * NU + lane];
  wsync();
  const size_t s0 = (size_t)pb * p.n_max;
  const int N = C.N;

  // input checks, in the first launch (the second one's problems passed them):
  // finiteness of the scalars and weights, then the bounds (a friction
  // coefficient must be positive: mu = 0 leaves the pyramid without f_z >= 0 and
  // its apex multipliers undefined), then finiteness of this problem's stage data
  const size_t ux = (size_t)C.b * C.n * NU, xx = (size_t)C.b * (C.n + 1) * NX;
  if (PHASE == 1) {
    const int Nraw = horizon_raw(p, C.b);
    int nonfinite = !isfinite(C.mu) || !isfinite(C.fz) || !isfinite(C.tm) || !isfinite(C.mg);
    for (int j = 0; j < NX; ++j) nonfinite |= !isfinite(C.Q[j]);
    for (int j = 0; j < NU; ++j) nonfinite |= !isfinite(C.R[j]);
    int bad = 0;
    if (!nonfinite) {
      bad = !(C.mu > 0.0) || !(C.fz >= 0.0) || !(C.tm >= 0.0) || !(C.mg > 0.0) || Nraw < 1 ||
            Nraw > C.n;
      for (int j = 0; j < NX; ++j) bad |= !(C.Q[j] > 0.0);
      for (int j = 0; j < NU; ++j) bad |= !(C.R[j] > 0.0);
    }
    if (!bad && !nonfinite) {
      int nf = any_nonfinite(uni(C.A), N * NX * NX) | any_nonfinite(uni(C.B), N * NX * NU) |
               any_nonfinite(uni(C.x_ref), N * NX);
      if (C.e) nf |= any_nonfinite(uni(C.e), N * NX);
      if (C.u_ref) nf |= any_nonfinite(uni(C.u_ref), N * NU);
      if (lane < NX) nf |= !isfinite(C.x0[lane]);
      if (p.u_prev && lane < NU) nf |= !isfinite(p.u_prev[(size_t)C.b * NU + lane]);
      nonfinite = wave_max_int(nf) > 0;
    }
    if (bad || nonfinite) {
      for (int e = fresh_lane(); e < C.n * NU; e += W64) out_u[ux + e] = 0.f;
      for (int e = fresh_lane(); e < (C.n + 1) * NX; e += W64) out_x[xx + e] = 0.f;
      if (lane == 0) {
        if (out_status) out_status[C.b] = bad ? PINMPC_ST_BADINPUT : PINMPC_ST_NONFINITE;
        if (out_iters) out_iters[C.b] = 0;
      }
      if (out_detail && lane < 4) out_detail[(size_t)C.b * 4 + lane] = 0;
      if (out_res && lane < PINMPC_NRES) out_res[(size_t)C.b * PINMPC_NRES + lane] = __builtin_nanf("");
      return;
    }
  }

  gcf zsrc = (gcf)((accel ? ws.cur : ws.hat) + s0 * NSTATE * NL);
  gcf sf = (gcf)(ws.sf + s0);
  const float tsc = ws.tsc[C.b];
  if (PHASE == 1) admm_point(C, zsrc, sf, tsc);

  // Passes until one certifies, the face set repeats or their number is spent;
  // then (second launch) the interior point with its crossover passes, then polish
  // passes again.  One loop, so that the pass is in the kernel once.  The first
  // launch takes pass_1 passes (all pass_a when pass_1 is 0) and leaves the rest to
  // the second.  Without refinement the ADMM point is evaluated as it is: rollout,
  // faces from slack, residuals.
  double res[PINMPC_NRES] = {0, 0, 0, 0, 0};
  Counts cnt = {0, 0, 0};
  bool ok = false, cycled = false;
  enum { PASSES, INTERIOR, POLISH } part = PASSES;
  const int p1 = (pass_1 > 0 && pass_1 < pass_a) ? pass_1 : pass_a;
  int left = refine ? p1 : 1;
  if (PHASE == 1) {
    faces_from_u(C, 1e-5);
    if (!refine) rollout_ru<LONG>(C, sh);
  } else {
    // resume from the faces the first launch left
    const int rp = __builtin_amdgcn_readfirstlane(ws.rpass[C.b]);
    cnt.eq = rp & 1023;
    cnt.stf = (rp >> 10) & ((1 << 20) - 1);
    left = ((rp >> 30) & 1) ? pass_a - cnt.eq : 0;
  }
  IpmState ist = {0, 0, 0.0, 0.0, 0.0};
  uint64_t hist[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // the last face sets
  int nh = 0, ktop = N;   // the first pass solves the whole horizon
  for (;;) {
    bool cross = false;
    if constexpr (PHASE == 2) {
      if (part == PASSES && (left <= 0 || cycled)) {
        if (ipm_max <= 0) break;
        // interior point from the ADMM point
        admm_point(C, zsrc, sf, tsc);
        rollout_ru<LONG>(C, sh);
        ipm_start<LONG>(C, sh, ist);
        part = INTERIOR;
      }
      if (part == INTERIOR) {
        cross = ipm_run<LONG, WV>(C, sh, ist, ipm_max);
        if (!cross) {
          part = POLISH;
          left = pass_c;
          cycled = false;
          nh = 0;
          ktop = N;
        }
      }
    }
    if (!cross && (left <= 0 || cycled)) break;
    FaceUpdate upd;
    const bool update = refine && !cross;
    const int kt = cross || ktop > N ? N : ktop;
    const double kkt = eq_pass<LONG, WV>(C, sh, res, PHASE == 2 || refine, kt, update, &upd);
    if (PHASE == 1 && !refine) break;
    ++cnt.eq;
    cnt.stf += kt;
    ok = scalar(kkt <= tol);
    if (ok) break;
    if (cross) {
      gsync();
      copy_doubles(uni(C.ru), C.rdu, N * NU);
      copy_doubles(uni(C.rx), C.rdx, (N + 1) * NX);
      continue;
    }
    ktop = __builtin_amdgcn_readfirstlane(upd.ktop);
    for (int i = 0; i < 8; ++i) cycled |= hist[i] == upd.hash && (i < nh || nh >= 8);
    cycled = scalar(cycled);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if ((nh & 7) == i) hist[i] = upd.hash;
    ++nh;
    --left;
  }
  cnt.ipm = ist.it;
  if (PHASE == 1 && refine && !ok && (ipm_max > 0 || (!cycled && p1 < pass_a))) {
    if (lane == 0) {
      const int slot = atomicAdd(ws.rcount, 1);
      ws.rlist[slot] = C.b;
      // passes (< 2^10, settings are capped at 1000) and stages factored
      // (< 2^20) so far, and whether active-set passes remain
      ws.rpass[C.b] = cnt.eq | (cnt.stf << 10) | (!cycled && p1 < pass_a ? (1 << 30) : 0);
    }
    return;
  }
  // the dynamics residual of the returned trajectory, checked independently
  // of the rollout that produced it
  res[0] = dyn_residual(C);
  ok = ok && res[0] <= tol;

  // outputs
  gsync();
  put_floats(out_u + ux, rsrc(uni(C.ru), N * NU * 8), C.n * NU);
  put_floats(out_x + xx, rsrc(uni(C.rx), (N + 1) * NX * 8), (C.n + 1) * NX);
  if (lane == 0) {
    // the solve's refinement work (stages of every pass and iteration)
    atomicAdd(ws.work, (unsigned long long)(cnt.eq + cnt.ipm) * (unsigned long long)N);
    if (out_status)
      out_status[C.b] = refine ? (ok ? PINMPC_ST_OK : PINMPC_ST_UNPOLISHED) : PINMPC_ST_MAXITER;
    if (out_iters) out_iters[C.b] = admm_iters + cnt.eq + cnt.ipm;
  }
  if (out_detail && lane < 4) {
    const int v = lane == 0 ? cnt.eq : lane == 1 ? cnt.ipm : lane == 2 ? cnt.stf : PHASE;
    out_detail[(size_t)C.b * 4 + lane] = v;
  }
  if (out_res) {
    for (int i = 0; i < PINMPC_NRES; ++i)
      if (lane == i) out_res[(size_t)C.b * PINMPC_NRES + i] = (float)res[i];
  }
}

}  // namespace

// The first launch runs a problem by two waves while two waves per SIMD hold the
// whole batch (the registers allow no more).  With more problems two single waves on
// a SIMD do the same work without the meetings.
// The second launch's problems are fewer, and each one's time is its chain, so pairs
// pay longer: 3001 problems of 8 to 60 stages, half of them listed, 7.8 ms with one
// wave each, 6.8 ms with two; 24 of 160 stages 35 and 28 ms.  From about 1.2 to 2.5
// listed problems per SIMD either may win by up to 15 %: pairs where the listed have
// different lengths or mostly need a few passes more, single waves where every one
// needs the interior point in 10 or 20 stages.  Beyond (first_passes or refine_passes of
// a few leave it most of a large batch) one wave is as fast or faster: both launches of
// 4096 x 20 with first_passes = 2 take 3.16 ms with one, 3.56 with two, of 3001 x 40
// 6.24 and 6.70, of 4096 x 10 without active-set passes 1.78 and 2.21.  The device alone
// knows the number, so above that batch both builds are launched and one exits at once
// (a few microseconds).
struct PairRule {
  int first, second;   // most problems run by pairs in either launch
};
PairRule pair_rule() {
  const int simds = 4 * device_cus();
  return {simds, simds * 5 / 2};
}

size_t scan_lds_bytes(int W) {
  return W > 1 ? (size_t)(W - 1) * sizeof(ShR) + (size_t)W * 4 * TILE_D * sizeof(double) : 0;
}

hipError_t refine_prepare() {
  // the scanning kernels may take more dynamic LDS than the default limit
  const int lds = (int)scan_lds_bytes(SCAN_WMAX);
  const void* k[] = {reinterpret_cast<const void*>(&refine_kernel<1, false, Waves::SCAN>),
                     reinterpret_cast<const void*>(&refine_kernel<1, true, Waves::SCAN>),
                     reinterpret_cast<const void*>(&refine_kernel<2, false, Waves::SCAN>),
                     reinterpret_cast<const void*>(&refine_kernel<2, true, Waves::SCAN>)};
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_refine(const Problem& p, const Workspace& w, const pinmpc_settings& s,
                         const pinmpc_out& out, hipStream_t st) {
  if (p.batch == 0) return hipSuccess;
  const bool second =
      s.refine && (s.ipm_iters > 0 || (s.first_passes > 0 && s.first_passes < s.refine_passes));
  if (second) {
    // the hand-off counter starts at zero (a fill kernel: graph-safe)
    const hipError_t e = launch_fill_i32(w.rcount, 1, 0, 0, st);
    if (e != hipSuccess) return e;
  }
  // the horizon scan: one wave per chunk, dynamic LDS for the helpers'
  // buffers, the summaries and the boundary values
  const int W = s.scan > 1 ? s.scan : 1;
  const size_t lds = scan_lds_bytes(W);
#define PINMPC_REFINE(PH, L, WV, T)                                                               \
  hipLaunchKernelGGL((refine_kernel<PH, L, Waves::WV>), dim3(p.batch), dim3(T), lds, st, p, w,     \
                     out.u, out.x, out.res, out.iters, out.status, out.detail, s.iters, s.accel,   \
                     s.refine, s.refine_passes, s.ipm_iters, s.polish_passes, s.kkt_tol,           \
                     s.first_passes, rule.second)
#define PINMPC_REFINE_L(PH, WV, T)              \
  do {                                          \
    if (lng) PINMPC_REFINE(PH, true, WV, T);    \
    else PINMPC_REFINE(PH, false, WV, T);       \
  } while (0)
  // horizons beyond PINMPC_NMAX keep the rollout's and the costates' stage
  // buffers in the scratch block (refine_block_doubles sizes it so)
  const bool lng = p.n_max > PINMPC_NMAX;
  const PairRule rule = pair_rule();
  if (W > 1) {
    PINMPC_REFINE_L(1, SCAN, 64 * W);
    if (second) PINMPC_REFINE_L(2, SCAN, 64 * W);
  } else {
    if (p.batch <= rule.first) PINMPC_REFINE_L(1, PAIR, 128);
    else PINMPC_REFINE_L(1, ONE, 64);
    if (second) PINMPC_REFINE_L(2, PAIR, 128);
    if (second && p.batch > rule.second) PINMPC_REFINE_L(2, ONE, 64);
  }
#undef PINMPC_REFINE_L
#undef PINMPC_REFINE
  return hipGetLastError();
}

}  // namespace pinmpc
