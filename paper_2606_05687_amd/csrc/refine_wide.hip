// FP64 refinement and certificate of problems with four contacts per stage
// (the feet and the hands of loco-manipulation, Sec. II-A: 24 inputs), one
// 64-lane wave per problem.
//
// The ADMM of Sec. III ends near the optimum; from its point the kernel runs a
// primal-dual interior point with Mehrotra's predictor-corrector on the QP
// (the same QP the two-contact refinement certifies), all in FP64:
//   rows     each stance contact's eleven wrench rows g_r . u_c <= h_r (Sec.
//            II-B, in the contact's own frame), scaled by m g (force rows) and
//            tau_max (moment rows), slacks s >= 0 and multipliers z >= 0;
//   Newton   every step is the LQ problem in (du, dx) with input Hessian
//            R' = R + G^T diag(z / s) G (per contact a 6 x 6 block; the
//            identity on a swing contact's inputs, which stay zero), linear
//            input term rho = R (u - u_ref) + G^T (z + (z rp - rc) / s) and
//            state term q = Q (x_{k+1} - r_k), solved by the backward Riccati
//            recursion over the horizon and a forward rollout of the gains;
//   stop     when the point's KKT residuals, with multipliers refitted to its
//            gradient, meet the tolerance.
// The returned u is the last iterate, x its rollout in FP64, and res its
// normalised residuals (r_dyn, r_ineq, r_stat, r_comp, r_sign).
//
// The 24 inputs are handled as two halves of 12 (a: contacts 0 and 1, b: 2 and
// 3), each the size the two-contact tiles and elimination are built for.  Per
// stage 51 matrix instructions form W Ba, W Bb, the blocks Haa, Hab, Hbb of
// H = R' + B^T W B, Hwx and the value function; half a is eliminated beside
// Hab and its right-hand sides, half b after the Schur update, and half a's
// gains follow by back substitution (H = U^T D U with U = [Ua, Tab; 0, Ub],
// whose factors the corrector keeps).  A stage built entry by entry through LDS
// (products on the vector units, a 24-column elimination broadcast by lane
// reads) took about 25 000 cycles, and each stage of the chains 6 000.
#include "refine_tiles.h"

namespace pinmpc {

namespace {

constexpr int C4 = 4;                 // contacts
constexpr int U4 = 6 * C4;            // 24 inputs
constexpr int L4 = NX + U4;           // 37 lifted rows of the ADMM iterates
// doubles per stage of the scratch blocks: the input blocks of four contacts,
// the gains [K | kap] of both halves (12 x 14 each), the factors Ua, Ub and Tab
constexpr int WT = C4 * 18, WK = 2 * NU * (NX + 1), WF = 3 * NU * NU;
constexpr int KB = NU * (NX + 1) * 8;   // byte offset of half b's gains in a stage
constexpr int FB = NU * NU * 8;         // of Ub (and twice that: Tab) in a stage

// The problem's FP64 scratch (refine_wide_block_doubles(n) doubles).
struct WCtx {
  int b, n, N;
  double mu, fz, tm, mg, scf, scm;   // bounds, force scale, row scales
  double isf, ism;                   // inverse row scales
  gcf A, B, e, x_ref, u_ref, x0;
  const GMEM uint8_t* contact;       // [n][4]
  gd T, K, F, u, s, z, ds, dz, rc, q, x;
};

static_assert(refine_wide_block_doubles(1) >=
                  (size_t)WT + WK + WF + U4 + 5 * C4 * NROW + NX + 2 * NX,
              "the carve below fits the scratch block");

__device__ inline void carve(WCtx& C, gd blk) {
  const int n = C.n;
  C.T = blk;    blk += (size_t)n * WT;
  C.K = blk;    blk += (size_t)n * WK;
  C.F = blk;    blk += (size_t)n * WF;
  C.u = blk;    blk += (size_t)n * U4;
  C.s = blk;    blk += (size_t)n * C4 * NROW;
  C.z = blk;    blk += (size_t)n * C4 * NROW;
  C.ds = blk;   blk += (size_t)n * C4 * NROW;
  C.dz = blk;   blk += (size_t)n * C4 * NROW;
  C.rc = blk;   blk += (size_t)n * C4 * NROW;
  C.q = blk;    blk += (size_t)n * NX;
  C.x = blk;
}

// LDS: the stage recursion's hand-off buffers (columns of 12 at stride GC), or
// the per-stage vectors of the chains; the two are never in use together.
constexpr int GC = 14;
struct WSh {
  union {
    struct {
      alignas(16) double G[(NU + 16) * GC];   // [H | right-hand sides] of a half
      alignas(16) double Tab[NU * GC];        // D^-1 Ua^-T Hab
      alignas(16) double Yab[NU * GC];        // Ua^-T Hab
      double ST[16 * 17];                     // a tile for its transpose
    } r;
    struct {
      double PV[PINMPC_NMAX * NX];   // dx_{k+1}, x_{k+1}, Q (x_{k+1} - r_k), p_{k+1}
      double GV[PINMPC_NMAX * U4];   // du_k, rho_k, hw_k, kap_k, B_k^T p_{k+1}
    } c;
  };
  double Q[NX], R[U4];
  uint32_t unit[PINMPC_NMAX];        // swing inputs of a stage, a byte per contact
};

__device__ inline bool stance(const WCtx& C, int k, int i) { return C.contact[k * C4 + i] != 0; }

// g_r . u for the eleven rows of one contact (u its six inputs), with h_r and
// the inverse row scale: pyramid sides, normal-force bound, moment box.
__device__ inline void rows_of(const WCtx& C, const double u[6], double gu[NROW], double h[NROW],
                               double isc[NROW]) {
  gu[0] = u[0] - C.mu * u[2];
  gu[1] = -u[0] - C.mu * u[2];
  gu[2] = u[1] - C.mu * u[2];
  gu[3] = -u[1] - C.mu * u[2];
  gu[4] = u[2];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    gu[5 + a] = u[3 + a];
    gu[8 + a] = -u[3 + a];
  }
#pragma unroll
  for (int r = 0; r < NROW; ++r) {
    h[r] = r < 4 ? 0.0 : (r == 4 ? C.fz : C.tm);
    isc[r] = r < 5 ? C.isf : C.ism;
  }
}

// G^T v for one contact (v one value per row).
__device__ inline void rows_T(const WCtx& C, const double v[NROW], double o[6]) {
  o[0] = v[0] - v[1];
  o[1] = v[2] - v[3];
  o[2] = -C.mu * (v[0] + v[1] + v[2] + v[3]) + v[4];
#pragma unroll
  for (int a = 0; a < 3; ++a) o[3 + a] = v[5 + a] - v[8 + a];
}

__device__ inline void ld6(gcd p, double v[6]) {
#pragma unroll
  for (int t = 0; t < 6; ++t) v[t] = p[t];
}
// A row's entries for consecutive contact-stages are consecutive in memory
// (rs = 4 n_max apart per row).
__device__ inline void ldr(gcd p, int rs, int e, double v[NROW]) {
#pragma unroll
  for (int r = 0; r < NROW; ++r) v[r] = p[r * rs + e];
}
__device__ inline void str(gd p, int rs, int e, const double v[NROW]) {
#pragma unroll
  for (int r = 0; r < NROW; ++r) p[r * rs + e] = v[r];
}

// The passes over the rows (one lane per contact-stage) load all they need before
// any branch on it: each trip to memory costs about as much as a pass's
// arithmetic, and a load under `if (u_ref)` or `if (stance)` is one more (six for
// the components of u_ref).
__device__ inline __amdgpu_buffer_rsrc_t uref_buf(const WCtx& C) {
  const gcf p = uni(C.u_ref);   // none: an empty buffer, which reads as zeros
  return rsrc(p ? p : uni(C.A), p ? C.N * U4 * 4 : 0);
}
struct RowLoads {
  bool on;
  double u[6], s[NROW], z[NROW];
  float ur[6];
};
__device__ inline void load_rows(const WCtx& C, __amdgpu_buffer_rsrc_t rR, int rs, int e,
                                 RowLoads& w) {
  w.on = uni(C.contact)[e] != 0;
  ldf3(rR, e * 24, 0, w.ur);
  ldf3(rR, e * 24 + 12, 0, w.ur + 3);
  ld6(uni(C.u) + e * 6, w.u);
  ldr(uni(C.s), rs, e, w.s);
  ldr(uni(C.z), rs, e, w.z);
}
__device__ inline void pin_rows(const RowLoads& w) {
#pragma unroll
  for (int r = 0; r < NROW; ++r) {
    pin(w.s[r]);
    pin(w.z[r]);
  }
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    pin(w.u[t]);
    asm volatile("" ::"v"(w.ur[t]));
  }
  pin_memory();
}

// Stage inputs of the Newton step, in parallel over (stage, contact): the R'
// block and rho of every contact at the affine target s z (identity and zero on
// a swing contact), and the state cost gradients q.
__device__ inline void build_terms(const WCtx& C, WSh& sh) {
  const int rs = C4 * C.n;
  const auto rR = uref_buf(C);
  __syncthreads();
  for (int e = fresh_lane(); e < C.N * C4; e += W64) {
    const int i = e % C4;
    RowLoads w;
    load_rows(C, rR, rs, e, w);
    pin_rows(w);
    InputBlock t;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      t.d[a] = 1.0;
#pragma unroll
      for (int b = 0; b < 3; ++b) t.m[a][b] = a == b ? 1.0 : 0.0;
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) t.v[a] = 0.0;
    if (w.on) {
      double gu[NROW], h[NROW], isc[NROW], d[NROW], c[NROW];
      rows_of(C, w.u, gu, h, isc);
#pragma unroll
      for (int r = 0; r < NROW; ++r) {
        const double rp = fma(gu[r] - h[r], isc[r], w.s[r]), zs = w.z[r] * recip(w.s[r]);
        d[r] = zs * (isc[r] * isc[r]);
        c[r] = zs * rp * isc[r];
      }
      const double m = C.mu;
      double rho[6];
      rows_T(C, c, rho);
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        const int j = 6 * i + a;
        t.v[a] = fma(sh.R[j], w.u[a] - (double)w.ur[a], rho[a]);
      }
      t.m[0][0] = d[0] + d[1] + sh.R[6 * i];
      t.m[0][1] = t.m[1][0] = 0.0;
      t.m[0][2] = t.m[2][0] = -m * (d[0] - d[1]);
      t.m[1][1] = d[2] + d[3] + sh.R[6 * i + 1];
      t.m[1][2] = t.m[2][1] = -m * (d[2] - d[3]);
      t.m[2][2] = m * m * (d[0] + d[1] + d[2] + d[3]) + d[4] + sh.R[6 * i + 2];
#pragma unroll
      for (int a = 0; a < 3; ++a) t.d[a] = d[5 + a] + d[8 + a] + sh.R[6 * i + 3 + a];
    }
    reinterpret_cast<uint8_t*>(sh.unit)[e] = w.on ? 0 : 0x3F;
    store_block(C.T + (size_t)e * 18, t);
  }
  const int nx = C.N * NX;
  const gd pq = uni(C.q), px = uni(C.x);
  const gcf pr = uni(C.x_ref);
  for (int e0 = fresh_lane(); e0 < nx; e0 += 8 * W64) {
    double x[8];
    float xr[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = e0 + t * W64 < nx ? e0 + t * W64 : e0;
      x[t] = px[NX + e];
      xr[t] = pr[e];
    }
    pin_memory();
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = e0 + t * W64;
      if (e < nx) pq[e] = sh.Q[e % NX] * (x[t] - (double)xr[t]);
    }
  }
  __syncthreads();
}

// Forward elimination of a half's system c1 = [H | right-hand sides] (as factor)
// with the columns c2 of Hab beside it (column j in lane j of every 16-lane row):
// y2 ends with Ua^-T Hab, c2 with D^-1 times that.  The pivot column comes from
// c1's lanes, so c2's update of a pivot goes first.
template <int p = 0>
__device__ inline void factor_beside(double (&c1)[12], double (&c2)[12], double (&y2)[12], int hc,
                                     uint32_t unit) {
  if constexpr (p < 12) {
    y2[p] = c2[p];
    if (!((unit >> p) & 1u)) {
      const double rd = recip(row_bcast<p>(c1[p]));
      const double t1 = c1[p] * rd, t2 = c2[p] * rd, n2 = -t2;
      if constexpr (p < 11) asm volatile("s_nop 1");
#pragma unroll
      for (int r = p + 1; r < 12; ++r)
        asm volatile(
            "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(c2[r])
            : "v"(c1[r]), "v"(n2), "i"(p));
      fmac_rows<p, p + 1, 12>(c1, -t1);
      c1[p] = hc == p ? rd : t1;
      c2[p] = t2;
    }
    factor_beside<p + 1>(c1, c2, y2, hc, unit);
  }
}

struct WideRaw {
  float a[4], ba[4], bb[4];
  double q[4], ta[3], tb[3];
};

// Backward recursion of the Newton step, stages N-1 .. 0: gains, feedforward and
// factors of every stage into the scratch.  Tiles are homogeneous (row and
// column VC carry the linear terms), as in the two-contact recursion.
__device__ __attribute__((always_inline)) inline void backward(const WCtx& C, WSh& sh) {
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const auto rA = rsrc(uni(C.A), N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * U4 * 4);
  const auto rQ = rsrc(uni(C.q), N * NX * 8), rT = rsrc(uni(C.T), N * WT * 8);
  const auto rK = rsrc(uni(C.K), N * WK * 8), rF = rsrc(uni(C.F), N * WF * 8);
  const int oA = j < NX ? (g * NX + j) * 4 : OOB;
  const int oA3 = (g == 0 && j < NX) ? (12 * NX + j) * 4 : OOB;
  const int oB = j < NU ? (g * U4 + j) * 4 : OOB;
  const int oB3 = (g == 0 && j < NU) ? (12 * U4 + j) * 4 : OOB;
  const int oV = j == VC ? g * 8 : OOB;
  const int oV3 = (g == 0 && j == VC) ? 96 : ((g == 1 && j < NX) ? j * 8 : OOB);
  int oT[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) oT[q] = t_offset(4 * q + g, j);
  const int oK = j <= VC ? (g * (NX + 1) + j) * 8 : OOB;
  const int oF = j < NU ? (g * NU + j) * 8 : OOB;
  d4 Qd;
#pragma unroll
  for (int q = 0; q < 4; ++q) Qd[q] = (4 * q + g == j && j < NX) ? sh.Q[clampi(j, NX - 1)] : 0.0;
  const SymWeights sw = sym_weights();
  const double one = (g == 1 && j == VC) ? 1.0 : 0.0;   // (VC, VC) as item 3
  const int hc = lane & 15, rhs = 4 * (lane >> 4) + hc - NU, jc = clampi(j, NU - 1);
  const bool is_h = hc < NU, in = j < NU;
  double* const gc = sh.r.G + (is_h ? hc : NU + rhs) * GC;
  auto fetch = [&](int k, WideRaw& s) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      s.a[q] = ldf(rA, oA + q * 4 * NX * 4, k * (NX * NX * 4));
      s.ba[q] = ldf(rB, oB + q * 4 * U4 * 4, k * (NX * U4 * 4));
      s.bb[q] = ldf(rB, oB + q * 4 * U4 * 4 + NU * 4, k * (NX * U4 * 4));
      s.q[q] = ldd(rQ, oV + q * 32, k * (NX * 8));
      s.ta[q] = ldd(rT, oT[q], k * (WT * 8));
      s.tb[q] = ldd(rT, oT[q] + WT * 4, k * (WT * 8));
    }
    s.a[3] = ldf(rA, oA3, k * (NX * NX * 4));
    s.ba[3] = ldf(rB, oB3, k * (NX * U4 * 4));
    s.bb[3] = ldf(rB, oB3 + NU * 4, k * (NX * U4 * 4));
    s.q[3] = ldd(rQ, oV3, k * (NX * 8));
  };
  WideRaw raw;
  fetch(N - 1, raw);
  d4 Ss = zero4();
  for (int k = N - 1; k >= 0; --k) {
    // this stage's data, the swing contacts' columns of B zero
    const uint32_t ub = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.unit[k]);
    const uint32_t ua = (ub & 0x3F) | ((ub >> 2) & 0xFC0), uc = ((ub >> 16) & 0x3F) | ((ub >> 18) & 0xFC0);
    const bool ka = in && !((ua >> jc) & 1u), kb = in && !((uc >> jc) & 1u);
    d4 At, Da, Db, Wt, Ta = zero4(), Tb = zero4();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      At[q] = (double)raw.a[q];
      Da[q] = ka ? (double)raw.ba[q] : 0.0;
      Db[q] = kb ? (double)raw.bb[q] : 0.0;
      Wt[q] = Ss[q] + (Qd[q] + raw.q[q]);
    }
    Da[3] += one;
    Db[3] += one;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      Ta[q] = raw.ta[q];
      Tb[q] = raw.tb[q];
    }
    pin(At); pin(Da); pin(Db); pin(Wt); pin(Ta); pin(Tb);
    pin_memory();
    if (k > 0) fetch(k - 1, raw);

    const d4 D3a = mmT<4>(Wt, Da, zero4());   // [W Ba | 0 | q + s], row VC Ba^T (q + s)
    const d4 Haa = mmT<4>(D3a, Da, Ta);       // [Haa | 0 | hwa]
    const d4 Hxa = mmT<4>(D3a, At, zero4());
    const d4 Hab = mmT<4>(D3a, Db, zero4());
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int r = 4 * q + g;
      if (in) {
        sh.r.G[j * GC + r] = Haa[q];
        sh.r.Tab[j * GC + r] = Hab[q];
      }
      sh.r.G[(NU + j) * GC + r] = -(j == VC ? Haa[q] : Hxa[q]);
    }
    const d4 D3b = mmT<4>(Wt, Db, zero4());
    d4 Hbb = mmT<4>(D3b, Db, Tb);             // [Hbb | 0 | hwb]
    const d4 Hxb = mmT<4>(D3b, At, zero4());
    d4 D2 = mmT<4>(Wt, At, zero4());          // [W A | q + s]
#pragma unroll
    for (int q = 0; q < 4; ++q) D2[q] = j == VC ? D3a[q] : D2[q];
    const d4 SA = mmT<4>(At, D2, zero4());
    wsync();
    // half a: lane 16 R + c holds column c of Haa (c < 12, the same in every row
    // R) or right-hand side 4 R + c - 12, and column c of Hab
    double c1[NU];
    {
      double c2[NU], y2[NU];
      const double* hb = sh.r.Tab + clampi(hc, NU - 1) * GC;
#pragma unroll
      for (int r = 0; r < NU; ++r) {
        c1[r] = gc[r];
        c2[r] = hb[r];
      }
      wsync();
      factor_beside(c1, c2, y2, hc, ua);
      if (!is_h || lane < NU) {
#pragma unroll
        for (int r = 0; r < NU; ++r) gc[r] = c1[r];
      }
      if (lane < NU) {
#pragma unroll
        for (int r = 0; r < NU; ++r) {
          sh.r.Tab[lane * GC + r] = c2[r];
          sh.r.Yab[lane * GC + r] = y2[r];
        }
      }
      wsync();
    }
    d4 Tx = zero4(), Tab = zero4(), nTt = zero4(), nY = zero4(), X = zero4();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int r = 4 * q + g;
      Tx[q] = sh.r.G[(NU + j) * GC + r];
      const double tab = sh.r.Tab[jc * GC + r], tt = sh.r.Tab[r * GC + jc];
      const double y = sh.r.Yab[jc * GC + r];
      const int hi = r > jc ? r : jc, lo = r > jc ? jc : r;
      Tab[q] = in ? tab : 0.0;
      nTt[q] = in ? -tt : 0.0;
      nY[q] = in ? -y : 0.0;
      std1(rF, oF + q * 4 * NU * 8, k * (WF * 8), sh.r.G[hi * GC + lo]);   // Ua, 1 / d
      std1(rF, oF + q * 4 * NU * 8 + 2 * FB, k * (WF * 8), tab);
      X[q] = -(j == VC ? Hbb[q] : Hxb[q]);
    }
    wsync();
    // half b after the Schur update
    Hbb = mmT<3>(nY, Tab, Hbb);
    X = mmT<3>(nY, Tx, X);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int r = 4 * q + g;
      if (in) sh.r.G[j * GC + r] = Hbb[q];
      sh.r.G[(NU + j) * GC + r] = X[q];
    }
    wsync();
    d4 Kb = zero4();
    {
      double c3[NU];
#pragma unroll
      for (int r = 0; r < NU; ++r) c3[r] = gc[r];
      wsync();
      factor(c3, hc, uc);
      back_substitute(c3, is_h, uc);
      if (!is_h || lane < NU) {
#pragma unroll
        for (int r = 0; r < NU; ++r) gc[r] = c3[r];
      }
      wsync();
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int r = 4 * q + g;
      const int hi = r > jc ? r : jc, lo = r > jc ? jc : r;
      Kb[q] = sh.r.G[(NU + j) * GC + r];
      std1(rK, oK + q * 4 * (NX + 1) * 8 + KB, k * (WK * 8), Kb[q]);
      std1(rF, oF + q * 4 * NU * 8 + FB, k * (WF * 8), sh.r.G[hi * GC + lo]);   // Ub, 1 / d
    }
    // half a's gains: Ua Ka = Tx - Tab Kb
    Tx = mmT<3>(nTt, Kb, Tx);
    wsync();
#pragma unroll
    for (int q = 0; q < 3; ++q) sh.r.G[(NU + j) * GC + 4 * q + g] = Tx[q];
    wsync();
    if (!is_h) {
#pragma unroll
      for (int r = 0; r < NU; ++r) c1[r] = gc[r];
    }
    back_substitute(c1, is_h, ua);
    wsync();
    if (!is_h) {
#pragma unroll
      for (int r = 0; r < NU; ++r) gc[r] = c1[r];
    }
    wsync();
    d4 Ka = zero4();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      Ka[q] = sh.r.G[(NU + j) * GC + 4 * q + g];
      std1(rK, oK + q * 4 * (NX + 1) * 8, k * (WK * 8), Ka[q]);
    }
    // S = A^T W A + Hwx^T K, s = A^T (q + s) + Hwx^T kap
    Ss = symmetrize(mmT<3>(Hxa, Ka, mmT<3>(Hxb, Kb, SA)), sw, sh.r.ST);
  }
}

// Forward rollout of the gains from dx_0 = 0: du_k = K_k dx_k + kap_k (into GV),
// dx_{k+1} = A_k dx_k + B_k du_k (into PV).  VECK: kap_k from GV (a corrector's)
// instead of the stored gains.
template <bool VECK>
__device__ __attribute__((always_inline)) inline void forward(const WCtx& C, WSh& sh) {
  __syncthreads();
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  double* const PV = sh.c.PV;
  double* const GV = sh.c.GV;
  const auto rA = rsrc(uni(C.A), N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * U4 * 4);
  const auto rK = rsrc(uni(C.K), N * WK * 8);
  const int oA = j < NX ? (j * NX + 3 * g) * 4 : OOB, oB = j < NX ? (j * U4 + 3 * g) * 4 : OOB;
  const int oK = j < NU ? (j * (NX + 1) + 3 * g) * 8 : OOB;
  const int oKap = (g == 0 && j < NU) ? (j * (NX + 1) + NX) * 8 : OOB;
  struct FwdRaw {
    double ka[4], kb[4], pa, pb;
    float a[4], ba[3], bb[3];
  };
  auto ffetch = [&](int k, FwdRaw& s) {
    ldd2(rK, oK, k * (WK * 8), s.ka);
    ldd2(rK, oK + 16, k * (WK * 8), s.ka + 2);
    ldd2(rK, oK + KB, k * (WK * 8), s.kb);
    ldd2(rK, oK + KB + 16, k * (WK * 8), s.kb + 2);
    s.pa = VECK ? 0.0 : ldd(rK, oKap, k * (WK * 8));
    s.pb = VECK ? 0.0 : ldd(rK, oKap + KB, k * (WK * 8));
    ldf4(rA, oA, k * (NX * NX * 4), s.a);
    ldf3(rB, oB, k * (NX * U4 * 4), s.ba);
    ldf3(rB, oB + NU * 4, k * (NX * U4 * 4), s.bb);
  };
  constexpr int FD = 2;
  FwdRaw ring[FD];
#pragma unroll
  for (int d = 0; d < FD; ++d) {
    ffetch(d < N ? d : N - 1, ring[d]);
    pin_memory();
  }
  double xv = 0.0;   // dx_k, entry j
  auto step = [&](int k, FwdRaw& r) __attribute__((always_inline)) {
    double ka[4], kb[4], a[4], ba[3], bb[3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ka[q] = (q == 0 && g) ? 0.0 : r.ka[q];
      kb[q] = (q == 0 && g) ? 0.0 : r.kb[q];
      a[q] = (q == 0 && g) ? 0.0 : (double)r.a[q];
      pin(ka[q]); pin(kb[q]); pin(a[q]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      ba[q] = (double)r.ba[q];
      bb[q] = (double)r.bb[q];
      pin(ba[q]); pin(bb[q]);
    }
    double pa = r.pa, pb = r.pb;
    pin(pa); pin(pb);
    pin_memory();
    ffetch(k + FD < N ? k + FD : N - 1, r);
    if constexpr (VECK) {
      pa = (g == 0 && j < NU) ? GV[k * U4 + clampi(j, NU - 1)] : 0.0;
      pb = (g == 0 && j < NU) ? GV[k * U4 + NU + clampi(j, NU - 1)] : 0.0;
    }
    const double xt = turn_rows(xv);
    const double wa = row_total(dot4(xt, ka, pa)), wb = row_total(dot4(xt, kb, pb));
    const double ax = dot4(xt, a, 0.0);
    xv = row_total(dot3(turn_rows(wb), bb, dot3(turn_rows(wa), ba, ax)));
    if (lane < NU) {
      GV[k * U4 + j] = wa;
      GV[k * U4 + NU + j] = wb;
    }
    if (lane < NX) PV[k * NX + j] = xv;
  };
  static_assert(FD == 2, "one line below per ring slot");
  for (int k = 0;; k += FD) {
    if (!(k < N)) break;
    step(k, ring[0]);
    if (!(k + 1 < N)) break;
    step(k + 1, ring[1]);
  }
  wsync();
}

// Second right-hand side of a Newton step with the stored factors (the corrector
// of an interior-point iteration): rho_k (in GV) to kap_k (in GV).  The
// recursion of the linear part, s <- A^T wv + K^T hw with wv = q + s and
// hw = B^T wv + rho, is a chain; the feedforwards kap = -H^{-1} hw then follow
// four stages at a time, by block triangular solves with Ua, Tab and Ub.
__device__ __attribute__((always_inline)) inline void newton_vector(const WCtx& C, WSh& sh) {
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  double* const GV = sh.c.GV;
  const auto rA = rsrc(uni(C.A), N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * U4 * 4);
  const auto rK = rsrc(uni(C.K), N * WK * 8), rQ = rsrc(uni(C.q), N * NX * 8);
  const auto rF = rsrc(uni(C.F), N * WF * 8);
  const int oA = j < NX ? (3 * g * NX + j) * 4 : OOB, oA0 = (g == 0 && j < NX) ? j * 4 : OOB;
  const int oB = j < NU ? (3 * g * U4 + j) * 4 : OOB, oB0 = (g == 0 && j < NU) ? j * 4 : OOB;
  const int oK = j < NX ? (3 * g * (NX + 1) + j) * 8 : OOB, oQ = j < NX ? j * 8 : OOB;
  struct VecRaw {
    float a[4], ba[4], bb[4];
    double ka[3], kb[3], q;
  };
  auto vfetch = [&](int k, VecRaw& s) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int ob = q == 0 ? oB0 : oB + q * U4 * 4;
      s.a[q] = ldf(rA, q == 0 ? oA0 : oA + q * NX * 4, k * (NX * NX * 4));
      s.ba[q] = ldf(rB, ob, k * (NX * U4 * 4));
      s.bb[q] = ldf(rB, ob + NU * 4, k * (NX * U4 * 4));
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      s.ka[q] = ldd(rK, oK + q * (NX + 1) * 8, k * (WK * 8));
      s.kb[q] = ldd(rK, oK + q * (NX + 1) * 8 + KB, k * (WK * 8));
    }
    s.q = ldd(rQ, oQ, k * (NX * 8));
  };
  constexpr int VD = 2;
  VecRaw ring[VD];
#pragma unroll
  for (int d = 0; d < VD; ++d) {
    vfetch(N - 1 - d >= 0 ? N - 1 - d : 0, ring[d]);
    pin_memory();
  }
  double s = 0.0;   // value function's linear part, entry j
  auto step = [&](int k, VecRaw& r) __attribute__((always_inline)) {
    double a[4], ba[4], bb[4], ka[3], kb[3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = (double)r.a[q];
      ba[q] = (double)r.ba[q];
      bb[q] = (double)r.bb[q];
      pin(a[q]); pin(ba[q]); pin(bb[q]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      ka[q] = r.ka[q];
      kb[q] = r.kb[q];
      pin(ka[q]); pin(kb[q]);
    }
    const double qk = r.q;
    pin(qk);
    pin_memory();
    vfetch(k - VD >= 0 ? k - VD : 0, r);
    const bool on = g == 0 && j < NU;
    const double rhoa = on ? GV[k * U4 + clampi(j, NU - 1)] : 0.0;
    const double rhob = on ? GV[k * U4 + NU + clampi(j, NU - 1)] : 0.0;
    const double wt = turn_rows(qk + s);
    const double ha = row_total(dot4(wt, ba, rhoa)), hb = row_total(dot4(wt, bb, rhob));
    const double aw = dot4(wt, a, 0.0);
    s = row_total(dot3(turn_rows(hb), kb, dot3(turn_rows(ha), ka, aw)));
    if (lane < NU) {
      GV[k * U4 + j] = ha;
      GV[k * U4 + NU + j] = hb;
    }
  };
  static_assert(VD == 2, "one line below per ring slot");
  for (int k = N - 1;; k -= VD) {
    if (!(k >= 0)) break;
    step(k, ring[0]);
    if (!(k - 1 >= 0)) break;
    step(k - 1, ring[1]);
  }
  wsync();
  const int oF = j < NU ? (g * WF + j * NU) * 8 : OOB;          // row j of a block
  const int oC = j < NU ? (g * WF + j) * 8 : OOB;               // column j of a block
  const int oD = j < NU ? (g * WF + j * (NU + 1)) * 8 : OOB;    // its diagonal
  for (int k0 = 0; k0 < N; k0 += 4) {
    const int k = k0 + g, at = k0 * (WF * 8);
    const bool on = j < NU && k < N;
    double f[NU], tc[NU], ya = 0.0, yb = 0.0;
    if (on && stance(C, k, j / 6)) ya = GV[k * U4 + j];
    if (on && stance(C, k, 2 + j / 6)) yb = GV[k * U4 + NU + j];
    const double da = ldd(rF, oD, at), db = ldd(rF, oD + FB, at);
#define PINMPC_ACC(y, src, p, m)                                                              \
  {                                                                                           \
    const double mm = (m);                                                                    \
    asm volatile(                                                                             \
        "s_nop 1\n"                                                                           \
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:" #p " row_mask:0xf bank_mask:0xf bound_ctrl:1" \
        : "+v"(y)                                                                             \
        : "v"(src), "v"(mm));                                                                 \
  }
// y += (y of lane p) * m: the destination is its own broadcast source
#define PINMPC_TRI(y, p, use)                                                                 \
  {                                                                                           \
    const double mm = (use) ? -f[p] : 0.0;                                                    \
    asm volatile(                                                                             \
        "s_nop 1\n"                                                                           \
        "v_fmac_f64_dpp %0, %0, %1 row_newbcast:" #p " row_mask:0xf bank_mask:0xf bound_ctrl:1" \
        : "+v"(y)                                                                             \
        : "v"(mm));                                                                           \
  }
#define PINMPC_DOWN(y)                                                                     \
  PINMPC_TRI(y, 0, j > 0) PINMPC_TRI(y, 1, j > 1) PINMPC_TRI(y, 2, j > 2)                  \
  PINMPC_TRI(y, 3, j > 3) PINMPC_TRI(y, 4, j > 4) PINMPC_TRI(y, 5, j > 5)                  \
  PINMPC_TRI(y, 6, j > 6) PINMPC_TRI(y, 7, j > 7) PINMPC_TRI(y, 8, j > 8)                  \
  PINMPC_TRI(y, 9, j > 9) PINMPC_TRI(y, 10, j > 10)
#define PINMPC_UP(y)                                                                       \
  PINMPC_TRI(y, 11, j < 11) PINMPC_TRI(y, 10, j < 10) PINMPC_TRI(y, 9, j < 9)              \
  PINMPC_TRI(y, 8, j < 8) PINMPC_TRI(y, 7, j < 7) PINMPC_TRI(y, 6, j < 6)                  \
  PINMPC_TRI(y, 5, j < 5) PINMPC_TRI(y, 4, j < 4) PINMPC_TRI(y, 3, j < 3)                  \
  PINMPC_TRI(y, 2, j < 2) PINMPC_TRI(y, 1, j < 1)
#define PINMPC_SUB(y, src, v)                                                              \
  PINMPC_ACC(y, src, 0, -v[0]) PINMPC_ACC(y, src, 1, -v[1]) PINMPC_ACC(y, src, 2, -v[2])   \
  PINMPC_ACC(y, src, 3, -v[3]) PINMPC_ACC(y, src, 4, -v[4]) PINMPC_ACC(y, src, 5, -v[5])   \
  PINMPC_ACC(y, src, 6, -v[6]) PINMPC_ACC(y, src, 7, -v[7]) PINMPC_ACC(y, src, 8, -v[8])   \
  PINMPC_ACC(y, src, 9, -v[9]) PINMPC_ACC(y, src, 10, -v[10]) PINMPC_ACC(y, src, 11, -v[11])
    // ya <- Ua^-T ya, yb <- Ub^-T (yb - Tab^T ya)
#pragma unroll
    for (int p = 0; p < NU; p += 2) ldd2(rF, oF + p * 8, at, f + p);
#pragma unroll
    for (int p = 0; p < NU; ++p) tc[p] = ldd(rF, oC + p * NU * 8 + 2 * FB, at);
    PINMPC_DOWN(ya)
    PINMPC_SUB(yb, ya, tc)
    double fa[NU];
#pragma unroll
    for (int p = 0; p < NU; ++p) fa[p] = f[p];
#pragma unroll
    for (int p = 0; p < NU; p += 2) ldd2(rF, oF + p * 8 + FB, at, f + p);
    PINMPC_DOWN(yb)
    ya *= da;
    yb *= db;
    // yb <- Ub^-1 yb, ya <- Ua^-1 (ya - Tab yb)
    PINMPC_UP(yb)
#pragma unroll
    for (int p = 0; p < NU; p += 2) ldd2(rF, oF + p * 8 + 2 * FB, at, tc + p);
    PINMPC_SUB(ya, yb, tc)
#pragma unroll
    for (int p = 0; p < NU; ++p) f[p] = fa[p];
    PINMPC_UP(ya)
#undef PINMPC_SUB
#undef PINMPC_UP
#undef PINMPC_DOWN
#undef PINMPC_TRI
#undef PINMPC_ACC
    if (on) {
      GV[k * U4 + j] = -ya;
      GV[k * U4 + NU + j] = -yb;
    }
  }
  wsync();
}

// s + sum_l u_l b[l] over a half's 12 inputs (u in lanes 0..11 of the row).
__device__ inline double dot_half(double u, const float (&b)[NU], double s) {
  double bd[NX];
#pragma unroll
  for (int l = 0; l < NX; ++l) bd[l] = l < NU ? (double)b[l < NU ? l : 0] : 0.0;
  return dot_row_bcast13(u, bd, s);
}

// x = rollout of u from x0, in FP64: the stage terms B u + e for four stages at
// a time, then the chain.  x_{k+1} is left in PV as well.
__device__ __attribute__((always_inline)) inline void rollout(const WCtx& C, WSh& sh) {
  __syncthreads();
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  double* const PV = sh.c.PV;
  const gcf pe = uni(C.e), pA = uni(C.A);
  const auto rA = rsrc(pA, N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * U4 * 4);
  const auto rE = rsrc(pe ? pe : pA, pe ? N * NX * 4 : 0), rU = rsrc(uni(C.u), N * U4 * 8);
  const int oB = j < NX ? (g * NX + j) * U4 * 4 : OOB, oE = j < NX ? (g * NX + j) * 4 : OOB;
  const int oU = j < NU ? (g * U4 + j) * 8 : OOB;
  for (int k0 = 0; k0 < N; k0 += 4) {
    float ba[NU], bb[NU];
#pragma unroll
    for (int l = 0; l < NU; l += 4) {
      ldf4(rB, oB + l * 4, k0 * (NX * U4 * 4), ba + l);
      ldf4(rB, oB + (NU + l) * 4, k0 * (NX * U4 * 4), bb + l);
    }
    const double u0 = ldd(rU, oU, k0 * (U4 * 8)), u1 = ldd(rU, oU + NU * 8, k0 * (U4 * 8));
    const double e = (double)ldf(rE, oE, k0 * (NX * 4));
    const double d = dot_half(u1, bb, dot_half(u0, ba, e));
    if (j < NX && k0 + g < N) PV[(k0 + g) * NX + j] = d;
  }
  wsync();
  const int oA = j < NX ? (j * NX + 3 * g) * 4 : OOB;
  constexpr int RD = 8;
  float ring[RD][4];
#pragma unroll
  for (int d = 0; d < RD; ++d) {
    ldf4(rA, oA, (d < N ? d : N - 1) * (NX * NX * 4), ring[d]);
    pin_memory();
  }
  double xv = j < NX ? (double)uni(C.x0)[clampi(j, NX - 1)] : 0.0;
  if (lane < NX) C.x[lane] = xv;
  auto step = [&](int k, float (&r)[4]) __attribute__((always_inline)) {
    double a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = (q == 0 && g) ? 0.0 : (double)r[q];
      pin(a[q]);
    }
    pin_memory();
    ldf4(rA, oA, (k + RD < N ? k + RD : N - 1) * (NX * NX * 4), r);
    const double t = j < NX ? PV[k * NX + clampi(j, NX - 1)] : 0.0;
    xv = row_total(dot4(turn_rows(xv), a, 0.0)) + t;
    if (lane < NX) PV[k * NX + j] = xv;
  };
  static_assert(RD == 8, "one line below per ring slot");
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
  }
  wsync();
  for (int e = fresh_lane(); e < N * NX; e += W64) C.x[NX + e] = PV[e];
  __syncthreads();
}

// Dynamics residual of the FP64 trajectory (x, u), normalised by the largest
// term of each entry.
__device__ __attribute__((always_inline)) inline double dyn_residual(const WCtx& C) {
  // four stages at a time (one per 16-lane row, state j in lane j)
  const int g = tg(), j = tj();
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const gcf pe = uni(C.e), pA = uni(C.A);
  const auto rA = rsrc(pA, N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * U4 * 4);
  const auto rE = rsrc(pe ? pe : pA, pe ? N * NX * 4 : 0);
  const auto rU = rsrc(uni(C.u), N * U4 * 8), rX = rsrc(uni(C.x), (N + 1) * NX * 8);
  const int oA = j < NX ? (g * NX + j) * NX * 4 : OOB, oB = j < NX ? (g * NX + j) * U4 * 4 : OOB;
  const int oX = j < NX ? (g * NX + j) * 8 : OOB, oU = j < NU ? (g * U4 + j) * 8 : OOB;
  const int oE = j < NX ? (g * NX + j) * 4 : OOB;
  double r = 0.0;
  for (int k0 = 0; k0 < N; k0 += 4) {
    float a[NX], ba[NU], bb[NU];
#pragma unroll
    for (int l = 0; l < NU; l += 4) {
      ldf4(rA, oA + l * 4, k0 * (NX * NX * 4), a + l);
      ldf4(rB, oB + l * 4, k0 * (NX * U4 * 4), ba + l);
      ldf4(rB, oB + (NU + l) * 4, k0 * (NX * U4 * 4), bb + l);
    }
    a[NU] = ldf(rA, oA + NU * 4, k0 * (NX * NX * 4));
    const double ee = (double)ldf(rE, oE, k0 * (NX * 4));
    const double x = ldd(rX, oX, k0 * (NX * 8)), xn = ldd(rX, oX + NX * 8, k0 * (NX * 8));
    const double ua = ldd(rU, oU, k0 * (U4 * 8)), ub = ldd(rU, oU + NU * 8, k0 * (U4 * 8));
    double ad[NX], bd[NX], cd[NX];
#pragma unroll
    for (int l = 0; l < NX; ++l) {
      ad[l] = (double)a[l];
      bd[l] = l < NU ? (double)ba[l < NU ? l : 0] : 0.0;
      cd[l] = l < NU ? (double)bb[l < NU ? l : 0] : 0.0;
    }
    const double ax = dot_row_bcast13(x, ad, 0.0);
    const double bu = dot_row_bcast13(ub, cd, dot_row_bcast13(ua, bd, 0.0));
    const double d = xn - ax - bu - ee;
    const double den = 1.0 + fmax(fabs(xn), fmax(fabs(ax), fabs(bu)));
    if (j < NX && k0 + g < N) r = fmax(r, no_nan(fabs(d) / den));
  }
  return wave_max(r);
}

// Gradient of force row r (0..4) of the pyramid with respect to f.
__device__ inline void frow(int r, double mu, double g[3]) {
  g[0] = r == 0 ? 1.0 : (r == 1 ? -1.0 : 0.0);
  g[1] = r == 2 ? 1.0 : (r == 3 ? -1.0 : 0.0);
  g[2] = r == 4 ? 1.0 : -mu;
}

// Multipliers m >= 0 of the force rows in the set `am` (bits 0..4) that best
// cancel the force gradient gf: min |gf + sum_r m_r g_r| (nonnegative least
// squares).  An optimal support has at most three independent rows, so the
// candidates are every subset of at most three rows of `am` with a
// nonsingular Gram matrix whose least-squares multipliers are nonnegative.
// Every loop below unrolls completely (the subset S is a constant in each
// copy), so no array is indexed at run time and all of them stay in registers.
__device__ void force_refit(int am, double mu, const double gf[3], double m[5]) {
  double best = gf[0] * gf[0] + gf[1] * gf[1] + gf[2] * gf[2];
#pragma unroll
  for (int t = 0; t < 5; ++t) m[t] = 0.0;
  const double scale = 1.0 + mu * mu;
#pragma unroll
  for (int S = 1; S < 32; ++S) {
    if (__builtin_popcount(S) > 3) continue;
    if ((S & am) != S) continue;
    int idx[3] = {0, 0, 0}, k = 0;
#pragma unroll
    for (int r = 0; r < 5; ++r)
      if ((S >> r) & 1) idx[k++] = r;
    double g[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j) frow(j < k ? idx[j] : 0, mu, g[j]);
    // Gram matrix and right-hand side -G_S gf (k x k, k <= 3), the identity
    // on the unused rows
    double M[3][3], b[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      b[a] = a < k ? -(g[a][0] * gf[0] + g[a][1] * gf[1] + g[a][2] * gf[2]) : 0.0;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        M[a][c] = (a < k && c < k) ? g[a][0] * g[c][0] + g[a][1] * g[c][1] + g[a][2] * g[c][2]
                                   : (a == c ? 1.0 : 0.0);
    }
    const double det = M[0][0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) -
                       M[0][1] * (M[1][0] * M[2][2] - M[1][2] * M[2][0]) +
                       M[0][2] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]);
    if (!(fabs(det) > 1e-10 * scale * scale * scale)) continue;   // dependent rows
    double x[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double D[3][3];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) D[i][c] = c == a ? b[i] : M[i][c];
      x[a] = (D[0][0] * (D[1][1] * D[2][2] - D[1][2] * D[2][1]) -
              D[0][1] * (D[1][0] * D[2][2] - D[1][2] * D[2][0]) +
              D[0][2] * (D[1][0] * D[2][1] - D[1][1] * D[2][0])) / det;
    }
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) ok = ok && (a >= k || x[a] >= 0.0);
    if (!ok) continue;
    double rv[3] = {gf[0], gf[1], gf[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) rv[c] += a < k ? x[a] * g[a][c] : 0.0;
    const double res = rv[0] * rv[0] + rv[1] * rv[1] + rv[2] * rv[2];
    if (res < best) {
      best = res;
#pragma unroll
      for (int t = 0; t < 5; ++t) {
        double v = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) v = (a < k && idx[a] == t) ? x[a] : v;
        m[t] = v;
      }
    }
  }
}

// The certificate of the iterate: x (rollout of u) and res.  The costates
// come from the adjoint recursion; each stance contact's row multipliers are
// refitted to its input gradient on the rows whose slack is at most tol times
// the row's scale (nonnegative least squares: the force rows by force_refit,
// each moment axis in closed form), so complementarity holds to tol by
// construction and stationarity measures how well u meets it.  (The interior
// point's own multipliers lose their accuracy as the slacks of active rows
// approach zero: their step divides by the slack.)  Returns max(res).
__device__ __attribute__((always_inline)) inline double certificate(const WCtx& C, WSh& sh,
                                                       double res[PINMPC_NRES], double tol) {
  rollout(C, sh);
  res[0] = dyn_residual(C);
  const int N = __builtin_amdgcn_readfirstlane(C.N);
  const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
  double* const PV = sh.c.PV;
  double* const GV = sh.c.GV;
  const gcf pr = uni(C.x_ref);
  for (int e0 = fresh_lane(); e0 < N * NX; e0 += 8 * W64) {
    float xr[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) xr[t] = pr[e0 + t * W64 < N * NX ? e0 + t * W64 : e0];
    pin_memory();
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = e0 + t * W64;
      if (e < N * NX) PV[e] = sh.Q[e % NX] * (PV[e] - (double)xr[t]);
    }
  }
  wsync();
  // costates, backwards: p_{k+1} = Q (x_{k+1} - r_k) + A_{k+1}^T p_{k+2}
  const auto rA = rsrc(uni(C.A), N * NX * NX * 4), rB = rsrc(uni(C.B), N * NX * U4 * 4);
  const int oA = j < NX ? (3 * g * NX + j) * 4 : OOB, oA0 = (g == 0 && j < NX) ? j * 4 : OOB;
  auto cfetch = [&](int k, float (&s)[4]) {
    const int at = clampi(k + 1, N - 1) * (NX * NX * 4);
    s[0] = ldf(rA, oA0, at);
#pragma unroll
    for (int q = 1; q < 4; ++q) s[q] = ldf(rA, oA + q * NX * 4, at);
  };
  constexpr int CD = 8;
  float ring[CD][4];
#pragma unroll
  for (int d = 0; d < CD; ++d) {
    cfetch(N - 1 - d >= 0 ? N - 1 - d : 0, ring[d]);
    pin_memory();
  }
  double p = 0.0, terms = 0.0;
  auto step = [&](int k, float (&r)[4]) __attribute__((always_inline)) {
    double a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = (double)r[q];
      pin(a[q]);
    }
    pin_memory();
    cfetch(k - CD >= 0 ? k - CD : 0, r);
    const double qx = j < NX ? PV[k * NX + clampi(j, NX - 1)] : 0.0;
    const double ap = row_total(dot4(turn_rows(p), a, 0.0));
    p = qx + ap;
    terms = fmax(terms, fmax(fabs(qx), fmax(fabs(p), fabs(ap))));
    if (lane < NX) PV[k * NX + j] = p;
  };
  static_assert(CD == 8, "one line below per ring slot");
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
  }
  wsync();
  // B^T p, four stages at a time
  const int oB = j < NU ? (g * NX * U4 + j) * 4 : OOB;
  for (int k0 = 0; k0 < N; k0 += 4) {
    const int k = k0 + g;
    double ba[NX], bb[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      ba[r] = (double)ldf(rB, oB + r * U4 * 4, k0 * (NX * U4 * 4));
      bb[r] = (double)ldf(rB, oB + r * U4 * 4 + NU * 4, k0 * (NX * U4 * 4));
    }
    const double pk = (j < NX && k < N) ? PV[k * NX + j] : 0.0;
    const double ga = dot_row_bcast13(pk, ba, 0.0), gb = dot_row_bcast13(pk, bb, 0.0);
    if (j < NU && k < N) {
      GV[k * U4 + j] = ga;
      GV[k * U4 + NU + j] = gb;
    }
  }
  wsync();
  // per (stage, contact): gradient, multipliers, feasibility, complementarity
  double stat = 0.0, rin = 0.0, mmax = 0.0, comp = 0.0;
  const auto rR = uref_buf(C);
  for (int e = fresh_lane(); e < N * C4; e += W64) {
    const int k = e / C4, i = e % C4;
    double u[6];
    float ur[6];
    const bool on = uni(C.contact)[e] != 0;
    ldf3(rR, e * 24, 0, ur);
    ldf3(rR, e * 24 + 12, 0, ur + 3);
    ld6(uni(C.u) + e * 6, u);
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      pin(u[t]);
      asm volatile("" ::"v"(ur[t]));
    }
    pin_memory();
    if (!on) {
#pragma unroll
      for (int t = 0; t < 6; ++t) rin = fmax(rin, fabs(u[t]) / C.mg);
      continue;
    }
    double gu[NROW], h[NROW], isc[NROW], mv[NROW], gr[6];
    rows_of(C, u, gu, h, isc);
    double tr = 0.0, tb = 0.0;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int jj = 6 * i + t;
      const double ru = sh.R[jj] * (u[t] - (double)ur[t]), bl = GV[k * U4 + jj];
      tr = fmax(tr, fabs(ru));
      tb = fmax(tb, fabs(bl));
      gr[t] = ru + bl;
    }
    // rows active within tol, their refitted multipliers
    int am = 0;
#pragma unroll
    for (int r = 0; r < NROW; ++r)
      if (h[r] - gu[r] <= tol * (r < 5 ? C.scf : C.scm)) am |= 1 << r;
    double mf[5];
    force_refit(am & 31, C.mu, gr, mf);
#pragma unroll
    for (int r = 0; r < 5; ++r) mv[r] = mf[r];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      mv[5 + a] = ((am >> (5 + a)) & 1) ? fmax(-gr[3 + a], 0.0) : 0.0;
      mv[8 + a] = ((am >> (8 + a)) & 1) ? fmax(gr[3 + a], 0.0) : 0.0;
    }
    double gm[6];
    rows_T(C, mv, gm);
    double tgm = 0.0, cmp = 0.0;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      tgm = fmax(tgm, fabs(gm[t]));
      stat = fmax(stat, no_nan(fabs(gr[t] + gm[t])));
    }
#pragma unroll
    for (int r = 0; r < NROW; ++r) {
      rin = fmax(rin, fmax(gu[r] - h[r], 0.0) / C.mg);
      mmax = fmax(mmax, mv[r]);
      cmp = fmax(cmp, mv[r] * fmax(h[r] - gu[r], 0.0));
    }
    comp = fmax(comp, cmp);
    terms = fmax(terms, fmax(tr, fmax(tb, tgm)));
  }
  terms = wave_max(terms);
  mmax = wave_max(mmax);
  comp = wave_max(comp) / (1.0 + mmax * C.mg);
  res[1] = wave_max(rin);
  res[2] = terms < __builtin_inf() ? wave_max(stat) / (1.0 + terms) : terms;
  res[3] = comp;
  res[4] = 0.0;   // the refitted multipliers are nonnegative
  double m = 0.0;
#pragma unroll
  for (int i = 0; i < PINMPC_NRES; ++i) m = fmax(m, no_nan(res[i]));
  return m;
}

// Interior point from the current u (its rollout in x).  Returns the
// iterations; *ok tells whether the certificate was met (then res is it).
__device__ __attribute__((always_inline)) inline int ipm(const WCtx& C, WSh& sh, int maxit, double tol,
                                            double res[PINMPC_NRES], bool* ok) {
  const int N = C.N, rs = C4 * C.n;
  double* const PV = sh.c.PV;
  double* const GV = sh.c.GV;
  *ok = false;
  // rows of stance contacts, starting slacks (at least 1) and multipliers 1
  double mloc = 0.0, smz = 0.0, rpn = 0.0;
  __syncthreads();
  for (int e = fresh_lane(); e < N * C4; e += W64) {
    const int k = e / C4, i = e % C4;
    if (!stance(C, k, i)) continue;
    double u[6], gu[NROW], h[NROW], isc[NROW], sv[NROW], zv[NROW];
    ld6(C.u + (size_t)k * U4 + 6 * i, u);
    rows_of(C, u, gu, h, isc);
#pragma unroll
    for (int r = 0; r < NROW; ++r) {
      sv[r] = fmax((h[r] - gu[r]) * isc[r], 1.0);
      zv[r] = 1.0;
      smz += sv[r] * zv[r];
      rpn = fmax(rpn, fabs(fma(gu[r] - h[r], isc[r], sv[r])));
    }
    mloc += NROW;
    str(C.s, rs, e, sv);
    str(C.z, rs, e, zv);
  }
  const double m = wave_sum(mloc);
  int it = 0;
  for (;; ++it) {
    const double sz = wave_sum(smz), muv = m > 0.0 ? sz / m : 0.0;
    rpn = wave_max(rpn);
    // (beyond 1e-20 the steps of the multipliers of active rows, divided by
    // slacks near zero, carry no accuracy)
    const bool last = it >= maxit;
    if (last || (muv <= 1e-8 && rpn <= 1e-8)) {
      *ok = certificate(C, sh, res, tol) <= tol;
      if (scalar(*ok || last || muv <= 1e-20)) return it;
    }
    // predictor: affine target s z
    build_terms(C, sh);
    backward(C, sh);
    forward<false>(C, sh);
    double a = 1.0;
    if (m > 0.0) {
      // its row steps, the largest step to the boundary, and the sums that give
      // the complementarity after any step
      double amax = 1.0, sm1 = 0.0, sm2 = 0.0;
      const auto rR = uref_buf(C);
      for (int e = fresh_lane(); e < N * C4; e += W64) {
        const int k = e / C4, i = e % C4;
        RowLoads w;
        load_rows(C, rR, rs, e, w);
        pin_rows(w);
        if (!w.on) continue;
        double du[6], gu[NROW], gdu[NROW], h[NROW], isc[NROW], cv[NROW];
        const double(&sv)[NROW] = w.s, (&zv)[NROW] = w.z;
#pragma unroll
        for (int t = 0; t < 6; ++t) du[t] = GV[k * U4 + 6 * i + t];
        rows_of(C, w.u, gu, h, isc);
        rows_of(C, du, gdu, h, isc);
#pragma unroll
        for (int r = 0; r < NROW; ++r) {
          const double rp = fma(gu[r] - h[r], isc[r], sv[r]);
          const double ds = -fma(gdu[r], isc[r], rp);
          const double dz = -(zv[r] + zv[r] * ds * recip(sv[r]));
          if (ds < 0.0) amax = fmin(amax, -sv[r] * recip(ds));
          if (dz < 0.0) amax = fmin(amax, -zv[r] * recip(dz));
          sm1 += sv[r] * dz + zv[r] * ds;
          sm2 += ds * dz;
          cv[r] = fma(ds, dz, sv[r] * zv[r]);   // corrector target, less sigma mu
        }
        str(C.rc, rs, e, cv);
      }
      const double aa = wave_min(amax);
      const double mu_aff = fmax(fma(aa, fma(aa, wave_sum(sm2), wave_sum(sm1)), sz), 0.0) / m;
      const double ratio = muv > 0.0 ? mu_aff / muv : 0.0, smu = ratio * ratio * ratio * muv;
      // corrector: rc = s z + ds_aff dz_aff - sigma mu, the same Newton matrix:
      // its linear input term, the recursion's vector part and the rollout with
      // the predictor's factors (triangular solves, as accurate near the optimum
      // as factoring again; a product with the inverse is not)
      for (int e = fresh_lane(); e < N * C4; e += W64) {
        const int k = e / C4, i = e % C4;
        double rho[6] = {0, 0, 0, 0, 0, 0}, cv[NROW];
        RowLoads w;
        load_rows(C, rR, rs, e, w);
        ldr(uni(C.rc), rs, e, cv);
#pragma unroll
        for (int r = 0; r < NROW; ++r) pin(cv[r]);
        pin_rows(w);
        if (w.on) {
          double gu[NROW], h[NROW], isc[NROW], c[NROW];
          const double(&sv)[NROW] = w.s, (&zv)[NROW] = w.z;
          rows_of(C, w.u, gu, h, isc);
#pragma unroll
          for (int r = 0; r < NROW; ++r) {
            cv[r] -= smu;
            const double rp = fma(gu[r] - h[r], isc[r], sv[r]);
            c[r] = (zv[r] + (zv[r] * rp - cv[r]) * recip(sv[r])) * isc[r];
          }
          str(C.rc, rs, e, cv);
          rows_T(C, c, rho);
#pragma unroll
          for (int t = 0; t < 6; ++t) {
            const int jj = 6 * i + t;
            rho[t] = fma(sh.R[jj], w.u[t] - (double)w.ur[t], rho[t]);
          }
        }
#pragma unroll
        for (int t = 0; t < 6; ++t) GV[k * U4 + 6 * i + t] = rho[t];
      }
      wsync();
      newton_vector(C, sh);
      forward<true>(C, sh);
      // the step's rows, and its length
      amax = 1.0;
      for (int e = fresh_lane(); e < N * C4; e += W64) {
        const int k = e / C4, i = e % C4;
        RowLoads w;
        double du[6], gu[NROW], gdu[NROW], h[NROW], isc[NROW], cv[NROW];
        load_rows(C, rR, rs, e, w);
        ldr(uni(C.rc), rs, e, cv);
#pragma unroll
        for (int r = 0; r < NROW; ++r) pin(cv[r]);
        pin_rows(w);
        if (!w.on) continue;
        const double(&sv)[NROW] = w.s, (&zv)[NROW] = w.z;
#pragma unroll
        for (int t = 0; t < 6; ++t) du[t] = GV[k * U4 + 6 * i + t];
        rows_of(C, w.u, gu, h, isc);
        rows_of(C, du, gdu, h, isc);
        double dsv[NROW], dzv[NROW];
#pragma unroll
        for (int r = 0; r < NROW; ++r) {
          const double rp = fma(gu[r] - h[r], isc[r], sv[r]);
          dsv[r] = -fma(gdu[r], isc[r], rp);
          dzv[r] = -fma(zv[r], dsv[r], cv[r]) * recip(sv[r]);
          if (dsv[r] < 0.0) amax = fmin(amax, -sv[r] * recip(dsv[r]));
          if (dzv[r] < 0.0) amax = fmin(amax, -zv[r] * recip(dzv[r]));
        }
        str(C.ds, rs, e, dsv);
        str(C.dz, rs, e, dzv);
      }
      a = fmin(1.0, 0.99 * wave_min(amax));
    }
    // step; residuals of the new point (a lane updates the inputs of its own
    // contact-stage; swing inputs stay 0)
    smz = 0.0;
    rpn = 0.0;
    for (int e = fresh_lane(); e < N * C4; e += W64) {
      const int k = e / C4, i = e % C4;
      double u[6], gu[NROW], h[NROW], isc[NROW], sv[NROW], zv[NROW], dsv[NROW], dzv[NROW];
      const bool on = uni(C.contact)[e] != 0;
      ld6(uni(C.u) + e * 6, u);
      ldr(uni(C.s), rs, e, sv);
      ldr(uni(C.z), rs, e, zv);
      ldr(uni(C.ds), rs, e, dsv);
      ldr(uni(C.dz), rs, e, dzv);
#pragma unroll
      for (int r = 0; r < NROW; ++r) {
        pin(sv[r]);
        pin(zv[r]);
        pin(dsv[r]);
        pin(dzv[r]);
      }
      pin_memory();
      if (!on) continue;
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        u[t] += a * GV[k * U4 + 6 * i + t];
        C.u[(size_t)k * U4 + 6 * i + t] = u[t];
      }
      rows_of(C, u, gu, h, isc);
#pragma unroll
      for (int r = 0; r < NROW; ++r) {
        sv[r] += a * dsv[r];
        zv[r] += a * dzv[r];
        smz += sv[r] * zv[r];
        rpn = fmax(rpn, fabs(fma(gu[r] - h[r], isc[r], sv[r])));
      }
      str(C.s, rs, e, sv);
      str(C.z, rs, e, zv);
    }
    const gd px = uni(C.x);
    for (int e0 = fresh_lane(); e0 < N * NX; e0 += 8 * W64) {
      double x[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] = px[NX + (e0 + t * W64 < N * NX ? e0 + t * W64 : e0)];
      pin_memory();
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int e = e0 + t * W64;
        if (e < N * NX) px[NX + e] = x[t] + a * PV[e];
      }
    }
    wsync();
  }
}

__global__ void __launch_bounds__(64, 2) refine_wide_kernel(Problem p, Workspace ws, float* out_u,
                                                         float* out_x, float* out_res,
                                                         int32_t* out_iters, int32_t* out_status,
                                                         int32_t* out_detail, int admm_iters,
                                                         int accel, int refine, int ipm_max,
                                                         double tol) {
  __shared__ WSh sh;
  const int lane = lane_id();
  // the problem's context lives in LDS (the phase functions read its fields
  // with LDS loads, which no wait for a global load in flight holds up)
  __shared__ WCtx C;
  const size_t s0 = (size_t)blockIdx.x * p.n_max;
  if (lane == 0) {
    C.b = blockIdx.x;
    C.n = p.n_max;
    C.N = horizon(p, C.b);
    C.mu = p.mu[C.b];
    C.fz = p.fz_max[C.b];
    C.tm = p.tau_max[C.b];
    C.mg = weight_of(p, C.b);
    C.scf = C.mg;
    C.scm = C.tm > 0.0 ? C.tm : 1.0;
    C.isf = 1.0 / C.scf;
    C.ism = 1.0 / C.scm;
    C.A = (gcf)(p.A + s0 * NX * NX);
    C.B = (gcf)(p.B + s0 * NX * U4);
    C.e = p.e ? (gcf)(p.e + s0 * NX) : nullptr;
    C.x_ref = (gcf)(p.x_ref + s0 * NX);
    C.u_ref = p.u_ref ? (gcf)(p.u_ref + s0 * U4) : nullptr;
    C.x0 = (gcf)(p.x0 + (size_t)C.b * NX);
    C.contact = (const GMEM uint8_t*)(p.contact + s0 * C4);
    carve(C, (gd)(ws.rblk + (size_t)C.b * refine_wide_block_doubles(C.n)));
  }
  __syncthreads();
  if (lane < NX) sh.Q[lane] = p.Q[(size_t)C.b * NX + lane];
  if (lane < U4) sh.R[lane] = p.R[(size_t)C.b * U4 + lane];
  __syncthreads();
  const int N = C.N;

  // input checks as in the two-contact refinement: finiteness of scalars and
  // weights, the bounds, then this problem's stage data
  const int Nraw = horizon_raw(p, C.b);
  int nonfinite = !isfinite(C.mu) || !isfinite(C.fz) || !isfinite(C.tm) || !isfinite(C.mg);
  #pragma unroll
  for (int j = 0; j < NX; ++j) nonfinite |= !isfinite(sh.Q[j]);
  #pragma unroll
  for (int j = 0; j < U4; ++j) nonfinite |= !isfinite(sh.R[j]);
  int bad = 0;
  if (!nonfinite) {
    bad = !(C.mu > 0.0) || !(C.fz >= 0.0) || !(C.tm >= 0.0) || !(C.mg > 0.0) || Nraw < 1 ||
          Nraw > C.n;
    #pragma unroll
    for (int j = 0; j < NX; ++j) bad |= !(sh.Q[j] > 0.0);
    #pragma unroll
    for (int j = 0; j < U4; ++j) bad |= !(sh.R[j] > 0.0);
  }
  if (!bad && !nonfinite) {
    int nf = any_nonfinite(uni(C.A), N * NX * NX) | any_nonfinite(uni(C.B), N * NX * U4) |
             any_nonfinite(uni(C.x_ref), N * NX);
    if (C.e) nf |= any_nonfinite(uni(C.e), N * NX);
    if (C.u_ref) nf |= any_nonfinite(uni(C.u_ref), N * U4);
    if (lane < NX) nf |= !isfinite(C.x0[lane]);
    if (p.u_prev && lane < U4) nf |= !isfinite(p.u_prev[(size_t)C.b * U4 + lane]);
    nonfinite = wave_max_int(nf) > 0;
  }
  const size_t ux = (size_t)C.b * C.n * U4, xx = (size_t)C.b * (C.n + 1) * NX;
  if (bad || nonfinite) {
    for (int e = fresh_lane(); e < C.n * U4; e += 64) out_u[ux + e] = 0.f;
    for (int e = fresh_lane(); e < (C.n + 1) * NX; e += 64) out_x[xx + e] = 0.f;
    if (lane == 0) {
      if (out_status) out_status[C.b] = bad ? PINMPC_ST_BADINPUT : PINMPC_ST_NONFINITE;
      if (out_iters) out_iters[C.b] = 0;
    }
    if (out_detail && lane < 4) out_detail[(size_t)C.b * 4 + lane] = 0;
    if (out_res && lane < PINMPC_NRES) out_res[(size_t)C.b * PINMPC_NRES + lane] = __builtin_nanf("");
    return;
  }

  // the ADMM point: unscaled inputs of the z iterate, zero on swing contacts
  const float* zsrc = (accel ? ws.cur : ws.hat) + s0 * NSTATE * L4;
  const float tsc = ws.tsc[C.b];
  for (int e = fresh_lane(); e < N * U4; e += 64) {
    const int k = e / U4, j = e % U4;
    const double sc = (j % 6 < 3) ? (double)ws.sf[s0 + k] : (double)tsc;
    const double v = (double)zsrc[(size_t)k * NSTATE * L4 + NX + j] * sc;
    C.u[e] = stance(C, k, j / 6) ? v : 0.0;
  }
  double res[PINMPC_NRES] = {0, 0, 0, 0, 0};
  int its = 0;
  bool ok = false;
  rollout(C, sh);
  if (refine) {
    its = ipm(C, sh, ipm_max, tol, res, &ok);   // res: the returned point's
  } else {
    // the ADMM point as it is
    (void)certificate(C, sh, res, tol);
  }

  // outputs
  __syncthreads();
  for (int e = fresh_lane(); e < C.n * U4; e += 64) out_u[ux + e] = (e < N * U4) ? (float)C.u[e] : 0.f;
  for (int e = fresh_lane(); e < (C.n + 1) * NX; e += 64)
    out_x[xx + e] = (e < (N + 1) * NX) ? (float)C.x[e] : 0.f;
  if (lane == 0) {
    atomicAdd(ws.work, (unsigned long long)its * (unsigned long long)N);
    if (out_status)
      out_status[C.b] = refine ? (ok ? PINMPC_ST_OK : PINMPC_ST_UNPOLISHED) : PINMPC_ST_MAXITER;
    if (out_iters) out_iters[C.b] = admm_iters + its;
  }
  if (out_detail && lane < 4) {
    // (every predictor factors the horizon, no corrector does)
    const int v = lane == 1 ? its : lane == 2 ? its * N : lane == 3 ? 1 : 0;
    out_detail[(size_t)C.b * 4 + lane] = v;
  }
  if (out_res && lane < PINMPC_NRES) out_res[(size_t)C.b * PINMPC_NRES + lane] = (float)res[lane];
}

}  // namespace

hipError_t launch_refine_wide(const Problem& p, const Workspace& w, const pinmpc_settings& s,
                              const pinmpc_out& out, hipStream_t st) {
  if (p.batch == 0) return hipSuccess;
  if (p.nc != C4 || p.n_max > PINMPC_NMAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(refine_wide_kernel, dim3(p.batch), dim3(64), 0, st, p, w, out.u, out.x,
                     out.res, out.iters, out.status, out.detail, s.iters, s.accel, s.refine,
                     s.ipm_iters, s.kkt_tol);
  return hipGetLastError();
}

}  // namespace pinmpc
