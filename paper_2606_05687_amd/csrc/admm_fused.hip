// Parallel-in-horizon ADMM (Sec. III), all sweeps of a problem in one launch,
// with every thread's share of the stage operators loaded once into registers
// and kept there across the sweeps.
//
// A workgroup owns PPW problems (one, or two or four short ones packed into one
// workgroup), each with its own group of threads and LDS buffers; with U = 6 NC
// inputs, thread (k, r) of a problem's group owns lifted row r of stage k:
//   r < 13 : row r of H_k, row r and column r of A_k, row r of Bt_k
//   r >= 13: row r of H_k, column j = r-13 of Bt_k, row j of M_k
// which is exactly what its share of the stage products needs:
//   (Abar^T y)_r, (Bt^T w)_j, (M t)_j, (H htilde)_r, (Abar xi)_r, (Bbar du)_r.
// Vectors that a product needs whole (w, y, t, htilde, xi_k of the
// neighbour stage, du) are exchanged through LDS; the iterates stay in
// registers and are written back once at the end.  HBM traffic per solve is
// the operators once plus the iterates once, independent of the sweep count.
//
// Bound by the latency of its phases: each waits at a barrier for the vectors
// the one before it wrote.  So a stage's vectors sit at a stride of 16 + U floats
// with the inputs at 16, read as 16-byte pieces (a quarter of the LDS
// instructions of single floats), and every thread forms the restart test's sum
// over the stages itself (no barrier for one thread's result): eight barriers a
// sweep.  Launching every sweep on its own, operators streamed, took 136 us a
// sweep at 4096 x 10 and 13 us at one problem of 10 stages.
#include "pinmpc_internal.h"

// Every multiply-add below is either an explicit fmaf or a separate multiply
// and add: no compiler contraction, so every instantiation of the sweep
// (plain or fused, any block size) computes bitwise the same iterates.
#pragma clang fp contract(off)

namespace pinmpc {

namespace {

// Stage stride and offset of lifted row r in the LDS vectors.
template <int NC>
constexpr int VS = 16 + Dims<NC>::U;
__device__ inline int vrow(int r) { return r < NX ? r : r + 3; }

// LDS floats of one problem for a capacity of n stages: five lifted vectors and
// four input vectors per stage, the stage sums of the restart test, and the
// fixed initial lifted state.
template <int NC>
__host__ __device__ inline size_t fused_lds_floats(int n) {
  return (size_t)(5 * n * VS<NC> + 4 * n * Dims<NC>::U + ((n + 3) & ~3) + VS<NC>);
}

// acc + sum_i o[i] p[i] in order, p 16-byte aligned LDS.
template <int COUNT>
__device__ inline float dot(const float* o, const float* p, float acc) {
#pragma unroll
  for (int i = 0; i < COUNT / 4; ++i) {
    const float4 t = ((const float4*)p)[i];
    acc = fmaf(o[4 * i], t.x, acc);
    acc = fmaf(o[4 * i + 1], t.y, acc);
    acc = fmaf(o[4 * i + 2], t.z, acc);
    acc = fmaf(o[4 * i + 3], t.w, acc);
  }
#pragma unroll
  for (int i = COUNT & ~3; i < COUNT; ++i) acc = fmaf(o[i], p[i], acc);
  return acc;
}
// acc + p[0] + p[1] + ... in order.
template <int COUNT>
__device__ inline float sum(const float* p, float acc) {
#pragma unroll
  for (int i = 0; i < COUNT / 4; ++i) {
    const float4 t = ((const float4*)p)[i];
    acc += t.x;
    acc += t.y;
    acc += t.z;
    acc += t.w;
  }
#pragma unroll
  for (int i = COUNT & ~3; i < COUNT; ++i) acc += p[i];
  return acc;
}

// WAVES: waves per SIMD that the registers must leave room for (see wants_room).
template <int MAXT, bool BF16, int PPW, int NC, int WAVES>
__global__ void __launch_bounds__(MAXT, WAVES) admm_fused_kernel(Problem p, Workspace ws, float rho,
                                                                 int accel, float eta, int iters,
                                                                 const int32_t* order,
                                                                 const int32_t* count, int lds_n) {
  constexpr int NU = Dims<NC>::U, NL = Dims<NC>::L, NH = Dims<NC>::H, NM = Dims<NC>::M;
  constexpr int V = VS<NC>;
  OpLoad<BF16> op;
  if constexpr (BF16) {
    op.A = ws.Abf; op.Bt = ws.Btbf; op.H = ws.Hbf; op.M = ws.Mbf;
  } else {
    op.A = p.A; op.Bt = ws.Bt; op.H = ws.Hp; op.M = ws.Mp;
  }
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int slots = count ? *count : p.batch;   // problems this launch walks
  if ((int)blockIdx.x * PPW >= slots) return;   // the whole workgroup: uniform
  // this thread's problem slot in the workgroup, and its index in that group
  const int tpp = PPW == 1 ? (int)blockDim.x : (int)blockDim.x / PPW;
  const int sub = PPW == 1 ? 0 : (int)threadIdx.x / tpp;
  const int slot = (int)blockIdx.x * PPW + sub;
  const int n = p.n_max;          // stage stride of the global arrays
  const int ln = lds_n;           // stage capacity of the LDS buffers
  // a slot past the end, or a horizon beyond the LDS capacity (never for a
  // valid packing), leaves its group idle: it still takes part in the barriers
  bool live = slot < slots;
  const int b = live ? (order ? order[slot] : slot) : 0;
  int N = live ? horizon(p, b) : 0;
  if constexpr (PPW == 1) {
    if (N > ln || N == 0) return;   // the whole (one-problem) workgroup
  }
  if (N > ln) N = 0;
  live = live && N > 0;
  // LDS: per stage vectors of this group's problem
  float* W = lds + (size_t)sub * (fused_lds_floats<NC>(ln));   // w = vhat - betahat; restart terms
  float* Y = W + ln * V;          // y = zhat - vhat - e + lamhat
  float* ATY = Y + ln * V;        // Abar^T y
  float* HT = ATY + ln * V;       // htilde
  float* XI = HT + ln * V;        // xi_{k+1}
  float* T1 = XI + ln * V;        // Bt^T w_x + w_u
  float* DU = T1 + ln * NU;       // du
  float* PIN = DU + ln * NU;      // projection input (u part)
  float* PO = PIN + ln * NU;      // projection output
  float* SS = PO + ln * NU;       // restart-test sum of each stage
  float* XI0 = SS + ((ln + 3) & ~3);

  const int tid = PPW == 1 ? (int)threadIdx.x : (int)threadIdx.x - sub * tpp;
  const bool act = tid < N * NL;
  const int k = act ? tid / NL : 0;
  const int r = act ? tid % NL : 0;
  const int at = k * V + vrow(r);
  const size_t s0 = (size_t)b * n;
  const size_t st = s0 + k;
  const float mu = live ? p.mu[b] : 0.f;
  const float tsc = live ? ws.tsc[b] : 1.f;

  // operators into registers
  float hrow[NL], o1[NX], o2[NX], o3[NU];
  float qb = 0.f, eb = 0.f;
  if (act) {
    const size_t H0 = st * NH, A0 = st * NX * NX, B0 = st * NX * NU, M0 = st * NM;
    for (int j = 0; j < NL; ++j) hrow[j] = op.h(H0 + pk(r, j, NL));
    if (r < NX) {
      for (int j = 0; j < NX; ++j) o1[j] = op.a(A0 + r * NX + j);    // row r of A
      for (int j = 0; j < NX; ++j) o2[j] = op.a(A0 + j * NX + r);    // column r of A
      for (int j = 0; j < NU; ++j) o3[j] = op.bt(B0 + r * NU + j);   // row r of Bt
    } else {
      const int jj = r - NX;
      for (int i = 0; i < NX; ++i) o1[i] = op.bt(B0 + i * NU + jj);  // column jj of Bt
      for (int i = 0; i < NX; ++i) o2[i] = 0.f;
      for (int l = 0; l < NU; ++l) o3[l] = op.m(M0 + pk(jj, l, NU)); // row jj of M
    }
    qb = ws.qb[st * NL + r];
    eb = (r < NX && p.e) ? p.e[st * NX + r] : 0.f;
  }
  if (live && tid < NL) {
    float v;
    if (tid < NX) v = p.x0[(size_t)b * NX + tid];
    else v = p.u_prev ? p.u_prev[(size_t)b * NU + tid - NX] /
                            ((tid - NX) % 6 < 3 ? ws.sf[s0] : tsc)
                      : 0.f;
    XI0[vrow(tid)] = v;
  }

  // iterates
  float zh = 0, vh = 0, th = 0, bh = 0, lh = 0;
  float zc = 0, vc = 0, tc = 0, bc = 0, lc = 0;
  if (act) {
    const size_t base = (st * NSTATE) * NL + r;
    zh = ws.hat[base]; vh = ws.hat[base + NL]; th = ws.hat[base + 2 * NL];
    bh = ws.hat[base + 3 * NL]; lh = ws.hat[base + 4 * NL];
    zc = ws.cur[base]; vc = ws.cur[base + NL]; tc = ws.cur[base + 2 * NL];
    bc = ws.cur[base + 3 * NL]; lc = ws.cur[base + 4 * NL];
  }
  float alpha = live ? ws.alpha[b] : 1.f, cprev = live ? ws.cprev[b] : 0.f;
  int restarts = 0;
  // the contact-stage this thread projects (one thread each), its bounds
  // (a group has at least 25 threads per stage, so one pass covers them)
  const bool proj = tid < NC * N;
  const int pks = proj ? tid / NC : 0;
  const bool stance = proj && p.contact[(s0 + pks) * NC + tid % NC];
  const float F = proj ? p.fz_max[b] / ws.sf[s0 + pks] : 0.f;
  const float tm = proj ? p.tau_max[b] / tsc : 0.f;
  __syncthreads();

  for (int it = 0; it < iters; ++it) {
    if (act) {
      W[at] = vh - bh;
      Y[at] = zh - vh - eb + lh;
    }
    __syncthreads();
    if (act) {
      float aty;
      if (r < NX) {
        aty = dot<NX>(o2, Y + k * V, 0.f);
      } else {
        aty = dot<NX>(o1, Y + k * V, Y[at]);
        T1[k * NU + r - NX] = dot<NX>(o1, W + k * V, W[at]);
      }
      ATY[at] = aty;
    }
    __syncthreads();
    if (act) {
      float h = zh - th;
      if (k + 1 < N) h += ATY[at + V];
      HT[at] = fmaf(rho, h, qb);
      if (r >= NX) DU[k * NU + r - NX] = dot<NU>(o3, T1 + k * NU, 0.f);
    }
    __syncthreads();
    float xi = 0.f;
    if (act) {
      xi = dot<NX>(hrow, HT + k * V, 0.f);
      xi = dot<NU>(hrow + NX, HT + k * V + 16, xi);
      XI[at] = xi;
    }
    __syncthreads();
    float s = 0.f, bb = 0.f, gam = 0.f, zin = 0.f;
    if (act) {
      const float* prev = (k == 0) ? XI0 : XI + (k - 1) * V;
      if (r < NX) {
        s = dot<NX>(o1, prev, 0.f);
        s = dot<NU>(o3, prev + 16, s);
        bb = dot<NU>(o3, DU + k * NU, 0.f);
      } else {
        s = prev[vrow(r)];
        bb = DU[k * NU + r - NX];
      }
      gam = bb + bh - s - eb + lh;
      const float gt = xi + th + s + eb - lh;
      zin = (2.f * gt + gam) * (1.f / 3.f);
      if (r >= NX) PIN[k * NU + r - NX] = zin;
    }
    __syncthreads();
    if (proj) {
      const float* yv = PIN + tid * 6;
      float* o = PO + tid * 6;
      if (stance) {
        float px, py, pz;
        project_pyramid<float>(mu, F, yv[0], yv[1], yv[2], &px, &py, &pz);
        o[0] = px; o[1] = py; o[2] = pz;
        for (int a = 3; a < 6; ++a) o[a] = fminf(fmaxf(yv[a], -tm), tm);
      } else {
        for (int a = 0; a < 6; ++a) o[a] = 0.f;
      }
    }
    __syncthreads();
    float zv = 0, vv = 0, tv = 0, bv = 0, lv = 0;
    if (act) {
      zv = (r < NX) ? zin : PO[k * NU + r - NX];
      vv = 0.5f * (zv + gam);
      tv = th + xi - zv;
      bv = bh + bb - vv;
      lv = lh + zv - s - vv - eb;
    }
    if (accel) {
      // the restart test: the terms summed over a stage's rows in order by one
      // thread, then over the stages in order by every thread (an order fixed by
      // N alone, as in the other sweep kernels)
      if (act) {
        const float dz = zv - zh, dv = vv - vh;
        const float d1 = tv - th, d2 = bv - bh, d3 = lv - lh;
        W[at] = d1 * d1 + d2 * d2 + d3 * d3 + dz * dz + dv * dv + (dz - dv) * (dz - dv);
      }
      __syncthreads();
      if (tid < N) {
        SS[tid] = sum<NU>(W + tid * V + 16, sum<NX>(W + tid * V, 0.f));
      }
      __syncthreads();
      float cm = 0.f;
      int kk = 0;
      for (; kk + 4 <= N; kk += 4) cm = sum<4>(SS + kk, cm);
      for (; kk < N; ++kk) cm += SS[kk];
      if (cm < eta * cprev) {
        const float an = 0.5f * (1.f + sqrtf(1.f + 4.f * alpha * alpha));
        const float f = (alpha - 1.f) / an;
        zh = zv + f * (zv - zc); vh = vv + f * (vv - vc); th = tv + f * (tv - tc);
        bh = bv + f * (bv - bc); lh = lv + f * (lv - lc);
        alpha = an;
        cprev = cm;
      } else {
        zh = zc; vh = vc; th = tc; bh = bc; lh = lc;
        alpha = 1.f;
        cprev = cprev / eta;
        ++restarts;
      }
      zc = zv; vc = vv; tc = tv; bc = bv; lc = lv;
    } else {
      zh = zv; vh = vv; th = tv; bh = bv; lh = lv;
    }
  }
  if (act) {
    const size_t base = (st * NSTATE) * NL + r;
    ws.hat[base] = zh; ws.hat[base + NL] = vh; ws.hat[base + 2 * NL] = th;
    ws.hat[base + 3 * NL] = bh; ws.hat[base + 4 * NL] = lh;
    if (accel) {
      ws.cur[base] = zc; ws.cur[base + NL] = vc; ws.cur[base + 2 * NL] = tc;
      ws.cur[base + 3 * NL] = bc; ws.cur[base + 4 * NL] = lc;
    }
  }
  if (live && tid == 0) {
    ws.alpha[b] = alpha;
    ws.cprev[b] = cprev;
    ws.restarts[b] += restarts;
  }
}

// Problems per workgroup that fit: ppw groups of round_up(nl n, 64) threads.
int fit_ppw(int ppw, int nl, int n) {
  const int tpp = ((nl * n + 63) / 64) * 64;
  while (ppw > 1 && ppw * tpp > 1024) ppw /= 2;
  return ppw < 1 ? 1 : ppw;
}

// Whether the two-contact kernel of up to 512 threads should run in its build for
// four waves per SIMD: a second workgroup's operator loads and barriers then fill the
// first one's waits (207 us instead of 373 for three sweeps at 4096 x 20, 1.33 ms
// instead of 1.68 for a hundred at 4096 x 10), against 8 spilled registers, or 30 with
// several problems per workgroup (none with room for two waves).  Where a CU's share
// of the launch is two waves per SIMD or less there is no second one to make room
// for: 274 us instead of 299 for a hundred sweeps of one problem of 10 stages, 310
// instead of 383 for 64 of them in pairs, 300 instead of 417 for 512 of 5 stages in
// fours.  With one problem per workgroup the build without spills takes 3 us longer to
// start, which about 15 sweeps make up.
bool wants_room(unsigned grid, int threads, int ppw, int iters) {
  const unsigned cus = (unsigned)device_cus();
  const unsigned waves = (grid + cus - 1) / cus * (unsigned)(threads / 64);   // of a CU
  return waves > 8 || (ppw == 1 && iters < 16);
}

template <bool BF16, int NC>
hipError_t fused(const Problem& p, const Workspace& w, const pinmpc_settings& s, int iters,
                 int cap, const int32_t* ord, const int32_t* cnt, hipStream_t st) {
  const int ppw = NC == 2 ? fit_ppw(s.group, Dims<NC>::L, cap) : 1;
  const int threads = ppw * (((Dims<NC>::L * cap + 63) / 64) * 64);
  const dim3 grid((unsigned)((p.batch + ppw - 1) / ppw));
  const size_t lds = (size_t)ppw * fused_lds_floats<NC>(cap) * sizeof(float);
  // a kernel bound to fewer threads may use more registers (one row's operators are
  // 63 floats, 87 with four contacts); those of 1024 threads spill
#define PINMPC_FUSED(T, G, W)                                                                    \
  hipLaunchKernelGGL((admm_fused_kernel<T, BF16, G, NC, W>), grid, dim3(threads), lds, st, p, w, \
                     s.rho, s.accel, s.restart_eta, iters, ord, cnt, cap)
  if constexpr (NC == 2) {
    if (threads > 512) {
      if (ppw == 1) PINMPC_FUSED(1024, 1, 1);
      else if (ppw == 2) PINMPC_FUSED(1024, 2, 1);
      else PINMPC_FUSED(1024, 4, 1);
    } else if (wants_room(grid.x, threads, ppw, iters)) {
      if (ppw == 1) PINMPC_FUSED(512, 1, 4);
      else if (ppw == 2) PINMPC_FUSED(512, 2, 4);
      else PINMPC_FUSED(512, 4, 4);
    } else {
      if (ppw == 1) PINMPC_FUSED(512, 1, 1);
      else if (ppw == 2) PINMPC_FUSED(512, 2, 1);
      else PINMPC_FUSED(512, 4, 1);
    }
  } else {
    if (threads <= 512) PINMPC_FUSED(512, 1, 1);
    else if (threads <= 768) PINMPC_FUSED(768, 1, 1);
    else PINMPC_FUSED(1024, 1, 1);
  }
#undef PINMPC_FUSED
  return hipGetLastError();
}

}  // namespace

// (Four contacts beyond 20 stages run the 1024-thread build, which spills 48
// registers, and are still faster than with their operators streamed: 59 us instead of
// 146 for five sweeps of one problem of 27 stages, 823 instead of 1957 for 2048,
// 9.3 ms instead of 33 for a hundred.)
bool fused_fits(int nc, int n_max) { return (NX + 6 * nc) * n_max <= 1024; }

hipError_t launch_admm_fused(const Problem& p, const Workspace& w, const pinmpc_settings& s,
                             int iters, hipStream_t st) {
  if (p.batch == 0 || iters == 0) return hipSuccess;
  if (!fused_fits(p.nc, p.n_max)) return hipErrorInvalidValue;
  if (p.nc == 4)
    return s.precision ? fused<true, 4>(p, w, s, iters, p.n_max, nullptr, nullptr, st)
                       : fused<false, 4>(p, w, s, iters, p.n_max, nullptr, nullptr, st);
  return s.precision ? fused<true, 2>(p, w, s, iters, p.n_max, nullptr, nullptr, st)
                     : fused<false, 2>(p, w, s, iters, p.n_max, nullptr, nullptr, st);
}

// Problems of horizon class cls, walked through the order array; the grid
// covers the whole batch and workgroups past the class count exit at once.
hipError_t launch_admm_fused_class(const Problem& p, const Workspace& w, const pinmpc_settings& s,
                                   int iters, int cls, hipStream_t st) {
  if (p.batch == 0 || iters == 0) return hipSuccess;
  const int cap = CLASS_N[cls] < p.n_max ? CLASS_N[cls] : p.n_max;
  const int32_t* ord = w.order + (size_t)cls * p.batch;
  const int32_t* cnt = w.counts + cls;
  return s.precision ? fused<true, 2>(p, w, s, iters, cap, ord, cnt, st)
                     : fused<false, 2>(p, w, s, iters, cap, ord, cnt, st);
}

}  // namespace pinmpc
