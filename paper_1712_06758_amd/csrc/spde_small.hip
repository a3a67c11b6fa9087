// Whole MINRES iterations of the small boxes (8^3 and 16^3) in one launch.
//
// One block per sample runs up to `iters` iterations with the Lanczos vectors on
// its compute unit: the current faces in LDS (their windows along the grid lines
// are what other threads read), the rest in registers, and one LDS array that
// the smoothing stages share.  Launched kernel by kernel, an iteration of a 16^3
// box is five launches of a few blocks each and takes 33 us (float64); here it is
// a chain of 16 block barriers and takes 12 us (28,900 cycles: the nine stages of
// the finest level 5,300, the 8^3 and 4^3 levels 7,000, the face windows and
// sums 11,300, the operator and the scalar step 5,300): a call on one 16^3 sample
// 1366 -> 648 us.  It is bound by the FP64 issue and the latencies of one compute
// unit; batches run side by side on the others.
//
// The arithmetic is that of the level, coarse, scalar and operator kernels,
// cell by cell; only the partial sums of gamma and delta are added in another
// order.  zhat goes to the ring and the update coefficients to its table, so
// that the direction pass follows as after the other kernels, and the Lanczos
// vectors are stored back when the launch ends.  Constant kappa only.
#include "spde_common.inc"
#include "spde_coarse8.inc"
#include "spde_scalar.inc"

namespace spde {

// Byte-offset store to a uniform base (as ld_off).
template <typename T>
__device__ __forceinline__ void st_off(T v, T* base, uint32_t byte_off) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + byte_off) = v;
}

struct SmallLevels {
  Level lv[2];        // the box's level and, below 16^3, the 8^3 one
  const void* cinv;   // inverse of the 4^3 level's operator (level precision, 64 x 64)
};

template <typename TM, int LN>
struct SmallLayout {
  // cells per thread: at 16^3 eight, whose state fits the registers of 512
  // threads (four by 1024 threads: 24.8 us an iteration, with spills)
  static constexpr int C = LN == 4 ? 8 : 4;
  static constexpr int n = 1 << LN, N = 1 << (3 * LN), T = N / C;
  // planes of the shared array end in a zero, which the neighbours outside the
  // box read
  static constexpr int PP = n * n + 1;
  static constexpr size_t faces = 3 * (size_t)N * sizeof(double);
  static constexpr size_t shared = (size_t)PP * n * sizeof(TM);
  static constexpr size_t coarse = (LN == 4 ? Coarse8<TM, false>::words() : 128) * sizeof(TM);
  static constexpr size_t bytes =
      faces + (2 * (T / 64) + 2) * sizeof(double) + sizeof(Scalars) + shared + coarse;
};

// Threads own columns of C cells along z (cells (i, j, C q .. C q + C - 1)), so
// that the z neighbours, the z window of the faces and the pairs of the
// restriction are mostly a thread's own.
// FIN: a sample that finishes gets the updates it has waiting before the launch ends.
template <typename TM, int LN, int POLY, bool FIN>
__global__ __launch_bounds__(LN == 4 ? 512 : 128) void k_small(Fields F, Box bx, SmallLevels P, int iters) {
  using S = SmallLayout<TM, LN>;
  constexpr int n = S::n, N = S::N, T = S::T, PL = n * n, PP = S::PP, C = S::C, Q = n / C;
  extern __shared__ __align__(16) unsigned char smem[];
  double* fs = reinterpret_cast<double*>(smem);                        // [3][N] faces of v_j
  double* red = fs + 3 * N;                                            // [T / 64][2]
  int* go = reinterpret_cast<int*>(red + 2 * (T / 64));                // whether the sample goes on
  Scalars* ss = reinterpret_cast<Scalars*>(red + 2 * (T / 64) + 2);    // the slot's scalars
  TM* sh = reinterpret_cast<TM*>(ss + 1);                              // [n][PP] shared by the stages
  TM* mem = sh + PP * n;                                               // the coarser levels
  const int slot = blockIdx.x;
  Scalars* SC = F.sc + slot;
  if (SC->state != ST_ACTIVE) return;
  const int tid = (int)threadIdx.x;
  const int pc = tid & (PL - 1), q = __builtin_amdgcn_readfirstlane(tid >> (2 * LN));
  static_assert(S::T == PL * Q && (LN == 3 || T == 512), "one column per thread, one cell of the 8^3 level");
  const int i = pc & (n - 1), j = pc >> LN;
  int c0 = pc + PL * C * q, s0 = pc + PP * C * q;                // the thread's first cell, and its place in sh
  const int64_t nc = N, co = cell_off(slot, nc);
  int jt = SC->it;
  double zs_prev = SC->zs;                                             // 1 / gamma_{j-1}
  if (tid == 0) *ss = *SC;
  if (tid < n) sh[tid * PP + PL] = (TM)0;
  TM *b4 = mem, *x4 = mem + 64;                                        // 8^3: the 4^3 level
  Coarse8<TM, false, LN == 4> K8(P.lv[1], P.cinv, mem, tid);                    // 16^3: the 8^3 and 4^3 levels

  // ---- constants of the thread's cells
  const Diag<TM> D(P.lv[0].k2, P.lv[0].a);
  const TM a = D.a;
  const int nxy = (i > 0) + (i < n - 1) + (j > 0) + (j < n - 1);
  TM dI = D.d(nxy + 2), dB = D.d(nxy + 1), vI = D.inv(nxy + 2), vB = D.inv(nxy + 1);
  auto edge = [&](int r) { return (r == 0 && q == 0) || (r == C - 1 && q == Q - 1); };
  auto dd = [&](int r) { return edge(r) ? dB : dI; };
  auto di = [&](int r) { return edge(r) ? vB : vI; };
  // places of the x and y neighbours of the thread's first cell (the others
  // follow at the plane pitch, the zeros too)
  const int z0 = PP * C * q + PL;
  int nxm = i > 0 ? s0 - 1 : z0, nxp = i < n - 1 ? s0 + 1 : z0;
  int nym = j > 0 ? s0 - n : z0, nyp = j < n - 1 ? s0 + n : z0;
  // sum over the neighbours of the thread's cells of the shared array, own[] the cells' values
  auto nbr = [&](const TM (&own)[C], TM (&sum)[C]) {
    const TM below = q > 0 ? sh[s0 - PP] : (TM)0, above = q < Q - 1 ? sh[s0 + C * PP] : (TM)0;
#pragma unroll
    for (int r = 0; r < C; ++r)
      sum[r] = sh[nxm + r * PP] + sh[nxp + r * PP] + sh[nym + r * PP] + sh[nyp + r * PP] +
               (r > 0 ? own[r > 0 ? r - 1 : 0] : below) + (r < C - 1 ? own[r < C - 1 ? r + 1 : 0] : above);
  };
  auto share = [&](const TM (&v)[C]) {
#pragma unroll
    for (int r = 0; r < C; ++r) sh[s0 + r * PP] = v[r];
  };
  // exact 4^3 solve: T / 64 lanes per row, each with 64 * 64 / T products
  constexpr int RL = T / 64, RP = 64 / RL;
  const TM* cinv = reinterpret_cast<const TM*>(P.cinv) + RP * tid;

  // ---- state: v_j's cell values and v_{j-1} in registers, v_j's faces in LDS
  // (global addresses: a uniform base and the lane's place in the plane)
  const uint32_t p8 = (uint32_t)pc * 8u, pm = (uint32_t)pc * (uint32_t)sizeof(TM);
  const int qo = PL * C * q;
  double vu[C], vuo[C], vo[3][C];
  {
    const int p = jt & 1;
#pragma unroll
    for (int r = 0; r < C; ++r) {
      vu[r] = ld_off(F.vu[p] + co + qo + r * PL, p8);
      vuo[r] = jt > 1 ? ld_off(F.vu[p ^ 1] + co + qo + r * PL, p8) : 0.0;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        fs[d * N + c0 + r * PL] = ld_off(F.vs[p] + face_off(slot, d, nc) + qo + r * PL, p8);
        vo[d][r] = jt > 1 ? ld_off(F.vs[p ^ 1] + face_off(slot, d, nc) + qo + r * PL, p8) : 0.0;
      }
    }
  }
  // x and y windows by odd reflection about the boundary faces 0 and n: the
  // index of each of the seven faces along the line, 4 bits each (the face n is
  // zero like the face 0, which is stored), and their signs
  uint32_t ox = 0, oy = 0, neg = 0;
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const int gx = i + k - 3, gy = j + k - 3;
    const int sx = gx < 0 ? -gx : (gx > n ? 2 * n - gx : gx), sy = gy < 0 ? -gy : (gy > n ? 2 * n - gy : gy);
    ox |= (uint32_t)(sx & (n - 1)) << (4 * k);
    oy |= (uint32_t)(sy & (n - 1)) << (4 * k);
    neg |= (uint32_t)(gx < 0 || gx > n) << k | (uint32_t)(gy < 0 || gy > n) << (k + 8);
  }
  auto signed_face = [&](double v, int bit) {
    const int hi = __double2hiint(v) ^ (int)((neg << (31 - bit)) & 0x80000000u);
    return __hiloint2double(hi, __double2loint(v));
  };
  int rowx = c0 - i, rowy = c0 - n * j, pz = pc;

  for (int it = 0; it < iters; ++it) {
    // what follows from these is formed anew in every iteration: the unpacked
    // offsets and the products with the diagonals would take registers that the
    // iteration needs
    asm volatile("" : "+v"(ox), "+v"(oy), "+v"(neg), "+v"(dI), "+v"(dB), "+v"(vI), "+v"(vB));
    asm volatile("" : "+v"(c0), "+v"(s0), "+v"(nxm), "+v"(nxp), "+v"(nym), "+v"(nyp), "+v"(rowx), "+v"(rowy),
                 "+v"(K8.at), "+v"(K8.zero), "+v"(pz));
    // pre-smoothing from zero: x = cA bhat + (cB / d) sum bhat
    TM bh[C], xs[C], t[C], w[C];
#pragma unroll
    for (int r = 0; r < C; ++r) bh[r] = (TM)vu[r] * di(r);
    share(bh);
    __syncthreads();
    nbr(bh, t);
#pragma unroll
    for (int r = 0; r < C; ++r) xs[r] = (TM)P.lv[0].cA * bh[r] + (TM)P.lv[0].cB * di(r) * t[r];
    __syncthreads();
    share(xs);
    __syncthreads();
    // the thread's entries of the 4^3 inverse, on their way during the residual
    TM sinv[RP];
#pragma unroll
    for (int u = 0; u < RP; ++u) sinv[u] = cinv[u];
    // residual, summed over the 8 children: pairs along z are the thread's own,
    // along x and y neighbouring lanes
    nbr(xs, t);
#pragma unroll
    for (int r = 0; r < C; ++r) w[r] = dd(r) * (bh[r] - xs[r]) + a * t[r];
#pragma unroll
    for (int u = 0; u < C / 2; ++u) {
      TM v = w[2 * u] + w[2 * u + 1];
      v += __shfl_xor(v, 1, 64);
      v += __shfl_xor(v, n, 64);
      if (!(i & 1) && !(j & 1)) {
        const int I = i >> 1, J = j >> 1, K = C / 2 * q + u;
        if constexpr (LN == 4) K8.y8[K8.place(I, J, K)] = v;
        else b4[I + 4 * (J + 4 * K)] = v;
      }
    }
    __syncthreads();
    if constexpr (LN == 4) {
      K8.solve(sinv);
    } else {   // exact solve on the 4^3 level
      const int part = tid & (RL - 1), row = tid / RL;
      TM v = sinv[0] * b4[RP * part];
#pragma unroll
      for (int u = 1; u < RP; ++u) v += sinv[u] * b4[RP * part + u];
#pragma unroll
      for (int o = 1; o < RL; o <<= 1) v += __shfl_xor(v, o, 64);
      if (part == 0) x4[row] = v;
      __syncthreads();
    }
    // x' = x + P e; r = d (bhat - x') + a sum x'; y = c0 D^-1 r
#pragma unroll
    for (int u = 0; u < C / 2; ++u) {
      const int I = i >> 1, J = j >> 1, K = C / 2 * q + u;
      const TM e = LN == 4 ? K8.x8[K8.place(I, J, K)] : x4[I + 4 * (J + 4 * K)];
      xs[2 * u] += e;
      xs[2 * u + 1] += e;
    }
    share(xs);
    __syncthreads();
    nbr(xs, t);
#pragma unroll
    for (int r = 0; r < C; ++r) {
      w[r] = dd(r) * (bh[r] - xs[r]) + a * t[r];
      bh[r] = (TM)P.lv[0].c0 * di(r) * w[r];      // y
    }
    __syncthreads();
    share(bh);
    __syncthreads();
    nbr(bh, t);
    // zhat = x' + c1 y + c2 D^-1 (r - S~ y), and the partial sums with the face
    // terms of v_j, which the operator takes too
    TM zh[C];
#pragma unroll
    for (int r = 0; r < C; ++r)
      zh[r] = xs[r] + (TM)P.lv[0].c1 * bh[r] + (TM)P.lv[0].c2 * di(r) * (w[r] - (dd(r) * bh[r] - a * t[r]));
    // (scheduling barriers: one cell's windows at a time, or the loads of all of
    // them together would not fit the registers)
    double mz[3][C], dv[C], sv = 0.0, sm = 0.0, p0 = 0.0, p1 = 0.0;
    __builtin_amdgcn_sched_barrier(0);
    {
      double wz[C + 6], zf[C + 1];
#pragma unroll
      for (int k = 0; k < C + 6; ++k) {   // z faces C q - 3 .. C q + C + 2 (q is uniform)
        const int g = C * q + k - 3, sg = g < 0 ? -g : (g > n ? 2 * n - g : g);
        const double v = fs[2 * N + pz + PL * (sg & (n - 1))];
        wz[k] = (g < 0 || g > n) ? -v : v;
      }
#pragma unroll
      for (int r = 0; r <= C; ++r)
        zf[r] = POLY ? 1.125 * wz[r + 3] - 0.25 * (wz[r + 2] + wz[r + 4]) +
                           0.0625 * (wz[r + 1] + wz[r + 5])
                     : wz[r + 3];
#pragma unroll
      for (int r = 0; r < C; ++r) {
        const double s1 = wz[r + 2] + wz[r + 4];
        mz[2][r] = POLY ? wz[r + 3] + 0.015625 * ((wz[r] + wz[r + 6]) + 3.0 * s1) : wz[r + 3] + 0.25 * s1;
        sv += zf[r] * wz[r + 3];
        sm += zf[r] * mz[2][r];
        dv[r] = zf[r + 1] - zf[r];
      }
    }
#pragma unroll
    for (int r = 0; r < C; ++r) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        double wd[7], zf, zhi;
#pragma unroll
        for (int k = 0; k < 7; ++k)
          wd[k] = d == 0 ? signed_face(fs[rowx + r * PL + ((ox >> (4 * k)) & 15)], k)
                         : signed_face(fs[N + rowy + r * PL + n * ((oy >> (4 * k)) & 15)], k + 8);
        line_terms_ext(wd, POLY, mz[d][r], zf, zhi);
        sv += zf * wd[3];
        sm += zf * mz[d][r];
        dv[r] += zhi - zf;
      }
      const double zc = (double)zh[r];
      p0 += zc * vu[r];
      p1 += 2.0 * zc * bx.h2q * dv[r] - bx.k2h3 * zc * zc;
    }
    p0 += bx.q * sv;
    p1 += bx.q * sm;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      p0 += __shfl_xor(p0, o, 64);
      p1 += __shfl_xor(p1, o, 64);
    }
    if ((tid & 63) == 0) {
      red[2 * (tid >> 6)] = p0;
      red[2 * (tid >> 6) + 1] = p1;
    }
    __syncthreads();   // (every stage has read y)
    share(zh);
    double a0 = 0.0, a1 = 0.0;
#pragma unroll
    for (int k = 0; k < T / 64; ++k) {
      a0 += red[2 * k];
      a1 += red[2 * k + 1];
    }
    __syncthreads();   // zhat is in the shared array
    // operator: v_{j+1} = A z_j - a_v v_j - b_v v_{j-1}, its coefficients from the
    // sums in every thread (as the scalar step forms them)
    const double gam = sqrt(a0), zs = 1.0 / gam, av = (a1 * zs) * zs * zs;
    const double bv = jt > 1 ? gam * zs_prev : 0.0;
    zs_prev = zs;
    const double zlow = q > 0 ? (double)sh[s0 - PP] : 0.0;
#pragma unroll
    for (int r = 0; r < C; ++r) {
      __builtin_amdgcn_sched_barrier(0);
      const int c = c0 + r * PL;
      const double zc = (double)zh[r];
      const double zlo[3] = {(double)sh[nxm + r * PP], (double)sh[nym + r * PP],
                             r > 0 ? (double)zh[r > 0 ? r - 1 : 0] : zlow};
      const bool inner[3] = {i > 0, j > 0, r > 0 || q > 0};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double w3 = fs[d * N + c];
        const double nv = zs * (mz[d][r] + bx.h2 * (zlo[d] - zc)) - av * w3 - bv * vo[d][r];
        fs[d * N + c] = inner[d] ? nv : 0.0;
        vo[d][r] = w3;
      }
      const double nu = zs * (bx.h2q * dv[r] - bx.k2h3 * zc) - av * vu[r] - bv * vuo[r];
      vuo[r] = vu[r];
      vu[r] = nu;
    }
    // zhat to the ring, here, where the stores have the whole V-cycle to complete
    __builtin_amdgcn_sched_barrier(0);
    TM* zr = reinterpret_cast<TM*>(F.z) + (jt & F.zm) * F.zstr + co + qo;
#pragma unroll
    for (int r = 0; r < C; ++r) st_off(zh[r], zr + r * PL, pm);
    // the rest of the scalar step follows the operator, whose registers it takes; a
    // sample that stops has no use for v_{j+1}
    if (tid == 0) {
      DirCoef dc{};
      if (scalar_step(*ss, a0, a1, dc)) F.dir[(int64_t)slot * (F.zm + 1) + (jt & F.zm)] = dc;
      *go = ss->state == ST_ACTIVE;
    }
    ++jt;
    __syncthreads();   // the shared array is free, the faces of v_{j+1} are complete
    if (!*go) break;
  }
  // a sample that goes on: v_j and v_{j-1} back to their buffers
  if (*go) {
    const int p = jt & 1;
#pragma unroll
    for (int r = 0; r < C; ++r) {
      st_off(vu[r], F.vu[p] + co + qo + r * PL, p8);
      st_off(vuo[r], F.vu[p ^ 1] + co + qo + r * PL, p8);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        st_off(fs[d * N + c0 + r * PL], F.vs[p] + face_off(slot, d, nc) + qo + r * PL, p8);
        st_off(vo[d][r], F.vs[p ^ 1] + face_off(slot, d, nc) + qo + r * PL, p8);
      }
    }
  }
  if constexpr (FIN) {
    if (ss->state == ST_DONE && ss->pit > ss->jf) {
      const int jf = ss->jf, m = ss->pit - jf;
      const int own = (int)(threadIdx.x & (PL - 1)) + PL * C * (int)(threadIdx.x >> (2 * LN));
      finish_cells<TM>(F, blockIdx.x, nc, jf, m, ss->flags & FL_ACCUM, own, own + PL * C, PL);   // (the zhat it wrote)
      __syncthreads();
      if (threadIdx.x == 0) ss->jf = jf + m;
    }
  }
  if (tid == 0) *SC = *ss;
}

bool small_box(const Box& bx, const Level& top) { return (bx.n == 8 || bx.n == 16) && !bx.kap && !top.dg; }

template <typename TM, int LN, int POLY, bool FIN>
static hipError_t launch_small_one(const Fields& F, const Box& bx, const SmallLevels& P, int batch, int iters,
                                   hipStream_t st) {
  using S = SmallLayout<TM, LN>;
  const hipError_t e = hipFuncSetAttribute((const void*)k_small<TM, LN, POLY, FIN>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_small<TM, LN, POLY, FIN>), dim3(batch), dim3(S::T), S::bytes, st, F, bx, P, iters);
  return hipGetLastError();
}

hipError_t launch_small(bool fp64, const Fields& F, const Box& bx, const Level& top, const Level& next,
                        const void* cinv, int batch, int iters, hipStream_t st) {
  if (!small_box(bx, top) || top.m != bx.n || next.m != bx.n / 2 || !cinv || iters > F.zm + 1)
    return hipErrorInvalidValue;
  SmallLevels P;
  P.lv[0] = top;
  P.lv[1] = next;
  P.cinv = cinv;
#define SPDE_SMALL(TM, LN)                                                                              \
  return F.finish ? (bx.poly ? launch_small_one<TM, LN, 1, true>(F, bx, P, batch, iters, st)            \
                             : launch_small_one<TM, LN, 0, true>(F, bx, P, batch, iters, st))           \
                  : (bx.poly ? launch_small_one<TM, LN, 1, false>(F, bx, P, batch, iters, st)           \
                             : launch_small_one<TM, LN, 0, false>(F, bx, P, batch, iters, st))
  if (bx.n == 16) {
    if (fp64) SPDE_SMALL(double, 4);
    SPDE_SMALL(float, 4);
  }
  if (fp64) SPDE_SMALL(double, 3);
  SPDE_SMALL(float, 3);
#undef SPDE_SMALL
}

}  // namespace spde
