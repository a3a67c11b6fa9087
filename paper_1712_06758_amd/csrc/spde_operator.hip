// Operator pass of the MINRES iteration (fused Lanczos recurrence),
// one-cell-per-thread and column forms.
#include "spde_common.inc"

namespace spde {

// ---------------------------------------------------------------------------
// operator pass of iteration j:
//   v_{j+1} = A z_j - a_v v_j - b_v v_{j-1},  z_j = (P_sigma^-1 v_sigma, zhat_u) / gamma_j.
// One thread per cell: the cell value and the three low faces of the cell.
//   (M z)_face = (M P_sigma^-1 v)_f / gamma              (line_terms)
//   (B^T z_u)_face = h^2 (zhat[c - e_d] - zhat[c]) / gamma
//   (A z)_cell = (h^2 q sum_d (z_hi - z_lo) / q - kappa^2 h^3 zhat) / gamma

// Slot and block of an operator launch.  Slots that all or nearly all iterate run
// in contiguous ranges, one range per XCD; a partly filled engine deals its slots
// out in turn.  (The turn costs the pass 15 % where every slot is busy: 64^3 x 32
// float64 148 -> 170 us; the level kernels run the same either way.)
__device__ __forceinline__ void operator_block(const Fields& F, int nb, int& slot, int& blk) {
  if (F.spread) {
    slot_block(blockIdx.x, gridDim.x, nb, slot, blk);
  } else {
    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    slot = lb >> ilog2(nb);
    blk = lb & (nb - 1);
  }
}

// POLY: face block of the preconditioner (0 diag(M)^-1, 1 Neumann series), a
// template parameter so that no window load sits behind a branch on it.
// VAR: cell-wise kappa (the reaction term kappa_c^2 h^3 of the cell row).
// FIN: the blocks of a finished slot apply the updates it has waiting (the last
// operator pass of a step of the slots; the sampling calls end with a direction pass).
// A launch of its own for that cost 1 % of a burst of requests (11.35 -> 11.46 ms);
// the instance costs a full 32^3 x 128 launch 4 of 45 us, once per step.
template <typename TZ, int POLY, bool VAR, bool FIN>
__global__ __launch_bounds__(kBlock) void k_operator(Fields F, Box bx, int nb) {
  int slot, blk;
  operator_block(F, nb, slot, blk);
  const Scalars* S = F.sc + slot;
  const int state = S->state;
  if (state != ST_ACTIVE) {
    if (FIN && state == ST_DONE)
      finish_block<TZ>(F, F.sc + slot, slot, nb, bx.nc, (int64_t)blk * kBlock, (int64_t)(blk + 1) * kBlock);
    return;
  }
  const int j = S->pit;
  const int p = j & 1, pq = p ^ 1;
  const int64_t nc = bx.nc;
  const int n = bx.n;
  const int64_t n2 = bx.n2;
  const int64_t c = (int64_t)blk * kBlock + threadIdx.x;
  if (c >= nc) return;
  const int i = (int)(c % n);
  const int jj = (int)((c / n) % n), k = (int)(c / n2);
  const int64_t co = cell_off(slot, nc);
  const bool has_prev = j > 1;
  const int idx[3] = {i, jj, k};
  const int64_t str[3] = {1, n, n2};
  // scalars before any store (after a store they could no longer be scalar loads)
  const double zs = S->zs, av = S->a_v, bv = S->b_v;
  // All loads first, unconditionally (the addresses are valid in every state;
  // values that a state does not need are discarded).  The stores go through
  // pointers that may alias the loads, so a load after a store, or inside a
  // branch the compiler may sink below the stores, would cost the wave another
  // memory round trip.
  const TZ* z = reinterpret_cast<const TZ*>(F.z) + (j & F.zm) * F.zstr + co;
  double w[3][7], vo[3], zlo[3];
  const double zc = (double)z[c];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    // radius 3 in either face-block mode (a branch here would split the
    // loads into groups that each wait for their own data)
    line_load_ext<3>(F.vs[p] + face_off(slot, d, nc), c, str[d], idx[d], n, w[d]);
    zlo[d] = (double)z[idx[d] > 0 ? c - str[d] : c];
    vo[d] = F.vs[pq][face_off(slot, d, nc) + c];
  }
  const double vuc = F.vu[p][co + c], vuo = F.vu[pq][co + c];
  // VAR: cell-wise kappa (shared by the slots), read with the other loads
  const double kc = VAR ? bx.kap[c] : 0.0;

  double dv = 0.0, nf[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double mz, zf, zh;
    line_terms_ext(w[d], POLY, mz, zf, zh);
    dv += zh - zf;
    const double a = zs * (mz + bx.h2 * (zlo[d] - zc));
    const double nv = a - av * w[d][3];
    nf[d] = idx[d] > 0 ? (has_prev ? nv - bv * vo[d] : nv) : 0.0;
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) F.vs[pq][face_off(slot, d, nc) + c] = nf[d];
  const double k2 = VAR ? (kc * kc) * bx.h3 : bx.k2h3;
  const double Au = zs * (bx.h2q * dv - k2 * zc);
  const double nu = Au - av * vuc;
  F.vu[pq][co + c] = has_prev ? nu - bv * vuo : nu;
}

// Column form of the operator pass for n a multiple of 64.  A block owns
// 64 x 4 cell columns (one grid row per wave) and walks ZC planes up z.  The
// z-window of the z faces slides in registers (one new plane per step), the z
// neighbour of zhat is the previous step's value, and each step stages the x
// faces of its 4 rows (with a 3-face halo along x) and the y faces of rows
// -3 .. +6 in LDS, from which the x and y windows are read.  Same arithmetic,
// in the same order, as k_operator.
// NT: the Lanczos vectors are streamed with the nontemporal hint (chosen by the
// launcher from the launch's working set).
template <typename TZ, int POLY, bool VAR, int ZC, bool NT, bool FIN>
__global__ __launch_bounds__(kBlock) void k_operator_col(Fields F, Box bx, int nb) {
  constexpr int XW = 64 + 6, AXF = XW * 4, RXF = (AXF + kBlock - 1) / kBlock;   // x faces, halo 3 in x
  constexpr int AYF = 64 * (4 + 6), RYF = (AYF + kBlock - 1) / kBlock;           // y faces, halo 3 in y
  __shared__ double sxf[2][AXF];
  __shared__ double syf[2][AYF];
  int slot, t;
  operator_block(F, nb, slot, t);
  const Scalars* S = F.sc + slot;
  const int state = S->state;
  if (state != ST_ACTIVE) {
    constexpr int64_t cells = 64 * 4 * ZC;   // of a block
    if (FIN && state == ST_DONE) finish_block<TZ>(F, F.sc + slot, slot, nb, bx.nc, t * cells, (t + 1) * cells);
    return;
  }
  const int j = S->pit;
  const int p = j & 1, pq = p ^ 1;
  const int64_t nc = bx.nc;
  const int n = bx.n;
  const int64_t n2 = bx.n2;
  int x0, y0, z0;
  tile_origin<64, 4, ZC>(t, n, x0, y0, z0);
  const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int i = x0 + lane;
  const int jj = __builtin_amdgcn_readfirstlane(y0 + wv);
  const int64_t col = i + (int64_t)n * jj;
  const int64_t co = cell_off(slot, nc);
  const bool has_prev = j > 1;
  const double zs = S->zs, av = S->a_v, bv = S->b_v;
  // staged items: byte offset within a plane and the odd-reflection factor
  uint32_t xo[RXF], yo[RYF];
  double xf[RXF], yf[RYF];
#pragma unroll
  for (int r = 0; r < RXF; ++r) {
    const int q = tid + r * kBlock;
    const int gx = x0 + q % XW - 3, gy = y0 + q / XW;
    const bool neg = gx < 0 || gx > n;
    const int src = gx < 0 ? -gx : (gx > n ? 2 * n - gx : gx);
    xo[r] = q < AXF ? (uint32_t)(min(src, n - 1) + n * gy) * 8u : 0u;
    xf[r] = (q >= AXF || src == n) ? 0.0 : (neg ? -1.0 : 1.0);
  }
#pragma unroll
  for (int r = 0; r < RYF; ++r) {
    const int q = tid + r * kBlock;
    const int gx = x0 + q % 64, gy = y0 + q / 64 - 3;
    const bool neg = gy < 0 || gy > n;
    const int src = gy < 0 ? -gy : (gy > n ? 2 * n - gy : gy);
    yo[r] = q < AYF ? (uint32_t)(gx + n * min(src, n - 1)) * 8u : 0u;
    yf[r] = (q >= AYF || src == n) ? 0.0 : (neg ? -1.0 : 1.0);
  }
  const TZ* z = reinterpret_cast<const TZ*>(F.z) + (j & F.zm) * F.zstr + co;
  const double* vs0 = F.vs[p] + face_off(slot, 0, nc);
  const double* vs1 = F.vs[p] + face_off(slot, 1, nc);
  const double* vz = F.vs[p] + face_off(slot, 2, nc) + col;
  // z face of plane g of this column, odd reflection about the boundary faces
  // 0 and n (the plane index is block-uniform, so the reflection is scalar)
  auto face_z = [&](int g) {
    const bool neg = g < 0 || g > n;
    const int src = g < 0 ? -g : (g > n ? 2 * n - g : g);
    const double x = vz[n2 * min(src, n - 1)];
    return x * (src == n ? 0.0 : (neg ? -1.0 : 1.0));
  };
  double wz[7];
#pragma unroll
  for (int q = 0; q < 6; ++q) wz[q] = face_z(z0 - 3 + q);
  double zprev = (double)z[col + n2 * max(z0 - 1, 0)];
  for (int kk = 0; kk < ZC; ++kk) {
    const int k = z0 + kk;
    const int64_t pk = n2 * k;
    const int64_t c = col + pk;
    const int b = kk & 1;
    // stage this plane's x and y faces (the buffer written two steps ago has
    // been read by everyone: the previous step's barrier lies between)
    const double* px = vs0 + pk;
    const double* py = vs1 + pk;
#pragma unroll
    for (int r = 0; r < RXF; ++r) {
      const int q = tid + r * kBlock;
      if ((r + 1) * kBlock <= AXF || q < AXF) sxf[b][q] = ld_off(px, xo[r]) * xf[r];
    }
#pragma unroll
    for (int r = 0; r < RYF; ++r) {
      const int q = tid + r * kBlock;
      if ((r + 1) * kBlock <= AYF || q < AYF) syf[b][q] = ld_off(py, yo[r]) * yf[r];
    }
    wz[6] = face_z(k + 3);
    double vo[3];
    const double zc = (double)z[c];
    const double zlo[3] = {(double)z[i > 0 ? c - 1 : c], (double)z[jj > 0 ? c - n : c], k > 0 ? zprev : zc};
#pragma unroll
    for (int d = 0; d < 3; ++d) vo[d] = ld_stream<NT>(&F.vs[pq][face_off(slot, d, nc) + c]);
    const double vuc = ld_stream<NT>(&F.vu[p][co + c]), vuo = ld_stream<NT>(&F.vu[pq][co + c]);
    const double kc = VAR ? bx.kap[c] : 0.0;
    __syncthreads();
    double w[2][7];
#pragma unroll
    for (int q = 0; q < 7; ++q) {
      w[0][q] = sxf[b][lane + q + XW * wv];
      w[1][q] = syf[b][lane + 64 * (wv + q)];
    }
    const int idx[3] = {i, jj, k};
    double dv = 0.0, nf[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double* wd = d == 2 ? wz : w[d];
      double mz, zf, zh;
      line_terms_ext(wd, POLY, mz, zf, zh);
      dv += zh - zf;
      const double a = zs * (mz + bx.h2 * (zlo[d] - zc));
      const double nv = a - av * wd[3];
      nf[d] = idx[d] > 0 ? (has_prev ? nv - bv * vo[d] : nv) : 0.0;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) st_stream<NT>(nf[d], &F.vs[pq][face_off(slot, d, nc) + c]);
    const double k2 = VAR ? (kc * kc) * bx.h3 : bx.k2h3;
    const double Au = zs * (bx.h2q * dv - k2 * zc);
    const double nu = Au - av * vuc;
    st_stream<NT>(has_prev ? nu - bv * vuo : nu, &F.vu[pq][co + c]);
#pragma unroll
    for (int q = 0; q < 6; ++q) wz[q] = wz[q + 1];
    zprev = zc;
  }
}


// Planes per block of the column form.  A launch whose vectors stream past the
// last-level cache has thousands of blocks and takes 16: deeper blocks read fewer
// planes of the z windows twice (128^3 x 2 mixed, a call: 7.82 ms with 16, 7.94
// with 4; 256^3 x 1: 25.9 and 26.2).  A launch that stays in the cache has few
// blocks, each a chain of one memory latency per plane, and takes 4, or 2 where
// 4 would leave fewer than four blocks per compute unit (64^3 x 1 mixed, a call:
// 2.77 ms with 16, 2.12 with 4, 2.06 with 2; 64^3 x 7: 5.08, 4.85, 4.86; 128^3 x 1
// float64: 7.42, 7.24, 7.26).
constexpr int kOpZC = 16, kOpZCShort = 4, kOpZCShortest = 2;

template <typename TZ, int ZC, bool NT, bool FIN>
static hipError_t launch_operator_col(const Fields& F, const Box& bx, int batch, hipStream_t st) {
  const int nb = (bx.n / 64) * (bx.n / 4) * (bx.n / ZC);   // 64 x 4 columns of ZC planes per block
  const dim3 grid(nb * batch), blk(kBlock);
  if (bx.kap) {
    if (bx.poly) hipLaunchKernelGGL((k_operator_col<TZ, 1, true, ZC, NT, FIN>), grid, blk, 0, st, F, bx, nb);
    else hipLaunchKernelGGL((k_operator_col<TZ, 0, true, ZC, NT, FIN>), grid, blk, 0, st, F, bx, nb);
  } else {
    if (bx.poly) hipLaunchKernelGGL((k_operator_col<TZ, 1, false, ZC, NT, FIN>), grid, blk, 0, st, F, bx, nb);
    else hipLaunchKernelGGL((k_operator_col<TZ, 0, false, ZC, NT, FIN>), grid, blk, 0, st, F, bx, nb);
  }
  return hipGetLastError();
}

template <typename TZ, bool FIN>
static hipError_t launch_operator_as(const Fields& F, const Box& bx, int batch, hipStream_t st) {
  if (bx.n % 64 == 0) {
    if (streams_past_cache(bx, batch)) return launch_operator_col<TZ, kOpZC, true, FIN>(F, bx, batch, st);
    // (a block of 4 planes has 1024 cells)
    if ((double)bx.nc * batch >= 4.0 * 256 * 1024)
      return launch_operator_col<TZ, kOpZCShort, false, FIN>(F, bx, batch, st);
    return launch_operator_col<TZ, kOpZCShortest, false, FIN>(F, bx, batch, st);
  }
  const int nb = operator_blocks(bx);
  const dim3 grid(nb * batch), blk(kBlock);
  if (bx.kap) {
    if (bx.poly) hipLaunchKernelGGL((k_operator<TZ, 1, true, FIN>), grid, blk, 0, st, F, bx, nb);
    else hipLaunchKernelGGL((k_operator<TZ, 0, true, FIN>), grid, blk, 0, st, F, bx, nb);
  } else {
    if (bx.poly) hipLaunchKernelGGL((k_operator<TZ, 1, false, FIN>), grid, blk, 0, st, F, bx, nb);
    else hipLaunchKernelGGL((k_operator<TZ, 0, false, FIN>), grid, blk, 0, st, F, bx, nb);
  }
  return hipGetLastError();
}

hipError_t launch_operator(bool z_fp64, const Fields& F, const Box& bx, int batch, hipStream_t st) {
  if (F.finish)
    return z_fp64 ? launch_operator_as<double, true>(F, bx, batch, st)
                  : launch_operator_as<float, true>(F, bx, batch, st);
  return z_fp64 ? launch_operator_as<double, false>(F, bx, batch, st)
                : launch_operator_as<float, false>(F, bx, batch, st);
}

}  // namespace spde
