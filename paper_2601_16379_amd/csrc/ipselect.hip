// Interpolation-point selection by pivoted Cholesky of the pair products
// (the IP-selection paragraph of the paper's section "Periodic k-point
// FFTISDF representation of integrals").  The products
// phi^{k_mu}_mu(r) conj(phi^{k_nu}_nu(r)) over all orbital pairs have the
// Gram matrix M(x, y) = |G(x, y)|^2 with G(x, y) = sum_k sum_mu
// phi^k_mu(x) conj(phi^k_mu(y)), whose diagonal is rho(x)^2.  The greedy
// (diagonally pivoted) Cholesky keeps a residual diagonal d and, at step i,
// takes the point p of largest residual (lowest index among equals), forms
//   L_i(x) = (|G(x, p)|^2 - sum_{j<i} L_j(x) L_j(p)) / sqrt(d(p))
// and lowers d(x) by L_i(x)^2; the chosen point leaves the candidate set
// (its residual is zero in exact arithmetic and is set to zero).  M is never
// formed.  Everything is FP64.
//
// Orbitals are rows phi_r(x), r = (k, mu), of length N_g (the context's
// [N_k][N_orb][N_g] layout).  A step is two launches and keeps the pivot in
// device memory:
//   sel_part   -- every workgroup reduces the block maxima of the last update
//                 to the step's pivot; when its column of G is not held, one
//                 pass over the orbitals forms the columns of the pivot and of
//                 the C - 1 points next in line (the largest residuals of
//                 other blocks): partial sums over a slice of rows, one thread
//                 per grid point, the slice's values at the C points in LDS;
//   sel_update -- sums the slices of the pivot's column, forms the column of
//                 the factor and the residual, writes L_i and d, and reduces
//                 its block's d to (max, argmax).
// Bound: a pass reads the orbitals once (N_k N_orb N_g 16 bytes); one
// with 8 columns takes 184 us against 152 for one (872 MB).  A greedy
// step takes the largest residual; the point next in line is usually taken
// soon, so a pass serves several steps: 8 columns leave about one pass in five
// to six steps (4x4x4 mesh, 32^3 grid, 520 points: 104 -> 31 ms; a pass a
// step was 152 us of the 201 us a step).  The update reads the previous columns
// once (i N_g 8 bytes): one wavefront a workgroup and 16 loads in flight a
// lane, so that a 32^3 grid has work for every CU (43 -> 21 us a step).
#include "kernels.hpp"

namespace {

constexpr int SEL_T = 256;       // threads of a sel_part workgroup (4 wavefronts)
constexpr int SEL_X = 512;       // grid points of a sel_part workgroup (two a thread)
constexpr int SEL_U = 64;        // threads of a sel_update workgroup
constexpr int SEL_ROWS = 128;    // rows staged per LDS pass of sel_part
constexpr int SEL_CHUNK = 1024;  // earlier columns' values at p staged per LDS pass of sel_update
constexpr int SEL_LD = 16;       // their loads in flight a lane

__global__ void sel_clear_kernel(int* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

// larger value wins; among equal values the lower index
__device__ inline void argmax_merge(double& v, long long& i, double v2, long long i2) {
  if (v2 > v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}

__device__ inline void wave_argmax(double& v, long long& i) {
  for (int off = 32; off > 0; off >>= 1) {
    const double v2 = __shfl_xor(v, off);
    const long long i2 = __shfl_xor(i, off);
    argmax_merge(v, i, v2, i2);
  }
}

// (max, argmax) over the SEL_T threads of a workgroup; every thread returns
// the result
__device__ inline void block_argmax(double& v, long long& i) {
  __shared__ double sv[SEL_T / 64];
  __shared__ long long si[SEL_T / 64];
  wave_argmax(v, i);
  __syncthreads();                       // the last call's results have been read
  if ((threadIdx.x & 63) == 0) {
    sv[threadIdx.x >> 6] = v;
    si[threadIdx.x >> 6] = i;
  }
  __syncthreads();
  for (int w = 0; w < SEL_T / 64; ++w) argmax_merge(v, i, sv[w], si[w]);
}

// Columns of G held in part: those of the points pt[0 .. n).
template <int C>
struct SelCols {
  int n, slot;        // slot: the one of the current pivot
  int pt[C];
};

// rho(x) over slice s = blockIdx.y of the rows: part[s][x] = (sum_r |phi_r(x)|^2, 0)
__global__ __launch_bounds__(SEL_T) void sel_rho_kernel(const cplx* __restrict__ phi, long long nrows, long long ng,
                                                      long long rows_per, cplx* __restrict__ part) {
  const long long r0 = (long long)blockIdx.y * rows_per;
  const long long r1 = r0 + rows_per < nrows ? r0 + rows_per : nrows;
  for (int h = 0; h < SEL_X; h += SEL_T) {
    const long long x = (long long)blockIdx.x * SEL_X + h + threadIdx.x;
    if (x >= ng) return;
    double gr = 0.0;
    for (long long r = r0; r < r1; ++r) {
      const cplx a = phi[r * ng + x];
      gr = fma(a.x, a.x, fma(a.y, a.y, gr));
    }
    part[(long long)blockIdx.y * ng + x] = cmk(gr, 0.0);
  }
}

// The pivot of `step` from the nb block maxima (bv, bi) into piv and dmax, and
// the state of the columns from st[step & 1] into st[(step + 1) & 1].  When
// the pivot's column is not held: slice s = blockIdx.y of the rows, part[c][s][x]
// = sum_r phi_r(x) conj(phi_r(pt[c])).
template <int C>
__global__ __launch_bounds__(SEL_T) void sel_part_kernel(const cplx* __restrict__ phi, long long nrows, long long ng,
                                                       long long rows_per, const double* __restrict__ bv,
                                                       const long long* __restrict__ bi, int nb, int* piv,
                                                       double* dmax, int step, SelCols<C>* st,
                                                       cplx* __restrict__ part) {
  __shared__ cplx sp[SEL_ROWS][C];
  __shared__ SelCols<C> cols;
  const SelCols<C>* old = st + (step & 1);
  // pivot and, for C > 1, the points next in line: the maxima of other blocks
  double v = -1.0;
  long long p = ng;
  for (int b = threadIdx.x; b < nb; b += SEL_T) argmax_merge(v, p, bv[b], bi[b]);
  block_argmax(v, p);
  const bool first = blockIdx.x == 0 && blockIdx.y == 0;
  if (first && threadIdx.x == 0) {
    piv[step] = (int)(p < ng ? p : -1);
    dmax[step] = p < ng ? v : -1.0;
  }
  // a pivot that is not valid reads point 0; sel_update then discards the column
  const int pv = p < ng && v > 0.0 ? (int)p : 0;
  int slot = -1;
  for (int c = 0; c < old->n; ++c)
    if (old->pt[c] == pv) slot = c;
  if (slot >= 0) {
    if (first && threadIdx.x == 0) {
      SelCols<C> o = *old;
      o.slot = slot;
      st[(step + 1) & 1] = o;
    }
    return;
  }
  if (threadIdx.x == 0) {
    cols.n = 1;
    cols.slot = 0;
    for (int c = 0; c < C; ++c) cols.pt[c] = pv;
  }
  for (int c = 1; c < C; ++c) {
    __syncthreads();
    double cv = -1.0;
    long long ci = ng;
    for (int b = threadIdx.x; b < nb; b += SEL_T) {
      bool taken = false;
      for (int e = 0; e < c; ++e) taken = taken || bi[b] == cols.pt[e];
      if (!taken) argmax_merge(cv, ci, bv[b], bi[b]);
    }
    block_argmax(cv, ci);
    if (threadIdx.x == 0 && ci < ng && cv > 0.0) {
      cols.pt[c] = (int)ci;
      cols.n = c + 1;
    }
  }
  __syncthreads();
  if (first && threadIdx.x == 0) st[(step + 1) & 1] = cols;
  // two grid points a thread: each value read from LDS serves both
  const long long x0 = (long long)blockIdx.x * SEL_X + threadIdx.x, x1 = x0 + SEL_T;
  const long long xa = x0 < ng ? x0 : ng - 1, xb = x1 < ng ? x1 : ng - 1;
  const long long r0 = (long long)blockIdx.y * rows_per;
  const long long r1 = r0 + rows_per < nrows ? r0 + rows_per : nrows;
  double gr[2][C], gi[2][C];
#pragma unroll
  for (int c = 0; c < C; ++c) gr[0][c] = gi[0][c] = gr[1][c] = gi[1][c] = 0.0;
  for (long long c0 = r0; c0 < r1; c0 += SEL_ROWS) {
    const int n = (int)(r1 - c0 < SEL_ROWS ? r1 - c0 : SEL_ROWS);
    __syncthreads();
    for (int e = threadIdx.x; e < n * C; e += SEL_T) sp[e / C][e % C] = phi[(c0 + e / C) * ng + cols.pt[e % C]];
    __syncthreads();
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const cplx* row = phi + (c0 + j) * ng;
      const cplx a[2] = {row[xa], row[xb]};
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const cplx b = sp[j][c];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          gr[h][c] = fma(a[h].x, b.x, fma(a[h].y, b.y, gr[h][c]));
          gi[h][c] = fma(a[h].y, b.x, fma(-a[h].x, b.y, gi[h][c]));
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    cplx* o = part + ((long long)c * gridDim.y + blockIdx.y) * ng;
    if (x0 < ng) o[x0] = cmk(gr[0][c], gi[0][c]);
    if (x1 < ng) o[x1] = cmk(gr[1][c], gi[1][c]);
  }
}

// INIT: d(x) = rho(x)^2.  Else column `step`:
//   l = (|G(x, p)|^2 - sum_{j<step} L_j(x) L_j(p)) / sqrt(d(p)),  L_step(x) = l,
//   d(x) -= l^2, and d(p) = 0.
// Both end with the workgroup's (max d, argmax) in bv[b], bi[b].
template <bool INIT, int C>
__global__ __launch_bounds__(SEL_U) void sel_update_kernel(const cplx* __restrict__ part, int nslice, long long ng,
                                                         double* __restrict__ lf, double* __restrict__ d,
                                                         const int* __restrict__ piv, const double* __restrict__ dmax,
                                                         int step, const SelCols<C>* st, double* __restrict__ bv,
                                                         long long* __restrict__ bi) {
  __shared__ double sl[SEL_CHUNK];
  const long long x = (long long)blockIdx.x * SEL_U + threadIdx.x;
  const bool in = x < ng;
  const long long xr = in ? x : ng - 1;              // a readable point
  double gr = 0.0, gi = 0.0;
  const cplx* col = part + (INIT ? 0 : (long long)st[(step + 1) & 1].slot * nslice * ng);
  for (int s = 0; s < nslice; ++s) {
    const cplx g = col[(long long)s * ng + xr];
    gr += g.x;
    gi += g.y;
  }
  double dn = 0.0;
  if (INIT) {
    dn = gr * gr;
    if (in) d[x] = dn;
  } else {
    const double dm = dmax[step];
    const long long pp = piv[step];
    const bool ok = dm > 0.0 && pp >= 0 && pp < ng;
    const long long p = ok ? pp : 0;
    double corr = 0.0;
    for (int j0 = 0; j0 < step; j0 += SEL_CHUNK) {
      const int n = step - j0 < SEL_CHUNK ? step - j0 : SEL_CHUNK;
      __syncthreads();
      for (int j = threadIdx.x; j < n; j += SEL_U) sl[j] = lf[(long long)(j0 + j) * ng + p];
      __syncthreads();
      const double* lc = lf + (long long)j0 * ng + xr;
      int j = 0;
      for (; j + SEL_LD <= n; j += SEL_LD) {
        double t[SEL_LD];
#pragma unroll
        for (int e = 0; e < SEL_LD; ++e) t[e] = lc[(long long)(j + e) * ng];
#pragma unroll
        for (int e = 0; e < SEL_LD; ++e) corr = fma(t[e], sl[j + e], corr);
      }
      for (; j < n; ++j) corr = fma(lc[(long long)j * ng], sl[j], corr);
    }
    if (in) {
      const double l = ok ? (gr * gr + gi * gi - corr) / sqrt(dm) : 0.0;
      lf[(long long)step * ng + x] = l;
      dn = (ok && x == p) ? 0.0 : d[x] - l * l;
      d[x] = dn;
    }
  }
  double v = in ? dn : -1.0;
  long long i = in ? x : ng;
  wave_argmax(v, i);
  if (threadIdx.x == 0) {
    bv[blockIdx.x] = v;
    bi[blockIdx.x] = i;
  }
}

template <int C>
hipError_t step_launch(const SelPlan& pl, const cplx* phi, long long nrows, long long ng, const SelBufs& b, int step,
                       hipStream_t s) {
  SelCols<C>* st = (SelCols<C>*)b.state;
  hipLaunchKernelGGL(sel_part_kernel<C>, dim3(pl.xblocks, pl.nslice), dim3(SEL_T), 0, s, phi, nrows, ng, pl.rows_per,
                     b.bv, b.bi, pl.ublocks, b.piv, b.dmax, step, st, b.part);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sel_update_kernel<false, C>), dim3(pl.ublocks), dim3(SEL_U), 0, s, b.part, pl.nslice, ng, b.lf,
                     b.d, b.piv, b.dmax, step, st, b.bv, b.bi);
  return hipGetLastError();
}

}  // namespace

SelPlan sel_plan(long long nrows, long long ng) {
  SelPlan p;
  p.xblocks = (int)((ng + SEL_X - 1) / SEL_X);
  p.ublocks = (int)((ng + SEL_U - 1) / SEL_U);
  // enough row slices that a pass has about 1024 workgroups, each slice at
  // least 16 rows long
  long long ns = (1024 + p.xblocks - 1) / p.xblocks;
  const long long most = (nrows + 15) / 16;
  if (ns > most) ns = most;
  if (ns < 1) ns = 1;
  p.rows_per = (nrows + ns - 1) / ns;
  p.nslice = (int)((nrows + p.rows_per - 1) / p.rows_per);
  return p;
}

hipError_t sel_start_launch(const SelPlan& pl, const cplx* phi, long long nrows, long long ng, const SelBufs& b,
                            hipStream_t s) {
  hipLaunchKernelGGL(sel_rho_kernel, dim3(pl.xblocks, pl.nslice), dim3(SEL_T), 0, s, phi, nrows, ng, pl.rows_per,
                     b.part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sel_update_kernel<true, 1>), dim3(pl.ublocks), dim3(SEL_U), 0, s, b.part, pl.nslice, ng, b.lf,
                     b.d, b.piv, b.dmax, 0, (const SelCols<1>*)nullptr, b.bv, b.bi);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // no column is held yet
  hipLaunchKernelGGL(sel_clear_kernel, dim3(1), dim3(64), 0, s, (int*)b.state, (int)(SEL_STATE_BYTES / sizeof(int)));
  return hipGetLastError();
}

hipError_t sel_step_launch(const SelPlan& pl, const cplx* phi, long long nrows, long long ng, const SelBufs& b,
                           int ncols, int step, hipStream_t s) {
  return ncols == SEL_COLS ? step_launch<SEL_COLS>(pl, phi, nrows, ng, b, step, s)
                           : step_launch<1>(pl, phi, nrows, ng, b, step, s);
}
