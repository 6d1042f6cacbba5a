// From the contraction of eq. (19) to the ERIs: the fold of partial blocks and
// the scatter G[(pq)][(sr)] -> (pq|rs).
#include "kernels.hpp"

namespace {

// One partial block a workgroup: C (+)= its chunks, in order.
__global__ __launch_bounds__(256) void nt_fold_kernel(const NtDesc* __restrict__ descs, int ndesc, int tile, int edge,
                                                      long long t0, long long nblk, int c0, int nc,
                                                      const cplx* __restrict__ part) {
  const int per = tile / edge, sub2 = per * per;
  const long long u = blockIdx.x;
  const NtTile tl = nt_tile(descs, ndesc, t0 + u / sub2);
  const NtDesc d = descs[tl.desc];
  const int sub = (int)(u % sub2);
  const int m0 = tl.tm * tile + (sub / per) * edge, n0 = tl.tn * tile + (sub % per) * edge;
  cplx* C = (cplx*)d.C + (long long)tl.b * d.sC_bat;
  const long long sz = (long long)edge * edge;
  for (int e = threadIdx.x; e < sz; e += blockDim.x) {
    const int m = m0 + e / edge, n = n0 + e % edge;
    // above the diagonal of a Hermitian product nothing is computed or read
    if (m >= d.M || n >= d.N || (d.herm && n > m)) continue;
    cplx* o = C + (long long)m * d.ldc + n;
    cplx x = c0 > 0 ? *o : cmk(0.0, 0.0);
    for (int c = 0; c < nc; ++c) x = cadd(x, part[((long long)c * nblk + u) * sz + e]);
    *o = x;
  }
}

// E[(pq)][(sr)] (lower triangle computed) -> eri[p][q][r][s], fragment f
// reading e + eoff[f] and writing eri[f]
__global__ void eri_scatter_batch_kernel(const cplx* __restrict__ e, const long long* __restrict__ eoff,
                                         cplx* const* __restrict__ eri, const int* __restrict__ nfa) {
  const int f = blockIdx.y;
  const int nf = nfa[f];
  const cplx* ef = e + eoff[f];
  cplx* out = eri[f];
  const long long n = (long long)nf * nf;
  const long long total = n * n;
  // G[a][b] from the computed lower triangle (G is Hermitian)
  auto g = [&](long long a, long long b) { return a >= b ? ef[a * n + b] : cconj(ef[b * n + a]); };
  // (pq|rs) = G[(pq)][(sr)] + conj(G[(qp)][(rs)]) = v; (qp|sr) = conj(v),
  // (rs|pq) = v, (sr|qp) = conj(v): one thread per orbit {o1, o2, o3, o4}
  // (the smallest of the four output indices) reads G twice and writes all
  for (long long o = blockIdx.x * (long long)blockDim.x + threadIdx.x; o < total;
       o += (long long)gridDim.x * blockDim.x) {
    const long long pq = o / n, rs = o - pq * n;
    const int p_ = (int)(pq / nf), q_ = (int)(pq - (long long)p_ * nf);
    const int r_ = (int)(rs / nf), s_ = (int)(rs - (long long)r_ * nf);
    const long long qp = (long long)q_ * nf + p_, sr = (long long)s_ * nf + r_;
    const long long o2 = qp * n + sr, o3 = rs * n + pq, o4 = sr * n + qp;
    if (o2 < o || o3 < o || o4 < o) continue;
    const cplx a = g(pq, sr), b = g(qp, rs);
    const cplx v = cmk(a.x + b.x, a.y - b.y), vc = cmk(v.x, -v.y);
    out[o] = v;
    out[o2] = vc;
    out[o3] = v;
    out[o4] = vc;
  }
}

}  // namespace

hipError_t nt_fold_launch(const NtDesc* descs_dev, int ndesc, int tile, int edge, long long t0, long long nt, int c0,
                          int nc, const cplx* part, hipStream_t s) {
  if (nt <= 0) return hipSuccess;
  const long long nblk = nt * (tile / edge) * (tile / edge);
  hipLaunchKernelGGL(nt_fold_kernel, dim3((unsigned)nblk), dim3(256), 0, s, descs_dev, ndesc, tile, edge, t0, nblk, c0,
                     nc, part);
  return hipGetLastError();
}

hipError_t eri_scatter_batch_launch(const cplx* e, const long long* eoff, cplx* const* eri, const int* nf,
                                    int n, int maxnf, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const long long m = (long long)maxnf * maxnf;
  long long bx = (m * m + 255) / 256;
  if (bx > 1024) bx = 1024;
  hipLaunchKernelGGL(eri_scatter_batch_kernel, dim3((unsigned)bx, n), dim3(256), 0, s, e, eoff, eri, nf);
  return hipGetLastError();
}
