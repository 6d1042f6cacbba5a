// Steps of the blocked Cholesky factor that the waves of a workgroup share
// through LDS: the unblocked factor of a 64 x 64 diagonal block and the forward
// substitution with its triangle.  (No includes: the host test compiles them on
// its own cplx, barriers and lane exchange.)
#pragma once

// Unblocked Cholesky of the diagonal block A[jb:jb+nb, jb:jb+nb].
// Bound: the chain of 64 columns, each a square root, a reciprocal and an
// update.  The block is held in registers, lane i of every wave its row i, wave
// w the columns w + 4 e; a column goes through LDS to the other waves, one
// barrier a column (two buffers in turn).  Each entry takes the same updates in
// the same order as in LDS with three barriers a column: 93 -> 35 us a block.
// The breakdown flag is one of two in turn as well: a wave that reads column
// J's late must not see column J + 1's, or it would leave before a barrier that
// the others still reach.
template <int J>
__device__ inline bool diag_steps(cplx (&d)[16], cplx (&col)[2][CHOL_NB], int (&bad)[2], double tol, int nb, int lane,
                                  int w) {
  if constexpr (J < CHOL_NB) {
    if (J >= nb) return true;
    constexpr int EJ = J / 4, WJ = J % 4;
    cplx* cj = col[J & 1];
    if (w == WJ) {
      const double djj = __shfl(d[EJ].x, J);
      if (!(djj > tol) || !(djj > 0.0)) {      // the same for the whole wave
        if (lane == 0) bad[J & 1] = 1;
      } else {
        const double r = sqrt(djj);
        d[EJ] = lane == J ? cmk(r, 0.0) : cscale(d[EJ], 1.0 / r);
        cj[lane] = d[EJ];
      }
    }
    __syncthreads();
    if (bad[J & 1]) return false;
    const cplx li = cj[lane];
#pragma unroll
    for (int e = EJ; e < 16; ++e) {
      if (e == EJ && w <= WJ) continue;
      const cplx lc = cj[4 * e + w];
      d[e].x -= fma(li.x, lc.x, li.y * lc.y);
      d[e].y -= fma(li.y, lc.x, -(li.x * lc.y));
    }
    return diag_steps<J + 1>(d, col, bad, tol, nb, lane, w);
  }
  return true;
}

// Forward substitution with a 64 x 64 lower triangle for 64 right hand sides,
//   x_c = (a_c - sum_{d<c} op(L[c][d]) x_d) / L[c][c],  d ascending,
// op the conjugate for CJ; unknowns at or past rb are zero.  Bound: the chain of
// 64 unknowns.  256 threads, four lanes (a quad) a right hand side, 8 unknowns
// at a time, two a lane in registers: the earlier unknowns' products first
// (T[d][c] = L[c][d], X and the reciprocals of the diagonal in LDS, the reads of
// several d in flight), then the 8 in turn, each sent through the quad by DPP.
// A block of the factor's panel 112-220 -> 35 us, a diagonal block's inverse
// 152-250 -> 29 us (one lane a right hand side, one unknown at a time).
struct Tri64 {
  cplx T[CHOL_NB][CHOL_NB];
  cplx X[64][CHOL_NB + 1];
  double rinv[CHOL_NB];
};
// the triangle at jb from lt (L transposed); nb rows and columns of it
__device__ inline void load_tri(Tri64& t, const cplx* lt, int n, int jb, int nb) {
  const int c = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int d = w; d < CHOL_NB; d += 4)
    t.T[d][c] = d <= c && c < nb ? lt[(long long)(jb + d) * n + jb + c] : cmk(0.0, 0.0);
  if (w == 0) t.rinv[c] = c < nb ? 1.0 / lt[(long long)(jb + c) * (n + 1)].x : 0.0;
}
template <int K> __device__ inline cplx quad_bcast(cplx v) {
  auto one = [](double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, K * 0x55, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), K * 0x55, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
  };
  return cmk(one(v.x), one(v.y));
}
// s -= op(l) x, the roundings written out so that every caller has the same
template <bool CJ>
__device__ inline void tri_sub(cplx& s, const cplx l, const cplx x) {
  if (CJ) {
    s.x -= fma(x.x, l.x, x.y * l.y);
    s.y -= fma(x.y, l.x, -(x.x * l.y));
  } else {
    s.x -= fma(l.x, x.x, -(l.y * x.y));
    s.y -= fma(l.y, x.x, l.x * x.y);
  }
}
template <bool CJ, int V>
__device__ inline void tri_step(Tri64& t, cplx (&acc)[2], int c0, int rb, int row, int g) {
  if constexpr (V < 8) {
    const cplx x = quad_bcast<V / 2>(c0 + V < rb ? cscale(acc[V & 1], t.rinv[c0 + V]) : cmk(0.0, 0.0));
    if (g == V / 2) t.X[row][c0 + V] = x;
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (2 * g + u > V) tri_sub<CJ>(acc[u], t.T[c0 + V][c0 + 2 * g + u], x);
    tri_step<CJ, V + 1>(t, acc, c0, rb, row, g);
  }
}
template <bool CJ>
__device__ inline void tri_solve64(Tri64& t, int rb) {
  const int row = threadIdx.x >> 2, g = threadIdx.x & 3;
  for (int c0 = 0; c0 < rb; c0 += 8) {
    cplx acc[2] = {t.X[row][c0 + 2 * g], t.X[row][c0 + 2 * g + 1]};
#pragma unroll 8
    for (int d = 0; d < c0; ++d) {
      const cplx x = t.X[row][d];
#pragma unroll
      for (int u = 0; u < 2; ++u) tri_sub<CJ>(acc[u], t.T[d][c0 + 2 * g + u], x);
    }
    tri_step<CJ, 0>(t, acc, c0, rb, row, g);
    wave_sync();                         // the next unknowns read what the quad's other lanes stored
  }
}
