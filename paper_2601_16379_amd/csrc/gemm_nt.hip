// FP64 complex "NT" GEMM on CDNA4 matrix cores for the large contractions of
// the path (V^q of eq. (7), U^q = R^q W^q and the fragment contraction of
// eq. (19), the factorisation updates and the two-sided solve of eq. (8)):
//
//   C[m][n] (+)= sum_{s < nseg} sum_{k} opA(A_s[m][k]) * opB(B_s[n][k])
//
// Both operands are complex128 interleaved, k-contiguous rows (no transposes
// anywhere); v_mfma_f64_16x16x4.  (The mixed formats have their own kernels in
// gemm_big.hip and gemm_x3.hip.)  K advances in stages of 16: MFMA step s
// of a stage takes k = 4 (l/16) + s from lane l, the same for A and B.
//
// Bound: the FP64 matrix cores (64 cycles a 16x16x4 MFMA), in practice the
// power they draw: with the cores busy 0.84 of the cycles the clock falls
// from 2.4 to 2.0-2.25 GHz.  A workgroup of 256 threads takes a 64 x 64 tile
// (four waves of 2 x 2 blocks of 16 x 16), two workgroups a CU.  A stage of
// both operands (2 x 16 KB) is copied from global memory straight into LDS
// (global_load_lds_dwordx4) one stage ahead, one barrier a stage; the
// fragments of MFMA step s + 1 are read from LDS under the MFMAs of step s.
// In LDS a row keeps its 16 values in an order XOR-permuted by the row, so the
// fragment reads (16 rows x 4 k) fall on distinct banks.  Measured on the
// tiles' own flops (random operands): 62.8 TFLOP/s for V^q products of 640 x
// 640 x 32768, 66.6 for 1024^3 products, 64.7 for U^q (3765 x 520 x 520),
// against 40, 49 and 49 with operands staged through registers, two barriers a
// stage; a vendor GEMM reaches 72-74.  A 128 x 128 tile of eight waves was
// 5 % faster on 1024^3 but loses more to the edges of 520 or 1040 rows.
//
// Tile size: products of few tiles take 32 x 32 tiles (one block of 16 x 16 a
// wave, four or five workgroups a CU) so that every CU has work; the MFMAs of
// an output element and their order are the same in both, so the results are
// too, bit for bit.  Tiles with at most 32 (16) valid rows or columns are
// dealt to the four waves as strips.
#include "kernels.hpp"

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;

constexpr int MT = 64;            // edge of the tiles that the tile list counts
constexpr int BK = 16;            // k per stage
constexpr int ROW_B = BK * 16;    // bytes of one row of one stage

__device__ inline int isqrt_floor(long long x) {
  long long r = (long long)sqrt((double)x);
  while (r * r > x) --r;
  while ((r + 1) * (r + 1) <= x) ++r;
  return (int)r;
}

// Values at or past the end of the K segment are copied from here.
__device__ __attribute__((aligned(16))) double kZeroC[2];

__device__ inline double flip(double x, unsigned long long sign) {
  return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, x) ^ sign);
}

// Position of a K stage: segment and first k of it.
struct KPos {
  int seg, k0;
};

// Sources of this lane's copies of one operand: a wave-instruction copies 4
// rows x 256 bytes; lane l copies value kk of row l/16 to position l%16.
template <int T>
struct Src {
  const cplx* p[T / 16];
  int kk[T / 16];
};

template <int T>
__device__ inline void make_src(Src<T>& s, const cplx* base, long long ld, int row0, int nrows, int wave, int lane) {
#pragma unroll
  for (int j = 0; j < T / 16; ++j) {
    const int row = (wave + 4 * j) * 4 + (lane >> 4);
    s.kk[j] = (lane & 15) ^ (row & 15);
    // rows past the end repeat the last one (their outputs are not stored)
    s.p[j] = base + (long long)min(row0 + row, nrows - 1) * ld + s.kk[j];
  }
}

template <int T>
__device__ inline void stage_copy(const Src<T>& s, long long off, int k0, int kcur, char* dst, int wave) {
  const bool tail = k0 + BK > kcur;      // the same for the whole workgroup
#pragma unroll
  for (int j = 0; j < T / 16; ++j) {
    const cplx* g = s.p[j] + off;
    if (tail && k0 + s.kk[j] >= kcur) g = (const cplx*)kZeroC;
    __builtin_amdgcn_global_load_lds((glb_void*)g, (lds_void*)(dst + (wave + 4 * j) * 4 * ROW_B), 16, 0, 0);
  }
}

// The K loop over segments [s0, s1) and the epilogue of one tile: this wave
// computes NI x NJ blocks of 16 x 16 at rows rb, columns cb of the T x T tile
// (idle: it only helps with the copies).  part: the block goes there (T x T,
// row-major) instead of into C; first: the first chunk of the K range.
template <int T, int NI, int NJ>
__device__ inline void tile_body(const NtDesc& d, const Src<T>& sa, const Src<T>& sb, int s0, int s1, int m0, int n0,
                                 int rb, int cb, bool idle, bool mirror, cplx* Cb, cplx* part, bool first,
                                 unsigned long long sx, unsigned long long sy, unsigned long long sz, char* smem,
                                 int wave, int lane) {
  constexpr int SA = T * ROW_B, STAGE = 2 * SA;
  const int lr = lane & 15, lk = lane >> 4;
  d4 re[NI][NJ], im[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      re[i][j] = d4{0, 0, 0, 0};
      im[i][j] = d4{0, 0, 0, 0};
    }
  const int sw = ((4 * lk) ^ lr) << 4;
  const int aoff = (rb + lr) * ROW_B + sw, boff = SA + (cb + lr) * ROW_B + sw;
  auto kcur_of = [&](int seg) { return seg == d.nseg - 1 ? d.Klast : d.Kseg; };
  auto copy = [&](const KPos& p, char* buf) {
    const int kcur = kcur_of(p.seg);
    stage_copy<T>(sa, (long long)p.seg * d.sA_seg + p.k0, p.k0, kcur, buf, wave);
    stage_copy<T>(sb, (long long)p.seg * d.sB_seg + p.k0, p.k0, kcur, buf + SA, wave);
  };
  auto rd = [&](const char* buf, int q, d2 (&a)[NI], d2 (&b)[NJ]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) a[i] = *(const d2*)(buf + ((aoff ^ (q << 4)) + i * 16 * ROW_B));
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[j] = *(const d2*)(buf + ((boff ^ (q << 4)) + j * 16 * ROW_B));
  };
  // re += a_r b_r - a_i b_i, im += a_r b_i + a_i b_r, the signs of the
  // conjugations on a copy of A's components
  auto mm = [&](const d2 (&a)[NI], const d2 (&b)[NJ]) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].x, re[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const double x = flip(a[i].x, sx);
#pragma unroll
      for (int j = 0; j < NJ; ++j) im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b[j].y, im[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const double x = flip(a[i].y, sy);
#pragma unroll
      for (int j = 0; j < NJ; ++j) re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b[j].y, re[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const double x = flip(a[i].y, sz);
#pragma unroll
      for (int j = 0; j < NJ; ++j) im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b[j].x, im[i][j], 0, 0, 0);
    }
  };
  // the stage after p (seg = s1: none)
  auto next = [&](KPos p) {
    p.k0 += BK;
    if (p.k0 >= kcur_of(p.seg)) {
      ++p.seg;
      p.k0 = 0;
    }
    return p;
  };
  KPos nx{s0, 0};                        // the stage to copy next
  __syncthreads();                       // LDS of the previous tile no longer read
  copy(nx, smem);
  nx = next(nx);
  int par = 0;
  for (bool more = true; more; par ^= 1) {
    const char* buf = smem + par * STAGE;
    // this stage's copies have landed; after the barrier everyone's have, and
    // every wave has read the previous stage, whose buffer takes the next
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    more = nx.seg < s1;
    d2 a0[NI], b0[NJ], a1[NI], b1[NJ];
    rd(buf, 0, a0, b0);
    if (more) {
      copy(nx, smem + (par ^ 1) * STAGE);
      nx = next(nx);
    }
    rd(buf, 1, a1, b1);
    if (!idle) {
      __builtin_amdgcn_sched_barrier(0);
      mm(a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      rd(buf, 2, a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      mm(a1, b1);
      __builtin_amdgcn_sched_barrier(0);
      rd(buf, 3, a1, b1);
      __builtin_amdgcn_sched_barrier(0);
      mm(a0, b0);
      mm(a1, b1);
    }
  }
  if (idle) return;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ml = rb + i * 16 + 4 * v + lk, nl = cb + j * 16 + lr;
        const int m = m0 + ml, n = n0 + nl;
        if (m >= d.M || n >= d.N) continue;
        cplx val = cmk(re[i][j][v], im[i][j][v]);
        if (part) {
          part[ml * T + nl] = val;
          continue;
        }
        const long long o = (long long)m * d.ldc + n;
        if (d.epi == 4) val = csub(Cb[o], val);
        else if (d.epi == 1 && !first) val = cadd(Cb[o], val);
        Cb[o] = val;
        if (mirror) Cb[(long long)n * d.ldc + m] = cconj(val);
      }
}

// KIND only names the call site in profiles (0 generic, 1 V^q, 2 U^q,
// 3 fragment contraction); the code is the same.  Units: the tiles
// [t0, t0 + nt) of the tile list (64 x 64 each; T = 32: four units a tile).
// With nch > 1 the K segments run in nch chunks of d.cseg segments, the
// chunks added one after the other: by the workgroup of the tile (C is
// stored by the first chunk, added to by the later ones), or, with part, by a
// unit of its own each, which leaves its partial block in part for
// nt_fold_kernel.
template <int T, int KIND>
__global__ __launch_bounds__(256, T == 64 ? 2 : 4) void zgemm_nt_kernel(const NtDesc* __restrict__ descs, int ndesc,
                                                                        long long t0, long long nt, int nch,
                                                                        cplx* part, int conj) {
  extern __shared__ __attribute__((aligned(16))) char smem[];   // two stages of (A, B)
  constexpr int SUB = (MT / T) * (MT / T);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr unsigned long long NEG = 0x8000000000000000ull;
  const bool ca = conj & 1, cb_ = (conj & 2) != 0;
  const unsigned long long sx = cb_ ? NEG : 0, sy = ca == cb_ ? NEG : 0, sz = ca ? NEG : 0;

  // XCD-aware order: workgroups are dispatched round-robin over the 8 XCDs,
  // so iteration `it` of workgroup b maps to a unit such that each XCD walks
  // a contiguous range of the units (tiles that share operand rows then
  // share that XCD's L2).  gridDim.x is a multiple of 8.
  const long long units = nt * SUB * (part ? nch : 1);
  const long long u8 = (units + 7) / 8 * 8;
  const long long per = u8 / 8;
  for (long long it = blockIdx.x; it < u8; it += gridDim.x) {
    const long long u = (it % 8) * per + it / 8;
    if (u >= units) continue;
    const int ch = part ? (int)(u / (nt * SUB)) : 0;
    const long long ut = u - (long long)ch * nt * SUB;
    const long long t = t0 + ut / SUB;
    const int sub = (int)(ut % SUB);
    int lo = 0, hi = ndesc - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (descs[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
    }
    const NtDesc d = descs[lo];
    const long long local = t - d.tile_begin;
    const int b = (int)(local / d.tiles_per_batch);
    const int lt = (int)(local - (long long)b * d.tiles_per_batch);
    int tm, tn;
    if (d.herm) {
      tm = (isqrt_floor(8LL * lt + 1) - 1) / 2;
      tn = lt - tm * (tm + 1) / 2;
    } else {
      tm = lt / d.tiles_n;
      tn = lt - tm * d.tiles_n;
    }
    const int m0 = tm * MT + (T == 32 ? 32 * (sub >> 1) : 0), n0 = tn * MT + (T == 32 ? 32 * (sub & 1) : 0);
    if (m0 >= d.M || n0 >= d.N) continue;            // a quarter outside the matrix
    // entries above the diagonal of a 64 x 64 diagonal tile: computed where
    // the matrix is wanted whole (herm 1: the other tiles are mirrored), left
    // out where the consumer reads the lower triangle only (herm 2)
    const bool diag2 = d.herm == 2 && tm == tn;
    if (T == 32 && diag2 && sub == 1) continue;
    const bool mirror = d.herm == 1 && tm != tn;
    const int rv = min(T, d.M - m0), cv = min(T, d.N - n0);
    Src<T> sa, sb;
    make_src<T>(sa, (const cplx*)d.A + (long long)b * d.sA_bat, d.lda, m0, d.M, wave, lane);
    make_src<T>(sb, (const cplx*)d.B + (long long)b * d.sB_bat, d.ldb, n0, d.N, wave, lane);
    cplx* Cb = (cplx*)d.C + (long long)b * d.sC_bat;
    cplx* pt = part ? part + (u * T) * T : nullptr;
    const int wm = wave >> 1, wn = wave & 1;
    for (int c = part ? ch : 0; c < (part ? ch + 1 : nch); ++c) {
      const int s0 = nch > 1 ? c * d.cseg : 0, s1 = nch > 1 ? min(d.nseg, s0 + d.cseg) : d.nseg;
      const bool first = c == 0;
#define NT_BODY(NI, NJ, RB, CB, IDLE) \
  tile_body<T, NI, NJ>(d, sa, sb, s0, s1, m0, n0, RB, CB, IDLE, mirror, Cb, pt, first, sx, sy, sz, smem, wave, lane)
      if constexpr (T == 32) {
        NT_BODY(1, 1, wm * 16, wn * 16, wm * 16 >= rv || wn * 16 >= cv || (diag2 && sub != 2 && wm < wn));
      } else {
        if (cv <= 16) NT_BODY(1, 1, wave * 16, 0, wave * 16 >= rv);
        else if (cv <= 32) NT_BODY(1, 2, wave * 16, 0, wave * 16 >= rv);
        else if (rv <= 16) NT_BODY(1, 1, 0, wave * 16, wave * 16 >= cv);
        else if (rv <= 32) NT_BODY(2, 1, 0, wave * 16, wave * 16 >= cv);
        else NT_BODY(2, 2, wm * 32, wn * 32, diag2 && wm < wn);
      }
#undef NT_BODY
    }
  }
}

template <int T>
hipError_t launch_kind(int kind, const NtDesc* descs, int ndesc, long long t0, long long nt, int nch, cplx* part,
                       int conj, int blocks, hipStream_t s) {
  dim3 g(blocks), b(256);
  const size_t lds = 4 * T * ROW_B;
  switch (kind) {
    case 1: hipLaunchKernelGGL((zgemm_nt_kernel<T, 1>), g, b, lds, s, descs, ndesc, t0, nt, nch, part, conj); break;
    case 2: hipLaunchKernelGGL((zgemm_nt_kernel<T, 2>), g, b, lds, s, descs, ndesc, t0, nt, nch, part, conj); break;
    case 3: hipLaunchKernelGGL((zgemm_nt_kernel<T, 3>), g, b, lds, s, descs, ndesc, t0, nt, nch, part, conj); break;
    default: hipLaunchKernelGGL((zgemm_nt_kernel<T, 0>), g, b, lds, s, descs, ndesc, t0, nt, nch, part, conj); break;
  }
  return hipGetLastError();
}

}  // namespace

long long nt_plan(NtDesc* d, int n) {
  long long acc = 0;
  for (int i = 0; i < n; ++i) {
    d[i].tiles_m = ceil_div(d[i].M, MT);
    d[i].tiles_n = ceil_div(d[i].N, MT);
    d[i].tiles_per_batch = d[i].herm ? d[i].tiles_m * (d[i].tiles_m + 1) / 2
                                     : d[i].tiles_m * d[i].tiles_n;
    if (d[i].Klast <= 0 || d[i].Klast > d[i].Kseg) d[i].Klast = d[i].Kseg;
    if (d[i].cseg <= 0) d[i].cseg = d[i].nseg;
    d[i].tile_begin = acc;
    acc += (long long)d[i].tiles_per_batch * d[i].batch;
  }
  return acc;
}

hipError_t nt_launch(int conj, const NtDesc* descs_dev, int ndesc, long long total, int max_blocks, hipStream_t s,
                     int kind) {
  if (total <= 0) return hipSuccess;
  max_blocks = max_blocks / 8 * 8;
  // 32 x 32 tiles where 64 x 64 would leave CUs idle or half filled: below
  // NT_SMALL_TILES tiles
  const bool small = total < NT_SMALL_TILES;
  const long long units = small ? 4 * total : total;
  const long long u8 = (units + 7) / 8 * 8;
  if (small) return launch_kind<32>(kind, descs_dev, ndesc, 0, total, 1, nullptr, conj, (int)(u8 < 2048 ? u8 : 2048), s);
  return launch_kind<64>(kind, descs_dev, ndesc, 0, total, 1, nullptr, conj, (int)(u8 < max_blocks ? u8 : max_blocks), s);
}
