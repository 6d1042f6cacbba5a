// Complex "NT" GEMM on CDNA4 matrix cores in FP64 (F = 0) and FP32 (F = 1) for
// the large contractions of the path (V^q of eq. (7), U^q = R^q W^q and the
// fragment contraction of eq. (19), the factorisation updates and the
// two-sided solve of eq. (8)):
//
//   C[m][n] (+)= sum_{s < nseg} sum_{k} opA(A_s[m][k]) * opB(B_s[n][k])
//
// Operands are k-contiguous rows (no transposes anywhere):
//   F = 0  complex128 interleaved; v_mfma_f64_16x16x4; stages of 16 k, MFMA
//          step s of a stage takes k = 4 (l/16) + s from lane l;
//   F = 1  two float planes (re, im), rows zero-padded to a multiple of 4;
//          v_mfma_f32_16x16x4; stages of 32 k, step s takes k = 8 (l/16) + s;
// the same k for A and B.  In both one row of one stage is 256 bytes.  (The
// bf16 formats have their own kernel in gemm_x3.hip.)
//
// Bound: the matrix cores; in FP64 (64 cycles a 16x16x4 MFMA) in practice the
// power they draw: with the cores busy 0.80 of the cycles the clock falls
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
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;

constexpr int MT = NT_TILE;       // edge of the tiles that the tile list counts
constexpr int ROW_B = 256;        // bytes of one row of one stage (16 slots of 16 bytes)

// BK: k per stage; EPS: elements per 16-byte slot; ESZ: bytes per element as
// addressed by the strides; NQ: fragment reads per stage
template <int F> struct Fm;
template <> struct Fm<0> {
  static constexpr int BK = 16, EPS = 1, ESZ = 16, NQ = 4;
  typedef d4 Acc;
  struct Frag { d2 v; };          // (re, im) of one k
};
template <> struct Fm<1> {
  static constexpr int BK = 32, EPS = 4, ESZ = 4, NQ = 2;
  typedef f4 Acc;
  struct Frag { f4 r, i; };       // four k
};

// Slots that start at or past the end of the K segment are copied from here.
__device__ __attribute__((aligned(16))) double kZeroC[2];

__device__ inline double flip(double x, bool neg) {
  return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, x) ^ (neg ? 0x8000000000000000ull : 0ull));
}
__device__ inline float flip(float x, bool neg) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned int, x) ^ (neg ? 0x80000000u : 0u));
}

// Position of a K stage: segment and first k of it.
struct KPos {
  int seg, k0;
};

// Sources of this lane's copies of one operand: a wave-instruction copies 4
// rows x 256 bytes; lane l copies the slot of its row whose LDS position is
// l%16; kk is the slot's first k.
template <int T>
struct Src {
  const char* p[T / 16];
  int kk[T / 16];
};

template <int F, int T>
__device__ inline void make_src(Src<T>& s, const char* base, long long ld, long long plane, int row0, int nrows,
                                int wave, int lane) {
#pragma unroll
  for (int j = 0; j < T / 16; ++j) {
    const int row = (wave + 4 * j) * 4 + (lane >> 4);
    const int slot = (lane & 15) ^ (row & 15);
    s.kk[j] = F == 0 ? slot : 4 * (slot & 7);
    // rows past the end repeat the last one (their outputs are not stored)
    s.p[j] = base + ((long long)min(row0 + row, nrows - 1) * ld + s.kk[j] + (F == 0 ? 0 : (slot >> 3) * plane)) *
                        Fm<F>::ESZ;
  }
}

template <int F, int T>
__device__ inline void stage_copy(const Src<T>& s, long long off, int k0, int kcur, char* dst, int wave) {
  const bool tail = k0 + Fm<F>::BK > kcur;      // the same for the whole workgroup
#pragma unroll
  for (int j = 0; j < T / 16; ++j) {
    const char* g = s.p[j] + off * Fm<F>::ESZ;
    if (tail && k0 + s.kk[j] >= kcur) g = (const char*)kZeroC;
    __builtin_amdgcn_global_load_lds((glb_void*)g, (lds_void*)(dst + (wave + 4 * j) * 4 * ROW_B), 16, 0, 0);
  }
}

// The K loop over segments [s0, s1) and the epilogue of one tile: this wave
// computes NI x NJ blocks of 16 x 16 at rows rb, columns cb of the T x T tile
// (idle: it only helps with the copies).  part: the block goes there (T x T,
// row-major) instead of into C; first: the first chunk of the K range.
template <int F, int T, int NI, int NJ>
__device__ inline void tile_body(const NtDesc& d, const Src<T>& sa, const Src<T>& sb, int s0, int s1, int kstart,
                                 int m0, int n0, int rb, int cb, bool idle, bool mirror, int b, cplx* part, bool first,
                                 bool nx_, bool ny, bool nz, char* smem, int wave, int lane) {
  constexpr int SA = T * ROW_B, STAGE = 2 * SA, BK = Fm<F>::BK;
  typedef typename Fm<F>::Acc Acc;
  typedef typename Fm<F>::Frag Frag;
  const int lr = lane & 15, lk = lane >> 4;
  Acc re[NI][NJ], im[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      re[i][j] = Acc{0, 0, 0, 0};
      im[i][j] = Acc{0, 0, 0, 0};
    }
  // slots of fragment read q: F = 0, 4 lk + q; F = 1, 2 lk + q (re) and 8 + 2 lk + q (im)
  const int sw = ((F == 0 ? 4 * lk : 2 * lk) ^ lr) << 4;
  const int aoff = (rb + lr) * ROW_B + sw, boff = SA + (cb + lr) * ROW_B + sw;
  // a triangular B (zero for k < n) contributes from kstart on
  auto kcur_of = [&](int seg) { return (seg == d.nseg - 1 ? d.Klast : d.Kseg) - kstart; };
  auto copy = [&](const KPos& p, char* buf) {
    const int kcur = kcur_of(p.seg);
    stage_copy<F, T>(sa, (long long)p.seg * d.sA_seg + p.k0, p.k0, kcur, buf, wave);
    stage_copy<F, T>(sb, (long long)p.seg * d.sB_seg + p.k0, p.k0, kcur, buf + SA, wave);
  };
  auto rd1 = [&](const char* p, Frag& f) {
    if constexpr (F == 0) f.v = *(const d2*)p;
    else f.r = *(const f4*)p;
  };
  auto rd = [&](const char* buf, int q, Frag (&a)[NI], Frag (&b_)[NJ]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) rd1(buf + ((aoff ^ (q << 4)) + i * 16 * ROW_B), a[i]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) rd1(buf + ((boff ^ (q << 4)) + j * 16 * ROW_B), b_[j]);
    if constexpr (F == 1) {
#pragma unroll
      for (int i = 0; i < NI; ++i) a[i].i = *(const f4*)(buf + ((aoff ^ ((8 + q) << 4)) + i * 16 * ROW_B));
#pragma unroll
      for (int j = 0; j < NJ; ++j) b_[j].i = *(const f4*)(buf + ((boff ^ ((8 + q) << 4)) + j * 16 * ROW_B));
    }
  };
  // re += a_r b_r - a_i b_i, im += a_r b_i + a_i b_r, the signs of the
  // conjugations on a copy of A's components
  auto mma = [](auto x, auto y, Acc c) {
    if constexpr (F == 0) return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);
  };
  auto mm1 = [&](auto ar, auto ai, auto br, auto bi) {   // component getters by block
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) re[i][j] = mma(ar(i), br(j), re[i][j]);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const auto x = flip(ar(i), nx_);
#pragma unroll
      for (int j = 0; j < NJ; ++j) im[i][j] = mma(x, bi(j), im[i][j]);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const auto x = flip(ai(i), ny);
#pragma unroll
      for (int j = 0; j < NJ; ++j) re[i][j] = mma(x, bi(j), re[i][j]);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const auto x = flip(ai(i), nz);
#pragma unroll
      for (int j = 0; j < NJ; ++j) im[i][j] = mma(x, br(j), im[i][j]);
    }
  };
  auto mm = [&](const Frag (&a)[NI], const Frag (&b_)[NJ]) {
    if constexpr (F == 0) {
      mm1([&](int i) { return a[i].v.x; }, [&](int i) { return a[i].v.y; }, [&](int j) { return b_[j].v.x; },
          [&](int j) { return b_[j].v.y; });
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        mm1([&](int i) { return a[i].r[t]; }, [&](int i) { return a[i].i[t]; }, [&](int j) { return b_[j].r[t]; },
            [&](int j) { return b_[j].i[t]; });
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
    Frag a0[NI], b0[NJ], a1[NI], b1[NJ];
    rd(buf, 0, a0, b0);
    if (more) {
      copy(nx, smem + (par ^ 1) * STAGE);
      nx = next(nx);
    }
    rd(buf, 1, a1, b1);
    if (!idle) {
      __builtin_amdgcn_sched_barrier(0);
      mm(a0, b0);
      if constexpr (Fm<F>::NQ == 4) {
        __builtin_amdgcn_sched_barrier(0);
        rd(buf, 2, a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        mm(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        rd(buf, 3, a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        mm(a0, b0);
      }
      mm(a1, b1);
    }
  }
  if (idle) return;
  // row and column of the first value; opaque, so that the addresses below are
  // formed here and not held in registers over the K loop
  int ml0 = rb + (F == 0 ? lk : 4 * lk), nl0 = cb + lr;
  asm volatile("" : "+v"(ml0), "+v"(nl0));
  constexpr int VS = F == 0 ? 4 : 1;     // rows between the values of a block
  if (part) {
    cplx* pp = part + ml0 * T + nl0;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) pp[(i * 16 + VS * v) * T + j * 16] = cmk(re[i][j][v], im[i][j][v]);
    return;
  }
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + ml0 + i * 16 + VS * v, n = n0 + nl0 + j * 16;
        if (m >= d.M) continue;
        if (F == 1 && d.epi == 3) {
          // operand format, zeros in the row padding
          if (n >= d.npad) continue;
          float* c = (float*)d.C + (long long)b * d.sC_bat + (long long)m * d.ldc + n;
          c[0] = n < d.N ? (float)re[i][j][v] : 0.f;
          c[d.c_plane] = n < d.N ? (float)im[i][j][v] : 0.f;
          continue;
        }
        if (n >= d.N) continue;
        cplx val = cmk(re[i][j][v], im[i][j][v]);
        cplx* Cb = (cplx*)d.C + (long long)b * d.sC_bat;
        const long long o = (long long)m * d.ldc + n;
        if (d.epi == 4) val = csub(Cb[o], val);
        else if (d.epi == 1) val = cadd(first ? cmk(0.0, 0.0) : Cb[o], val);
        Cb[o] = val;
        if (mirror) Cb[(long long)n * d.ldc + m] = cconj(val);
      }
}

// KIND only names the call site in profiles (0 generic, 1 V^q, 2 U^q,
// 3 fragment contraction); the code is the same.  Units: the tiles
// [t0, t0 + nt) of the tile list (64 x 64 each; T = 32: four units a tile),
// and the chunks [c0, c0 + nc) of the K segments (chunk c: the d.cseg
// segments from c d.cseg on).  The workgroup of a tile runs its chunks one
// after the other (epi 1: the first chunk of all stores C, the later ones add
// to it); with part every chunk is a unit of its own, which leaves its partial
// block in part for the fold (nt_fold_kernel).
template <int F, int T, int KIND>
__global__ __launch_bounds__(256, T == 64 ? 2 : 4) void zgemm_nt_kernel(const NtDesc* __restrict__ descs, int ndesc,
                                                                        long long t0, long long nt, int c0, int nc,
                                                                        cplx* part, int conj) {
  extern __shared__ __attribute__((aligned(16))) char smem[];   // two stages of (A, B)
  constexpr int SUB = (MT / T) * (MT / T);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool ca = conj & 1, cb_ = (conj & 2) != 0;

  // XCD-aware order: workgroups are dispatched round-robin over the 8 XCDs,
  // so iteration `it` of workgroup b maps to a unit such that each XCD walks
  // a contiguous range of the units (tiles that share operand rows then
  // share that XCD's L2).  gridDim.x is a multiple of 8.
  const long long units = nt * SUB * (part ? nc : 1);
  const long long u8 = (units + 7) / 8 * 8;
  const long long per = u8 / 8;
  for (long long it = blockIdx.x; it < u8; it += gridDim.x) {
    const long long u = (it % 8) * per + it / 8;
    if (u >= units) continue;
    const int pc = part ? (int)(u / (nt * SUB)) : 0;
    const long long ut = u - (long long)pc * nt * SUB;
    const NtTile tl = nt_tile(descs, ndesc, t0 + ut / SUB);
    const NtDesc d = descs[tl.desc];
    const int sub = (int)(ut % SUB), tm = tl.tm, tn = tl.tn, b = tl.b;
    const int m0 = tm * MT + (T == 32 ? 32 * (sub >> 1) : 0), n0 = tn * MT + (T == 32 ? 32 * (sub & 1) : 0);
    if (m0 >= d.M || n0 >= d.N) continue;            // a quarter outside the matrix
    // entries above the diagonal of a 64 x 64 diagonal tile: computed where
    // the matrix is wanted whole (herm 1: the other tiles are mirrored), left
    // out where the consumer reads the lower triangle only (herm 2)
    const bool diag2 = d.herm == 2 && tm == tn;
    if (T == 32 && diag2 && sub == 1) continue;
    const bool mirror = d.herm == 1 && tm != tn;
    const int rv = min(T, d.M - m0), cv = min(T, d.N - n0);
    const int kstart = d.ktri ? n0 : 0;
    Src<T> sa, sb;
    make_src<F, T>(sa, (const char*)d.A + ((long long)b * d.sA_bat + kstart) * Fm<F>::ESZ, d.lda, d.a_plane, m0, d.M,
                   wave, lane);
    make_src<F, T>(sb, (const char*)d.B + ((long long)b * d.sB_bat + kstart) * Fm<F>::ESZ, d.ldb, d.b_plane, n0, d.N,
                   wave, lane);
    cplx* pt = part ? part + (u * T) * T : nullptr;
    const int wm = wave >> 1, wn = wave & 1;
    for (int c = c0 + pc; c < (part ? c0 + pc + 1 : c0 + nc); ++c) {
      const int s0 = c * d.cseg, s1 = min(d.nseg, s0 + d.cseg);
#define NT_BODY(NI, NJ, RB, CB, IDLE)                                                                            \
  tile_body<F, T, NI, NJ>(d, sa, sb, s0, s1, kstart, m0, n0, RB, CB, IDLE, mirror, b, pt, c == 0, cb_, ca == cb_, \
                          ca, smem, wave, lane)
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

template <int F, int T>
hipError_t launch_kind(int kind, const NtDesc* descs, int ndesc, long long t0, long long nt, int c0, int nc,
                       cplx* part, int conj, int blocks, hipStream_t s) {
  dim3 g(blocks), b(256);
  const size_t lds = 4 * T * ROW_B;
#define NT_LAUNCH(K) \
  hipLaunchKernelGGL((zgemm_nt_kernel<F, T, K>), g, b, lds, s, descs, ndesc, t0, nt, c0, nc, part, conj)
  if (F == 1) {                          // FP32: the two fragment products only
    if (kind == 2) NT_LAUNCH(2);
    else if (kind == 3) NT_LAUNCH(3);
    else return hipErrorInvalidValue;
  } else {
    switch (kind) {
      case 1: NT_LAUNCH(1); break;
      case 2: NT_LAUNCH(2); break;
      case 3: NT_LAUNCH(3); break;
      default: NT_LAUNCH(0); break;
    }
  }
#undef NT_LAUNCH
  return hipGetLastError();
}

template <int F>
hipError_t launch_tiles(bool small, int kind, const NtDesc* descs, int ndesc, long long t0, long long nt, int c0,
                        int nc, cplx* part, int conj, int max_blocks, hipStream_t s) {
  if (nt <= 0) return hipSuccess;
  const long long units = (small ? 4 : 1) * nt * (part ? nc : 1);
  const long long u8 = (units + 7) / 8 * 8;
  const int cap = small ? 2048 : max_blocks / 8 * 8;
  const int blocks = (int)(u8 < cap ? u8 : cap);
  return small ? launch_kind<F, 32>(kind, descs, ndesc, t0, nt, c0, nc, part, conj, blocks, s)
               : launch_kind<F, 64>(kind, descs, ndesc, t0, nt, c0, nc, part, conj, blocks, s);
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
    if (d[i].npad <= 0) d[i].npad = (int)d[i].ldc;
    d[i].tile_begin = acc;
    acc += (long long)d[i].tiles_per_batch * d[i].batch;
  }
  return acc;
}

hipError_t nt_launch(int prec, int conj, const NtDesc* descs_dev, int ndesc, long long t0, long long nt, int c0,
                     int nc, cplx* part, int max_blocks, hipStream_t s, int kind) {
  if (nt <= 0 || nc <= 0) return hipSuccess;
  if (prec > 1) return hipErrorInvalidValue;
  // A whole number of rounds of two workgroups a CU runs as 64 x 64 tiles,
  // the rest as 32 x 32 ones when it would fill less than three quarters of
  // a round: a 64 x 64 tile of a nearly empty last round holds its CU for a
  // whole tile.  The same for launches of few tiles altogether.
  const long long round = 512, units = nt * (part ? nc : 1);
  long long big = 0;
  if (units >= NT_SMALL_TILES) {
    const long long rem = units % round;
    big = part || rem >= round * 3 / 4 ? nt : nt - rem;
  }
  hipError_t e = hipSuccess;
  auto go = [&](bool small, long long a, long long n) {
    return prec == 0 ? launch_tiles<0>(small, kind, descs_dev, ndesc, a, n, c0, nc, part, conj, max_blocks, s)
                     : launch_tiles<1>(small, kind, descs_dev, ndesc, a, n, c0, nc, part, conj, max_blocks, s);
  };
  e = go(false, t0, big);
  if (e == hipSuccess) e = go(true, t0 + big, nt - big);
  return e;
}

int nt_part_tile(long long nt, int nc) { return nt * nc >= NT_SMALL_TILES ? 64 : 32; }
