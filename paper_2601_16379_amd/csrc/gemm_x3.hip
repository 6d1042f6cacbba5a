// Complex "NT" GEMM on bf16 operands with the 32x32x16 bf16 matrix cores of
// gfx950, in two operand formats: F = 2, bf16 hi+lo (the bf16x3 precision),
// and F = 3, single bf16 (re, im) (the bf16 precision):
//
//   C[m][n] (+)= sum_k opA(A_seg[m][k]) opB(B_seg[n][k])
//
// F = 2: x = hi + lo per real component; every real product keeps hi*hi +
// hi*lo + lo*hi (three bf16 MFMAs, FP32 accumulation), and a complex product
// is four real ones, so one 32x32 complex block costs 12 MFMAs per 16 k.
// F = 3: one bf16 MFMA per real product, 8 MFMAs per 32 k.  In both formats
// one row of one stage is 128 contiguous bytes: 16 k x 4 planes (F = 2) or
// 32 k x 2 planes (F = 3), so the copies and the LDS layout are shared.
//
// Workgroup: 256 threads (4 waves, 2 x 2), 128 x 128 output tile, each wave
// 64 x 64 (2 x 2 blocks of 32 x 32); two workgroups per CU.  K advances in
// stages of 16 (one MFMA step).  In the operand format (bf16 hi/lo
// interleaved by 8-element groups) the 16 k of one row are 128 contiguous
// bytes, so a stage of a 128-row operand tile is 128 whole cache lines; it is
// copied from global memory straight into LDS (global_load_lds_dwordx4, no
// register staging) into one of two LDS stage buffers, one stage ahead of
// the one being multiplied.  Each stage: wait for its copies, one barrier
// (after it every wave has also read the previous stage, whose buffer then
// takes the copies of the next stage, issued first), read the fragments,
// MFMAs.  The stalls of one workgroup's waves are filled by the other
// workgroup's MFMAs.  (Two barriers a stage with the copies two stages
// ahead measured 8 % slower on the 1000-k contraction; so did issuing the
// fragment reads before the copies.)  A launch with fewer tiles than two
// rounds of workgroups leaves workgroups alone on their CUs; its
// contraction runs the two-barrier loop, which hides more latency
// (zgemm_c2b_kernel: 0.143 against 0.126 of peak at 216 k).  Both loops
// issue the same MFMAs in the same order: the results do not depend on the
// choice.  The single-bf16 contraction always runs the two-barrier loop.  U^q
// (but for bf16x3 rows far apart, run_u16) and products of few tiles have kernels
// of their own below.  In LDS a row keeps its eight 16-byte slots (2 k-groups x 4
// planes) in an order XOR-permuted by the row, so that the 32x32 fragment reads
// (lane -> row l%32, k-group l/32) hit distinct banks.
//
// Rows beyond M / N are loaded from the last valid row (their outputs are
// dropped); 16-byte vectors that start beyond the segment length are copied
// from a zero block.  Each lane's copy sources are computed once per tile.
// One K segment per launch, or with partial blocks several; epilogues: the
// operand format, FP64 accumulation across launches, or a partial block.
#include "kernels.hpp"

namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;

constexpr int XT = 128;               // tile edge
// k per stage, u16 per element in the global layout, and log2 of the
// planes per 8-element group, by format
template <int F> struct Fmt;
template <> struct Fmt<2> { static constexpr int K = 16, EU = 4, PL = 2; };
template <> struct Fmt<3> { static constexpr int K = 32, EU = 2, PL = 1; };
constexpr int NBUF = 2;               // LDS stages (two workgroups per CU)
constexpr int XNT = 256;              // threads
constexpr int ROW_B = 128;             // bytes of one row of one stage
constexpr int OPER_B = XT * ROW_B;     // one operand tile of a stage (16 KB)
constexpr int STAGE_B = 2 * OPER_B;    // A and B (32 KB)
constexpr int NCOPY = 4;               // copy instructions per wave per operand and stage

// LDS position of 16-byte slot `slot` (k-group * 4 + plane) of a row
__device__ inline int lds_slot(int row, int slot) { return slot ^ ((row ^ (row >> 3)) & 7); }

__device__ inline bf8 as_bf8(u4 v) { return __builtin_bit_cast(bf8, v); }

// wait until at most n stages of copies (2 * NCOPY instructions each) are in flight
__device__ inline void wait_copies(int n) {
  static_assert(2 * NCOPY == 8, "vmcnt below counts 8 copies a stage");
  if (n >= 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else if (n == 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The ring pipeline: one workgroup a CU, RING LDS stage buffers
constexpr int RING = 4;

// Vectors that start at or past the end of the K segment are copied from
// this zero block instead, so that LDS holds zeros there.
__device__ __attribute__((aligned(16))) unsigned short kZeroVec[8];

// Issue the copies of one operand's stage (128 or 64 rows x 128 bytes) into
// LDS at `dst`: wave-instructions of 8 rows, N (4 or 2) per wave.  src[j]: this lane's
// 16-byte source of the wave's j-th instruction at k = 0 (row base plus the
// slot gslot[j] whose LDS position is this lane's); the address advances by
// 4 u16 an element of k.  In the last stage of a segment, vectors that start
// at or past its end are copied from the zero block.
template <int F, int N>
__device__ inline void stage_copy(const unsigned short* const (&src)[N], const int (&gslot)[N], int k0,
                                  int kcur, char* dst, int wave) {
  const bool tail = k0 + Fmt<F>::K > kcur;    // the same for the whole workgroup
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const int rc = wave + 4 * j;          // rows rc*8 .. rc*8+7
    const unsigned short* g = src[j] + Fmt<F>::EU * k0;
    if (tail && k0 + 8 * (gslot[j] >> Fmt<F>::PL) >= kcur) g = kZeroVec;
    __builtin_amdgcn_global_load_lds((glb_void*)g, (lds_void*)(dst + rc * 8 * ROW_B), 16, 0, 0);
  }
}

// Fragments of one stage for this lane: NI 32-row blocks of A (rows rb0 +
// i * 32) and NJ 32-row blocks of B (rows cb0 + j * 32), four planes each
// (16 bytes = 8 k of the lane's k-group l/32).
template <int NI, int NJ>
struct Frag {
  u4 a[NI][4], b[NJ][4];
};

// The four 16-byte slots of a lane's row: F = 2, planes rh rl ih il of k-group
// lk; F = 3, (re, im) of k-group lk for the first MFMA step, then of k-group
// 2 + lk for the second.
template <int F>
__device__ inline int frag_slot(int lk, int x) {
  return F == 2 ? 4 * lk + x : 4 * (x >> 1) + 2 * lk + (x & 1);
}
template <int F, int NI, int NJ>
__device__ inline void read_frags_a(const char* buf, Frag<NI, NJ>& f, int rb0, int lr, int lk) {
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int row = rb0 + i * 32 + lr;
    const char* p = buf + row * ROW_B;
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) f.a[i][pl] = *(const u4*)(p + (lds_slot(row, frag_slot<F>(lk, pl)) << 4));
  }
}
template <int F, int OPB = OPER_B, int NI, int NJ>
__device__ inline void read_frags_b(const char* buf, Frag<NI, NJ>& f, int cb0, int lr, int lk) {
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int row = cb0 + j * 32 + lr;
    const char* p = buf + OPB + row * ROW_B;
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) f.b[j][pl] = *(const u4*)(p + (lds_slot(row, frag_slot<F>(lk, pl)) << 4));
  }
}

// Pin a stage's fragments: their reads have completed here, and later uses
// do not depend on the loads any more.
template <int NI, int NJ>
__device__ inline void settle(Frag<NI, NJ>& f) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int p = 0; p < 4; ++p) asm volatile("" : "+v"(f.a[i][p]));
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int p = 0; p < 4; ++p) asm volatile("" : "+v"(f.b[j][p]));
}

__device__ inline u4 neg_bf(u4 v) {
  return u4{v.x ^ 0x80008000u, v.y ^ 0x80008000u, v.z ^ 0x80008000u, v.w ^ 0x80008000u};
}

// The 12 MFMAs of one 32x32 block pair (i, j) and one 16-k step, as six
// (re, im) term pairs: re += a_r b_r - a_i b_i, im += a_r b_i + a_i b_r,
// each real product as hi*hi + hi*lo + lo*hi; conjugation flips the sign of
// the imaginary planes of that operand.
struct BFr {
  bf8 rh, rl, ih, il, nih, nil;
};
template <bool CONJ>
__device__ inline BFr split_a(const u4 (&a)[4]) {
  const u4 ih = CONJ ? neg_bf(a[2]) : a[2];
  const u4 il = CONJ ? neg_bf(a[3]) : a[3];
  return BFr{as_bf8(a[0]), as_bf8(a[1]), as_bf8(ih), as_bf8(il), as_bf8(neg_bf(ih)), as_bf8(neg_bf(il))};
}
#define X3_TERMS(A, BRH, BRL, BIH, BIL, CR, CI, T)                          \
  if ((T) == 0) { CR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.rl, BRH, CR, 0, 0, 0);  \
                  CI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.rl, BIH, CI, 0, 0, 0); }\
  if ((T) == 1) { CR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.rh, BRL, CR, 0, 0, 0);  \
                  CI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.rh, BIL, CI, 0, 0, 0); }\
  if ((T) == 2) { CR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.nil, BIH, CR, 0, 0, 0); \
                  CI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.il, BRH, CI, 0, 0, 0); }\
  if ((T) == 3) { CR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.nih, BIL, CR, 0, 0, 0); \
                  CI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.ih, BRL, CI, 0, 0, 0); }\
  if ((T) == 4) { CR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.rh, BRH, CR, 0, 0, 0);  \
                  CI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.rh, BIH, CI, 0, 0, 0); }\
  if ((T) == 5) { CR = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.nih, BIH, CR, 0, 0, 0); \
                  CI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.ih, BRH, CI, 0, 0, 0); }

// MFMAs of one stage for the wave's column block j; with two row blocks
// their four accumulator chains are interleaved (a chain every fourth MFMA).
template <int NI, int NJ, bool A_CONJ, bool B_CONJ>
__device__ inline void mma_half(const Frag<NI, NJ>& f, int j, f16v (&c_re)[NI][NJ], f16v (&c_im)[NI][NJ]) {
  const u4 bi = B_CONJ ? neg_bf(f.b[j][2]) : f.b[j][2];
  const u4 bl = B_CONJ ? neg_bf(f.b[j][3]) : f.b[j][3];
  const bf8 brh = as_bf8(f.b[j][0]), brl = as_bf8(f.b[j][1]), bih = as_bf8(bi), bil = as_bf8(bl);
  if constexpr (NI == 2) {
    const BFr x0 = split_a<A_CONJ>(f.a[0]), x1 = split_a<A_CONJ>(f.a[1]);
    f16v cr0 = c_re[0][j], ci0 = c_im[0][j], cr1 = c_re[1][j], ci1 = c_im[1][j];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      X3_TERMS(x0, brh, brl, bih, bil, cr0, ci0, t)
      X3_TERMS(x1, brh, brl, bih, bil, cr1, ci1, t)
    }
    c_re[0][j] = cr0;
    c_im[0][j] = ci0;
    c_re[1][j] = cr1;
    c_im[1][j] = ci1;
  } else {
    const BFr x0 = split_a<A_CONJ>(f.a[0]);
    f16v cr0 = c_re[0][j], ci0 = c_im[0][j];
#pragma unroll
    for (int t = 0; t < 6; ++t) { X3_TERMS(x0, brh, brl, bih, bil, cr0, ci0, t) }
    c_re[0][j] = cr0;
    c_im[0][j] = ci0;
  }
}
#undef X3_TERMS

// The 8 MFMAs of one stage of the single-bf16 format for the wave's column
// block j: two k steps (fragment slots 0, 1 and 2, 3 hold re, im), each
// re += a_r b_r - a_i b_i, im += a_r b_i + a_i b_r.
// The accumulator chains (re and im of each row block) are issued round
// robin, so that dependent MFMAs are 2 NI apart.
template <int NI, int NJ, bool A_CONJ, bool B_CONJ>
__device__ inline void mma_single(const Frag<NI, NJ>& f, int j, f16v (&c_re)[NI][NJ], f16v (&c_im)[NI][NJ]) {
  f16v cr[NI], ci[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    cr[i] = c_re[i][j];
    ci[i] = c_im[i][j];
  }
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    const u4 bi = B_CONJ ? neg_bf(f.b[j][2 * st + 1]) : f.b[j][2 * st + 1];
    const bf8 br = as_bf8(f.b[j][2 * st]), bim = as_bf8(bi);
    bf8 ar[NI], aim[NI], naim[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const u4 ai = A_CONJ ? neg_bf(f.a[i][2 * st + 1]) : f.a[i][2 * st + 1];
      ar[i] = as_bf8(f.a[i][2 * st]);
      aim[i] = as_bf8(ai);
      naim[i] = as_bf8(neg_bf(ai));
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) cr[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar[i], br, cr[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) ci[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar[i], bim, ci[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) cr[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(naim[i], bim, cr[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) ci[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aim[i], br, ci[i], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    c_re[i][j] = cr[i];
    c_im[i][j] = ci[i];
  }
}

// Epilogue of one tile (32x32 layout: lane l, register v -> row
// 8(v/4) + 4(l/32) + v%4, column l%32).  epi 3: each wave assembles its
// block 32 rows at a time in LDS (16 KB a wave) in the operand format (a row
// of NJ*32 points is NJ*256 contiguous bytes) and writes it with 16-byte
// stores; otherwise FP64 accumulation across launches (the first K segment,
// `first`, stores).  One branch for all kernels: compiled for one use each, the
// contraction took 2.5 % longer and the two-workgroup U^q 4 % (10^3 mesh, N_IP
// 1040, 259.7 against 253.5 ms and 89.5 against 85.8).
template <int F, int NI, int NJ, int T = XT>
__device__ inline void tile_epilogue(const NtDesc& d, int b, int m0, int n0, int rb0, int cb0,
                                     const f16v (&c_re)[NI][NJ], const f16v (&c_im)[NI][NJ], char* smem, int wave,
                                     int lane, bool first, cplx* part) {
  const int lr = lane & 31, lk = lane >> 5;
  if (d.epi == 3) {
    __syncthreads();                      // every wave is past its last stage reads
    unsigned short* st = (unsigned short*)(smem + wave * 16384);
    const int npad = d.npad ? d.npad : (int)d.ldc;
    constexpr int EU = Fmt<F>::EU;
    constexpr int RU = NJ * 32 * EU;      // u16 per staged row
    constexpr int PPR = NJ * 4 * EU;      // 16-byte parts per row
    unsigned short* C = (unsigned short*)d.C + EU * ((long long)b * d.sC_bat + n0 + cb0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int ml = 8 * (v >> 2) + 4 * lk + (v & 3);
          const int nl = j * 32 + lr;
          const bool in = n0 + cb0 + nl < d.N;
          const float re = in ? c_re[i][j][v] : 0.f, im = in ? c_im[i][j][v] : 0.f;
          const unsigned short rh = bf16_bits_of(re), ih = bf16_bits_of(im);
          unsigned short* e = st + ml * RU + (nl >> 3) * (8 * EU) + (nl & 7);
          if constexpr (F == 2) {
            e[0] = rh;
            e[8] = bf16_bits_of(re - bf16_value(rh));
            e[16] = ih;
            e[24] = bf16_bits_of(im - bf16_value(ih));
          } else {
            e[0] = rh;
            e[8] = ih;
          }
        }
      __builtin_amdgcn_wave_barrier();
      // 32 staged rows of PPR parts, 64 lanes a pass
#pragma unroll 4
      for (int h = 0; h < PPR / 2; ++h) {
        const int c = h * 64 + lane, ml = c / PPR, part = c % PPR;
        const int m = m0 + rb0 + i * 32 + ml;
        if (m < d.M && n0 + cb0 + (part >> Fmt<F>::PL) * 8 < npad)
          *(u4*)(C + EU * (long long)m * d.ldc + part * 8) = *(const u4*)(st + ml * RU + part * 8);
      }
      __builtin_amdgcn_wave_barrier();
    }
  } else if (part) {
    // partial block of the tile, row-major; the offset is opaque so that the
    // addresses are formed here and not held over the K loop
    int o0 = (rb0 + 4 * lk) * T + cb0 + lr;
    asm volatile("" : "+v"(o0));
    cplx* pp = part + o0;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          pp[(i * 32 + 8 * (v >> 2) + (v & 3)) * T + j * 32] =
              cmk((double)c_re[i][j][v], (double)c_im[i][j][v]);
  } else {
    int mr = m0 + rb0 + 4 * lk;
    asm volatile("" : "+v"(mr));
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = mr + i * 32 + 8 * (v >> 2) + (v & 3);
          const int n = n0 + cb0 + j * 32 + lr;
          if (m >= d.M || n >= d.N) continue;
          cplx* cp = (cplx*)d.C + (long long)b * d.sC_bat + (long long)m * d.ldc + n;
          cplx x = first ? cmk(0.0, 0.0) : *cp;   // FP64 accumulation across launches
          x.x += (double)c_re[i][j][v];
          x.y += (double)c_im[i][j][v];
          *cp = x;
        }
  }
}

// The MFMAs of one stage of fragments (both column blocks).
template <int F, int NI, int NJ, bool A_CONJ, bool B_CONJ>
__device__ inline void stage_mma(const Frag<NI, NJ>& f, f16v (&c_re)[NI][NJ], f16v (&c_im)[NI][NJ]) {
  if constexpr (F == 2) {
    mma_half<NI, NJ, A_CONJ, B_CONJ>(f, 0, c_re, c_im);
    if (NJ == 2) mma_half<NI, NJ, A_CONJ, B_CONJ>(f, NJ - 1, c_re, c_im);
  } else {
    mma_single<NI, NJ, A_CONJ, B_CONJ>(f, 0, c_re, c_im);
    if (NJ == 2) mma_single<NI, NJ, A_CONJ, B_CONJ>(f, NJ - 1, c_re, c_im);
  }
}

// The same with a triangular B (U^q in the factor form, kind 2): a column
// block whose B rows are all zero over the stage's k range (live0 / live1
// false) is skipped; it would add exact zeros.
template <int F, int NI, int NJ, bool A_CONJ, bool B_CONJ>
__device__ inline void stage_mma_tri(const Frag<NI, NJ>& f, f16v (&c_re)[NI][NJ], f16v (&c_im)[NI][NJ],
                                     bool live0, bool live1) {
  if constexpr (F == 2) {
    if (live0) mma_half<NI, NJ, A_CONJ, B_CONJ>(f, 0, c_re, c_im);
    if (NJ == 2 && live1) mma_half<NI, NJ, A_CONJ, B_CONJ>(f, NJ - 1, c_re, c_im);
  } else {
    if (live0) mma_single<NI, NJ, A_CONJ, B_CONJ>(f, 0, c_re, c_im);
    if (NJ == 2 && live1) mma_single<NI, NJ, A_CONJ, B_CONJ>(f, NJ - 1, c_re, c_im);
  }
}

// With a triangular B (B[n][k] = 0 for k < n; the K range starts at the
// tile's first column), column block j of the wave (columns cb0 + 32 j on)
// has only zeros in B over stage s when (s + 1) SK <= cb0 + 32 j.
__device__ inline void tri_live(bool tri, int s, int sk, int cb0, bool& l0, bool& l1) {
  l0 = !tri || (s + 1) * sk > cb0;
  l1 = !tri || (s + 1) * sk > cb0 + 32;
}

// K loop and epilogue of one tile.  The wave owns the (NI*32) x (NJ*32)
// block at rows rb0, columns cb0 of the tile: 64 x 64 in full tiles (2 x 2
// waves); in tiles with at most 32 valid rows (columns) each wave takes a
// 32 x 32 block of the one 32-row (32-column) strip, so edge tiles cost a
// quarter of the matrix-core work.  Two workgroups share a CU (64 KB of LDS
// each): two LDS stages, each stage's fragments read from LDS at its start
// (the waves of the other workgroup keep the matrix cores busy meanwhile),
// copies one stage ahead, one barrier a stage.
template <int F, int NI, int NJ, bool A_CONJ, bool B_CONJ, int KIND>
__device__ inline void tile_body(const NtDesc& d, int b, int m0, int n0, int kcur,
                                 const unsigned short* const (&asrc)[NCOPY], const unsigned short* const (&bsrc)[NCOPY],
                                 const int (&gslot)[NCOPY], int rb0, int cb0, char* smem, int wave, int lane,
                                 bool idle, bool first, cplx* part) {
  const int lr = lane & 31, lk = lane >> 5;
  f16v c_re[NI][NJ], c_im[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        c_re[i][j][v] = 0.f;
        c_im[i][j][v] = 0.f;
      }
  constexpr int SK = Fmt<F>::K;
  const int nst = (kcur + SK - 1) / SK;
  __syncthreads();                        // LDS of the previous tile no longer read
  stage_copy<F>(asrc, gslot, 0, kcur, smem, wave);
  stage_copy<F>(bsrc, gslot, 0, kcur, smem + OPER_B, wave);
  for (int s = 0; s < nst; ++s) {
    char* buf = smem + (s & 1) * STAGE_B;
    // stage s landed (nothing else in flight); after the barrier every wave
    // has read stage s - 1, so its buffer takes stage s + 1
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + 1 < nst) {
      char* nb = smem + ((s + 1) & 1) * STAGE_B;
      stage_copy<F>(asrc, gslot, (s + 1) * SK, kcur, nb, wave);
      stage_copy<F>(bsrc, gslot, (s + 1) * SK, kcur, nb + OPER_B, wave);
    }
    Frag<NI, NJ> f;
    read_frags_a<F>(buf, f, rb0, lr, lk);
    read_frags_b<F>(buf, f, cb0, lr, lk);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    settle(f);
    if constexpr (KIND == 2) {
      bool l0, l1;
      tri_live(d.ktri != 0, s, SK, cb0, l0, l1);
      stage_mma_tri<F, NI, NJ, A_CONJ, B_CONJ>(f, c_re, c_im, l0, l1);
    } else {
      if (!idle) stage_mma<F, NI, NJ, A_CONJ, B_CONJ>(f, c_re, c_im);
    }
  }
  if (!idle) tile_epilogue<F, NI, NJ>(d, b, m0, n0, rb0, cb0, c_re, c_im, smem, wave, lane, first, part);
}

// One step of the ring pipeline: the MFMAs of stage s (fragments in `cur`)
// while the fragments of stage s + 1 are read from LDS into `nxt`.  Before
// them: stage s + 1 has landed (this wave's copies, then the barrier for
// everyone's), and every wave has read stage s, so its buffer takes the
// copies of stage s + RING.  One barrier a stage; the copies run up to
// RING - 1 stages ahead of the MFMAs.
template <int F, int NI, int NJ, bool A_CONJ, bool B_CONJ>
__device__ inline void ring_step(int s, int nst, int kcur, Frag<NI, NJ>& cur, Frag<NI, NJ>& nxt,
                                 f16v (&c_re)[NI][NJ], f16v (&c_im)[NI][NJ],
                                 const unsigned short* const (&asrc)[NCOPY],
                                 const unsigned short* const (&bsrc)[NCOPY], const int (&gslot)[NCOPY],
                                 int rb0, int cb0, char* smem, int wave, int lr, int lk, bool idle) {
  constexpr int SK = Fmt<F>::K;
  const bool more = s + 1 < nst;
  if (more) {
    // copies issued so far: stages up to min(nst, s + RING) - 1
    const int last = (nst < s + RING ? nst : s + RING) - 1;
    wait_copies(last - (s + 1));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + RING < nst) {
      char* buf = smem + (s % RING) * STAGE_B;
      stage_copy<F>(asrc, gslot, (s + RING) * SK, kcur, buf, wave);
      stage_copy<F>(bsrc, gslot, (s + RING) * SK, kcur, buf + OPER_B, wave);
    }
    const char* nb = smem + ((s + 1) % RING) * STAGE_B;
    read_frags_a<F>(nb, nxt, rb0, lr, lk);
    read_frags_b<F>(nb, nxt, cb0, lr, lk);
  }
  if (!idle) stage_mma<F, NI, NJ, A_CONJ, B_CONJ>(cur, c_re, c_im);
  if (more) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    settle(nxt);
  }
}

// K loop and epilogue of one tile on the ring pipeline (same blocks, MFMA
// order and epilogues as tile_body, so the same results bit for bit).
template <int F, int NI, int NJ, bool A_CONJ, bool B_CONJ>
__device__ inline void tile_body_ring(const NtDesc& d, int b, int m0, int n0, int kcur,
                                      const unsigned short* const (&asrc)[NCOPY],
                                      const unsigned short* const (&bsrc)[NCOPY], const int (&gslot)[NCOPY],
                                      int rb0, int cb0, char* smem, int wave, int lane, bool idle, bool first, cplx* part) {
  const int lr = lane & 31, lk = lane >> 5;
  f16v c_re[NI][NJ], c_im[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        c_re[i][j][v] = 0.f;
        c_im[i][j][v] = 0.f;
      }
  constexpr int SK = Fmt<F>::K;
  const int nst = (kcur + SK - 1) / SK;
  __syncthreads();                        // LDS of the previous tile no longer read
#pragma unroll
  for (int s = 0; s < RING; ++s)
    if (s < nst) {
      stage_copy<F>(asrc, gslot, s * SK, kcur, smem + s * STAGE_B, wave);
      stage_copy<F>(bsrc, gslot, s * SK, kcur, smem + s * STAGE_B + OPER_B, wave);
    }
  // stage 0 landed: the later stages of the prologue may be in flight
  wait_copies((nst < RING ? nst : RING) - 1);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  Frag<NI, NJ> f0, f1;
  read_frags_a<F>(smem, f0, rb0, lr, lk);
  read_frags_b<F>(smem, f0, cb0, lr, lk);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  settle(f0);
  for (int s = 0; s < nst; s += 2) {
    ring_step<F, NI, NJ, A_CONJ, B_CONJ>(s, nst, kcur, f0, f1, c_re, c_im, asrc, bsrc, gslot, rb0,
                                              cb0, smem, wave, lr, lk, idle);
    if (s + 1 < nst)
      ring_step<F, NI, NJ, A_CONJ, B_CONJ>(s + 1, nst, kcur, f1, f0, c_re, c_im, asrc, bsrc, gslot,
                                                rb0, cb0, smem, wave, lr, lk, idle);
  }
  if (!idle) tile_epilogue<F, NI, NJ>(d, b, m0, n0, rb0, cb0, c_re, c_im, smem, wave, lane, first, part);
}

// The same K loop with two barriers a stage and the copies two stages
// ahead (a buffer is refilled only after every wave has read the stage it
// holds): more tolerant of a workgroup that has its CU to itself, the case
// of launches with fewer tiles than two rounds of workgroups.
template <int F, int NI, int NJ, bool A_CONJ, bool B_CONJ>
__device__ inline void tile_body_2b(const NtDesc& d, int b, int m0, int n0, int kcur,
                                 const unsigned short* const (&asrc)[NCOPY], const unsigned short* const (&bsrc)[NCOPY],
                                 const int (&gslot)[NCOPY], int rb0, int cb0, char* smem, int wave, int lane,
                                 bool idle, bool first, cplx* part) {
  const int lr = lane & 31, lk = lane >> 5;
  f16v c_re[NI][NJ], c_im[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        c_re[i][j][v] = 0.f;
        c_im[i][j][v] = 0.f;
      }
  constexpr int SK = Fmt<F>::K;
  const int nst = (kcur + SK - 1) / SK;
  __syncthreads();                        // LDS of the previous tile no longer read
#pragma unroll
  for (int s = 0; s < NBUF; ++s)
    if (s < nst) {
      stage_copy<F>(asrc, gslot, s * SK, kcur, smem + s * STAGE_B, wave);
      stage_copy<F>(bsrc, gslot, s * SK, kcur, smem + s * STAGE_B + OPER_B, wave);
    }
  for (int s = 0; s < nst; ++s) {
    char* buf = smem + (s & 1) * STAGE_B;
    // stage s landed: at most the copies of stage s+1 still in flight
    wait_copies(s + 1 < nst ? 1 : 0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    Frag<NI, NJ> f;
    read_frags_a<F>(buf, f, rb0, lr, lk);
    read_frags_b<F>(buf, f, cb0, lr, lk);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    settle(f);
    // every wave holds its fragments of stage s: its buffer takes stage s+2
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + NBUF < nst) {
      stage_copy<F>(asrc, gslot, (s + NBUF) * SK, kcur, buf, wave);
      stage_copy<F>(bsrc, gslot, (s + NBUF) * SK, kcur, buf + OPER_B, wave);
    }
    if (!idle) stage_mma<F, NI, NJ, A_CONJ, B_CONJ>(f, c_re, c_im);
  }
  if (!idle) tile_epilogue<F, NI, NJ>(d, b, m0, n0, rb0, cb0, c_re, c_im, smem, wave, lane, first, part);
}

// Small tiles: 64 x 64, a 32 x 32 block a wave, SRING stages of 16 KB.
constexpr int SOPER_B = X3_SMALL * ROW_B;
constexpr int SSTAGE_B = 2 * SOPER_B;
constexpr int SCOPY = X3_SMALL / 32;
constexpr int SRING = 8;

// One stage of a small tile: as ring_step, without conditions.  Copies past the
// last stage repeat it into buffers no longer read (so the count in flight stays
// the same), and the fragments read after the last stage are not used.
template <int F, bool A_CONJ, bool B_CONJ>
__device__ inline void small_step(int s, int nst, int kcur, bool live, Frag<1, 1>& cur, Frag<1, 1>& nxt,
                                  f16v (&c_re)[1][1], f16v (&c_im)[1][1], const unsigned short* const (&asrc)[SCOPY],
                                  const unsigned short* const (&bsrc)[SCOPY], const int (&gslot)[SCOPY], int rb0,
                                  int cb0, char* smem, int wave, int lr, int lk) {
  static_assert(2 * SCOPY * (SRING - 2) == 24, "the count below");
  // stage s + 1 has landed, and this wave holds its fragments of stage s
  asm volatile("s_waitcnt vmcnt(24) lgkmcnt(0)" ::: "memory");
  settle(cur);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  const int k0 = min(s + SRING, nst - 1) * Fmt<F>::K;
  char* buf = smem + (s % SRING) * SSTAGE_B;
  const char* nb = smem + ((s + 1) % SRING) * SSTAGE_B;
  read_frags_a<F>(nb, nxt, rb0, lr, lk);
  read_frags_b<F, SOPER_B>(nb, nxt, cb0, lr, lk);
  __builtin_amdgcn_sched_barrier(0);
  if (k0 + Fmt<F>::K <= kcur) {
#pragma unroll
    for (int j = 0; j < SCOPY; ++j) {
      char* dst = buf + (wave + 4 * j) * 8 * ROW_B;
      __builtin_amdgcn_global_load_lds((glb_void*)(asrc[j] + Fmt<F>::EU * k0), (lds_void*)dst, 16, 0, 0);
      __builtin_amdgcn_global_load_lds((glb_void*)(bsrc[j] + Fmt<F>::EU * k0), (lds_void*)(dst + SOPER_B), 16, 0, 0);
    }
  } else {
    stage_copy<F>(asrc, gslot, k0, kcur, buf, wave);
    stage_copy<F>(bsrc, gslot, k0, kcur, buf + SOPER_B, wave);
  }
  if (live) stage_mma<F, 1, 1, A_CONJ, B_CONJ>(cur, c_re, c_im);
  __builtin_amdgcn_sched_barrier(0);
}

template <int F, bool A_CONJ, bool B_CONJ, bool TRI>
__device__ inline void tile_body_small(const NtDesc& d, int b, int m0, int n0, int kcur,
                                       const unsigned short* const (&asrc)[SCOPY],
                                       const unsigned short* const (&bsrc)[SCOPY], const int (&gslot)[SCOPY], int rb0,
                                       int cb0, char* smem, int wave, int lane, bool idle, bool first, cplx* part) {
  const int lr = lane & 31, lk = lane >> 5;
  f16v c_re[1][1], c_im[1][1];
#pragma unroll
  for (int v = 0; v < 16; ++v) c_re[0][0][v] = c_im[0][0][v] = 0.f;
  constexpr int SK = Fmt<F>::K;
  const int nst = (kcur + SK - 1) / SK;
  // with a triangular B, the first stage whose B rows are not all zero (tri_live)
  const int s0 = TRI && d.ktri ? cb0 / SK : 0;
  __syncthreads();                        // LDS of the previous tile no longer read
#pragma unroll
  for (int s = 0; s < SRING; ++s) {
    const int k0 = min(s, nst - 1) * SK;
    stage_copy<F>(asrc, gslot, k0, kcur, smem + s * SSTAGE_B, wave);
    stage_copy<F>(bsrc, gslot, k0, kcur, smem + s * SSTAGE_B + SOPER_B, wave);
  }
  static_assert(2 * SCOPY * (SRING - 1) == 28, "the count below");
  asm volatile("s_waitcnt vmcnt(28)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  Frag<1, 1> f0, f1;
  read_frags_a<F>(smem, f0, rb0, lr, lk);
  read_frags_b<F, SOPER_B>(smem, f0, cb0, lr, lk);
  const int even = nst & ~1;              // one exit: the accumulators stay where they are
  for (int s = 0; s < even; s += 2) {
    small_step<F, A_CONJ, B_CONJ>(s, nst, kcur, !TRI || s >= s0, f0, f1, c_re, c_im, asrc, bsrc, gslot, rb0, cb0, smem,
                                  wave, lr, lk);
    small_step<F, A_CONJ, B_CONJ>(s + 1, nst, kcur, !TRI || s + 1 >= s0, f1, f0, c_re, c_im, asrc, bsrc, gslot, rb0, cb0,
                                  smem, wave, lr, lk);
  }
  if (even < nst)
    small_step<F, A_CONJ, B_CONJ>(even, nst, kcur, true, f0, f1, c_re, c_im, asrc, bsrc, gslot, rb0, cb0, smem, wave, lr,
                                  lk);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // before LDS is used for anything else
  if (!idle) tile_epilogue<F, 1, 1, X3_SMALL>(d, b, m0, n0, rb0, cb0, c_re, c_im, smem, wave, lane, first, part);
}

// ---- U^q = R^q W^q on 128 x 128 tiles as one stream of stages ----
// One workgroup a CU; the stages of its tiles follow one another in UR LDS
// buffers, copied up to UR - 1 ahead across the tile boundaries, and a tile's
// outputs go to the operand format straight from the accumulators (quad_store),
// past the LDS.  The MFMAs and their order are those of tile_body.
constexpr int UR = 4;

// The copy side: the tile being copied and its next stage.
template <int F>
struct UFlow {
  const unsigned short *a[NCOPY], *b[NCOPY];
  int gslot[NCOPY];
  int kcur, k0;                           // of the tile
  int it;                                 // its place in the workgroup's sequence
  int gi;                                 // stages copied in all
  bool more;
};

struct UTile {
  int b, m0, n0;
};
__device__ inline int u_unit(int it, int nt) { return (it & 7) * ((nt + 7) >> 3) + (it >> 3); }   // XCD-contiguous
__device__ inline bool u_valid(int it, int nt) { return it < ((nt + 7) & ~7) && u_unit(it, nt) < nt; }
// (the quotients are formed in vector registers and read back: everything that
// steers the stream stays scalar)
__device__ inline int u_div(int x, int y) { return __builtin_amdgcn_readfirstlane((unsigned)x / (unsigned)y); }
__device__ inline UTile u_tile(const NtDesc& d, int nt, int it) {
  const int u = u_unit(it, nt), b = u_div(u, d.tiles_per_batch), lt = u - b * d.tiles_per_batch;
  const int tm = u_div(lt, d.tiles_n);
  int tn = lt - tm * d.tiles_n;
  if (d.rot) {
    tn += u_div(b * d.tiles_m + tm, d.rot);
    tn -= u_div(tn, d.tiles_n) * d.tiles_n;
  }
  return UTile{b, tm * XT, tn * XT};
}

template <int F>
__device__ inline void u_start(UFlow<F>& f, const NtDesc& d, int nt, int wave, int lane) {
  constexpr int EU = Fmt<F>::EU;
  const UTile t = u_tile(d, nt, f.it);
  const int kstart = d.ktri ? t.n0 : 0;   // a triangular B contributes from k = n0 on
  const unsigned short* As = (const unsigned short*)d.A + EU * (t.b * d.sA_bat + kstart);
  const unsigned short* Bs = (const unsigned short*)d.B + EU * (t.b * d.sB_bat + kstart);
#pragma unroll
  for (int j = 0; j < NCOPY; ++j) {
    const int row = (wave + 4 * j) * 8 + (lane >> 3);
    f.a[j] = As + EU * ((long long)min(t.m0 + row, d.M - 1) * d.lda) + 8 * f.gslot[j];
    f.b[j] = Bs + EU * ((long long)min(t.n0 + row, d.N - 1) * d.ldb) + 8 * f.gslot[j];
  }
  f.kcur = d.Klast - kstart;
  f.k0 = 0;
}

// Copy the next stage of the stream, if there is one.
template <int F>
__device__ inline void u_issue(UFlow<F>& f, const NtDesc& d, int nt, char* smem, int wave, int lane) {
  if (!f.more) return;
  char* buf = smem + (f.gi % UR) * STAGE_B;
  if (f.k0 + Fmt<F>::K <= f.kcur) {
#pragma unroll
    for (int j = 0; j < NCOPY; ++j) {
      char* dst = buf + (wave + 4 * j) * 8 * ROW_B;
      __builtin_amdgcn_global_load_lds((glb_void*)(f.a[j] + Fmt<F>::EU * f.k0), (lds_void*)dst, 16, 0, 0);
      __builtin_amdgcn_global_load_lds((glb_void*)(f.b[j] + Fmt<F>::EU * f.k0), (lds_void*)(dst + OPER_B), 16, 0, 0);
    }
  } else {
    stage_copy<F>(f.a, f.gslot, f.k0, f.kcur, buf, wave);
    stage_copy<F>(f.b, f.gslot, f.k0, f.kcur, buf + OPER_B, wave);
  }
  ++f.gi;
  f.k0 += Fmt<F>::K;
  if (f.k0 >= f.kcur) {
    f.more = u_valid(f.it + gridDim.x, nt);
    if (f.more) {
      f.it += gridDim.x;
      u_start<F>(f, d, nt, wave, lane);
    }
  }
}

// Wait until a stage has landed: `newer` stages were copied after it.  Where a
// whole tile's outputs (64 store instructions, counted in order with the copies)
// were stored after it as well, 40 in flight leave it landed.
__device__ inline void u_wait(int newer, bool stored) {
  static_assert(2 * NCOPY == 8 && UR == 4, "the counts below");
  if (stored) asm volatile("s_waitcnt vmcnt(40)" ::: "memory");
  else if (newer >= 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else if (newer == 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Stage g of the stream: fragments in `cur`; those of the next stage go to
// `nxt` (not used after a tile's last).  l0, l1: column blocks that are not
// zero in B (tri_live), used unless WHOLE.
template <int F, int NI, int NJ, bool WHOLE>
__device__ inline void u_step(UFlow<F>& f, const NtDesc& d, int nt, int& g, int ge, bool l0, bool l1,
                              Frag<NI, NJ>& cur, Frag<NI, NJ>& nxt, f16v (&c_re)[NI][NJ], f16v (&c_im)[NI][NJ],
                              int rb0, int cb0, char* smem, int wave, int lane) {
  const int lr = lane & 31, lk = lane >> 5;
  u_wait(f.gi - 2 - g, g + 1 < ge);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  settle(cur);
  // stage g + 1 is there and every wave has read stage g: its buffer is free
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  u_issue<F>(f, d, nt, smem, wave, lane);
  const char* nb = smem + ((g + 1) % UR) * STAGE_B;
  __builtin_amdgcn_sched_barrier(0);
  read_frags_a<F>(nb, nxt, rb0, lr, lk);
  read_frags_b<F>(nb, nxt, cb0, lr, lk);
  if constexpr (WHOLE) {
    // the reads spread over the MFMAs: issued ahead of them they fill the LDS
    // queue, and the MFMAs wait for their turn
    stage_mma<F, NI, NJ, false, false>(cur, c_re, c_im);
#pragma unroll
    for (int i = 0; i < 4 * (NI + NJ); ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                             // a read of LDS
      __builtin_amdgcn_sched_group_barrier(0x8, NI * NJ * (F == 2 ? 12 : 8) / (4 * (NI + NJ)), 0);   // MFMAs
    }
  } else {
    stage_mma_tri<F, NI, NJ, false, false>(cur, c_re, c_im, l0, l1);
  }
  __builtin_amdgcn_sched_barrier(0);
  ++g;
}

// The outputs of a wave's block (tile_epilogue's layout) in the operand format;
// columns up to npad are stored, zero from N on.
template <int F, int NI, int NJ, bool FULL>
__device__ inline void u_store(const NtDesc& d, int b, int m0, int n0, const f16v (&c_re)[NI][NJ],
                               const f16v (&c_im)[NI][NJ], int npad, int lane) {
  constexpr int EB = 2 * Fmt<F>::EU;      // bytes per element
  const int lr = lane & 31, lk = lane >> 5;
  char* C = (char*)d.C + EB * ((long long)b * d.sC_bat + (long long)m0 * d.ldc + n0);
  long long part = 2 * quad_part<F>(4 * lk * d.ldc + lr);
  asm volatile("" : "+v"(part));          // formed here, not held over the K loop
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const bool in = FULL || n0 + j * 32 + lr < d.N;
      const bool col = FULL || n0 + j * 32 + (lr & ~7) < npad;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = i * 32 + 8 * (v >> 2) + (v & 3);
        const float re = in ? c_re[i][j][v] : 0.f, im = in ? c_im[i][j][v] : 0.f;
        if (FULL || (col && m0 + row + 4 * lk < d.M))
          quad_store<F>(C + (long long)row * d.ldc * EB + j * 32 * EB + part, re, im);
      }
    }
}

// The stages and outputs of one tile.
template <int F, int NI, int NJ>
__device__ inline void u_body(UFlow<F>& f, const NtDesc& d, int nt, const UTile& t, int& g, int& ge, int rb0, int cb0,
                              char* smem, int wave, int lane) {
  constexpr int SK = Fmt<F>::K;
  const int lr = lane & 31, lk = lane >> 5;
  const int kcur = d.Klast - (d.ktri ? t.n0 : 0);
  const int nst = (kcur + SK - 1) / SK;
  // from this stage on every column block of the wave counts (tri_live)
  const int s1 = d.ktri ? min(nst, (cb0 + (NJ - 1) * 32) / SK) : 0;
  f16v c_re[NI][NJ], c_im[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) c_re[i][j][v] = c_im[i][j][v] = 0.f;
  Frag<NI, NJ> f0, f1;
  read_frags_a<F>(smem + (g % UR) * STAGE_B, f0, rb0, lr, lk);
  read_frags_b<F>(smem + (g % UR) * STAGE_B, f0, cb0, lr, lk);
  int s = 0;
#pragma unroll 1
  for (; s < s1; ++s) {
    bool l0, l1;
    tri_live(true, s, SK, cb0, l0, l1);
    u_step<F, NI, NJ, false>(f, d, nt, g, ge, l0, l1, f0, f1, c_re, c_im, rb0, cb0, smem, wave, lane);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    settle(f1);
    f0 = f1;
  }
  // pairs, then an odd one: a loop of one exit keeps the accumulators in place
  const int pairs = (nst - s) >> 1;
#pragma unroll 1
  for (int i = 0; i < pairs; ++i) {
    u_step<F, NI, NJ, true>(f, d, nt, g, ge, true, true, f0, f1, c_re, c_im, rb0, cb0, smem, wave, lane);
    u_step<F, NI, NJ, true>(f, d, nt, g, ge, true, true, f1, f0, c_re, c_im, rb0, cb0, smem, wave, lane);
  }
  if ((nst - s) & 1)
    u_step<F, NI, NJ, true>(f, d, nt, g, ge, true, true, f0, f1, c_re, c_im, rb0, cb0, smem, wave, lane);
  const int npad = d.npad ? d.npad : (int)d.ldc;
  if (NI == 2 && t.m0 + XT <= d.M && t.n0 + XT <= d.N) {
    u_store<F, NI, NJ, true>(d, t.b, t.m0 + rb0, t.n0 + cb0, c_re, c_im, npad, lane);
    ge = f.gi;
  } else {
    u_store<F, NI, NJ, false>(d, t.b, t.m0 + rb0, t.n0 + cb0, c_re, c_im, npad, lane);
  }
}

// Bound: the matrix cores and what one wave a SIMD cannot lay beside them (busy
// 0.50 of the cycles in bf16x3 and 0.38 in single bf16 at 216 k, N_IP 800; the
// rest outputs, 17 operations a value, and the steps between stages).  Whole tiles
// one after the other with two workgroups a CU, outputs staged through LDS and
// every tile's first stages waited for -> now: bf16x3 47.5 k pairs on 4x4x4 (N_IP
// 520) 6.8 -> 6.5 ms; single bf16 at 216 k (N_IP 520) 5.9 -> 4.8 ms; 1000 k (N_IP
// 416) 10.0 ms both; bf16x3 rows 4 MB apart are slower and keep the former loop
// (run_u16).  Two workgroups a CU with two stages each measured 7.6, 6.6 and 10.7
// ms.
template <int F>
__global__ __launch_bounds__(XNT, 1) void zgemm_u16_kernel(NtDesc d, int nt) {
  extern __shared__ __attribute__((aligned(16))) char smem[];   // UR stages x (A, B)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (!u_valid(blockIdx.x, nt)) return;
  UFlow<F> f;
#pragma unroll
  for (int j = 0; j < NCOPY; ++j) f.gslot[j] = lds_slot((wave + 4 * j) * 8 + (lane >> 3), lane & 7);
  f.it = blockIdx.x;
  f.gi = 0;
  f.more = true;
  u_start<F>(f, d, nt, wave, lane);
#pragma unroll 1
  for (int i = 0; i < UR; ++i) u_issue<F>(f, d, nt, smem, wave, lane);
  int g = 0, ge = 0;                      // stages done; stages copied before the last whole tile's stores
  u_wait(f.gi - 1, false);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  for (int it = blockIdx.x; u_valid(it, nt); it += gridDim.x) {
    const UTile t = u_tile(d, nt, it);
    const int wm = wave >> 1, wn = wave & 1;
    // strips of at most 32 rows or columns: a 32 x 32 block a wave
    if (d.M - t.m0 <= 32) u_body<F, 1, 1>(f, d, nt, t, g, ge, 0, wave * 32, smem, wave, lane);
    else if (d.N - t.n0 <= 32) u_body<F, 1, 1>(f, d, nt, t, g, ge, wave * 32, 0, smem, wave, lane);
    else u_body<F, 2, 2>(f, d, nt, t, g, ge, wm * 64, wn * 64, smem, wave, lane);
  }
}

template <int F, bool A_CONJ, bool B_CONJ, int KIND, bool RINGP, bool TWOB = false, int T = XT>
__device__ inline void x3_tiles(const NtDesc* __restrict__ descs, int ndesc, long long t0, long long nt, int seg0,
                                int nseg, cplx* part) {
  extern __shared__ __attribute__((aligned(16))) char smem[];   // NBUF (RING) stages x (A, B)
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // units: the tiles [t0, t0 + nt) of the K segment seg0, or with part those
  // of each of nseg segments, segment by segment
  const long long units = nt * nseg;
  const long long u8 = (units + 7) / 8 * 8;
  const long long per = u8 / 8;
  for (long long it = blockIdx.x; it < u8; it += gridDim.x) {
    const long long u = (it % 8) * per + it / 8;   // XCD-contiguous ranges
    if (u >= units) continue;
    const int seg = seg0 + (int)(u / nt);
    const NtTile tl = nt_tile(descs, ndesc, t0 + u % nt);
    const NtDesc d = descs[tl.desc];
    const int b = tl.b, tm = tl.tm;
    int tn = tl.tn;
    if constexpr (KIND == 2 && T == XT)
      if (d.rot) tn = (tn + (b * d.tiles_m + tm) / d.rot) % d.tiles_n;
    cplx* pt = part ? part + u * (T * T) : nullptr;
    const int m0 = tm * T, n0 = tn * T;
    // interleaved formats: logical element e at u16 EU*e (e a multiple of 8)
    constexpr int EU = Fmt<F>::EU;
    // a triangular B (zero for k < n) contributes from k = n0 on
    const int kstart = d.ktri ? n0 : 0;
    const unsigned short* As =
        (const unsigned short*)d.A + EU * (b * d.sA_bat + (long long)seg * d.sA_seg + kstart);
    const unsigned short* Bs =
        (const unsigned short*)d.B + EU * (b * d.sB_bat + (long long)seg * d.sB_seg + kstart);
    const int kcur = ((seg == d.nseg - 1) ? d.Klast : d.Kseg) - kstart;

    // this lane's sources and slots in its copy instructions; rows past M / N
    // read the last valid row (their outputs are not stored)
    constexpr int NC = T / 32;
    const unsigned short* asrc[NC];
    const unsigned short* bsrc[NC];
    int gslot[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int row = (wave + 4 * j) * 8 + (lane >> 3);
      gslot[j] = lds_slot(row, lane & 7);     // the slot whose LDS position is lane & 7
      const int ra = min(m0 + row, d.M - 1), rb = min(n0 + row, d.N - 1);
      asrc[j] = As + EU * ((long long)ra * d.lda) + 8 * gslot[j];
      bsrc[j] = Bs + EU * ((long long)rb * d.ldb) + 8 * gslot[j];
    }
    // Hermitian outputs (lower tiles; the upper triangle is mirrored later):
    // in a diagonal tile, a wave whose block lies strictly above the
    // diagonal only helps with the copies (FP64 epilogues only; the entries it
    // skips lie above the diagonal, which the consumers never read)
    const bool diag = d.herm && tm == tn && d.epi != 3;
    const bool first = seg == 0;
    if constexpr (T != XT) {
      // a block outside the product stores nothing
      const bool idle = (diag && wm < wn) || (d.epi != 3 && (m0 + wm * 32 >= d.M || n0 + wn * 32 >= d.N));
      tile_body_small<F, A_CONJ, B_CONJ, KIND == 2>(d, b, m0, n0, kcur, asrc, bsrc, gslot, wm * 32, wn * 32, smem, wave,
                                                    lane, idle, first, pt);
    } else if constexpr (RINGP) {
      if (d.M - m0 <= 32)
        tile_body_ring<F, 1, 1, A_CONJ, B_CONJ>(d, b, m0, n0, kcur, asrc, bsrc, gslot, 0, wave * 32, smem, wave,
                                                lane, diag && wave > 0, first, pt);
      else if (d.N - n0 <= 32)
        tile_body_ring<F, 1, 1, A_CONJ, B_CONJ>(d, b, m0, n0, kcur, asrc, bsrc, gslot, wave * 32, 0, smem, wave,
                                                lane, false, first, pt);
      else
        tile_body_ring<F, 2, 2, A_CONJ, B_CONJ>(d, b, m0, n0, kcur, asrc, bsrc, gslot, wm * 64, wn * 64, smem,
                                                wave, lane, diag && wm < wn, first, pt);
    } else if constexpr (TWOB) {
      if (d.M - m0 <= 32)
        tile_body_2b<F, 1, 1, A_CONJ, B_CONJ>(d, b, m0, n0, kcur, asrc, bsrc, gslot, 0, wave * 32, smem, wave, lane,
                                              diag && wave > 0, first, pt);
      else if (d.N - n0 <= 32)
        tile_body_2b<F, 1, 1, A_CONJ, B_CONJ>(d, b, m0, n0, kcur, asrc, bsrc, gslot, wave * 32, 0, smem, wave, lane,
                                              false, first, pt);
      else
        tile_body_2b<F, 2, 2, A_CONJ, B_CONJ>(d, b, m0, n0, kcur, asrc, bsrc, gslot, wm * 64, wn * 64, smem, wave,
                                              lane, diag && wm < wn, first, pt);
    } else {
      if (d.M - m0 <= 32)
        tile_body<F, 1, 1, A_CONJ, B_CONJ, KIND>(d, b, m0, n0, kcur, asrc, bsrc, gslot, 0, wave * 32, smem, wave, lane,
                                           diag && wave > 0, first, pt);
      else if (d.N - n0 <= 32)
        tile_body<F, 1, 1, A_CONJ, B_CONJ, KIND>(d, b, m0, n0, kcur, asrc, bsrc, gslot, wave * 32, 0, smem, wave, lane,
                                           false, first, pt);
      else
        tile_body<F, 2, 2, A_CONJ, B_CONJ, KIND>(d, b, m0, n0, kcur, asrc, bsrc, gslot, wm * 64, wn * 64, smem, wave,
                                           lane, diag && wm < wn, first, pt);
    }
  }
}

// the two call sites of the path: U^q = R^q W^q (kind 2, no conjugation) and
// the fragment contraction (kind 3, B conjugated)
#define X3_ARGS const NtDesc *__restrict__ descs, int ndesc, long long t0, long long nt, int seg0, int nseg, cplx *part

__global__ __launch_bounds__(XNT, 2) void zgemm_x3_kernel(X3_ARGS) {
  x3_tiles<2, false, true, 3, false>(descs, ndesc, t0, nt, seg0, nseg, part);
}

// U^q in bf16x3 where zgemm_u16_kernel is the slower one (run_u16)
__global__ __launch_bounds__(XNT, 2) void zgemm_x3u_kernel(X3_ARGS) {
  x3_tiles<2, false, false, 2, false>(descs, ndesc, t0, nt, seg0, nseg, part);
}

// two barriers a stage: the fragment contraction of launches with few tiles
// (bf16x3), or always (single bf16)
template <int F>
__global__ __launch_bounds__(XNT, 2) void zgemm_c2b_kernel(X3_ARGS) {
  x3_tiles<F, false, true, 3, false, true>(descs, ndesc, t0, nt, seg0, nseg, part);
}

// ring pipeline (one workgroup a CU), both formats
template <int F>
__global__ __launch_bounds__(XNT, 1) void zgemm_ring_kernel(X3_ARGS) {
  x3_tiles<F, false, true, 3, true>(descs, ndesc, t0, nt, seg0, nseg, part);
}

// 64 x 64 tiles, a 32 x 32 block a wave, eight LDS stages (one workgroup a CU):
// launches of few tiles, which leave most CUs idle and wait out every stage's
// latency.  The K chain of an element stays whole and in order (the bits do not
// change); its stage falls from 1.2 us (128 x 128 tile alone on its CU: 48 MFMAs
// a wave and two stages ahead) to 0.39 us (12 MFMAs, seven ahead): contraction
// of one 16-orbital fragment at N_IP = 256 on the 2x2x2 mesh, 128 stages, 154 ->
// 50 us; its U^q 30 -> 15 us.
template <int F, int KIND>
__global__ __launch_bounds__(XNT, 1) void zgemm_small16_kernel(X3_ARGS) {
  x3_tiles<F, false, KIND == 3, KIND, true, false, X3_SMALL>(descs, ndesc, t0, nt, seg0, nseg, part);
}
#undef X3_ARGS

}  // namespace

long long x3_plan(NtDesc* d, int n, int tile) {
  long long acc = 0;
  for (int i = 0; i < n; ++i) {
    d[i].tiles_m = ceil_div(d[i].M, tile);
    d[i].tiles_n = ceil_div(d[i].N, tile);
    d[i].tiles_per_batch = d[i].herm ? d[i].tiles_m * (d[i].tiles_m + 1) / 2
                                     : d[i].tiles_m * d[i].tiles_n;
    if (d[i].Klast <= 0 || d[i].Klast > d[i].Kseg) d[i].Klast = d[i].Kseg;
    d[i].tile_begin = acc;
    acc += (long long)d[i].tiles_per_batch * d[i].batch;
  }
  return acc;
}

hipError_t u16_launch(int fmt, const NtDesc& d, long long nt, int max_blocks, hipStream_t s) {
  if (nt <= 0) return hipSuccess;
  if ((fmt != 2 && fmt != 3) || nt > (1LL << 30) || d.nseg != 1 || d.epi != 3 || d.herm) return hipErrorInvalidValue;
  const long long u8 = (nt + 7) / 8 * 8;
  max_blocks = max_blocks / 8 * 8;
  const dim3 g((unsigned)(u8 < max_blocks ? u8 : max_blocks)), b(XNT);
  if (fmt == 2) hipLaunchKernelGGL(zgemm_u16_kernel<2>, g, b, UR * STAGE_B, s, d, (int)nt);
  else hipLaunchKernelGGL(zgemm_u16_kernel<3>, g, b, UR * STAGE_B, s, d, (int)nt);
  return hipGetLastError();
}

hipError_t x3_launch(int fmt, const NtDesc* descs_dev, int ndesc, long long t0, long long nt, int seg0, int nseg,
                     cplx* part, int max_blocks, hipStream_t s, int kind, bool ring, int tile) {
  if (nt <= 0 || nseg <= 0) return hipSuccess;
  if ((fmt != 2 && fmt != 3) || (kind != 2 && kind != 3) || (!part && nseg != 1) ||
      (tile != XT && tile != X3_SMALL) || (kind == 2 && tile != X3_SMALL && (fmt != 2 || ring)))
    return hipErrorInvalidValue;
  const long long units = nt * nseg, u8 = (units + 7) / 8 * 8;
  max_blocks = max_blocks / 8 * 8;
  const dim3 g((unsigned)(u8 < max_blocks ? u8 : max_blocks)), b(XNT);
#define COMMA ,
#define X3_GO(KERNEL, LDS) \
  hipLaunchKernelGGL((KERNEL), g, b, LDS, s, descs_dev, ndesc, t0, nt, seg0, nseg, part)
  if (tile == X3_SMALL) {
    if (fmt == 2 && kind == 2) X3_GO(zgemm_small16_kernel<2 COMMA 2>, SRING * SSTAGE_B);
    else if (fmt == 2) X3_GO(zgemm_small16_kernel<2 COMMA 3>, SRING * SSTAGE_B);
    else if (kind == 2) X3_GO(zgemm_small16_kernel<3 COMMA 2>, SRING * SSTAGE_B);
    else X3_GO(zgemm_small16_kernel<3 COMMA 3>, SRING * SSTAGE_B);
  } else if (kind == 2) {
    X3_GO(zgemm_x3u_kernel, NBUF * STAGE_B);
  } else if (ring) {
    if (fmt == 2) X3_GO(zgemm_ring_kernel<2>, RING * STAGE_B);
    else X3_GO(zgemm_ring_kernel<3>, RING * STAGE_B);
  } else if (fmt == 3) {
    // single bf16: 32 MFMAs a stage (against 48 in bf16x3) leave less time to
    // cover a one-stage prefetch; the contraction always takes the two-barrier
    // loop (0.378 against 0.354 of bf16 peak on the 120-orbital 1000-k shape)
    X3_GO(zgemm_c2b_kernel<3>, NBUF * STAGE_B);
  } else if (units < 2LL * g.x) {
    X3_GO(zgemm_c2b_kernel<2>, NBUF * STAGE_B);
  } else {
    X3_GO(zgemm_x3_kernel, NBUF * STAGE_B);
  }
#undef X3_GO
#undef COMMA
  return hipGetLastError();
}
