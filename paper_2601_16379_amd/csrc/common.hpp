// Shared device helpers of the gfx950 ISDF library: complex arithmetic on
// interleaved float64 pairs and small launch utilities.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef double2 cplx;   // (re, im)

__host__ __device__ inline cplx cmk(double r, double i) { cplx z; z.x = r; z.y = i; return z; }
__host__ __device__ inline cplx cadd(cplx a, cplx b) { return cmk(a.x + b.x, a.y + b.y); }
__host__ __device__ inline cplx csub(cplx a, cplx b) { return cmk(a.x - b.x, a.y - b.y); }
__host__ __device__ inline cplx cmul(cplx a, cplx b) {
  return cmk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
__host__ __device__ inline cplx cmulc(cplx a, cplx b) {
  return cmk(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__host__ __device__ inline cplx cconj(cplx a) { return cmk(a.x, -a.y); }
__host__ __device__ inline cplx cscale(cplx a, double s) { return cmk(a.x * s, a.y * s); }
// acc += a * b
__host__ __device__ inline void cfma(cplx& acc, cplx a, cplx b) {
  acc.x = fma(a.x, b.x, fma(-a.y, b.y, acc.x));
  acc.y = fma(a.x, b.y, fma(a.y, b.x, acc.y));
}

// exp(i * pi * x) in FP64
__device__ inline cplx cexpipi(double x) {
  double s, c;
  sincospi(x, &s, &c);
  return cmk(c, s);
}

// LDS values stored by lanes of this wavefront are there for its other lanes.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

static inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

// Store one complex value in one of the operand formats of the NT GEMMs:
//   0  complex128 at element off;
//   1  float planes re | im, element off of each plane (plane stride `plane`);
//   2  bf16 hi + lo (x = hi + lo per real component), interleaved by groups
//      of 8 elements: element off at u16 index bf16x3_index(off, p) with
//      p = 0 re_hi, 1 re_lo, 2 im_hi, 3 im_lo, so that the 16 k of one
//      matrix-core step of a row are 128 contiguous bytes (rows start at
//      multiples of 8 elements; `plane` is not used);
//   3  single bf16 (re, im), interleaved by groups of 8 elements: element off
//      at u16 index (off >> 3) * 16 + p * 8 + (off & 7), p = 0 re, 1 im, so
//      that the 32 k of one stage of a row are 128 contiguous bytes.
__device__ inline unsigned short bf16_bits_of(float x) {
  __bf16 h = (__bf16)x;
  return __builtin_bit_cast(unsigned short, h);
}
__device__ inline float bf16_value(unsigned short b) { return (float)__builtin_bit_cast(__bf16, b); }
__host__ __device__ inline long long bf16x3_index(long long off, int p) { return (off >> 3) * 32 + p * 8 + (off & 7); }

__device__ inline void store_bf16x3(unsigned short* o, long long off, float re, float im) {
  const unsigned short rh = bf16_bits_of(re), ih = bf16_bits_of(im);
  const long long b = (off >> 3) * 32 + (off & 7);
  o[b] = rh;
  o[b + 8] = bf16_bits_of(re - bf16_value(rh));
  o[b + 16] = ih;
  o[b + 24] = bf16_bits_of(im - bf16_value(ih));
}

// ---- 16-bit operand stores of four consecutive points by the lanes of a quad ----
// Each lane holds the values of one point (the quad's four are consecutive, the
// first a multiple of four); the quad exchanges them by DPP so that each lane
// stores one whole part: 8 bytes (4 points of one of the four planes) in bf16
// hi+lo, 4 bytes (2 points of one of the two) in single bf16, against four
// (two) 2-byte stores a lane.
__device__ inline unsigned bf16_pair(float lo, float hi) {      // bits of lo and hi in bf16, one conversion
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f2{lo, hi}), b2));
}
template <int CTRL> __device__ inline unsigned quad_mov(unsigned v) {
  return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}
// quad_part: u16 offset of the part this lane stores, for its point's element
// offset off; output rows further on add a multiple of 8 elements.
template <int FMT> __device__ inline long long quad_part(long long off) {
  const int t = threadIdx.x & 3;
  return FMT == 2 ? (off >> 3) * 32 + t * 8 + (off & 4) : (off >> 3) * 16 + (t >> 1) * 8 + (off & 4) + 2 * (t & 1);
}
template <int FMT> __device__ inline void quad_store(char* o, float re, float im) {
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(1))) v2u glb_v2u;        // global, not flat, stores
  typedef __attribute__((address_space(1))) unsigned glb_u;
  constexpr int X1 = 0xB1, X2 = 0x4E, SWAP12 = 0xD8;   // quad_perm [1,0,3,2], [2,3,0,1], [0,2,1,3]
  const int t = threadIdx.x & 3;
  const unsigned h = bf16_pair(re, im);
  // byte selectors of v_perm (s0, s1): even lanes (own.lo, other.lo), odd (other.hi, own.hi)
  const unsigned sel = (t & 1) ? 0x07060302u : 0x01000504u;
  if constexpr (FMT == 2) {
    const unsigned l = bf16_pair(re - __uint_as_float(h << 16), im - __uint_as_float(h & 0xffff0000u));
    const unsigned d0 = __builtin_amdgcn_perm(l, h, 0x05040100u), d1 = __builtin_amdgcn_perm(l, h, 0x07060302u);
    // points (2i, 2i + 1) of planes t & 1 (n0) and 2 + (t & 1) (n1)
    const unsigned n0 = __builtin_amdgcn_perm(d0, quad_mov<X1>(d0), sel);
    const unsigned n1 = __builtin_amdgcn_perm(d1, quad_mov<X1>(d1), sel);
    const unsigned r = quad_mov<X2>(t < 2 ? n1 : n0);
    *(glb_v2u*)o = t < 2 ? v2u{n0, r} : v2u{r, n1};
  } else {
    const unsigned n = __builtin_amdgcn_perm(h, quad_mov<X1>(h), sel);   // lanes: re01, im01, re23, im23
    *(glb_u*)o = quad_mov<SWAP12>(n);
  }
}

__device__ inline void store_fmt(void* out, long long off, long long plane, int fmt, cplx v) {
  if (fmt == 0) {
    ((cplx*)out)[off] = v;
  } else if (fmt == 1) {
    float* o = (float*)out;
    o[off] = (float)v.x;
    o[plane + off] = (float)v.y;
  } else if (fmt == 2) {
    store_bf16x3((unsigned short*)out, off, (float)v.x, (float)v.y);
  } else {
    unsigned short* o = (unsigned short*)out;
    const long long b = (off >> 3) * 16 + (off & 7);
    o[b] = bf16_bits_of((float)v.x);
    o[b + 8] = bf16_bits_of((float)v.y);
  }
}
