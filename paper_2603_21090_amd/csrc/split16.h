// fp32 matrix products on the f16 matrix units, both operands split in two:  a s = h + l / 2048 with h = f16(a s) and
// l = f16(2048 (a s - h)), s a power of two.  h and l hold 11 significant bits each, so a is represented to 2^-23 to 2^-24 of
// itself, and
//     a b = (h_a h_b + (h_a l_b + l_a h_b) / 2048) / (s_a s_b)        [l_a l_b, at most 2^-24 of the product, left out]
// takes three v_mfma_f32_16x16x32_f16 of 16 cycles for 32 elements of K where v_mfma_f32_16x16x4_f32 takes eight of 32
// cycles: 48 against 256.  Products of f16 are exact in fp32 and each instruction adds 32 of them to its accumulator, so a sum over
// K is rounded a fraction as often as in the fp32 form: the errors of whole embeddings against 64 bits are
// smaller than with it (the figures stand in layer_kernel.h).
//
// Range: f16 is normal from 2^-14 to 2^16, so s brings a bound of the operand's magnitudes to 2^13 .. 2^14 and whatever is
// more than 2^-27 of the bound keeps all of its bits (below, h and l together are exact to 2^-36 absolute, 2^-49 of the bound).
// Weights have one s per matrix, chosen when they are packed; activations one per row, from the row's largest magnitude
// or a bound of it.  Rows that hold an infinity or a NaN come out as NaN; no other row is touched by them.
//
// Layouts.  An operand takes the bytes that the fp32 form would take: eight columns are 16 bytes of h and, behind
// them, 16 bytes of l.  Lane (i, c) = (lane / 16, lane % 16) owns, in step u of a 64-element chunk, the elements
// 32 u + 8 i .. + 7 of K: of row c for the A operand (LDS, row-major), of column c for the B operand.  B is packed per
// 16-column tile and chunk as four blocks of 1 KiB (h of step 0, l of step 0, h of step 1, l of step 1), 16 bytes
// per lane, so a wave's request is contiguous.
#pragma once
#include <hip/hip_runtime.h>

namespace stgn {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kChunkK = 64;              // elements of K per chunk
constexpr uint32_t kChunkFloats = 1024;       // floats of one (column tile, chunk) block of packed B
constexpr float kLoScale = 2048.0f;

__host__ __device__ inline uint32_t chunks64(uint32_t K) { return (K + kChunkK - 1) / kChunkK; }

// accumulator register r of lane l: row 4 (l / 16) + r, column l % 16
__device__ inline uint32_t s16_row(uint32_t lane, uint32_t r) { return 4u * (lane >> 4) + r; }
__device__ inline uint32_t s16_col(uint32_t lane) { return lane & 15u; }

// Power of two that brings magnitudes up to `bound` (>= 0, infinite or NaN) below 2^14, and its inverse.
__device__ inline float pow2_scale(float bound) {
  uint32_t e = (__builtin_bit_cast(uint32_t, bound) >> 23) & 0xFFu;
  e = e < 20u ? 20u : e > 254u ? 254u : e;
  return __builtin_bit_cast(float, (267u - e) << 23);
}
__device__ inline float inv_pow2(float s) { return __builtin_bit_cast(float, 0x7F000000u - __builtin_bit_cast(uint32_t, s)); }

// largest of each 16-lane row's magnitudes (every lane of a row receives it): as integers, whose order is theirs, with
// no quieting of NaNs between the steps (a NaN comes out as the largest)
template <int CTRL>
__device__ inline uint32_t dpp_max(uint32_t x) {
  return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false));
}
__device__ inline float row16_max(float m) {
  uint32_t x = __builtin_bit_cast(uint32_t, m);
  x = dpp_max<0xB1>(x); x = dpp_max<0x4E>(x); x = dpp_max<0x141>(x); x = dpp_max<0x140>(x);
  return __builtin_bit_cast(float, x);
}
__device__ inline float bits_max(float a, float b) {
  return __builtin_bit_cast(float, max(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b)));
}

__device__ inline float max4(const float4& v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))); }

// Pairs of elements through the mixed-precision multiply-add: h = f16(a s), r = a s - h (exact), l = f16(2048 r), three
// instructions an element with the packing done by them (conversions, a subtraction and a multiplication each took six
// and a pack).  In the halves of `hi` and `lo`: element 0 low, element 1 high.
__device__ inline void split2(float a0, float a1, float s, uint32_t& hi, uint32_t& lo) {
  float r0, r1;
  const float k = kLoScale;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(hi) : "v"(a0), "v"(s));
  asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(hi) : "v"(a1), "v"(s));
  asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(r0) : "v"(a0), "v"(s), "v"(hi));
  asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(r1) : "v"(a1), "v"(s), "v"(hi));
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(lo) : "v"(r0), "s"(k));
  asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(lo) : "v"(r1), "s"(k));
}

// four consecutive columns (the first a multiple of four) of a row in LDS that starts at `row`
__device__ inline float* split_at(float* row, uint32_t col) { return row + (col & ~7u) + ((col & 4u) >> 1); }
__device__ inline void split_store4(float* row, uint32_t col, const float4& v, float s) {
  uint2 h, l;
  split2(v.x, v.y, s, h.x, l.x);
  split2(v.z, v.w, s, h.y, l.y);
  float* p = split_at(row, col);
  *reinterpret_cast<uint2*>(p) = h;
  *reinterpret_cast<uint2*>(p + 4) = l;
}
__device__ inline float4 split_load4(const float* row, uint32_t col, float inv) {
  const float* p = split_at(const_cast<float*>(row), col);
  const halfx4 h = *reinterpret_cast<const halfx4*>(p), l = *reinterpret_cast<const halfx4*>(p + 4);
  const float c = 1.0f / kLoScale;
  return make_float4(fmaf((float)l[0], c, (float)h[0]) * inv, fmaf((float)l[1], c, (float)h[1]) * inv,
                     fmaf((float)l[2], c, (float)h[2]) * inv, fmaf((float)l[3], c, (float)h[3]) * inv);
}
// one element
__device__ inline void split_store1(float* row, uint32_t col, float v, float s) {
  uint32_t h, l;
  float r;
  const float k = kLoScale;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(v), "v"(s));
  asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(r) : "v"(v), "v"(s), "v"(h));
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(l) : "v"(r), "s"(k));
  uint16_t* p = reinterpret_cast<uint16_t*>(row + (col & ~7u)) + (col & 7u);
  p[0] = (uint16_t)h;
  p[8] = (uint16_t)l;
}

// per-lane offset (floats) into an A tile in LDS with rows of lda floats
__device__ inline uint32_t s16_off(uint32_t lane, uint32_t lda) { return (lane & 15u) * lda + 8u * (lane >> 4); }

// Operands of one chunk: h and l of step 0, h and l of step 1.  Reads of A past the last element of K land in
// neighbouring split data and meet zero weights.
__device__ inline void load_a64(const float* Ap, uint32_t ch, float4 (&a)[4]) {
  const float* p = Ap + kChunkK * ch;
  a[0] = *reinterpret_cast<const float4*>(p);
  a[1] = *reinterpret_cast<const float4*>(p + 4);
  a[2] = *reinterpret_cast<const float4*>(p + 32);
  a[3] = *reinterpret_cast<const float4*>(p + 36);
}
// (the lane is an argument so that a caller with a long loop can pass an opaque copy of it: from threadIdx.x alone the
// compiler computes one 64-bit address per lane and matrix ahead of the loop and keeps, or spills, them all)
__device__ inline void load_b64(const float* __restrict__ Bt, uint32_t ch, float4 (&b)[4], uint32_t lane) {
  const char* p = reinterpret_cast<const char*>(Bt) + (size_t)ch * (4u * kChunkFloats);
  const uint32_t off = lane * 16u;
#pragma unroll
  for (int c = 0; c < 4; ++c) b[c] = *reinterpret_cast<const float4*>(p + c * 1024 + off);
}

template <int NTL>
struct AccS { floatx4 h[NTL] = {}, l[NTL] = {}; };          // h_a h_b, and 2048 times the rest

template <int NTL>
__device__ inline void mfma_chunk(const float4 (&a)[4], const float4 (&b)[NTL][4], AccS<NTL>& acc) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const halfx8 ah = __builtin_bit_cast(halfx8, a[2 * u]), al = __builtin_bit_cast(halfx8, a[2 * u + 1]);
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      const halfx8 bh = __builtin_bit_cast(halfx8, b[t][2 * u]), bl = __builtin_bit_cast(halfx8, b[t][2 * u + 1]);
      acc.l[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bl, acc.l[t], 0, 0, 0);
      acc.h[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bh, acc.h[t], 0, 0, 0);
      acc.l[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, bh, acc.l[t], 0, 0, 0);
    }
  }
}
// the product's column tile t, row r of the lane's four (still scaled by s_a s_b)
template <int NTL>
__device__ inline float acc_value(const AccS<NTL>& acc, int t, int r) { return fmaf(acc.l[t][r], 1.0f / kLoScale, acc.h[t][r]); }

template <int NTL>
struct OpsS { float4 a[4]; float4 b[NTL][4]; };

// Chunks [c0, c1) of a product with one buffer: for what a shape has beyond the products its kernel is tuned for, where the
// registers of a second buffer would cost those.
template <int NTL>
__device__ __forceinline__ void mfma_lean(const float* Ap, uint32_t c0, uint32_t c1, const float* const (&Bt)[NTL],
                                          AccS<NTL>& acc, uint32_t lane) {
#pragma unroll 1
  for (uint32_t ch = c0; ch < c1; ++ch) {
    OpsS<NTL> o;
#pragma unroll
    for (int t = 0; t < NTL; ++t) load_b64(Bt[t], ch, o.b[t], lane);
    load_a64(Ap, ch, o.a);
    mfma_chunk<NTL>(o.a, o.b, acc);
  }
}

// The weight chunks of a short product requested in one go, typically a phase ahead.  Requests are unconditional (behind a
// branch the compiler would wait for more than it needs): chunks past the end repeat the last one and are never multiplied.
template <int NTL, int MAXC>
struct Upfront {
  float4 b[MAXC][NTL][4];
  __device__ __forceinline__ void request(const float* const (&Bt)[NTL], uint32_t nchunks, uint32_t lane) {
#pragma unroll
    for (int ch = 0; ch < MAXC; ++ch) {
      const uint32_t c = (uint32_t)ch < nchunks ? (uint32_t)ch : nchunks - 1u;
#pragma unroll
      for (int t = 0; t < NTL; ++t) load_b64(Bt[t], c, b[ch][t], lane);
    }
  }
  // the whole product, also where K has more chunks than were requested
  __device__ __forceinline__ void multiply(const float* Ap, uint32_t nchunks, const float* const (&Bt)[NTL], AccS<NTL>& acc,
                                           uint32_t lane) {
#pragma unroll
    for (int ch = 0; ch < MAXC; ++ch) {
      if ((uint32_t)ch < nchunks) {                  // wave-uniform; only LDS reads and products inside
        float4 a[4];
        load_a64(Ap, ch, a);
        mfma_chunk<NTL>(a, b[ch], acc);
      }
    }
    mfma_lean<NTL>(Ap, MAXC, nchunks, Bt, acc, lane);
  }
};

}  // namespace stgn
