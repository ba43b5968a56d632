// fp32 matrix-core tiles for gfx950 with 16-row operands: C[16 x 16] += A[16 x K] * B[K x 16]
// using v_mfma_f32_16x16x4_f32 (K advances by 4 per instruction, one "k-step").
//
// K is cut into GROUPS of 16 elements = four k-steps.  Inside a group the four lane groups
// (lane / 16 = i) own the elements 16 g + 4 i + u, u = 0..3 being the k-step: the matrix
// instruction does not care which element of K a lane group contributes as long as A and B agree,
// and this assignment makes both operands of four consecutive k-steps one 16-byte value per lane:
//   A (LDS, row-major, stride lda = 4 mod 8 floats):  one ds_read_b128 at row * lda + 16 g + 4 i
//   B (weights, global): packed GROUP-MAJOR per 16-column tile at create time -- for column tile n
//     and group g, 64 lanes x 4 floats, lane (i, col) holding B[16 g + 4 i + u][16 n + col] for
//     u = 0..3; the groups of one column tile follow each other.  A wave's load of one group is one
//     contiguous 1 KiB read at an immediate offset.
// Four groups (64 elements of K) form a CHUNK, the unit of register double buffering: while the
// matrix pipe works on one chunk the operands of the next one are in flight.  K is padded to whole
// chunks with zero weights.  Two column tiles
// that share the A operand are multiplied together (independent accumulators, so consecutive
// matrix instructions never wait for each other).
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>

namespace stgn {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kGrpK = 16;            // elements of K per group
constexpr uint32_t kGrpFloats = 256;      // floats of one (column tile, group) block of packed B
constexpr int kCG = 4;                    // groups per chunk
constexpr uint32_t kChunkSteps = 4 * kCG; // k-steps per chunk
constexpr uint32_t kChunkK = kGrpK * kCG; // elements of K per chunk
constexpr uint32_t kChunkFloats = kGrpFloats * kCG;   // floats of one (column tile, chunk) block of packed B

// number of groups that cover K elements, rounded up to whole chunks
__host__ __device__ inline uint32_t chunks_of(uint32_t K) { return (K + kGrpK * kCG - 1) / (kGrpK * kCG); }
__host__ __device__ inline uint32_t groups_of(uint32_t K) { return kCG * chunks_of(K); }

// Operand layout of v_mfma_f32_16x16x4_f32 for lane l:
//   A element: row l % 16, lane group l / 16        B element: lane group l / 16, column l % 16
//   accumulator register r (0..3): row 4 * (l / 16) + r, column l % 16
__device__ inline uint32_t m16_row(uint32_t lane, uint32_t r) { return 4u * (lane >> 4) + r; }
__device__ inline uint32_t m16_col(uint32_t lane) { return lane & 15u; }

// per-lane element offset into an A tile in LDS with stride lda
__device__ inline uint32_t a16_off(uint32_t lane, uint32_t lda) { return (lane & 15u) * lda + 4u * (lane >> 4); }
__device__ inline uint32_t a16_lane_off(uint32_t lda) {
  const uint32_t lane = threadIdx.x & 63u;
  return (lane & 15u) * lda + 4u * (lane >> 4);
}

template <int U>
__device__ inline float comp4(const float4& v) {
  if constexpr (U == 0) return v.x;
  else if constexpr (U == 1) return v.y;
  else if constexpr (U == 2) return v.z;
  else return v.w;
}

// A operands of groups [g0, g0 + kCG) of the tile row range this lane serves (Ap = tile + lane offset).  Groups past `last`,
// the last one inside the row, repeat it: they meet zero weights, but the next row's data could hold a NaN, and a
// NaN times zero is one.  (Rows of whole chunks need no limit.)
constexpr uint32_t kNoLimit = 0xFFFFFFFFu;
__device__ inline void load_a16(const float* Ap, uint32_t g0, float4 (&a)[kCG], uint32_t last = kNoLimit) {
#pragma unroll
  for (int c = 0; c < kCG; ++c) a[c] = *reinterpret_cast<const float4*>(Ap + kGrpK * (g0 + c < last ? g0 + c : last));
}
// that group of a row of `ld` floats, 4 of them padding
__host__ __device__ inline uint32_t last_group(uint32_t ld) { return ld / kGrpK - 1u; }

// B operands of groups [g0, g0 + kCG) of the column tile whose group 0 is Bt (wave-uniform).  The lane is an argument so
// that a caller with a long loop can pass an opaque copy of it: from threadIdx.x alone the compiler computes one 64-bit
// address per lane and matrix ahead of the loop and keeps (or spills) them all; with it a load takes its matrix's address
// from scalar registers and 16 lane as the offset.
__device__ inline void load_b16(const float* __restrict__ Bt, uint32_t g0, float4 (&b)[kCG], uint32_t lane) {
  const char* p = reinterpret_cast<const char*>(Bt) + (size_t)g0 * 1024u;
  const uint32_t off = lane * 16u;
#pragma unroll
  for (int c = 0; c < kCG; ++c) b[c] = *reinterpret_cast<const float4*>(p + c * 1024 + off);
}
__device__ inline void load_b16(const float* __restrict__ Bt, uint32_t g0, float4 (&b)[kCG]) {
  load_b16(Bt, g0, b, threadIdx.x & 63u);
}

template <int U, int NTL>
__device__ inline void mfma16_one(const float4& a, const float4 (&b)[NTL][kCG], int c, floatx4 (&acc)[NTL]) {
#pragma unroll
  for (int t = 0; t < NTL; ++t)
    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(comp4<U>(a), comp4<U>(b[t][c]), acc[t], 0, 0, 0);
}

// all 16 k-steps of one chunk, for NTL column tiles sharing the A operand (memory update, projections).  Straight-line code:
// K is padded to whole chunks (zero weights, finite A), which costs a few surplus products and buys a
// loop body without branches that the compiler can schedule around the outstanding loads.
template <int NTL>
__device__ inline void mfma16_chunk(const float4 (&a)[kCG], const float4 (&b)[NTL][kCG], floatx4 (&acc)[NTL]) {
#pragma unroll
  for (int c = 0; c < kCG; ++c) {
    mfma16_one<0, NTL>(a[c], b, c, acc);
    mfma16_one<1, NTL>(a[c], b, c, acc);
    mfma16_one<2, NTL>(a[c], b, c, acc);
    mfma16_one<3, NTL>(a[c], b, c, acc);
  }
}

// Groups of a chunk that hold elements of K: `used` of the product's groups, the chunk starting at g0 (uniform).
__device__ inline uint32_t groups_in(uint32_t used, uint32_t g0) { return used <= g0 ? 0u : min(used - g0, (uint32_t)kCG); }

// ... and all of them, where asking would take longer than the products
struct AllGroups {};

// The same for RT row tiles (`rs` floats apart in LDS) that share the B operand: every B register meets RT A registers.  Only
// the first ng groups are multiplied, the others hold zero weights: K of 100 has 7 of two chunks' 8 groups, a head of 32 two
// of four.  Batches with these products left out: four heads of 32 171 -> 164 us, 100,000 nodes of two heads of 50 426 -> 415,
// 1,000,000 nodes 1,941 -> 1,894.
template <int RT, int NTL, class NG>
__device__ inline void mfma16_chunk_rows(const float* Ap, uint32_t rs, uint32_t g0, const float4 (&b)[NTL][kCG],
                                         floatx4 (&acc)[RT][NTL], NG groups, uint32_t last = kNoLimit) {
  constexpr bool all = std::is_same<NG, AllGroups>::value;
  uint32_t ng = kCG;
  if constexpr (!all) {
    ng = (uint32_t)__builtin_amdgcn_readfirstlane((int)groups);
    asm volatile("" : "+s"(ng));                              // (else a caller's loop holds every comparison with it in scalar registers)
  }
  auto load = [&](int c, float4 (&a)[RT]) {
    const uint32_t g = g0 + c < last ? g0 + c : last;
#pragma unroll
    for (int r = 0; r < RT; ++r) a[r] = *reinterpret_cast<const float4*>(Ap + r * rs + kGrpK * g);
  };
  auto mul = [&](int c, const float4 (&a)[RT]) {
#pragma unroll
    for (int r = 0; r < RT; ++r) mfma16_one<0, NTL>(a[r], b, c, acc[r]);
#pragma unroll
    for (int r = 0; r < RT; ++r) mfma16_one<1, NTL>(a[r], b, c, acc[r]);
#pragma unroll
    for (int r = 0; r < RT; ++r) mfma16_one<2, NTL>(a[r], b, c, acc[r]);
#pragma unroll
    for (int r = 0; r < RT; ++r) mfma16_one<3, NTL>(a[r], b, c, acc[r]);
  };
  if constexpr (RT == 1) {
    float4 a[kCG][RT];
#pragma unroll
    for (int c = 0; c < kCG; ++c) load(c, a[c]);
#pragma unroll
    for (int c = 0; c < kCG; ++c)
      if (all || (uint32_t)c < ng) mul(c, a[c]);                     // (uniform)
  } else {
    static_assert(kCG == 4, "written out for four groups");   // (two groups of A in flight: all four would cost 16 registers more and spill)
    float4 a0[RT], a1[RT];
    load(0, a0);
    load(1, a1);
    __builtin_amdgcn_sched_barrier(0);
    if (all || ng > 0u) mul(0, a0);
    __builtin_amdgcn_sched_barrier(0);
    load(2, a0);
    __builtin_amdgcn_sched_barrier(0);
    if (all || ng > 1u) mul(1, a1);
    __builtin_amdgcn_sched_barrier(0);
    load(3, a1);
    __builtin_amdgcn_sched_barrier(0);
    if (all || ng > 2u) mul(2, a0);
    if (all || ng > 3u) mul(3, a1);
  }
}

// Operands of one chunk for NTL column tiles.
template <int NTL>
struct Ops16 {
  float4 a[kCG];
  float4 b[NTL][kCG];
};

template <int NTL>
__device__ inline void mfma16_chunk(const Ops16<NTL>& o, floatx4 (&acc)[NTL]) { mfma16_chunk<NTL>(o.a, o.b, acc); }

// Runs compute(i, buf) for i = 0 .. n - 1 (n >= 1) with two operand buffers: the operands of item
// i + 1 are requested (load(i + 1, buf)) before the work on item i is issued, so every load has one
// whole item of work to arrive.  P already holds item 0.  Scheduling fences keep the requests ahead
// of the work they are meant to overlap.
//
// Loads inside the steady-state loop are never conditional: the memory counter a wave waits on
// counts requests in issue order, and after a branch that may or may not have issued requests the
// compiler must wait for the youngest of them -- which would drain the prefetch it was meant to hide.
//
// Peeled form: the tail is written out, so no request is wasted (three more copies of `compute`).
template <class Buf, class LoadF, class ComputeF>
__device__ __forceinline__ void pingpong_peeled(uint32_t n, Buf& P, LoadF load, ComputeF compute) {
  Buf Q;
  uint32_t i = 0;
  for (; i + 2 < n; i += 2) {
    load(i + 1, Q);
    __builtin_amdgcn_sched_barrier(0);
    compute(i, P);
    __builtin_amdgcn_sched_barrier(0);
    load(i + 2, P);
    __builtin_amdgcn_sched_barrier(0);
    compute(i + 1, Q);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (i + 1 < n) {
    load(i + 1, Q);
    __builtin_amdgcn_sched_barrier(0);
    compute(i, P);
    __builtin_amdgcn_sched_barrier(0);
    compute(i + 1, Q);
  } else {
    compute(i, P);
  }
}

// Clamped form: two copies of `compute` only; past the end the last item is requested again (a
// cache hit) and ignored.
template <class Buf, class LoadF, class ComputeF>
__device__ __forceinline__ void pingpong_clamped(uint32_t n, Buf& P, LoadF load, ComputeF compute) {
  Buf Q;
  for (uint32_t i = 0; i < n; i += 2) {
    load(i + 1 < n ? i + 1 : n - 1, Q);
    __builtin_amdgcn_sched_barrier(0);
    compute(i, P);
    __builtin_amdgcn_sched_barrier(0);
    load(i + 2 < n ? i + 2 : n - 1, P);
    __builtin_amdgcn_sched_barrier(0);
    if (i + 1 < n) compute(i + 1, Q);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// acc[t] += A[16 x 64 nchunks] * (column tile Bt[t]), nchunks >= 1; the weights of the first chunk are
// already in P.b -- callers request them ahead of the barrier that makes A valid.
template <int NTL>
__device__ __forceinline__ void mfma16_gemm_pre(const float* Ap, uint32_t nchunks, const float* const (&Bt)[NTL],
                                                floatx4 (&acc)[NTL], Ops16<NTL>& P, uint32_t last) {
  load_a16(Ap, 0, P.a, last);
  pingpong_peeled<Ops16<NTL>>(
      nchunks, P,
      [&](uint32_t ch, Ops16<NTL>& o) {
        load_a16(Ap, ch * kCG, o.a, last);
#pragma unroll
        for (int t = 0; t < NTL; ++t) load_b16(Bt[t], ch * kCG, o.b[t]);
      },
      [&](uint32_t, const Ops16<NTL>& o) { mfma16_chunk<NTL>(o, acc); });
}

template <int NTL>
__device__ __forceinline__ void mfma16_gemm(const float* Ap, uint32_t nchunks, const float* const (&Bt)[NTL],
                                            floatx4 (&acc)[NTL], uint32_t last) {
  Ops16<NTL> P;
#pragma unroll
  for (int t = 0; t < NTL; ++t) load_b16(Bt[t], 0, P.b[t]);
  mfma16_gemm_pre<NTL>(Ap, nchunks, Bt, acc, P, last);
}

// Chunks [c0, c1) of a product for RT row tiles with one buffer: for what a shape has beyond the products its kernel is tuned
// for, where the registers of a second buffer would cost those.
template <int RT, int NTL, class Groups>
__device__ __forceinline__ void mfma16_lean_rows(const float* Ap, uint32_t rs, uint32_t c0, uint32_t c1, const float* const (&Bt)[NTL],
                                                 floatx4 (&acc)[RT][NTL], uint32_t lane, Groups ng, uint32_t last = kNoLimit) {
#pragma unroll 1
  for (uint32_t ch = c0; ch < c1; ++ch) {
    float4 b[NTL][kCG];
#pragma unroll
    for (int t = 0; t < NTL; ++t) load_b16(Bt[t], ch * kCG, b[t], lane);
    mfma16_chunk_rows<RT, NTL>(Ap, rs, ch * kCG, b, acc, ng(ch), last);
  }
}

// All weight chunks of a short product at once: for K of at most MAXC chunks the whole B operand of
// NTL column tiles is requested in one go (MAXC * NTL * 16 registers), typically ahead of the barrier
// that completes A, and the products then run as the chunks arrive -- one memory latency per product
// instead of one per chunk.  For workgroups that run alone on a CU and cannot hide latencies.
template <int NTL, int MAXC>
struct Upfront16 {
  float4 b[MAXC][NTL][kCG];
  // requests are unconditional: chunks past the end repeat the last one and are never multiplied
  __device__ __forceinline__ void request(const float* const (&Bt)[NTL], uint32_t nchunks) { request(Bt, nchunks, threadIdx.x & 63u); }
  __device__ __forceinline__ void request(const float* const (&Bt)[NTL], uint32_t nchunks, uint32_t lane) {
#pragma unroll
    for (int ch = 0; ch < MAXC; ++ch) {
      const uint32_t c = (uint32_t)ch < nchunks ? (uint32_t)ch : nchunks - 1u;
#pragma unroll
      for (int t = 0; t < NTL; ++t) load_b16(Bt[t], c * kCG, b[ch][t], lane);
    }
  }
  __device__ __forceinline__ void multiply(const float* Ap, uint32_t nchunks, floatx4 (&acc)[NTL], uint32_t last) {
#pragma unroll
    for (int ch = 0; ch < MAXC; ++ch) {
      if ((uint32_t)ch < nchunks) {                  // wave-uniform; only LDS reads and products inside
        float4 a[kCG];
        load_a16(Ap, ch * kCG, a, last);
        mfma16_chunk<NTL>(a, b[ch], acc);
      }
    }
  }
  // ... for RT row tiles, also where K has more chunks than were requested; ng(ch): groups of chunk ch that count
  template <int RT, class Groups>
  __device__ __forceinline__ void multiply_rows(const float* Ap, uint32_t rs, uint32_t nchunks, const float* const (&Bt)[NTL],
                                                floatx4 (&acc)[RT][NTL], uint32_t lane, Groups ng, uint32_t last = kNoLimit) {
#pragma unroll
    for (int ch = 0; ch < MAXC; ++ch)
      if ((uint32_t)ch < nchunks) mfma16_chunk_rows<RT, NTL>(Ap, rs, ch * kCG, b[ch], acc, ng((uint32_t)ch), last);
    mfma16_lean_rows<RT, NTL>(Ap, rs, MAXC, nchunks, Bt, acc, lane, ng, last);
  }
};

}  // namespace stgn
