// Temporal-attention layer for a list of target rows (paper Eq. attn_detail; Sec. 3.3 "Stage 4:
// Incremental Embedding Generation", exact recomputation of the affected rows; Sec. 3.6 "Parallel
// Batch Processing", one batched kernel over the affected set), one fused kernel per layer.
//
// Keys and values are linear in z_j = [h_{u_j} | e_j | phi(t_v - t_j)].  Their node and edge terms are
// cached rows (per node / per edge, [keys | values], see LayerDev); the time term is re-associated so
// that its dense products run over rows instead of (row, neighbour) pairs:
//     score_{h,j} = q_h . (kn_{u_j} + ke_j)_h + qt_h . phi_j ,     qt_h = W_K,h[time] q_h      (q carries 1/sqrt(dk))
//     o_h         = sum_j a_{h,j} (vn_{u_j} + ve_j)_h + pb_h W_V,h[time] ,   pb_h = sum_j a_{h,j} phi_j
// Edge features of at most one 64-float slot are not cached at all (ES variants): the raw row rides with the
// time encoding, z_j = [phi_j | e_j] in place of phi_j and W[time | edge] in place of W[time] above, and the
// cached rows hold the node terms alone.
// A workgroup of eight waves (four: rows of one slot, delta mode) owns 16 target rows, or 32 of a long list, and runs its phases without
// leaving the CU:
//   1. q  = h_v W_Q(node block) + phi(0) W_Q(time block)                           (MFMA 16x16x4)
//   2. qt_h = q_h W_K,h[time]^T                                                     (MFMA)
//   3. gather the cached rows of the ring entries, time encodings, scores, softmax, weighted sums;
//      a row is served by one 16-lane group per key slot, lane x float4               (HBM / vector ALU)
//   4. o_h += pb_h W_V,h[time]                                                       (MFMA)
//   5. h_v' = [o_1 | .. | o_H] W_O + b_O, written into the layer cache               (MFMA)
//   6. unless this is the last layer: the row's own cached keys|values for the next layer,
//      h_v' [W_K | W_V](node rows of layer l + 1)                                     (MFMA)
// Weights stream from L2 (group-major packing, see mfma16.h), each phase's requested ahead of its barrier; several
// workgroups per CU overlap one's gather with another's products.
//
// The products of phases 1, 2, 4, 5 and 6 are fp32 matrix instructions, which keep the matrix pipes busy for 26 to 43 % of
// a launch.  Operands split into two f16 under one power-of-two scale per row and per matrix took a fifth of those cycles
// and 12 to 24 % off a launch, but an f16 pair holds 22 bits, and those only within 2^27 of the scale's bound: a large
// feature with small weights in a row of ordinary ones cost its other columns their bits (queries 4e-5 off with one
// feature of 1.7e9).  So the operands stay in 32 bits.  Layer launches, with a 16-lane group per row and with one per key
// slot (tiles of sixteen rows; for tiles of 32 see layer32_kernel): 1,000,000 nodes, d_edge 100, 1,082 -> 1,003 us and (query
// cache) 1,052 -> 924; 1,300,000 nodes, raw edge rows, k = 20, 1,048 -> 952; 100,000 nodes, d_edge 172, 190 -> 180 and 204 ->
// 188; a rebuild of 200,000 nodes 662 + 429 -> 585 + 396.  Whole tables lie 1e-7 to 2.9e-7 (2-norm) and up to 2.6e-6 of the
// root mean square (largest) off 64-bit results.
#pragma once
#include <algorithm>
#include <mutex>
#include <type_traits>
#include "stgn_internal.h"
#include "mfma16.h"

namespace stgn {

namespace layer_impl {

constexpr uint32_t kTM = 16;   // rows of a row tile
constexpr uint32_t kFixedLds = 3072;   // bytes allowed for the kernels' LDS beside the tiles

template <int CTRL>
__device__ inline float dpp_mov(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}

// sum over each 16-lane row; every lane of a row receives its row's sum
__device__ inline float row16_sum(float x) {
  x += dpp_mov<0xB1>(x);    // quad_perm [1,0,3,2]
  x += dpp_mov<0x4E>(x);    // quad_perm [2,3,0,1]
  x += dpp_mov<0x141>(x);   // row_half_mirror
  x += dpp_mov<0x140>(x);   // row_mirror
  return x;
}

// 1 / x to about half a unit in the last place, 0 for 0 (x >= 0)
__device__ inline float reciprocal(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return x > 0.0f ? fmaf(fmaf(-x, r, 1.0f), r, r) : 0.0f;
}

// cos(2 pi frac(x)) with the argument reduced in fp64: timestamps reach 1e7 and beyond
__device__ inline float cos_rev(double x) {
  const double f = __builtin_amdgcn_fract(x);
  return __builtin_amdgcn_cosf((float)f);
}

__device__ inline float dot4(const float4 a, const float4 b, float acc) {
  acc = fmaf(a.x, b.x, acc);
  acc = fmaf(a.y, b.y, acc);
  acc = fmaf(a.z, b.z, acc);
  return fmaf(a.w, b.w, acc);
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): register arrays indexed by constants
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

struct LayerLds {
  uint32_t ldx, ldq, ldz;        // strides (floats) of the input tile, the Q / H' tile and the qt / pb tile
  uint32_t wx;                   // floats of an input row that are written and read
  uint32_t off_x, off_q, off_z, off_r, off_sc, total;
};

// Every stride is 4 (mod 8) floats: rows stay 16-byte aligned and the 16 rows of an operand read
// fall into distinct banks.  ks = key slots (heads * slots per head), nz = slots of z = [phi | raw edge row].
//
// Sixteen rows: the input tile and the cached part of the head outputs share storage.  Thirty-two: both move in with others, so
// that two workgroups of the widest common shapes fit a CU (two slots, two heads, two time slots, raw edge rows, k = 20: 79 KB,
// where storage of its own for each makes 94).  The cached part of the head outputs lies where q was and is completed in place,
// and a row's input lies behind the columns of its output row in the row's share of the qt / pb tile.
__host__ __device__ constexpr LayerLds layer_lds(uint32_t d_in, uint32_t d_emb, uint32_t heads, uint32_t ks, uint32_t nz, uint32_t k, bool delta, uint32_t tm) {
  LayerLds l{};
  const uint32_t wx = round_up(d_in, kGrpK), wo = kSlot * ks, wh = round_up(d_emb, kChunkK);
  l.ldq = wo + 4;                                 // q in the padded-head layout, later the head outputs
  l.ldz = heads * kSlot * nz + 4;
  if (tm == 16) {
    l.ldx = (wx > wo ? wx : wo) + 4;
    l.wx = l.ldx - 4;
    l.off_x = 0;
    l.off_q = tm * l.ldx;
    l.off_z = l.off_q + tm * l.ldq;
  } else {
    if (l.ldz < wh + wx + 4) l.ldz = wh + wx + 4;
    l.ldx = l.ldz;
    l.wx = wx;
    l.off_q = 0;
    l.off_z = tm * l.ldq;
    l.off_x = l.off_z + wh;
  }
  l.off_r = l.off_z + tm * l.ldz;
  l.off_sc = l.off_r + tm * k * 4;                // the ring records of the tile's rows, 16 bytes each
  l.total = l.off_sc + (delta ? tm * k * heads : 0u);        // delta mode: the scores of a row's entries until its weights are known
  return l;
}

// Everything the kernel needs, and nothing else (keeps the scalar register file uncrowded).
struct LayerArgs {
  const float* Hin; float* Hout;
  const float* KVn; const float* KVe;              // cached key|value rows of the input table's nodes / of the edges
                                                   // (ES variants: KVe holds the raw feature rows, one slot each)
  float* KVout;                                    // the next layer's node table (null for the last layer)
  // root-node inference (read by the ROOTS variants only): list row r is the source (r even) or destination (r odd) of edge
  // r / 2, queried at the edge's time instead of the node's last-interaction time; an id past `nodes` is a dead
  // row.  The rows are not stored: their tile holds both ends of its eight edges, and the link score
  // y = h_u . head[0 : d) + h_v . head[d : 2d) + head[2d] leaves the kernel in their place (NaN with a dead end).
  // One launch for what took three (roots listed, rows stored, rows read back by the head): 4,000 candidates on
  // 100,000 nodes 35.1 -> 29.9 us, 28.1 with variants of their own (ROOTS), 25.2 with a lane group per key slot.
  const uint32_t *root_src, *root_dst; const double* root_ts; uint32_t nodes;
  const float* head; float* scores;
  double window;                                   // ring entries older than the query time minus this are ignored (+inf: none)
  const RingEntry* ring; const uint32_t* deg; const double* t_last;
  const double* om_rev; const double* ph_rev;
  Ctrl* ctrl;
  uint32_t* tile_next;                             // streamed exact launches: tiles handed out beyond the first one of every workgroup (zero before the launch)
  uint64_t* gathered_slots;                        // statistic: ring entries gathered, one plain counter per workgroup index
  const float *WQ, *cQ, *WKT, *WV, *WO, *bO, *WKVnext;   // matrices group-major (mfma16.h)
  uint32_t ld_in, ld_out, ld_kv, ld_kve, hs;       // hs: floats of a head's keys in a cached row (values are heads hs further on); ld_kve = 0 without edge features (every edge reads one zero row)
  uint32_t k, d_in, d_emb, dk, d_time, d_edge;
  uint32_t k_inv;                                  // (2^32 - 1) / k
  // query cache (null: off): this layer's cached q | qt rows, [node][64 (KS + H NZ)], and per tile of the row list whether
  // every row's input row is unchanged (then q and qt are read back, not projected); a launch that must recompute everything
  // takes the variant without the cache, which still refreshes QC.  Link scores read every root's row back: nothing changed.
  float* QC; const uint8_t* tile_clean;
  // delta mode (read by the delta variant only): the batch's dirty flags and the highest flag whose owner's
  // input row of this layer changed (a row at or below it, or an endpoint, is recomputed exactly; an entry whose
  // neighbour is at or below it is a changed entry); the attention cache of this layer; the drift estimator
  const uint8_t* flags;
  uint32_t thr_in, force_exact, is_final;
  float gamma;
  float *ac_S, *ac_P, *ac_ZM, *ac_W, *ac_V;
  DriftCtl* drift; float* dsum; uint32_t* dlast; uint8_t* dseen;
};

// One 16-lane group's share of the cached rows of JC ring entries, one float4 per lane and piece: the neighbour's key slot
// and value slot, the edge's likewise (ES: the edge's raw feature row, one slot, instead), and the entry's time.
template <int JC, int ES>
struct GatherBuf {
  float4 nk[JC], nv[JC];
  float4 e[JC][ES ? 1 : 2];
  double t[JC];
};

// exchanges between the 16-lane groups of a wave: {groups 0 and 2, groups 1 and 3} of x, each in both groups of its pair;
// {lanes 0 - 31, lanes 32 - 63} of x, each in both halves
struct Two { float lo, hi; };
__device__ inline Two both_of_pair(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  return {__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1])};
}
__device__ inline Two both_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  return {__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1])};
}

// what the compiler may not move across a wave's own LDS traffic (the LDS serves one wave's requests in order)
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Waves of a workgroup.  Rows of two and four key slots: eight waves of at most 128 registers, two workgroups per CU;
// rows of one slot and the delta mode: four.  What bounds the kernel is the latency of a tile's dependent phases, so what
// counts is waves in flight and work per wave.  With one 16-lane group per row (all slots of all heads in one lane) a wave
// needed 240 registers, eight waves fitted a CU, and the time parameters and qt went through LDS once per entry; with
// a group per slot it needs 88 - 128, sixteen fit, and the entry loop reads nothing from LDS but the ring
// record.  Layer launches by this alone: 100,000 nodes, d_edge 172, 197 -> 173 us; 1,000,000 nodes, d_edge 100,
// 1,087 -> 971 and (query cache) 1,054 -> 1,012; 1,300,000 nodes, raw edge rows, k = 20, 1,053 -> 973; four
// heads of 32, 20,000 nodes, 110 -> 75; 10,000 nodes, one tile per workgroup, 33 -> 31.
__host__ __device__ constexpr int layer_waves(int ks, bool delta) { return delta || ks == 1 ? 4 : 8; }

// How a workgroup's tiles are chosen: in a fixed order, by the counter, by the one or the other as the list is short or long, or
// in a rotating order (see `advance`).  A short list: at most kShortTiles tiles of sixteen rows for every workgroup.
enum { kFixed, kCounted, kByLength, kRotated };
constexpr uint32_t kShortTiles = 4;

// The kernel's own LDS, in front of the tiles: one block, whatever bodies a kernel holds (a body's own arrays would lie there
// once for every body, the compiler does not overlay them).  kFixedLds is what the launches allow for it.
template <int NT, int NW, uint32_t TM>
struct FixedLds {
  uint32_t node[2][TM], sum[NW], next[2];
  __attribute__((aligned(16))) double om[NT * kSlot], ph[NT * kSlot];
};

// KS key slots in total (heads x slots per head), NT time slots; JC ring entries fetched together.
// ES = 1: raw edge rows.  The vector z_j = [phi(dt_j) | f_j] of NZ = NT + 1 slots takes the place of phi(dt_j)
// in the re-associated time products (scores: (W_K,h[time | edge] q_h) . z_j; values: (sum_j a_j z_j)
// W_V,h[time | edge]), and the cached rows hold the node parts alone.
// DELTA: the approximate mode of Sec. 3.3 "Stage 4" (attention cache, delta update of changed entries).
// QCACHE: rows may read q and qt back from the query cache.
// ROOTS: root-node inference (LayerArgs::root_src and on).  A variant of its own and not a test at run time: the
// places that differ would cost every streamed launch registers.
// RT: row tiles of a workgroup.
template <int KS, int NT, int ES, int H, int JC, bool DELTA, bool QCACHE, bool ROOTS, int RT, int ORDER, class Fixed>
__device__ __forceinline__
void layer_body(const LayerArgs& a, const uint32_t* __restrict__ rows, const uint32_t n, Fixed& fixed) {
  constexpr uint32_t TM = kTM * RT;           // rows of a workgroup
  extern __shared__ __align__(16) float lds[];
  constexpr int NW = layer_waves(KS, DELTA);  // waves
  constexpr uint32_t TH = 64u * NW;           // threads
  constexpr int NTL = 8 / NW;                 // column tiles a wave multiplies together in the dense phases
  constexpr int RPW = (int)TM / NW;          // rows a wave serves
  constexpr uint32_t LS = 64u / RPW;          // lanes per row while the rows are staged
  constexpr int NI = RPW / 2;                 // ring slots and input quads per lane that are fetched a tile ahead
  constexpr int GPR = DELTA ? 1 : KS;         // 16-lane groups per row in phase 3: one per key slot
  constexpr int RPP = 4 / GPR;                // rows a wave works on at a time there
  constexpr int PASSES = RPW / RPP;
  auto& s_node = fixed.node;
  auto& s_sum = fixed.sum;
  auto& s_next = fixed.next;
  auto& s_om = fixed.om;
  auto& s_ph = fixed.ph;
  static_assert(KS % H == 0, "whole slots per head");
  static_assert(!(DELTA && ES), "the delta mode keeps projected edge rows");
  static_assert(!(DELTA && ROOTS), "root rows are computed exactly");
  constexpr int SH = KS / H;                  // slots per head
  constexpr int NZ = NT + ES;                 // slots of z
  constexpr uint32_t Ztp = NZ * kSlot;        // floats of one head's qt / pb vector
  // (a batch that failed validation leaves every per-layer count at zero: nothing to test here, and the
  // control block's batch fields may already belong to the next batch, whose front part runs concurrently)
  const uint32_t ntiles = (n + TM - 1) / TM;
  if (blockIdx.x >= ntiles) return;           // (a workgroup's first tile is the one of its index)
  // The lane index and everything derived from it are derived anew at the top of every tile and of its phases, from
  // the lane counter and behind the compiler's back: otherwise it hoists dozens of loop-invariant address registers out
  // of the persistent tile loop and keeps them alive (or spilled) across all phases.
  uint32_t lane, sub, grp;
  // wave index, made provably uniform so that tile indices and weight addresses stay in scalar registers
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t k = a.k, dk = a.dk;
  const uint32_t c_in = chunks_of(a.d_in), c_de = chunks_of(a.d_emb);                                     // chunks of K
  const uint32_t ntd = round_up(a.d_emb, 16) >> 4, ntk = round_up(dk, 16) >> 4;                           // column tiles
  constexpr uint32_t ntz = Ztp >> 4;                                                                       // tiles of a qt vector
  const uint32_t nzt_t = (a.d_time + 15u) >> 4, nzt = nzt_t + (ES ? (a.d_edge + 15u) >> 4 : 0u);           // ... that hold valid columns
  const LayerLds ll = layer_lds(a.d_in, a.d_emb, H, KS, NZ, k, DELTA, TM);
  float* Xs = lds + ll.off_x;                 // input rows (phase 1)
  float* Qs = lds + ll.off_q;                 // q (phases 1-3), then the head outputs (phases 4-5)
  float* As = RT == 1 ? Xs : Qs;              // the cached-value part of the head outputs (phases 3-4)
  const uint32_t ldas = RT == 1 ? ll.ldx : ll.ldq;
  float* Zs = lds + ll.off_z;                 // qt (phases 2-3), then pb (phases 3-4), then the output rows (phases 5-6)
  RingEntry* Rs = reinterpret_cast<RingEntry*>(__builtin_assume_aligned(lds + ll.off_r, 16));   // [row][j], j = 0 the most recent entry
  using ZBuf = GatherBuf<JC, ES>;

  // time-encoding parameters (omega, phase in revolutions) live in LDS, zero past d_time
  for (uint32_t q = threadIdx.x; q < NT * kSlot; q += TH) {
    s_om[q] = q < a.d_time ? a.om_rev[q] : 0.0;
    s_ph[q] = q < a.d_time ? a.ph_rev[q] : 0.0;
  }
  // operand padding (columns nobody writes) must be finite: clear the tiles once
  for (uint32_t x = threadIdx.x; x < ll.off_r; x += TH) lds[x] = 0.0f;
  uint32_t gathered = 0;                      // ring entries of this wave's rows
  double drift_sum = 0.0;                     // delta mode: this wave's share of the drift estimator's sum and member count
  uint32_t drift_new = 0;
  // Arguments that a phase needs once a tile: fetched from the argument block there (a scalar load that the phase's products
  // cover), not held, or spilled, through the tile loop.
  typedef const __attribute__((address_space(4))) LayerArgs* ArgBlock;
  auto args = [&]() {
    ArgBlock p = (ArgBlock)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
  };
  auto derive_lane = [&]() {
    uint32_t x;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
    lane = x; sub = x & 15u; grp = x >> 4;
  };
  derive_lane();

  // groups of a chunk that count, where a chunk is a slot: of a head's columns, of z
  // (link scores, a tile or two per workgroup: all of them, the arguments' way to the scalar registers takes longer, 25.7 -> 26.2 us;
  // delta mode with one slot, whose 168 registers are all in use: all of them, the branches cost sixteen spilled ones)
  auto groups_used = [&](auto used, uint32_t g0) {
    if constexpr (ROOTS || (DELTA && KS == 1)) return AllGroups{};
    else return groups_in((used(args()) + 15u) >> 4, g0);
  };
  auto groups_head = [&](uint32_t slot) { return groups_used([](ArgBlock p) { return p->dk; }, (SH == 1 ? 0u : slot % SH) * kCG); };
  auto groups4 = [&](uint32_t slot) {
    if constexpr (ES) {                                       // (two closures without captures: a captured flag went through scratch memory)
      if (slot == NT) return groups_used([](ArgBlock p) { return p->d_edge; }, 0u);
    }
    return groups_used([](ArgBlock p) { return p->d_time; }, slot * kCG);
  };

  // ---- phase-2 work units: (head, NTL valid qt column tiles); wave w owns units w, w + NW, ...
  // Lane i of `udesc` holds the description of the wave's i-th unit (head, first tile, second tile, whether there is a
  // second one), worked out once; inside the tile loop a unit costs one cross-lane read.  Lanes past the last unit describe the
  // first again (an idle wave's: head 0, tile 0).
  const uint32_t npr = (nzt + NTL - 1u) / NTL, nunits2 = H * npr;
  const uint32_t nu2 = wave < nunits2 ? (nunits2 - wave + (NW - 1u)) / NW : 0u;     // units of this wave
  struct Unit2 { uint32_t h, t0, t1; bool two; };
  uint32_t udesc = 0;
  auto describe2 = [&]() {
    // the i-th valid tile: time tiles first, then (raw edge rows) the tiles of slot NT
    auto vt = [&](uint32_t i) { return i < nzt_t ? i : 4u * NT + (i - nzt_t); };
    const uint32_t x = wave + NW * (lane < nu2 ? lane : 0u);
    const uint32_t h = (H > 1 && x >= npr ? 1u : 0u) + (H > 2 && x >= 2u * npr ? 1u : 0u) + (H > 2 && x >= 3u * npr ? 1u : 0u), i0 = NTL * (x - h * npr);
    const uint32_t two = NTL == 2 && i0 + 1u < nzt ? 1u : 0u;
    udesc = nu2 ? h | (vt(i0) << 8) | (vt(i0 + two) << 16) | (two << 24) : 0u;
  };
  describe2();
  auto decode2 = [&](uint32_t i) {
    const uint32_t dsc = (uint32_t)__builtin_amdgcn_readlane((int)udesc, (int)i);
    Unit2 u;
    u.h = dsc & 0xFFu; u.t0 = (dsc >> 8) & 0xFFu; u.t1 = (dsc >> 16) & 0xFFu; u.two = (dsc >> 24) != 0u;
    return u;
  };
  auto wkt = [&](uint32_t h, uint32_t t) { return a.WKT + (size_t)(h * ntz + t) * SH * kChunkFloats; };
  auto request2 = [&](const Unit2& u, float4 (&b)[NTL][kCG]) {
    load_b16(wkt(u.h, u.t0), 0, b[0], lane);
    if constexpr (NTL == 2) load_b16(wkt(u.h, u.t1), 0, b[1], lane);
  };
  auto store2 = [&](const Unit2& u, const floatx4 (&acc)[RT][NTL]) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float* zp = Zs + u.h * Ztp + (kTM * rt + m16_row(lane, 0)) * ll.ldz + m16_col(lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) zp[u.t0 * 16 + r * ll.ldz] = acc[rt][0][r];
      if constexpr (NTL == 2) {
        if (u.two) {
#pragma unroll
          for (int r = 0; r < 4; ++r) zp[u.t1 * 16 + r * ll.ldz] = acc[rt][1][r];
        }
      }
    }
  };
  // ---- phase-4 work units: (head, NTL head-output column tiles)
  constexpr int N4 = KS == 1 ? 1 : NTL;       // (one slot: at most as many tiles as waves)
  const uint32_t np4 = (ntk + N4 - 1u) / N4, nunits4 = H * np4;
  // ---- phases 1 and 5: column tiles nt (and nt + 4) of the d_emb outputs form a unit
  // column tile of a product's t-th operand: past the end the unit's first tile again (its result is not stored)
  auto tile_b = [&](const float* W, uint32_t nt, int t, uint32_t limit, uint32_t chunks) {
    const uint32_t x = nt + NW * t < limit ? nt + NW * t : nt;
    return W + (size_t)x * chunks * kChunkFloats;
  };
  __syncthreads();

  // ---- staging of a tile, one tile ahead, every wave its own rows: lane -> (row lane / LS of the wave's, item lane % LS).
  // While a tile is worked on, the next one is made ready in steps, each behind requests that are waited for earlier
  // (loads return in order): stage A requests the rows' ids at the top of the tile; stage B, behind the entry loop and
  // the weights of phases 4 and 5, the lane's share of the rows' ring slots, degrees, query times and own input rows;
  // `commit`, between phases 4 and 5, moves those into LDS (the ring records and input tile of this tile are no longer
  // needed); and where q and qt are read back, they and the first gather are requested right behind it, so that phase 5
  // hides them.  All but a workgroup's first tile start without waiting for memory.  Shapes whose share does not
  // fit the registers fetch it inside `commit` instead.
  const uint32_t qpr = round_up(a.d_in, kGrpK) >> 2;          // 16-byte quads per staged input row
  const bool pf_ok = QCACHE || (k <= LS * NI && qpr <= LS * NI);   // (the query cache is kept for such shapes only)
  RingEntry p_ring[NI];
  uint32_t p_deg = 0;
  double p_tl = 0.0;
  float4 p_x[NI];                                             // own input rows (one address for all while q | qt are read back)
  constexpr uint32_t kQC = kSlot * (KS + H * NZ);             // floats per cached q | qt row
  uint32_t p_row = 0xFFFFFFFFu, p_clean = 0u;
  double p_tqn = 0.0;
  auto stage_a = [&](uint32_t t) {
    const uint32_t r = t * TM + wave * RPW + lane / LS;
    const uint32_t rc = r < n ? r : n - 1u;                   // (past the list: its last row, dropped in stage B)
    if constexpr (ROOTS) {
      p_row = ((rc & 1u) ? a.root_dst : a.root_src)[rc >> 1];
      p_tqn = a.root_ts[rc >> 1];
    } else {
      p_row = rows ? rows[rc] : rc;
    }
    if constexpr (QCACHE && !ROOTS) {                         // (a byte of a word that no lane has to hold: scalar)
      const uint32_t tc = t < ntiles ? t : ntiles - 1u;
      typedef const __attribute__((address_space(4))) uint32_t* ScalarWords;
      if constexpr (RT == 1) {
        p_clean = (((ScalarWords)(uintptr_t)a.tile_clean)[tc >> 2] >> (8u * (tc & 3u))) & 0xFFu;
      } else {                                                // (a byte per 16 rows; one past the list's end may be either)
        p_clean = ((((ScalarWords)(uintptr_t)a.tile_clean)[tc >> 1] >> (16u * (tc & 1u))) & 0x0101u) == 0x0101u ? 1u : 0u;
      }
    }
  };
  // (requests without conditions: behind a branch the compiler would wait for more than it needs to)
  auto stage_b = [&](uint32_t t) {
    const bool cl = QCACHE && (ROOTS || p_clean != 0u);
    const uint32_t it = lane % LS;
    const ArgBlock ab = args();
    if (t * TM + wave * RPW + lane / LS >= n || (ROOTS && p_row >= a.nodes)) p_row = 0xFFFFFFFFu;
    const size_t nn = p_row != 0xFFFFFFFFu ? p_row : 0u;
    p_deg = ab->deg[nn];
    p_tl = ROOTS ? p_tqn : ab->t_last[nn];
#pragma unroll
    for (int e = 0; e < NI; ++e) {
      const uint32_t sl = it + LS * e;
      p_ring[e] = ab->ring[nn * k + (sl < k ? sl : 0u)];
    }
#pragma unroll
    for (int e = 0; e < NI; ++e) {
      const uint32_t q = it + LS * e;
      // columns past d_in are row padding of the table (zero)
      p_x[e] = *reinterpret_cast<const float4*>(ab->Hin + (cl ? 0u : nn * ab->ld_in + 4u * (q < qpr ? q : 0u)));
    }
  };
  // the staged tile's rows: id, entry count and query time of this lane's row
  uint32_t node_s = 0xFFFFFFFFu, cnt_s = 0u;
  double tq_s = 0.0;
  // Input rows into Xs.  Columns up to the end of the last chunk are written (zero past d_in): what else lies there need
  // not be a number.
  const uint32_t qpz = min(kChunkK / 4u * c_in, ll.wx >> 2);
  auto place_x = [&](uint32_t q, float4 v) {
    if (q >= qpr || node_s == 0xFFFFFFFFu) v = make_float4(0.f, 0.f, 0.f, 0.f);
    *reinterpret_cast<float4*>(Xs + (wave * RPW + lane / LS) * ll.ldx + 4u * q) = v;
  };
  auto commit_x = [&](bool staged) {
    const uint32_t it = lane % LS;
    if (staged) {
#pragma unroll
      for (int e = 0; e < NI; ++e) if (it + LS * e < qpz) place_x(it + LS * e, p_x[e]);
    } else {
      const float* xr = a.Hin + (size_t)(node_s != 0xFFFFFFFFu ? node_s : 0u) * a.ld_in;
      for (uint32_t q = it; q < qpz; q += LS) place_x(q, *reinterpret_cast<const float4*>(xr + 4u * (q < qpr ? q : 0u)));
    }
  };
  auto commit = [&](uint32_t round) {
    const uint32_t local = wave * RPW + lane / LS, it = lane % LS;
    node_s = p_row;
    const bool live = node_s != 0xFFFFFFFFu;
    const size_t nn = live ? node_s : 0u;
    const uint32_t dg0 = pf_ok ? p_deg : a.deg[nn];
    tq_s = pf_ok || ROOTS ? p_tl : a.t_last[nn];
    const uint32_t dg = live ? dg0 : 0u;
    cnt_s = dg < k ? dg : k;
    // (dg - 1) mod k.  A division here, like one anywhere in the tile loop, is a reciprocal that the compiler keeps in a vector
    // register through the whole loop and spills; its reload then waited for every request in flight.
    uint32_t newest = dg ? dg - 1u : 0u;
    newest -= __umulhi(newest, args()->k_inv) * k;            // (the quotient is exact or one short)
    newest = newest >= k ? newest - k : newest;
    // the record of adjacency position p sits in ring slot p mod k; with the row's degree known, slot
    // sl holds the j-th most recent entry, j = (newest - sl) mod k; places past the row's entry count
    // name node 0 / edge 0, whose cached rows are there to be gathered (they may be NaN: such places are left out of every sum)
    auto place_ring = [&](uint32_t sl, RingEntry e) {
      const uint32_t j = newest >= sl ? newest - sl : newest + k - sl;
      if (j >= cnt_s) { e.nbr = 0u; e.eid = 0u; e.t = 0.0; }
      Rs[local * k + j] = e;
    };
    if (it == 0u) s_node[round & 1u][local] = node_s;
    if (pf_ok) {
#pragma unroll
      for (int e = 0; e < NI; ++e) if (it + LS * e < k) place_ring(it + LS * e, p_ring[e]);
    } else {
      for (uint32_t sl = it; sl < k; sl += LS) place_ring(sl, a.ring[nn * k + sl]);
    }
    wave_lds_fence();
#pragma unroll
    for (int r = 0; r < RPW; ++r) gathered += (uint32_t)__builtin_amdgcn_readlane((int)cnt_s, r * (int)LS);
  };

  // Tiles of a workgroup.  The first one is that of its index.  On long lists further ones are handed out by a counter, asked a
  // tile ahead: workgroups that find their place late (the next batch's front part holds CUs when a launch starts) then take
  // fewer tiles, where with a fixed share they hold up the launch.  On lists of up to four tiles a workgroup a counter only
  // adds its own latency (10,000 nodes, a tile each: 122 -> 128 us a batch; 20,000 nodes, two or three: 217 -> 221): rounds
  // go through the workgroups forwards and backwards in turn, since the list may be regrouped by entry count in windows of
  // 4,096 rows (long rows first) and a fixed position would hand the same workgroups every long tile, and the last round
  // forwards, since the workgroups of low index start first (backwards: 119 -> 128 and 188 -> 208 us).  The other modes
  // give workgroup b the tile i G + (b + 37 i) mod G in round i (G workgroups), to the same end.
  const uint32_t G = gridDim.x, step37 = 37u % G;
  uint32_t tile_base = 0, tile_pos = blockIdx.x, next_tile = blockIdx.x, taken = 0;
  auto counted = [&]() { return ORDER == kCounted || (ORDER == kByLength && ntiles > kShortTiles * G); };
  auto take = [&]() {
    taken = 0u;                                               // (not carried from tile to tile)
    if (ORDER != kRotated && counted() && wave == 0u && lane == 0u)
      taken = G + __hip_atomic_fetch_add(args()->tile_next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto publish = [&](uint32_t round) { if (ORDER != kRotated && counted() && wave == 0u && lane == 0u) s_next[round & 1u] = taken; };
  auto advance = [&](uint32_t round) {                        // next_tile: this workgroup's tile of the next round
    if constexpr (ORDER != kRotated) {
      if (counted()) next_tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_next[round & 1u]);
      else {
        const uint32_t last = (ntiles >= G) + (ntiles >= 2u * G) + (ntiles >= 3u * G);   // the round that is not full
        next_tile = (round + 1u) * G + (((last - round) & 1u) ? blockIdx.x : G - 1u - blockIdx.x);
      }
    } else {
      tile_base += G;
      tile_pos += step37;
      if (tile_pos >= G) tile_pos -= G;
      next_tile = tile_base + tile_pos;
    }
  };

  // ---- phase 3's rows: pass p works on rows p RPP .. p RPP + RPP - 1 of the wave's, GPR groups of 16 lanes each,
  // group g on key slot g.  With one pass a lane's row is the one it staged, else the pass has one row.
  constexpr bool LAZY = RT > 1;                               // a pass's query and first gather are requested when the pass before is over
  static_assert(PASSES == 1 || RPP == 1 || (RPP == 2 && PASSES == 2), "rows of a pass");
  uint32_t g = 0, head = 0, sg = 0;                           // this lane's key slot, its head and its place among the head's slots
  uint32_t kv_at = 0;                                         // ... and the lane's four keys in a cached row
  auto derive_slot = [&]() {
    g = GPR == 1 ? 0u : grp % GPR; head = g / SH; sg = g - head * SH;
    kv_at = head * a.hs + min(kSlot * sg + 4u * sub, a.hs - 4u);   // (past the head's floats: its last four; see in_head)
  };
  // Whether a lane's quad of slot s of its head lies among the head's floats.  Past them the query is zero, but the keys read
  // there are the head's last four again, not padding: one that has overflowed would make the product a NaN, where the score
  // is minus infinity and the entry has no weight.
  auto in_head = [&](uint32_t s) { return kSlot * s + 4u * sub < a.hs; };
  auto row_of = [&](int p) { return wave * RPW + (uint32_t)(p * RPP) + (RPP == 1 ? 0u : grp / GPR); };
  // the staged value of the row that this lane works on in pass p
  auto of_pass = [&](uint32_t x, int p) -> uint32_t {
    if constexpr (PASSES == 1) return x;
    else if constexpr (RPP == 1) return (uint32_t)__builtin_amdgcn_readlane((int)x, p * (int)LS);
    else {                                                    // groups {0, 0, 1, 1} in pass 0, {2, 2, 3, 3} in pass 1
      const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
      const auto q = __builtin_amdgcn_permlane32_swap((uint32_t)r[0], (uint32_t)r[1], false, false);
      return p ? (uint32_t)q[1] : (uint32_t)q[0];
    }
  };
  auto node_of = [&](int p) { return of_pass(node_s, p); };
  auto cnt_of = [&](int p) { return of_pass(cnt_s, p); };
  auto tq_of = [&](int p) {
    const uint64_t u = __builtin_bit_cast(uint64_t, tq_s);
    const uint32_t lo = of_pass((uint32_t)u, p), hi = of_pass((uint32_t)(u >> 32), p);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
  };
  auto cmax_of = [&](int p) {
    uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)cnt_s, p * RPP * (int)LS);
#pragma unroll
    for (int r = 1; r < RPP; ++r) m = max(m, (uint32_t)__builtin_amdgcn_readlane((int)cnt_s, (p * RPP + r) * (int)LS));
    return m;
  };
  auto gather_row = [&](uint32_t row, uint32_t c, ZBuf& zb) {
    const RingEntry* rrow = Rs + row * k;
#pragma unroll
    for (int jc = 0; jc < JC; ++jc) {
      const uint32_t j = c * JC + jc;
      const RingEntry e = rrow[JC == 1 || j < k ? j : k - 1u];   // (a chunk of one never runs past the longest row's entries, but for a wave without any: the record of place 0)
      // (byte addresses: one multiply-add a row)
      const float* nrow = reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.KVn + kv_at) + (uint64_t)e.nbr * (4u * a.ld_kv));
      zb.nk[jc] = *reinterpret_cast<const float4*>(nrow);
      zb.nv[jc] = *reinterpret_cast<const float4*>(nrow + H * a.hs);
      if constexpr (ES) {
        zb.e[jc][0] = *reinterpret_cast<const float4*>(a.KVe + (size_t)e.eid * kSlot + 4u * sub);
      } else {
        const float* erow = reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.KVe + kv_at) + (uint64_t)e.eid * (4u * a.ld_kve));
        zb.e[jc][0] = *reinterpret_cast<const float4*>(erow);
        zb.e[jc][1] = *reinterpret_cast<const float4*>(erow + H * a.hs);
      }
      zb.t[jc] = e.t;
    }
  };
  auto gather = [&](int p, uint32_t c, ZBuf& zb) { gather_row(row_of(p), c, zb); };
  // z slots a lane works with: all of them when a head is one slot (every head needs them all); shared out over the
  // head's slots otherwise, slot t to the lanes of key slot t mod SH
  constexpr int NZL = SH == 1 ? NZ : (NZ + SH - 1) / SH;
  constexpr int NP = LAZY ? 1 : PASSES;                       // passes whose first gather and query are held at once
  ZBuf z0[NP];                                                // the first gather
  float4 qk[NP], qt[NP][NZL];                                 // this lane's share of the row's q and qt vectors
  auto request_first = [&](auto P) { gather(decltype(P)::value, 0, z0[decltype(P)::value % NP]); };
  // the pass's q and qt from the query cache, each lane what it needs, and its first gather
  auto request_query = [&](auto P) {
    constexpr int p = decltype(P)::value;
    const uint32_t node = node_of(p);
    const float* qrow = a.QC + (size_t)(node != 0xFFFFFFFFu ? node : 0u) * kQC + 4u * sub;
    qk[p % NP] = *reinterpret_cast<const float4*>(qrow + kSlot * g);
#pragma unroll
    for (int i = 0; i < NZL; ++i) {
      const uint32_t t = SH == 1 ? (uint32_t)i : sg + SH * i;
      qt[p % NP][i] = *reinterpret_cast<const float4*>(qrow + kSlot * KS + head * Ztp + (t < NZ ? t : 0u) * kSlot);
    }
  };
  auto request_back = [&](auto P) { request_query(P); request_first(P); };
  constexpr std::integral_constant<int, 0> kPass0{};

  // Weights of phases 1 and 2: the first units' chunks, requested together.
  const uint32_t w1 = wave < ntd ? wave : 0u;                // loads are unconditional (clamped), products are not
  constexpr int C1 = KS == 1 && !DELTA ? 1 : 2;               // chunks of W_Q requested up front
  Upfront16<NTL, C1> u1;
  float c1v[NTL];                                             // this lane's c_Q of the first unit
  constexpr int U2 = SH == 1 ? 2 : 1;                         // phase 2's units requested up front
  float4 o2[U2][NTL][kCG];
  auto request12 = [&]() {
    const float* const wq = args()->WQ;
    const float* B1[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) B1[t] = tile_b(wq, w1, t, ntd, c_in);
    u1.request(B1, c_in, lane);
#pragma unroll
    for (int t = 0; t < NTL; ++t) { const uint32_t col = (w1 + NW * t) * 16 + m16_col(lane); c1v[t] = a.cQ[col < a.d_emb ? col : 0u]; }
#pragma unroll
    for (int i = 0; i < U2; ++i) request2(decode2((uint32_t)i), o2[i]);
  };

  // the first tile
  take();
  stage_a(blockIdx.x);
  stage_b(blockIdx.x);
  commit(0u);
  publish(0u);
  commit_x(pf_ok);
  derive_slot();
  if constexpr (QCACHE) request_back(kPass0);
  __syncthreads();

  // (Sixteen rows; for 32 rows see below.)  What separates a tile's uses of the LDS from the next tile's.  Ring records: a wave reads only its own rows'.  Xs holds the
  // input rows (phase 1), then the cached-value part of the head outputs (read in phase 4), and takes the next tile's
  // input rows behind the barrier in front of phase 5.  Qs holds q, then the whole head outputs (phase 5): a projecting tile has a
  // barrier ahead of its phase 1, a tile that reads q back writes Qs behind its first barrier.  Zs holds qt, pb, then the output
  // rows (phase 6, link scores): projecting tiles have two barriers ahead of their qt, and where tiles may read theirs back, a
  // tile that stored output rows there ends with one.
  // Thirty-two rows (layer_lds): Qs also takes the cached-value part and is completed in place, so every tile of a variant
  // that may read q back ends with a barrier; input rows lie behind the output row's columns of the same row of Zs, whose
  // last reader is phase 4, and phase 2 writes there behind the barrier that ends phase 1.
  const bool kv = !ROOTS && a.KVout != nullptr, rows_in_lds = ROOTS || kv;
  constexpr bool kRowsInZ = RT > 1 || H * NZ >= KS;                     // (wide heads of few time slots: Zs is narrower than a row, they take Xs)
  float* const Hs = kRowsInZ ? Zs : Xs;                       // output rows
  const uint32_t ldh = kRowsInZ ? ll.ldz : ll.ldx;
  // One tile.  CLEAN: every row of it has its q and qt in the query cache.  Two copies of the body and not tests inside
  // one: merged, the query cache's variants spilled 29 to 51 registers, and a spilled prefetch is waited for.
  auto work_tile = [&](auto CLEAN, const uint32_t tile, const uint32_t round) __attribute__((always_inline)) {
    constexpr bool clean = decltype(CLEAN)::value;
    derive_lane();
    derive_slot();
    const uint32_t* nodes_s = s_node[round & 1u];
    const uint32_t local_s = wave * RPW + lane / LS;
    const bool live_s = node_s != 0xFFFFFFFFu;
    bool ex = false;
    if constexpr (DELTA) {
      // exact recomputation for endpoints of the batch (query time and entries moved), for rows whose own
      // input row changed (every score moves), and whenever the caller asks for it
      const uint32_t fl = live_s ? a.flags[node_s] : 0u;
      ex = a.force_exact || fl == 1u || (fl != 0u && fl <= a.thr_in);
    }
    if constexpr (clean) {
      if constexpr (NP == 2) request_back(std::integral_constant<int, 1>{});
      stage_a(next_tile);                          // row ids of this workgroup's next tile
    } else {
    // ================================================================ phase 1: q = x W_Q + c_Q
    if constexpr (QCACHE) describe2();                        // (one register less through the other tiles)
    request12();
    stage_a(next_tile);
    if (!kRowsInZ && rows_in_lds && round) {                  // (the previous tile had its output rows where the input rows go)
      __syncthreads();
      commit_x(false);
    }
    __syncthreads();                                          // input rows there, the previous tile's head outputs read
    auto groups1 = [&](uint32_t ch) { return groups_used([](ArgBlock p) { return p->d_in; }, ch * kCG); };
    auto store1 = [&](uint32_t nt, const floatx4 (&acc)[RT][NTL]) {
#pragma unroll
      for (int t = 0; t < NTL; ++t) {
        const uint32_t col = (nt + NW * t) * 16 + m16_col(lane);
        if (nt + NW * t < ntd && col < a.d_emb) {
          const float cq = nt == wave ? c1v[t] : a.cQ[col];
          const uint32_t h = H == 1 ? 0u : H == 2 ? (col >= dk ? 1u : 0u) : (col >= dk ? 1u : 0u) + (col >= 2u * dk ? 1u : 0u) + (col >= 3u * dk ? 1u : 0u);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            float* qp = Qs + (kTM * rt + m16_row(lane, 0)) * ll.ldq + h * (SH * kSlot) + (col - h * dk);
#pragma unroll
            for (int r = 0; r < 4; ++r) qp[r * ll.ldq] = acc[rt][t][r] + cq;
          }
        }
      }
    };
    if (wave < ntd) {
      const float* B1[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) B1[t] = tile_b(a.WQ, w1, t, ntd, c_in);
      floatx4 acc[RT][NTL] = {};
      u1.template multiply_rows<RT>(Xs + a16_off(lane, ll.ldx), kTM * ll.ldx, c_in, B1, acc, lane, groups1, ll.wx / kGrpK - 1u);
      store1(wave, acc);
    }
    for (uint32_t nt = wave + 8; nt < ntd; nt += 8) {
      const float* Bt[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) Bt[t] = tile_b(a.WQ, nt, t, ntd, c_in);
      floatx4 acc[RT][NTL] = {};
      mfma16_lean_rows<RT, NTL>(Xs + a16_off(lane, ll.ldx), kTM * ll.ldx, 0u, c_in, Bt, acc, lane, groups1, ll.wx / kGrpK - 1u);
      store1(nt, acc);
    }
    __syncthreads();
    // ================================================================ phase 2: qt_h = q_h W_K,h[time]^T
    {
      const float* qa = Qs + a16_off(lane, ll.ldq);
      auto products2 = [&](uint32_t i, float4 (&b)[NTL][kCG]) {
        const Unit2 u = decode2(i);
        floatx4 acc[RT][NTL] = {};
        const float* qh = qa + u.h * (SH * kSlot);
        mfma16_chunk_rows<RT, NTL>(qh, kTM * ll.ldq, 0, b, acc, groups_head(0u));
        if constexpr (SH > 1) {
          const float* Bt[NTL];
          Bt[0] = wkt(u.h, u.t0);
          if constexpr (NTL == 2) Bt[1] = wkt(u.h, u.t1);
          mfma16_lean_rows<RT, NTL>(qh, kTM * ll.ldq, 1u, SH, Bt, acc, lane, groups_head);
        }
        store2(u, acc);
      };
      if constexpr (U2 == 2) {
        for (uint32_t i = 0; i < nu2; i += 2) {
          products2(i, o2[0]);
          if (i + 2 < nu2) request2(decode2(i + 2), o2[0]);
          if (i + 1 < nu2) {
            products2(i + 1, o2[1]);
            if (i + 3 < nu2) request2(decode2(i + 3), o2[1]);
          }
        }
      } else {
        for (uint32_t i = 0; i < nu2; ++i) {
          products2(i, o2[0]);
          if (i + 1 < nu2) request2(decode2(i + 1), o2[0]);
        }
      }
    }
    if constexpr (!DELTA) static_for<NP>(request_first);
    __syncthreads();
    }  // q and qt: read back, or projected
    // The time encodings are not masked per entry: a column past d_time has omega = phase = 0 and comes out as
    // cos(0) = 1.  In the scores it meets an exact zero of qt and in phase 4 one of pb: both are cleared there once
    // per row.
    // A raw edge row's own padding is zero, but qt's there is whatever an earlier tile left (phase 2 writes the tiles that
    // hold valid columns), and 0 x NaN is NaN: qt is cleared there too.
    // (the last time slot's alone: d_time > 64 (NT - 1))
    auto clear_padding = [&](float4& o, uint32_t t) {
      const uint32_t c0 = 4u * sub, end = t == NT - 1 ? a.d_time - (NT - 1) * kSlot : ES && t == NT ? a.d_edge : kSlot;
      o.x = c0 < end ? o.x : 0.0f;
      o.y = c0 + 1u < end ? o.y : 0.0f;
      o.z = c0 + 2u < end ? o.z : 0.0f;
      o.w = c0 + 3u < end ? o.w : 0.0f;
    };
    auto read_query = [&](auto P) {                           // a projected row's q and qt
          constexpr int p = decltype(P)::value;
          const uint32_t node = node_of(p), local = row_of(p);
          qk[p % NP] = *reinterpret_cast<const float4*>(Qs + local * ll.ldq + kSlot * g + 4u * sub);
          float* qrow = a.QC + (size_t)node * kQC + 4u * sub;
          const bool keep = !ROOTS && a.QC && node != 0xFFFFFFFFu;             // the rows' q | qt for later batches
          if (keep) *reinterpret_cast<float4*>(qrow + kSlot * g) = qk[p % NP];
#pragma unroll
          for (int i = 0; i < NZL; ++i) {
            // (a lane without a slot of its own reads slot 0 against zeros: that slot's padding is cleared there too)
            const uint32_t t = SH == 1 ? (uint32_t)i : sg + SH * i, tz = t < NZ ? t : 0u, at = head * Ztp + tz * kSlot;
            qt[p % NP][i] = *reinterpret_cast<const float4*>(Zs + local * ll.ldz + at + 4u * sub);
            if (SH > 1 || i >= NT - 1) clear_padding(qt[p % NP][i], tz);
            if (keep && t < NZ) *reinterpret_cast<float4*>(qrow + kSlot * KS + at) = qt[p % NP][i];
          }
    };
    if constexpr (!DELTA && !clean) static_for<NP>(read_query);
    // ================================================================ phase 3: gather + attention
    if constexpr (DELTA) {
      // ---- delta mode.  An exact row runs the same online softmax as the exact mode and leaves its attention
      // cache behind: per entry score, weight and the neighbour|edge part of the value, per row the sums S and
      // pb, the denominator and its reference score.  A delta row starts from its cached sums and visits only
      // the entries whose neighbour's input row changed: new score, denominator Z' = Z - e_old + e_new, new
      // weight e_new / Z', sums corrected by (new weight x new value) - (old weight x old value); the
      // other entries keep the weight they have (Eq. delta_embedding, "updated neighbours").
      float* Sc = lds + ll.off_sc;
      const uint32_t local = local_s, node = node_s, cnt = cnt_s, cmax = cmax_of(0);
      const double tq = tq_s;
      const RingEntry* rrow = Rs + local * k;
      const bool live = live_s;
      const uint32_t nn = live ? node : 0u;
      float* acS = a.ac_S + (size_t)nn * (kSlot * KS) + 4u * sub;
      float* acP = a.ac_P + (size_t)nn * (kSlot * NT * H) + 4u * sub;
      float* acZM = a.ac_ZM + (size_t)nn * (2 * H);
      // (first, and behind a fence of its own: a fence further down would wait for the cache reads below)
      for (uint32_t j = sub; j < cnt; j += 16)
#pragma unroll
        for (int h = 0; h < H; ++h) Sc[(local * k + j) * H + h] = -INFINITY;
      wave_lds_fence();
      float4 accv[KS], accp[H][NT];
      float mref[H], lrun[H];                                 // exact row: running reference and denominator; delta row: m and Z
#pragma unroll
      for (int s = 0; s < KS; ++s) accv[s] = ex ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<const float4*>(acS + s * kSlot);
#pragma unroll
      for (int h = 0; h < H; ++h) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
          accp[h][t] = ex ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<const float4*>(acP + (h * NT + t) * kSlot);
        mref[h] = ex ? -INFINITY : acZM[2 * h + 1];
        lrun[h] = ex ? 0.0f : acZM[2 * h];
      }
      float4 qk[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) qk[s] = *reinterpret_cast<const float4*>(Qs + local * ll.ldq + s * kSlot + 4u * sub);
      float* zq = Zs + local * ll.ldz + 4u * sub;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        float4* o = reinterpret_cast<float4*>(zq + h * Ztp + (NT - 1) * kSlot);
        float4 v = *o;
        clear_padding(v, NT - 1);
        *o = v;
      }
      uint32_t nch = 0, nvalid = 0;
      const bool any_delta = __any(!ex);                      // (exact rows take every entry: no flags needed)
      struct DBuf { float4 n[2 * KS], e[2 * KS]; uint32_t j; };
      for (uint32_t jb = 0; jb < cmax; jb += 32u) {
        // Which of the entries jb .. jb + 31 each row takes, worked out at once (lane s of a row looks at entries
        // jb + s and jb + 16 + s: their window test and the flag of their neighbour), instead of one dependent
        // flag read per entry: an exact row takes its valid entries, a delta row the valid ones whose
        // neighbour's input row changed.
        uint32_t vmask = 0, cmask = 0;
#pragma unroll
        for (uint32_t half = 0; half < 2; ++half) {
          const uint32_t jj = jb + 16u * half + sub;
          bool v = false, c = false;
          if (jj < cnt) {
            const RingEntry e = rrow[jj];
            v = tq - e.t <= a.window;
            if (any_delta) { const uint32_t fl = a.flags[e.nbr]; c = fl != 0u && fl <= a.thr_in; }
          }
          const uint64_t bv = __ballot(v), bc = __ballot(c);
          vmask |= ((uint32_t)(bv >> (16u * grp)) & 0xFFFFu) << (16u * half);
          cmask |= ((uint32_t)(bc >> (16u * grp)) & 0xFFFFu) << (16u * half);
        }
        const uint32_t amask = ex ? vmask : (vmask & cmask);
        nvalid += (uint32_t)__popc(vmask);
        if (!ex) nch += (uint32_t)__popc(amask);
        // entries some row of the wave takes, in entry order; the cached rows of the next one are in flight
        // while the current one is worked on
        const uint32_t wmask = (uint32_t)__builtin_amdgcn_readlane((int)amask, 0) | (uint32_t)__builtin_amdgcn_readlane((int)amask, 16) |
                               (uint32_t)__builtin_amdgcn_readlane((int)amask, 32) | (uint32_t)__builtin_amdgcn_readlane((int)amask, 48);
        const uint32_t n_items = (uint32_t)__popc(wmask);
        if (n_items == 0u) continue;
        uint32_t cur_idx = 0, cur_mask = wmask;               // item c = the c-th set bit (requests come in ascending c)
        auto fetch = [&](uint32_t c, DBuf& bf) {
          while (cur_idx < c) { cur_mask &= cur_mask - 1u; ++cur_idx; }
          const uint32_t j = jb + (uint32_t)__builtin_ctz(cur_mask);
          bf.j = j;
          const RingEntry e = rrow[j];
          const bool act = (amask >> (j - jb)) & 1u;
          const float* nrow = a.KVn + (size_t)(act ? e.nbr : 0u) * a.ld_kv;
          const float* erow = a.KVe + (size_t)(act ? e.eid : 0u) * a.ld_kve;
#pragma unroll
          for (int s = 0; s < 2 * KS; ++s) {                  // keys of all heads, then values
            if (s && s % SH == 0) { nrow += a.hs; erow += a.hs; }
            const uint32_t at = min(kSlot * (s % SH) + 4u * sub, a.hs - 4u);
            bf.n[s] = *reinterpret_cast<const float4*>(nrow + at);
            bf.e[s] = *reinterpret_cast<const float4*>(erow + at);
          }
        };
        auto work = [&](uint32_t, const DBuf& bf) {
        const uint32_t j = bf.j;
        const RingEntry e = rrow[j];
        const bool act = (amask >> (j - jb)) & 1u;
        const double dt = tq - e.t;
        float4 kk[KS], vv[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          kk[s] = make_float4(bf.n[s].x + bf.e[s].x, bf.n[s].y + bf.e[s].y, bf.n[s].z + bf.e[s].z, bf.n[s].w + bf.e[s].w);
          vv[s] = make_float4(bf.n[KS + s].x + bf.e[KS + s].x, bf.n[KS + s].y + bf.e[KS + s].y,
                              bf.n[KS + s].z + bf.e[KS + s].z, bf.n[KS + s].w + bf.e[KS + s].w);
        }
        float4 zt[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const double2 oa = *reinterpret_cast<const double2*>(s_om + t * kSlot + 4u * sub), ob = *reinterpret_cast<const double2*>(s_om + t * kSlot + 4u * sub + 2);
          const double2 pa = *reinterpret_cast<const double2*>(s_ph + t * kSlot + 4u * sub), pb = *reinterpret_cast<const double2*>(s_ph + t * kSlot + 4u * sub + 2);
          const float c0 = cos_rev(oa.x * dt + pa.x), c1 = cos_rev(oa.y * dt + pa.y);
          const float c2 = cos_rev(ob.x * dt + pb.x), c3 = cos_rev(ob.y * dt + pb.y);
          zt[t] = make_float4(c0, c1, c2, c3);           // (columns past d_time: see the exact variant)
        }
        float sc[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
          float p = 0.0f;
#pragma unroll
          for (int s = h * SH; s < (h + 1) * SH; ++s) { const float with = dot4(qk[s], kk[s], p); p = in_head(s - h * SH) ? with : p; }
#pragma unroll
          for (int t = 0; t < NT; ++t) p = dot4(*reinterpret_cast<const float4*>(zq + h * Ztp + t * kSlot), zt[t], p);
          sc[h] = row16_sum(p);
        }
        if (act && live) {
          float* w = a.ac_W + ((size_t)nn * k + j) * (2 * H);
          float* vc = a.ac_V + ((size_t)nn * k + j) * (kSlot * KS) + 4u * sub;
          if (ex) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
              const bool mv = sc[h] > mref[h] + 30.0f;
              const float mnew = mv ? sc[h] : mref[h];
              const float scale = mv ? __expf(mref[h] - mnew) : 1.0f;     // exp(-inf) = 0 on the first move
              mref[h] = mnew;
              const float p = __expf(sc[h] - mnew);
              lrun[h] = fmaf(lrun[h], scale, p);
#pragma unroll
              for (int s = h * SH; s < (h + 1) * SH; ++s) {
                accv[s].x = fmaf(accv[s].x, scale, p * vv[s].x); accv[s].y = fmaf(accv[s].y, scale, p * vv[s].y);
                accv[s].z = fmaf(accv[s].z, scale, p * vv[s].z); accv[s].w = fmaf(accv[s].w, scale, p * vv[s].w);
              }
#pragma unroll
              for (int t = 0; t < NT; ++t) {
                accp[h][t].x = fmaf(accp[h][t].x, scale, p * zt[t].x); accp[h][t].y = fmaf(accp[h][t].y, scale, p * zt[t].y);
                accp[h][t].z = fmaf(accp[h][t].z, scale, p * zt[t].z); accp[h][t].w = fmaf(accp[h][t].w, scale, p * zt[t].w);
              }
              if (sub == 0) Sc[(local * k + j) * H + h] = sc[h];
            }
          } else {
#pragma unroll
            for (int h = 0; h < H; ++h) {
              const float s_old = w[2 * h], a_old = w[2 * h + 1];
              const float e_old = __expf(s_old - mref[h]), e_new = __expf(sc[h] - mref[h]);
              const float Zn = lrun[h] - e_old + e_new;
              const float a_new = e_new / Zn;
              lrun[h] = Zn;
#pragma unroll
              for (int s = h * SH; s < (h + 1) * SH; ++s) {
                const float4 vo = *reinterpret_cast<const float4*>(vc + s * kSlot);
                accv[s].x += a_new * vv[s].x - a_old * vo.x; accv[s].y += a_new * vv[s].y - a_old * vo.y;
                accv[s].z += a_new * vv[s].z - a_old * vo.z; accv[s].w += a_new * vv[s].w - a_old * vo.w;
              }
              const float da = a_new - a_old;
#pragma unroll
              for (int t = 0; t < NT; ++t) {
                accp[h][t].x = fmaf(da, zt[t].x, accp[h][t].x); accp[h][t].y = fmaf(da, zt[t].y, accp[h][t].y);
                accp[h][t].z = fmaf(da, zt[t].z, accp[h][t].z); accp[h][t].w = fmaf(da, zt[t].w, accp[h][t].w);
              }
              if (sub == 0) { w[2 * h] = sc[h]; w[2 * h + 1] = a_new; }
            }
          }
#pragma unroll
          for (int s = 0; s < KS; ++s) *reinterpret_cast<float4*>(vc + s * kSlot) = vv[s];
        }
        };
        DBuf b0;
        fetch(0u, b0);
        pingpong_clamped<DBuf>(n_items, b0, fetch, work);
      }
      // ---- the row's sums: normalised by the denominator after an exact recomputation, as they stand after a delta update
      wave_lds_fence();
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const float inv = ex ? reciprocal(lrun[h]) : 1.0f;
#pragma unroll
        for (int s = h * SH; s < (h + 1) * SH; ++s) {
          float4 o = accv[s];
          o.x *= inv; o.y *= inv; o.z *= inv; o.w *= inv;
          *reinterpret_cast<float4*>(Xs + local * ll.ldx + s * kSlot + 4u * sub) = o;
          if (live) *reinterpret_cast<float4*>(acS + s * kSlot) = o;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float4 o = accp[h][t];
          o.x *= inv; o.y *= inv; o.z *= inv; o.w *= inv;
          if (t == NT - 1) clear_padding(o, t);
          *reinterpret_cast<float4*>(zq + h * Ztp + t * kSlot) = o;
          if (live) *reinterpret_cast<float4*>(acP + (h * NT + t) * kSlot) = o;
        }
        if (live && sub == 0) { acZM[2 * h] = lrun[h]; acZM[2 * h + 1] = mref[h]; }
        if (ex && live)
          for (uint32_t j = sub; j < cnt; j += 16) {          // the weights in effect after the exact recomputation
            const float sj = Sc[(local * k + j) * H + h];
            float* w = a.ac_W + ((size_t)nn * k + j) * (2 * H);
            w[2 * h] = sj;
            w[2 * h + 1] = lrun[h] > 0.0f ? __expf(sj - mref[h]) * inv : 0.0f;
          }
      }
      // ---- drift estimator (Sec. 3.5), final layer: an exact recomputation restarts the node's estimate, a
      // delta update adds the changed fraction of its entries to the decayed estimate
      // (the changes of the sum and of the member count are collected per wave and added once, at the end of
      // the launch: one update of the same word per row serialises -- 860 K of them took half of a launch)
      float dg = 0.0f;
      uint32_t dc = 0u;
      if (a.is_final && live && sub == 0) {
        const uint32_t tau = a.drift->tau;
        const float old = a.dseen[nn] ? a.dsum[nn] * __powf(a.gamma, (float)(tau - a.dlast[nn])) : 0.0f;
        const float nw = ex ? 0.0f : old + (nvalid ? (float)nch / (float)nvalid : 0.0f);
        if (!a.dseen[nn]) { a.dseen[nn] = 1; dc = 1u; }
        a.dsum[nn] = nw; a.dlast[nn] = tau;
        dg = nw - old;
      }
      drift_sum += (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(dg), 0)) +
                   (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(dg), 16)) +
                   (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(dg), 32)) +
                   (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(dg), 48));
      drift_new += (uint32_t)__builtin_amdgcn_readlane((int)dc, 0) + (uint32_t)__builtin_amdgcn_readlane((int)dc, 16) +
                   (uint32_t)__builtin_amdgcn_readlane((int)dc, 32) + (uint32_t)__builtin_amdgcn_readlane((int)dc, 48);
    } else {
      // ---- exact mode.  A row is served by one 16-lane group per key slot: a lane holds four columns of one slot of one
      // head, so sums, query and gathered rows take a quarter to a half of the registers that a group per row would need,
      // and all of q and qt and the time parameters stay in registers through the entry loop.  The time encodings,
      // which every head needs, are worked out once per row: each group evaluates its share of the columns and the groups
      // exchange them (SH = 1), or the slots of z are shared out over a head's slots (SH > 1).
      constexpr int CP = SH == 1 ? 4 * NT / KS : 4;           // cosines a lane evaluates per entry
      double om[CP], ph[CP];
      {
        const uint32_t i0 = SH == 1 ? g * CP : 4u * (sg < NT ? sg : 0u);   // first (slot, column of the quad) = (i0 / 4, i0 % 4)
        const uint32_t at = (i0 >> 2) * kSlot + 4u * sub + (i0 & 3u);
#pragma unroll
        for (int c = 0; c < CP; ++c) {
          om[c] = s_om[at + (c & 3) + (c >> 2) * kSlot];
          ph[c] = s_ph[at + (c & 3) + (c >> 2) * kSlot];
        }
      }
      static_for<PASSES>([&](auto P) {
      constexpr int p = decltype(P)::value;
      const uint32_t local = row_of(p), cnt = cnt_of(p), cmax = cmax_of(p);
      const double tq = tq_of(p);
      const uint32_t nchunk3 = (cmax + JC - 1) / JC;
      float4 accv = make_float4(0.f, 0.f, 0.f, 0.f), accp[NZL];
#pragma unroll
      for (int i = 0; i < NZL; ++i) accp[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      float mref = -INFINITY, lrun = 0.0f;
      auto attend = [&](uint32_t c, const ZBuf& zb) {
        float4 zt[JC][NZL];
        float sc[JC];
        bool vj[JC];
#pragma unroll
        for (int jc = 0; jc < JC; ++jc) {
          const double dt = tq - zb.t[jc];
          vj[jc] = c * JC + jc < cnt && dt <= a.window;       // inside the temporal window [tq - T_w, tq] (Sec. 3.3.2)
          float cs[CP], all[4 * NT];
#pragma unroll
          for (int i = 0; i < CP; ++i) cs[i] = cos_rev(__builtin_fma(om[i], dt, ph[i]));
          if constexpr (SH == 1) {
#pragma unroll
            for (int i = 0; i < CP; ++i) {
              if constexpr (KS == 1) {
                all[i] = cs[i];
              } else if constexpr (KS == 2) {
                const Two w = both_of_pair(cs[i]);
                all[i] = w.lo; all[CP + i] = w.hi;
              } else {
                const Two w = both_of_pair(cs[i]);
                const Two lo = both_halves(w.lo), hi = both_halves(w.hi);
                all[i] = lo.lo; all[CP + i] = hi.lo; all[2 * CP + i] = lo.hi; all[3 * CP + i] = hi.hi;
              }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) zt[jc][t] = make_float4(all[4 * t], all[4 * t + 1], all[4 * t + 2], all[4 * t + 3]);
            if constexpr (ES) zt[jc][NT] = zb.e[jc][0];
          } else {
            // (SH >= NT: time slots come first in a lane's share)
            const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < NZL; ++i) {
              const uint32_t t = sg + SH * i;
              zt[jc][i] = i == 0 && t < NT ? make_float4(cs[0], cs[1], cs[2], cs[3]) : ES && t == NT ? zb.e[jc][0] : zero;
            }
          }
          // score: q . (cached node keys + cached edge keys) + qt . phi  (raw edge rows: q . node keys + qt . z)
          float4 kk = zb.nk[jc];
          if constexpr (!ES) { kk.x += zb.e[jc][0].x; kk.y += zb.e[jc][0].y; kk.z += zb.e[jc][0].z; kk.w += zb.e[jc][0].w; }
          float s = dot4(qk[p % NP], kk, 0.0f);
          s = in_head(sg) ? s : 0.0f;
#pragma unroll
          for (int i = 0; i < NZL; ++i) s = dot4(qt[p % NP][i], zt[jc][i], s);
          s = row16_sum(s);
          if constexpr (SH >= 2) { const Two w = both_of_pair(s); s = w.lo + w.hi; }
          if constexpr (SH == 4) { const Two w = both_halves(s); s = w.lo + w.hi; }
          sc[jc] = vj[jc] ? s : -INFINITY;
        }
        // softmax against a reference score that only moves when a score exceeds it by a wide
        // margin (any reference gives the same quotient; the margin keeps exp() in range)
        float smax = sc[0];
#pragma unroll
        for (int jc = 1; jc < JC; ++jc) smax = fmaxf(smax, sc[jc]);
        const bool mv = smax > mref + 30.0f;
        if (__any(mv)) {
          const float mnew = mv ? smax : mref;
          const float scale = mv ? __expf(mref - mnew) : 1.0f;            // exp(-inf) = 0 on the first move
          lrun *= scale;
          accv.x *= scale; accv.y *= scale; accv.z *= scale; accv.w *= scale;
#pragma unroll
          for (int i = 0; i < NZL; ++i) {
            accp[i].x *= scale; accp[i].y *= scale; accp[i].z *= scale; accp[i].w *= scale;
          }
          mref = mnew;
        }
#pragma unroll
        for (int jc = 0; jc < JC; ++jc) {
          if (!vj[jc]) continue;                              // (a branch, and not a weight of zero: what does not count may be NaN)
          const float w = __expf(sc[jc] - mref);
          lrun += w;
          float4 vv = zb.nv[jc];
          if constexpr (!ES) { vv.x += zb.e[jc][1].x; vv.y += zb.e[jc][1].y; vv.z += zb.e[jc][1].z; vv.w += zb.e[jc][1].w; }
          accv.x = fmaf(w, vv.x, accv.x); accv.y = fmaf(w, vv.y, accv.y);
          accv.z = fmaf(w, vv.z, accv.z); accv.w = fmaf(w, vv.w, accv.w);
#pragma unroll
          for (int i = 0; i < NZL; ++i) {
            accp[i].x = fmaf(w, zt[jc][i].x, accp[i].x); accp[i].y = fmaf(w, zt[jc][i].y, accp[i].y);
            accp[i].z = fmaf(w, zt[jc][i].z, accp[i].z); accp[i].w = fmaf(w, zt[jc][i].w, accp[i].w);
          }
        }
      };
      if constexpr (LAZY && p + 1 < PASSES) {
        // the next pass's first gather takes the place of the request past this one's end
        constexpr std::integral_constant<int, p + 1> kNext{};
        ZBuf& P = z0[0];
        ZBuf Q;
        if (nchunk3 == 0u) gather(p + 1, 0, P);
        for (uint32_t i = 0; i < nchunk3; i += 2) {
          gather(p, i + 1 < nchunk3 ? i + 1 : nchunk3 - 1, Q);
          __builtin_amdgcn_sched_barrier(0);
          attend(i, P);
          __builtin_amdgcn_sched_barrier(0);
          gather_row(i + 2 < nchunk3 ? row_of(p) : row_of(p + 1), i + 2 < nchunk3 ? i + 2 : 0u, P);
          __builtin_amdgcn_sched_barrier(0);
          if (i + 1 < nchunk3) attend(i + 1, Q);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (clean) request_query(kNext); else read_query(kNext);
      } else {
        if (nchunk3) pingpong_clamped<ZBuf>(nchunk3, z0[p % NP], [&](uint32_t c, ZBuf& zb) { gather(p, c, zb); }, attend);
      }
      // the cached-value part of the head outputs goes into Xs (padded-head layout; what lanes past a head's floats leave in
      // its padding columns is not read), pb where qt is (each lane owns its columns)
      const float inv = reciprocal(lrun);                     // no entry, or none inside the window: b_O alone
      accv.x *= inv; accv.y *= inv; accv.z *= inv; accv.w *= inv;
      if constexpr (RT > 1) {
        // (the next tile's q comes to lie here, and phase 2 reads its padding columns, against zero weights: they must not
        // be this row's, whose sums may be NaN)
        const uint32_t c0 = kSlot * sg + 4u * sub;
        accv.x = c0 < dk ? accv.x : 0.0f;
        accv.y = c0 + 1u < dk ? accv.y : 0.0f;
        accv.z = c0 + 2u < dk ? accv.z : 0.0f;
        accv.w = c0 + 3u < dk ? accv.w : 0.0f;
      }
      *reinterpret_cast<float4*>(As + local * ldas + kSlot * g + 4u * sub) = accv;
#pragma unroll
      for (int i = 0; i < NZL; ++i) {
        const uint32_t t = SH == 1 ? (uint32_t)i : sg + SH * i;
        float4 o = accp[i];
        o.x *= inv; o.y *= inv; o.z *= inv; o.w *= inv;
        if (SH > 1 || i == NT - 1) clear_padding(o, t);    // (a raw edge row's padding is zero, and so are its sums)
        if (t < NZ) *reinterpret_cast<float4*>(Zs + local * ll.ldz + head * Ztp + t * kSlot + 4u * sub) = o;
      }
      });
    }
    // ================================================================ phase 4: o_h += pb_h W_V,h[time | raw edge]
    // K runs over the slots of z, one chunk per slot.  The weights of this phase and of the next are requested ahead of its
    // barrier, and behind them the next tile's rows.
    derive_lane();
    auto wv = [&](uint32_t h, uint32_t nt) { return a.WV + (size_t)(h * ntk + nt) * NZ * kChunkFloats; };
    uint32_t x4 = wave < nunits4 ? wave : nunits4 - 1u;
    Upfront16<N4, NZ> u4;
    const float* B4[N4];
    auto head4 = [&]() { return H == 1 ? 0u : H == 2 ? (x4 >= np4 ? 1u : 0u) : (x4 >= np4 ? 1u : 0u) + (x4 >= 2u * np4 ? 1u : 0u) + (x4 >= 3u * np4 ? 1u : 0u); };
    auto request4 = [&]() {
      const uint32_t h4 = head4(), n0 = N4 * (x4 - h4 * np4);
#pragma unroll
      for (int t = 0; t < N4; ++t) B4[t] = wv(h4, n0 + t < ntk ? n0 + t : n0);
      u4.request(B4, NZ, lane);
    };
    constexpr int U5 = NTL == 1 ? (KS < 2 ? KS : 2) : KS <= 2 ? KS : 1;   // chunks of W_O requested up front
    Upfront16<NTL, U5> u5;
    const float* B5[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) B5[t] = tile_b(a.WO, w1, t, ntd, KS);
    float b5v[NTL];                                           // this lane's bias of the first unit
    auto request5 = [&]() {
      u5.request(B5, KS, lane);
#pragma unroll
      for (int t = 0; t < NTL; ++t) { const uint32_t col = (w1 + NW * t) * 16 + m16_col(lane); b5v[t] = a.bO[col < a.d_emb ? col : 0u]; }
    };
    request4();
    stage_b(next_tile);
    take();                                // (behind what this tile waits for)
    __syncthreads();
    if (wave < nunits4) {
      for (;;) {
        const uint32_t h4 = head4(), n0 = N4 * (x4 - h4 * np4);
        floatx4 acc[RT][N4] = {};
        u4.template multiply_rows<RT>(Zs + h4 * Ztp + a16_off(lane, ll.ldz), kTM * ll.ldz, NZ, B4, acc, lane, groups4);
#pragma unroll
        for (int t = 0; t < N4; ++t) {
          const uint32_t col = (n0 + t) * 16 + m16_col(lane);
          if (n0 + t < ntk && col < dk) {
            const uint32_t at = h4 * (SH * kSlot) + col;      // one lane per (row, column)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const uint32_t row = kTM * rt + m16_row(lane, r);
                Qs[row * ll.ldq + at] = As[row * ldas + at] + acc[rt][t][r];
              }
          }
        }
        x4 += NW;
        if (x4 >= nunits4) break;
        request4();
      }
    }
    // ================================================================ phase 5: h' = o W_O + b_O
    derive_lane();
    request5();
    commit(round + 1u);
    publish(round + 1u);
    if constexpr (QCACHE) { derive_slot(); request_back(kPass0); }           // (a tile that projects does not use them)
    __syncthreads();
    if (kRowsInZ || !rows_in_lds) {                           // the next tile's input rows, if it projects
      if (!QCACHE || (!ROOTS && p_clean == 0u)) commit_x(pf_ok);
    }
    // a load behind a store waits for it: the first units' results stay in registers until everything that the following
    // phases read has been requested
    auto bias5 = [&](uint32_t nt, const floatx4 (&acc)[RT][NTL], floatx4 (&o)[RT][NTL]) {
#pragma unroll
      for (int t = 0; t < NTL; ++t) {
        const uint32_t col = (nt + NW * t) * 16 + m16_col(lane);
        const float b = nt == wave ? b5v[t] : a.bO[col < a.d_emb ? col : 0u];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            o[rt][t][r] = acc[rt][t][r] + b;
            if (rows_in_lds && nt + NW * t < ntd && col < a.d_emb) Hs[(kTM * rt + m16_row(lane, r)) * ldh + col] = o[rt][t][r];   // for the link scores; operand of phase 6
          }
      }
    };
    auto store5 = [&](uint32_t nt, const floatx4 (&acc)[RT][NTL]) {
      if constexpr (!ROOTS) {
        float* const hout = args()->Hout;
#pragma unroll
        for (int t = 0; t < NTL; ++t) {
          const uint32_t col = (nt + NW * t) * 16 + m16_col(lane);
          if (nt + NW * t < ntd && col < a.d_emb) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const uint32_t node = nodes_s[kTM * rt + m16_row(lane, r)];
                if (node != 0xFFFFFFFFu) hout[(size_t)node * a.ld_out + col] = acc[rt][t][r];
              }
          }
        }
      }
    };
    floatx4 out5[RT][NTL] = {};
    if (wave < ntd) {
      floatx4 acc[RT][NTL] = {};
      u5.template multiply_rows<RT>(Qs + a16_off(lane, ll.ldq), kTM * ll.ldq, KS, B5, acc, lane, groups_head);
      bias5(wave, acc, out5);
    }
    for (uint32_t nt = wave + 8; nt < ntd; nt += 8) {
      const float* Bt[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) Bt[t] = tile_b(a.WO, nt, t, ntd, KS);
      floatx4 acc[RT][NTL] = {}, o[RT][NTL];
      mfma16_lean_rows<RT, NTL>(Qs + a16_off(lane, ll.ldq), kTM * ll.ldq, 0u, KS, Bt, acc, lane, groups_head);
      bias5(nt, acc, o);
      store5(nt, o);
    }
    if (!kRowsInZ && kv) {                                    // (Xs: what lies past the output row need not be a number)
      const uint32_t w = 64u * c_de - a.d_emb;
      for (uint32_t x = threadIdx.x; x < TM * w; x += TH) Xs[(x / w) * ll.ldx + a.d_emb + x % w] = 0.0f;
    }
    if constexpr (ROOTS) {
      // link scores: a wave takes edges w and on of the tile (the list holds whole edges)
      __syncthreads();
      for (uint32_t e = wave; e < TM / 2; e += NW) {
        const uint32_t i = tile * (TM / 2) + e;
        const float* hu = Hs + 2u * e * ldh;
        const float* hv = hu + ldh;
        float acc = 0.0f;
        for (uint32_t c = lane; c < a.d_emb; c += 64) acc = fmaf(hu[c], a.head[c], fmaf(hv[c], a.head[a.d_emb + c], acc));
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
        const bool ok = nodes_s[2u * e] != 0xFFFFFFFFu && nodes_s[2u * e + 1u] != 0xFFFFFFFFu;
        if (lane == 0 && 2u * i < n) a.scores[i] = ok ? acc + a.head[2u * a.d_emb] : __builtin_nanf("");
      }
    }
    // ================================================================ phase 6: next layer's cached keys | values of these rows
    // A wave takes column tiles w, w + NW, ... of a cached row.  The second tile's chunks follow the first's into the same
    // registers.
    const uint32_t ntkv = args()->ld_kv >> 4;
    auto store6 = [&](uint32_t nt, const floatx4 (&acc)[RT][1]) {
      float* const kvout = args()->KVout;
      const uint32_t col = nt * 16 + m16_col(lane);           // every column is written: padding columns get exact zeros
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const uint32_t node = nodes_s[kTM * rt + m16_row(lane, r)];
          if (node != 0xFFFFFFFFu) kvout[(size_t)node * (16u * ntkv) + col] = acc[rt][0][r];
        }
    };
    floatx4 out6[2][RT][1] = {};
    if (kv) {
      const float* const wkv0 = args()->WKVnext;
      auto wkv = [&](uint32_t nt) { return wkv0 + (size_t)(nt < ntkv ? nt : ntkv - 1u) * c_de * kChunkFloats; };
      const bool two = wave + NW < ntkv;                      // (uniform)
      const float* Ha = Hs + a16_off(lane, ldh);
      const uint32_t c1 = c_de > 1 ? 1u : 0u;
      float4 b6[2][1][kCG];
      load_b16(wkv(wave), 0, b6[0][0], lane);
      load_b16(wkv(wave), c1 * kCG, b6[1][0], lane);
      __syncthreads();
      auto groups6 = [&](uint32_t ch) { return groups_used([](ArgBlock p) { return p->d_emb; }, ch * kCG); };
      auto chunk6 = [&](uint32_t ch, const float4 (&b)[1][kCG], floatx4 (&acc)[RT][1]) {
        mfma16_chunk_rows<RT, 1>(Ha, kTM * ldh, ch * kCG, b, acc, groups6(ch));
      };
      chunk6(0, b6[0], out6[0]);
      if (two) load_b16(wkv(wave + NW), 0, b6[0][0], lane);
      if (c1) chunk6(1, b6[1], out6[0]);
      if (two) {
        load_b16(wkv(wave + NW), c1 * kCG, b6[1][0], lane);
        chunk6(0, b6[0], out6[1]);
        if (c1) chunk6(1, b6[1], out6[1]);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const float* const Bt[1] = {wkv(wave + NW * t)};
        mfma16_lean_rows<RT, 1>(Ha, kTM * ldh, 2u, c_de, Bt, out6[t], lane, groups6);
      }
      for (uint32_t nt = wave + 2 * NW; nt < ntkv; nt += NW) {
        const float* const Bt[1] = {wkv(nt)};
        floatx4 acc[RT][1] = {};
        mfma16_lean_rows<RT, 1>(Ha, kTM * ldh, 0u, c_de, Bt, acc, lane, groups6);
        store6(nt, acc);
      }
    }
    if (wave < ntd) store5(wave, out5);
    if (kv) {
      if (wave < ntkv) store6(wave, out6[0]);
      if (wave + NW < ntkv) store6(wave + NW, out6[1]);
    }
    if (QCACHE && (RT > 1 || rows_in_lds)) __syncthreads();
  };
  for (uint32_t round = 0;; ++round) {
    const uint32_t tile = next_tile;
    if (tile >= ntiles) break;                                // wave-uniform; only in a workgroup's last round
    advance(round);
    // (set by the staging of a tile ago; uniform)
    if constexpr (QCACHE) {
      if (ROOTS || p_clean != 0u) { work_tile(std::true_type{}, tile, round); continue; }
    }
    if constexpr (!(QCACHE && ROOTS)) work_tile(std::false_type{}, tile, round);
  }
  if constexpr (DELTA) {
    if (lane == 0 && a.is_final) {
      if (drift_sum != 0.0) atomicAdd(&a.drift->G, drift_sum);
      if (drift_new) atomicAdd(&a.drift->count, drift_new);
    }
  }
  // statistics: the workgroup's count goes into the slot of its index with a plain update (launches
  // on one stream follow each other, and no other workgroup of a launch has this index); thousands of
  // same-address atomic updates at the end of a launch were measured to cost a third of its duration
  if constexpr (!ROOTS) {
    if (lane == 0) s_sum[wave] = gathered;
    __syncthreads();
    if (wave == 0u && lane == 0u) {                           // (threadIdx.x would be held, or spilled, through the tile loop)
      uint32_t tot = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) tot += s_sum[w];
      if (tot) a.gathered_slots[blockIdx.x] += tot;
      if (blockIdx.x == 0 && n) a.ctrl->tot_rows += n;
    }
  }
}

template <int KS, int NT, int ES, int H, int JC, int WGS, bool DELTA, bool QCACHE, bool ROOTS>
__global__ __launch_bounds__(64 * layer_waves(KS, DELTA), WGS * layer_waves(KS, DELTA) / 4)
void layer_kernel(LayerArgs a, const uint32_t* __restrict__ rows, const uint32_t* count_ptr, uint32_t count_max) {
  uint32_t n = count_max;
  if (count_ptr) { const uint32_t c = *count_ptr; n = c < count_max ? c : count_max; }
  __shared__ FixedLds<NT, layer_waves(KS, DELTA), kTM> fixed;
  static_assert(sizeof(fixed) <= kFixedLds, "the launches allow for it");
  layer_body<KS, NT, ES, H, JC, DELTA, QCACHE, ROOTS, 1, DELTA || ROOTS ? kRotated : kByLength>(a, rows, n, fixed);
}

// Launches whose list may be long: tiles of 32 rows if it is, of 16 if not (the list's length is known on the device alone).
// A tile streams every weight from L2 once whatever its rows (232 KB a tile of two slots, where its sixteen rows gather
// 190 KB), passes its barriers once and waits once for each phase's requests: 39 K cycles a tile of sixteen rows, half of
// them such waits.  With two row tiles each weight register meets both, the waits are shared by twice the rows, and a
// wave serves its four rows in two passes (four slots: four), a pass's first gather in flight through the end of the one before.
// Layer launches of 1,000,000 nodes (mean of both layers) 922 -> 847 us (794 with compact cached rows and without the products
// of zero weights; first layer, last layer, of 200,000 rebuilt nodes 585, 396 -> 481, 332).  Whole batches: 1,000,000 nodes, d_edge 100, 2,146 ->
// 2,001 us; 1,300,000 nodes, raw edge rows, k = 20, 1,292 -> 1,220; 200,000 nodes rebuilt 1,152 -> 1,093; 100,000 nodes,
// five to six tiles a workgroup, 446 -> 444.  Where a workgroup has a tile or two, the longer tile loses more than it
// shares: 10,000 nodes 113 -> 130 us, 20,000 nodes 188 -> 195, 30,000 nodes 252 -> 248, hence the line at kShortTiles.
template <int KS, int NT, int ES, int H, bool QCACHE>
__global__ __launch_bounds__(512, 4)
void layer32_kernel(LayerArgs a, const uint32_t* __restrict__ rows, const uint32_t* count_ptr, uint32_t count_max) {
  uint32_t n = count_max;
  if (count_ptr) { const uint32_t c = *count_ptr; n = c < count_max ? c : count_max; }
  __shared__ FixedLds<NT, 8, 2 * kTM> fixed;
  static_assert(sizeof(fixed) <= kFixedLds, "the launches allow for it");
  if (n > kShortTiles * kTM * gridDim.x) layer_body<KS, NT, ES, H, 1, false, QCACHE, false, 2, kCounted>(a, rows, n, fixed);
  else layer_body<KS, NT, ES, H, 1, false, QCACHE, false, 1, kFixed>(a, rows, n, fixed);
}

// Whether tiles of 32 rows of the narrowest model of these slots leave room for two workgroups per CU (else there is no such kernel).
constexpr bool layer32_fits(int ks, int nz, int heads) {
  return layer_lds(1, heads, heads, ks, nz, 1, false, 32).total * sizeof(float) + kFixedLds <= kMaxLds / 2;
}

// ---- dispatch over (heads, key slots, time slots)
struct LaunchArgs {
  LayerArgs k;
  hipStream_t s; const uint32_t* rows; const uint32_t* cp; uint32_t cm;
  uint32_t ks, nt, heads;
  bool es;                          // raw edge rows (never together with delta)
  bool delta;                       // the delta-mode variant of the kernel
  bool roots;                       // the root-node variant (the exact one also in delta mode)
  uint32_t num_cu;                  // compute units of the device
  bool set_attr; size_t lds; hipError_t err;
  bool tall; size_t lds32;
  int query_wgs; uint32_t wgs;      // query_wgs: only report the workgroups per CU of the variant in `wgs`
};

template <int KS, int NT, int ES, int H, int JC, int WGS, bool DELTA, bool QCACHE, bool ROOTS>
void go_k(LaunchArgs& a) {
  auto kern = layer_kernel<KS, NT, ES, H, JC, WGS, DELTA, QCACHE, ROOTS>;
  if (a.query_wgs) { a.wgs = WGS; return; }
  if (a.set_attr) {
    // never lowered: other layers of this context and other contexts of the process may launch the same variant
    static std::mutex mu;
    static size_t granted = 0;
    std::lock_guard<std::mutex> lock(mu);
    a.err = hipSuccess;
    if (a.lds > granted) {
      a.err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds);
      if (a.err == hipSuccess) granted = a.lds;
    }
    if constexpr (!DELTA && !ROOTS && KS >= 2 && layer32_fits(KS, NT + ES, H)) {
      if (a.err == hipSuccess && a.tall) a.err = hipFuncSetAttribute((const void*)layer32_kernel<KS, NT, ES, H, QCACHE>, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
    }
    return;
  }
  if constexpr (!DELTA && !ROOTS && KS >= 2 && layer32_fits(KS, NT + ES, H)) {
    if (a.tall && a.cm > kShortTiles * kTM * std::min(2u * (a.num_cu ? a.num_cu : 256u), kStatSlots)) {
      auto kern = layer32_kernel<KS, NT, ES, H, QCACHE>;
      const uint32_t cap = std::min(2u * (a.num_cu ? a.num_cu : 256u), kStatSlots);
      hipLaunchKernelGGL(kern, dim3(cap), dim3(512), std::max(a.lds32, a.lds), a.s, a.k, a.rows, a.cp, a.cm);
      return;
    }
  }
  uint64_t blocks = ((uint64_t)a.cm + kTM - 1) / kTM;
  uint64_t cap = (uint64_t)WGS * (a.num_cu ? a.num_cu : 256u);         // persistent: each workgroup strides over the tiles,
  if (cap > kStatSlots) cap = kStatSlots;                              // staging one tile ahead
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(64 * layer_waves(KS, DELTA)), a.lds, a.s, a.k, a.rows, a.cp, a.cm);
}

template <int KS, int NT, int H, int JC, int WGS, bool ROOTS>
void go_exact(LaunchArgs& a) {
  if (a.es) {
    if (a.k.tile_clean) go_k<KS, NT, 1, H, JC, WGS, false, true, ROOTS>(a); else go_k<KS, NT, 1, H, JC, WGS, false, false, ROOTS>(a);
    return;
  }
  if (a.k.tile_clean) { go_k<KS, NT, 0, H, JC, WGS, false, true, ROOTS>(a); return; }
  go_k<KS, NT, 0, H, JC, WGS, false, false, ROOTS>(a);
}

template <int KS, int NT, int H, int JC, int WGS>
void go(LaunchArgs& a) {
  if (a.roots) go_exact<KS, NT, H, JC, WGS, true>(a);
  else if (a.delta) go_k<KS, NT, 0, H, 1, WGS, true, false, false>(a);
  else go_exact<KS, NT, H, JC, WGS, false>(a);
}

// Ring entries per chunk and workgroups per CU are bounded by registers.  Exact mode, a lane per column quad of one key
// slot: two chunks of JC entries are in flight, 3 (raw edge rows) or 4 float4 each, beside 1 + NZL float4 of sums and as many
// of q and qt.  One slot: four waves of 168 registers, three workgroups per CU; more: eight of 128, two.  The delta mode, a lane per
// row's column quad of every slot, holds 4 KS float4 per entry and 2 KS + H NT beside them: four waves of 256 (one slot: 168).
template <int KS, int NT, int H>
void go_jc(LaunchArgs& a) {
  if constexpr (KS == 1) go<KS, NT, H, 2, 3>(a);
  else go<KS, NT, H, 1, 2>(a);
}

template <int H>
void go_h(LaunchArgs& a) {
  const uint32_t sh = a.ks / H;
  if (a.nt == 1) {
    if (sh == 1) go_jc<H, 1, H>(a);
    else if constexpr (H <= 2) { if (sh == 2) go_jc<2 * H, 1, H>(a); else if constexpr (H == 1) go_jc<4, 1, 1>(a); }
  } else {
    if (sh == 1) go_jc<H, 2, H>(a);
    else if constexpr (H <= 2) { if (sh == 2) go_jc<2 * H, 2, H>(a); else if constexpr (H == 1) go_jc<4, 2, 1>(a); }
  }
}

}  // namespace layer_impl

// one translation unit per head count instantiates this (keeps the build parallel)
template <int H>
void layer_entry(layer_impl::LaunchArgs& a) { layer_impl::go_h<H>(a); }

}  // namespace stgn
