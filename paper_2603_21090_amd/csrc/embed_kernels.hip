// Launch plumbing of the fused attention-layer kernel (defined in layer_kernel.h, instantiated per
// head count in layer_h*.hip) and the cached-row gather behind stgn_get_embeddings.
#include "layer_kernel.h"

namespace stgn {

extern template void layer_entry<1>(layer_impl::LaunchArgs&);
extern template void layer_entry<2>(layer_impl::LaunchArgs&);
extern template void layer_entry<4>(layer_impl::LaunchArgs&);

namespace {

using layer_impl::LaunchArgs;
using layer_impl::LayerArgs;

// Rows of a table for a list of node ids; an id past the node count (device-resident lists are not
// checked on the host) yields a row of NaN instead of a read outside the table.
//
// A copy, bound by HBM for long lists and by the launch for short ones.  A workgroup takes `per` consecutive list
// positions (and again `per`, a grid further on, when the list outgrows the largest grid) and its threads stride over
// their pieces of V floats; eight pieces per thread are requested before the first is stored, and the (row, piece) pair
// advances by additions.  One million rows of 100 floats: 173 us = 4.6 TB/s of ids, rows read and rows stored, 5.3 with
// the padding of the tables' rows to 512 bytes, where a large copy reaches 6.0 (four pieces together: 185 us; one float
// per thread and a 64-bit division each: 284 us).
// Results are stored past the caches: nothing here reads them again, and the tables keep their place.
constexpr uint32_t kGatherBlocks = 1u << 16;
template <int V> struct Piece;
template <> struct Piece<4> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct Piece<2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct Piece<1> { typedef float type; };

template <int V>
__global__ __launch_bounds__(256) void gather_rows_kernel(Table T, uint32_t N, uint32_t width, uint32_t n, uint32_t per,
                                                          const uint32_t* __restrict__ nodes, float* __restrict__ out) {
  using P = typename Piece<V>::type;
  constexpr int U = 8;
  const uint32_t q = width / V;                               // pieces per row
  const uint32_t dr = 256u / q, dc = 256u - dr * q;
  for (uint64_t i0 = (uint64_t)blockIdx.x * per; i0 < n; i0 += (uint64_t)gridDim.x * per) {   // (uniform)
    const uint32_t rows = (uint32_t)min((uint64_t)per, n - i0), tot = rows * q;
    const uint32_t* ids = nodes + i0;
    P* dst = reinterpret_cast<P*>(out) + (size_t)i0 * q;
    uint32_t x = threadIdx.x, r = x / q, c = x - r * q;
    while (x < tot) {
      P v[U];
      uint32_t id[U], rr[U], cc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        rr[u] = r < rows ? r : rows - 1u;                     // (pieces past the end repeat the last row and are not stored)
        cc[u] = c;
        id[u] = ids[rr[u]];
        c += dc; r += dr;
        if (c >= q) { c -= q; ++r; }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        v[u] = *reinterpret_cast<const P*>(T.base + (size_t)(id[u] < N ? id[u] : 0u) * T.ld + V * cc[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const P nan = (P)(__builtin_nanf(""));
        if (x + 256u * u < tot) __builtin_nontemporal_store(id[u] < N ? v[u] : nan, dst + x + 256u * u);
      }
      x += 256u * U;
    }
  }
}

__global__ void gather_times_kernel(const double* __restrict__ t, uint32_t N, uint32_t n, const uint32_t* __restrict__ nodes,
                                    double* __restrict__ out) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t v = nodes[i];
    out[i] = v < N ? t[v] : __builtin_nan("");
  }
}

// Linear link score (Algorithm 1, "Link prediction"): one 64-lane wave per edge,
// y = h_u . w[0 : d) + h_v . w[d : 2d) + b over the cached final-layer rows.  (Scores at the edges' own times
// come out of the final layer's kernel.)
__global__ __launch_bounds__(256) void predict_head_kernel(Dev d, uint32_t n, const uint32_t* __restrict__ src,
                                                           const uint32_t* __restrict__ dst,
                                                           float* __restrict__ scores) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nwaves = (gridDim.x * blockDim.x) >> 6;
  const uint32_t de = d.d_emb;
  const Table HL = d.H[d.layers];
  for (uint32_t i = wave; i < n; i += nwaves) {
    const uint32_t u = src[i], v = dst[i];
    const bool ok = u < d.N && v < d.N;
    const float* hu = HL.base + (size_t)(ok ? u : 0u) * HL.ld;
    const float* hv = HL.base + (size_t)(ok ? v : 0u) * HL.ld;
    float acc = 0.0f;
    for (uint32_t c = lane; c < de; c += 64) acc = fmaf(hu[c], d.pred_w[c], fmaf(hv[c], d.pred_w[de + c], acc));
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) scores[i] = ok ? acc + d.pred_w[2 * de] : __builtin_nanf("");
  }
}

LaunchArgs make_args(const Dev& d, uint32_t layer) {
  const LayerDev& L = d.L[layer];
  LaunchArgs a{};
  LayerArgs& k = a.k;
  k.Hin = d.H[layer].base; k.Hout = d.H[layer + 1].base;
  k.KVn = d.KV[layer].base; k.KVe = d.KVE[layer].base;
  k.KVout = layer + 1 < d.layers ? d.KV[layer + 1].base : nullptr;
  k.WKVnext = layer + 1 < d.layers ? d.L[layer + 1].WKVn : nullptr;
  k.ring = d.ring; k.deg = d.deg; k.t_last = d.t_last;
  k.om_rev = d.om_rev; k.ph_rev = d.ph_rev; k.ctrl = d.ctrl; k.gathered_slots = d.gathered_slots;
  k.WQ = L.WQn; k.cQ = L.cQ; k.WKT = L.WKT; k.WV = L.WV; k.WO = L.WO; k.bO = L.bO;
  k.ld_in = d.H[layer].ld; k.ld_out = d.H[layer + 1].ld; k.ld_kv = d.ld_kv; k.hs = d.hs; k.ld_kve = d.KVE[layer].ld;
  k.window = d.window;
  k.tile_next = d.tile_next + layer * kStatLine;
  k.k = d.k; k.k_inv = 0xFFFFFFFFu / d.k; k.d_in = L.d_in; k.d_emb = d.d_emb; k.dk = d.dk; k.d_time = d.d_time; k.d_edge = d.d_edge;
  if (d.delta) {
    k.flags = d.flags_kept;
    k.thr_in = d.d_mem ? layer + 1u : layer;                  // flags at or below: the owner's input row of this layer changed
    k.force_exact = 1u; k.is_final = layer + 1 == d.layers ? 1u : 0u;
    k.gamma = d.gamma;
    k.ac_S = d.ac_S[layer]; k.ac_P = d.ac_P[layer]; k.ac_ZM = d.ac_ZM[layer]; k.ac_W = d.ac_W[layer]; k.ac_V = d.ac_V[layer];
    k.drift = d.drift; k.dsum = d.dsum; k.dlast = d.dlast; k.dseen = d.dseen;
  }
  k.QC = d.qcache ? d.QC[layer] : nullptr;                     // (null for the layers that keep none)
  k.tile_clean = d.qcache ? d.tile_clean[layer] : nullptr;
  a.delta = d.delta != 0;
  a.es = d.es != 0;
  a.ks = d.ks; a.nt = d.nt; a.heads = d.heads;
  a.num_cu = d.num_cu;
  a.lds = (size_t)layer_impl::layer_lds(L.d_in, d.d_emb, d.heads, d.ks, d.nz, d.k, d.delta != 0, 16).total * sizeof(float);
  a.lds32 = (size_t)layer_impl::layer_lds(L.d_in, d.d_emb, d.heads, d.ks, d.nz, d.k, false, 32).total * sizeof(float);
  a.tall = !d.delta && d.ks >= 2 && a.lds32 + layer_impl::kFixedLds <= kMaxLds / 2;
  a.err = hipSuccess;
  return a;
}

void go_heads(LaunchArgs& a) {
  switch (a.heads) {
    case 1: layer_entry<1>(a); break;
    case 2: layer_entry<2>(a); break;
    default: layer_entry<4>(a); break;
  }
}

}  // namespace

// heads in {1, 2, 4}; every head takes whole slots of 64 floats in the kernels, at most four in total;
// the time encoding takes at most two
int attn_supported(uint32_t d_emb, uint32_t d_time, uint32_t heads) {
  if (!(heads == 1 || heads == 2 || heads == 4) || d_emb == 0 || d_emb % heads) return 0;
  uint32_t sh = (d_emb / heads + kSlot - 1) / kSlot;
  if (sh == 3) sh = 4;
  return d_time >= 1 && d_time <= kMaxTimeSlots * kSlot && heads * sh <= kMaxKeySlots;
}

void launch_layer(const Dev& d, hipStream_t s, uint32_t layer, const uint32_t* rows, const uint32_t* cp, uint32_t cm,
                  bool force_exact) {
  LaunchArgs a = make_args(d, layer);
  a.k.force_exact = force_exact ? 1u : 0u;
  if (force_exact) a.k.tile_clean = nullptr;                   // every row projects its query again (and refreshes the cache):
                                                               // the variant that reads nothing back
  a.s = s; a.rows = rows; a.cp = cp; a.cm = cm; a.set_attr = false;
  go_heads(a);
}

// link scores of n edges at their own times: the final layer for the 2 n roots
void launch_layer_scores(const Dev& d, hipStream_t s, uint32_t n, const uint32_t* src, const uint32_t* dst, const double* ts,
                         float* scores) {
  LaunchArgs a = make_args(d, d.layers - 1);
  a.roots = true;                                             // (at their own times; q and qt, which do not depend on the time, are read back where a query cache is kept)
  a.k.root_src = src; a.k.root_dst = dst; a.k.root_ts = ts; a.k.nodes = d.N;
  a.k.head = d.pred_w; a.k.scores = scores;
  a.s = s; a.rows = nullptr; a.cp = nullptr; a.cm = 2 * n; a.set_attr = false;
  go_heads(a);
}

void launch_predict_head(const Dev& d, hipStream_t s, uint32_t n, const uint32_t* src, const uint32_t* dst, float* scores) {
  hipLaunchKernelGGL(predict_head_kernel, dim3((n + 3) / 4), dim3(256), 0, s, d, n, src, dst, scores);
}

hipError_t launch_gather_rows(const Dev& d, hipStream_t s, uint32_t layer, uint32_t n, const uint32_t* nodes, float* out) {
  uint32_t width = layer == 0 ? d.d0 : d.d_emb;
  // 16-byte pieces where the width and the caller's buffer allow (table rows are aligned to 256 bytes), else 8, else 4
  const uintptr_t at = reinterpret_cast<uintptr_t>(out);
  const int v = width % 4 == 0 && at % 16 == 0 ? 4 : width % 2 == 0 && at % 8 == 0 ? 2 : 1;
  // rows per workgroup: one round of eight pieces per thread for long lists, fewer rows while the list would not fill the
  // chip otherwise
  uint32_t per = 2048u * (uint32_t)v / width;
  const uint32_t fill = n / 2048u;
  if (per > fill) per = fill;
  if (per < 8) per = 8;
  // a launch may hold 2^24 workgroups of 256 threads: the grid stops far below that and far above what fills the chip
  const uint32_t blocks = (uint32_t)std::min<uint64_t>(((uint64_t)n + per - 1) / per, kGatherBlocks);
  Table T = d.H[layer];
  uint32_t N = d.N;
  void* args[] = {&T, &N, &width, &n, &per, &nodes, &out};
  const auto kern = v == 4 ? gather_rows_kernel<4> : v == 2 ? gather_rows_kernel<2> : gather_rows_kernel<1>;
  return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(blocks), dim3(256), args, 0, s);
}

void launch_gather_times(const Dev& d, hipStream_t s, uint32_t n, const uint32_t* nodes, double* out) {
  uint32_t blocks = (n + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(gather_times_kernel, dim3(blocks), dim3(256), 0, s, d.t_last, d.N, n, nodes, out);
}

// ---- drift estimator (Sec. 3.5)
__global__ __launch_bounds__(256) void drift_reset_kernel(Dev d) {
  const uint32_t nth = gridDim.x * blockDim.x, tid = blockIdx.x * blockDim.x + threadIdx.x;
  for (uint32_t v = tid; v < d.N; v += nth) { d.dsum[v] = 0.0f; d.dlast[v] = 0u; d.dseen[v] = 0; }
  if (tid == 0) { d.drift->G = 0.0; d.drift->count = 0u; d.drift->n_list = 0u; }
}

// nodes whose decayed estimate exceeds the threshold, in no particular order
__global__ __launch_bounds__(256) void drift_list_kernel(Dev d, float threshold) {
  const uint32_t nth = gridDim.x * blockDim.x, tid = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t tau = d.drift->tau;
  // (grid-stride with a uniform trip count: every lane of a wave takes part in the ballots; one reservation
  // of list places per wave and round)
  const uint32_t lane = threadIdx.x & 63u;
  for (uint32_t v0 = tid - lane; v0 < d.N; v0 += nth) {
    const uint32_t v = v0 + lane;
    bool hit = false;
    if (v < d.N && d.dseen[v]) hit = d.dsum[v] * __powf(d.gamma, (float)(tau - d.dlast[v])) > threshold;
    const uint64_t m = __ballot(hit);
    if (m == 0ull) continue;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&d.drift->n_list, (uint32_t)__popcll(m));
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    if (hit) d.dlist[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = v;
  }
}

// every node's decayed estimate (0 for nodes outside the cumulative affected set)
__global__ __launch_bounds__(256) void drift_values_kernel(Dev d, float* out) {
  const uint32_t nth = gridDim.x * blockDim.x, tid = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t tau = d.drift->tau;
  for (uint32_t v = tid; v < d.N; v += nth)
    out[v] = d.dseen[v] ? d.dsum[v] * __powf(d.gamma, (float)(tau - d.dlast[v])) : 0.0f;
}

void launch_drift_values(const Dev& d, hipStream_t s, float* out) {
  uint32_t blocks = (d.N + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(drift_values_kernel, dim3(blocks ? blocks : 1), dim3(256), 0, s, d, out);
}

void launch_drift_reset(const Dev& d, hipStream_t s) {
  uint32_t blocks = (d.N + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(drift_reset_kernel, dim3(blocks ? blocks : 1), dim3(256), 0, s, d);
}

void launch_drift_list(const Dev& d, hipStream_t s, float threshold) {
  uint32_t blocks = (d.N + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(drift_list_kernel, dim3(blocks ? blocks : 1), dim3(256), 0, s, d, threshold);
}

// Whether the layer kernel's tiles fit its share of the LDS at every layer with nz slots of z (d: the
// configuration fields and ks, nt).
int layer_tiles_fit(const Dev& d, uint32_t nz) {
  LaunchArgs a{};
  a.ks = d.ks; a.nt = d.nt; a.heads = d.heads; a.query_wgs = 1;
  go_heads(a);
  if (a.wgs == 0) return 0;
  for (uint32_t l = 0; l < d.layers; ++l) {
    const size_t lds = (size_t)layer_impl::layer_lds(l ? d.d_emb : d.d0, d.d_emb, d.heads, d.ks, nz, d.k, false, 16).total * sizeof(float);
    if (lds + layer_impl::kFixedLds > kMaxLds / a.wgs) return 0;
  }
  return 1;
}

// ---- bare gather (diagnostic): 16 lanes per row piece of 256 B, as in the layer kernel's entry loop, and
// nothing else -- few registers, full occupancy
template <int SLOTS>
__global__ __launch_bounds__(256) void gather_probe_kernel(const float* __restrict__ table, const uint32_t* __restrict__ idx,
                                                           uint32_t n_groups, uint32_t per, float* __restrict__ out) {
  const uint32_t g = (blockIdx.x * 256u + threadIdx.x) >> 4, sub = threadIdx.x & 15u;
  if (g >= n_groups) return;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  const uint32_t* ip = idx + (size_t)g * per;
  for (uint32_t j = 0; j < per; ++j) {
    const float* row = table + (size_t)ip[j] * (SLOTS * kSlot) + 4u * sub;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const float4 v = *reinterpret_cast<const float4*>(row + s * kSlot);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
  }
  out[(size_t)g * 16u + sub] = acc.x + acc.y + acc.z + acc.w;
}

void launch_gather_probe(hipStream_t s, const float* table, uint32_t slots, const uint32_t* idx, uint32_t n_groups,
                         uint32_t per, float* out) {
  const dim3 grid((uint32_t)(((uint64_t)n_groups * 16u + 255u) / 256u)), blk(256);
  if (slots == 1) hipLaunchKernelGGL(gather_probe_kernel<1>, grid, blk, 0, s, table, idx, n_groups, per, out);
  else hipLaunchKernelGGL(gather_probe_kernel<4>, grid, blk, 0, s, table, idx, n_groups, per, out);
}

int setup_embed_attributes(const Dev& d) {
  for (uint32_t l = 0; l < d.layers; ++l) {
    LaunchArgs a = make_args(d, l);
    a.query_wgs = 1;
    go_heads(a);
    if (a.wgs == 0) return -1;                                    // no kernel variant for this shape
    if (a.lds + layer_impl::kFixedLds > kMaxLds / a.wgs) return -1;   // that many workgroups per CU
    a.query_wgs = 0;
    a.set_attr = true;
    go_heads(a);
    if (a.err != hipSuccess) return -1;
    if (const uint8_t* clean = a.k.tile_clean) {                  // rebuilds run the variant that reads nothing back
      a.k.tile_clean = nullptr;
      go_heads(a);
      if (a.err != hipSuccess) return -1;
      a.k.tile_clean = clean;
    }
    if (l + 1 == d.layers) {                                      // the final layer's root rows
      a.roots = true;
      go_heads(a);
      if (a.err != hipSuccess) return -1;
    }
  }
  return 0;
}

}  // namespace stgn
