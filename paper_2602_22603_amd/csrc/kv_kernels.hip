// kv_kernels.hip - gfx950 kernels that write and move KV-cache pages:
//   append (Algorithm 1, Phase 3: the context grows by the response R and the
//   tool output O), the fork's tail-page copy (Phase 2, C_aux <- C + p), and
//   span eviction clear_kv (Phase 1): keep-mask -> exclusive prefix sum ->
//   inverse map -> page-level gather into fresh pages.
//
// Layouts (elements are bf16 stored as uint16_t):
//   K pool [NL][Hkv][NP][P][D]   one 16-token page of one head is P*D
//                                 contiguous values, token-major; the pages
//                                 of one head are contiguous (head-major)
//   V pool [NL][Hkv][NP][D][P]   the same page stored channel-major: the P
//                                 tokens of one channel are contiguous
//   pos    [NP][P]               int32 position of each cached token
// The page size is 16 throughout.
#include "fp8.hpp"
#include "kv_args.hpp"

#include <type_traits>

namespace sq {
namespace {

constexpr int P = kPage;

__device__ inline uint16_t *k_chunk_w(const Pools &p, int layer, int page, int head) {
  return p.k + layer * p.layer_stride + (int64_t)page * p.page_stride + head * p.head_stride;
}
__device__ inline uint16_t *v_chunk_w(const Pools &p, int layer, int page, int head) {
  return p.v + layer * p.layer_stride + (int64_t)page * p.page_stride + head * p.head_stride;
}

// Element E of the pools (bf16 bits, or E4M3 bytes): the chunk of one
// (layer, page, head), strides counted in elements.
template <class E> __device__ inline E *chunk_of(uint16_t *pool, const Pools &p, int layer, int page,
                                                 int head) {
  return reinterpret_cast<E *>(pool) + layer * p.layer_stride + (int64_t)page * p.page_stride +
         head * p.head_stride;
}

// Non-temporal 16- and 8-byte moves.
typedef uint32_t nt4_t __attribute__((ext_vector_type(4)));
typedef uint32_t nt2_t __attribute__((ext_vector_type(2)));
template <bool NT> __device__ inline uint4 load16(const void *src) {
  if constexpr (!NT) return *static_cast<const uint4 *>(src);
  const nt4_t x = __builtin_nontemporal_load(static_cast<const nt4_t *>(src));
  return make_uint4(x.x, x.y, x.z, x.w);
}
__device__ inline void store_nt(void *dst, uint4 x) {
  __builtin_nontemporal_store(nt4_t{x.x, x.y, x.z, x.w}, static_cast<nt4_t *>(dst));
}
__device__ inline void store_nt(void *dst, uint2 x) {
  __builtin_nontemporal_store(nt2_t{x.x, x.y}, static_cast<nt2_t *>(dst));
}
template <bool NT, class T> __device__ inline void store_as(void *dst, T x) {
  if constexpr (NT) store_nt(dst, x);
  else *static_cast<T *>(dst) = x;
}

// ---------------------------------------------------------------------------
// Append.  New tokens come token-major [NL][n_total][Hkv][D]; K rows are
// copied as 16-byte units, V is transposed through LDS when a whole page is
// written and scattered per element when only some slots of a page are (the
// other slots of that page already hold earlier tokens of the sequence).  In
// an 8-bit store each bf16 value x becomes the E4M3 code of
// float(x) * (1 / scale) of its layer (K and V scales apart).
//
// The kernel is bound by HBM: each byte is read once and written once.  A
// workgroup takes one 8 KB unit of work (a page of 128 channels, two of 64)
// with every load in flight before the first store; groups of twice that were
// 1-4% slower.  NT says what passes the caches by, against the 256 MB
// memory-side cache.  0, source and pages fit it together: nothing, since the
// decode that follows reads the pages, and the projection before wrote the
// source (512 tokens of 24 layers of 8 heads of 128, then a decode of each layer:
// 253 us of GPU time, 267 with NT 1).  1, they do not: the pages, which would
// push the source out (8192 tokens of 24 layers 322 -> 294 us; 2048, with the
// decodes, 332 -> 319).  2, the source alone is larger: its loads too (294 ->
// 280 us, 5.8 TB/s; 3000 tokens of 12 layers, 147 MB, just read: 48 us, 51 with
// NT 2).
__device__ inline float bf16_val(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ inline uint2 quant8(uint4 w, float inv) { // 8 bf16 -> 8 codes
  const uint32_t x[4] = {w.x, w.y, w.z, w.w};
  uint32_t c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    c[i] = e4m3_encode2(__uint_as_float(x[i] << 16) * inv, __uint_as_float(x[i] & 0xffff0000u) * inv);
  return make_uint2(c[0] | c[1] << 16, c[2] | c[3] << 16);
}

template <int D> constexpr int kAppendGroup = 128 / D; // pages of one workgroup

template <int D, class E, int NT>
__global__ __launch_bounds__(256) void k_append(Pools p, AppendArgs a,
                                                const uint16_t *__restrict__ kn,
                                                const uint16_t *__restrict__ vn) {
  constexpr bool KV8 = sizeof(E) == 1;
  constexpr int U = D / 8;                       // 16-byte units per source row
  constexpr int NPG = kAppendGroup<D>;           // pages per workgroup
  constexpr int PT = P * U;                      // threads that load a page's K (and V)
  __shared__ uint16_t tile[NPG][P][D + 8];
  const int p0 = blockIdx.x * NPG;
  const int layer = blockIdx.y / p.hkv, head = blockIdx.y % p.hkv;
  float inv_k = 1.f, inv_v = 1.f;
  if constexpr (KV8) {
    inv_k = p.scales[4 * layer + 2];
    inv_v = p.scales[4 * layer + 3];
  }
  const int64_t tok_stride = (int64_t)p.hkv * D;
  const uint16_t *ks = kn + ((int64_t)layer * a.n_total + a.tok0) * tok_stride + head * D;
  const uint16_t *vs = vn + ((int64_t)layer * a.n_total + a.tok0) * tok_stride + head * D;
  auto kpage = [&](int i) { return chunk_of<E>(p.k, p, layer, a.page_ids[p0 + i], head); };
  auto vpage = [&](int i) { return chunk_of<E>(p.v, p, layer, a.page_ids[p0 + i], head); };
  // launch-local token of slot 0 of page p0
  const int tok = p0 * P - a.slot0;
  // N whole pages from page p0 + i0 on: all loads in flight together
  auto move_whole = [&](auto n_pages, int i0) {
    constexpr int N = decltype(n_pages)::value;
    constexpr int NR = (N * PT + 255) / 256; // units per thread
    const int t0 = tok + i0 * P;
    uint4 kr[NR], vr[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int idx = r * 256 + threadIdx.x;
      if (N * PT < 256 && idx >= N * PT) break;
      const int64_t src = (t0 + idx / U) * tok_stride + idx % U * 8;
      kr[r] = load16<NT == 2>(ks + src);
      vr[r] = load16<NT == 2>(vs + src);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int idx = r * 256 + threadIdx.x;
      if (N * PT < 256 && idx >= N * PT) break;
      *reinterpret_cast<uint4 *>(&tile[idx / PT][idx / U % P][idx % U * 8]) = vr[r];
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int idx = r * 256 + threadIdx.x;
      if (N * PT < 256 && idx >= N * PT) break;
      E *kd = kpage(i0 + idx / PT) + idx % PT * 8;
      if constexpr (KV8) store_as<NT != 0>(kd, quant8(kr[r], inv_k));
      else store_as<NT != 0>(kd, kr[r]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int idx = r * 256 + threadIdx.x;
      if (N * PT < 256 && idx >= N * PT) break;
      const int i = idx / PT, d = idx % PT / 2, h = idx & 1;
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = (uint32_t)tile[i][h * 8 + 2 * e][d] | (uint32_t)tile[i][h * 8 + 2 * e + 1][d] << 16;
      const uint4 o = make_uint4(w[0], w[1], w[2], w[3]);
      E *vd = vpage(i0 + i) + d * P + h * 8;
      if constexpr (KV8) store_as<NT != 0>(vd, quant8(o, inv_v));
      else store_as<NT != 0>(vd, o);
    }
  };
  if (tok >= 0 && tok + NPG * P <= a.n_tok) {
    move_whole(std::integral_constant<int, NPG>(), 0);
  } else {
    const int n_pg = min(NPG, a.n_pages - p0);
    for (int i = 0; i < n_pg; ++i) {
      const int t0 = tok + i * P; // token of the page's slot 0
      const int s0 = max(0, -t0), ns = min(P, a.n_tok - t0) - s0;
      if (ns == P) {
        move_whole(std::integral_constant<int, 1>(), i);
        __syncthreads(); // the next page reuses the tile
        continue;
      }
      const int64_t src = (t0 + s0) * tok_stride;
      E *kd = kpage(i) + s0 * D;
      for (int idx = threadIdx.x; idx < ns * U; idx += 256) {
        const int j = idx / U, u = idx % U;
        const uint4 val = *reinterpret_cast<const uint4 *>(ks + src + j * tok_stride + 8 * u);
        if constexpr (KV8) *reinterpret_cast<uint2 *>(kd + j * D + 8 * u) = quant8(val, inv_k);
        else *reinterpret_cast<uint4 *>(kd + j * D + 8 * u) = val;
      }
      E *vd = vpage(i) + s0;
      for (int idx = threadIdx.x; idx < ns * D; idx += 256) {
        const int d = idx % D, j = idx / D;
        const uint16_t val = vs[src + j * tok_stride + d];
        if constexpr (KV8) vd[d * P + j] = (E)e4m3_encode(bf16_val(val) * inv_v);
        else vd[d * P + j] = val;
      }
    }
  }

  if (layer == 0 && head == 0) {
    for (int idx = threadIdx.x; idx < NPG * P; idx += 256) {
      const int t = tok + idx;
      if (t >= 0 && t < a.n_tok) p.pos[(int64_t)a.page_ids[p0 + idx / P] * P + idx % P] = a.pos0 + t;
    }
    const int pi = p0 + threadIdx.x;
    if (threadIdx.x < NPG && pi < a.n_pages && pi >= a.new_from) a.pt_row[a.pt_first + pi] = a.page_ids[pi];
  }
}

// One token for each of n sequences: block (b, layer * Hkv + head).
template <int D>
__global__ __launch_bounds__(64) void k_append_batch(Pools p, AppendBatchArgs a,
                                                     const uint16_t *__restrict__ kn,
                                                     const uint16_t *__restrict__ vn) {
  constexpr int U = D / 8;
  const int b = blockIdx.x;
  const int lh = blockIdx.y;
  const int layer = lh / p.hkv;
  const int head = lh % p.hkv;
  const int page = a.page[b];
  const int slot = a.slot[b];
  const int64_t src = (((int64_t)layer * a.n + b) * p.hkv + head) * D;
  uint16_t *kd = k_chunk_w(p, layer, page, head) + slot * D;
  for (int u = threadIdx.x; u < U; u += blockDim.x)
    *(reinterpret_cast<uint4 *>(kd) + u) = *(reinterpret_cast<const uint4 *>(kn + src) + u);
  uint16_t *vd = v_chunk_w(p, layer, page, head) + slot;
  for (int d = threadIdx.x; d < D; d += blockDim.x) vd[d * P] = vn[src + d];
  if (lh == 0 && threadIdx.x == 0) {
    p.pos[(int64_t)page * P + slot] = a.pos[b];
    if (a.pt_index[b] >= 0) a.pt[a.pt_index[b]] = page;
  }
}

template <int D>
__global__ __launch_bounds__(64) void k_append_batch8(Pools p, AppendBatchArgs a,
                                                      const uint16_t *__restrict__ kn,
                                                      const uint16_t *__restrict__ vn) {
  constexpr int U = D / 8;
  const int b = blockIdx.x;
  const int lh = blockIdx.y;
  const int layer = lh / p.hkv;
  const int head = lh % p.hkv;
  const float inv_k = p.scales[4 * layer + 2], inv_v = p.scales[4 * layer + 3];
  const int page = a.page[b];
  const int slot = a.slot[b];
  const int64_t src = (((int64_t)layer * a.n + b) * p.hkv + head) * D;
  const int64_t chunk = layer * p.layer_stride + (int64_t)page * p.page_stride + head * p.head_stride;
  uint8_t *kd = reinterpret_cast<uint8_t *>(p.k) + chunk + slot * D;
  for (int u = threadIdx.x; u < U; u += blockDim.x)
    *reinterpret_cast<uint2 *>(kd + 8 * u) = quant8(*(reinterpret_cast<const uint4 *>(kn + src) + u), inv_k);
  uint8_t *vd = reinterpret_cast<uint8_t *>(p.v) + chunk + slot;
  for (int d = threadIdx.x; d < D; d += blockDim.x)
    vd[d * P] = (uint8_t)e4m3_encode(bf16_val(vn[src + d]) * inv_v);
  if (lh == 0 && threadIdx.x == 0) {
    p.pos[(int64_t)page * P + slot] = a.pos[b];
    if (a.pt_index[b] >= 0) a.pt[a.pt_index[b]] = page;
  }
}

// A step's plan from pinned host memory, and its new page-table entries.  (A
// kernel, 3 us, and no hipMemcpyAsync: the copy engine's hand-over to the kernels
// around it cost 10.)
__global__ __launch_bounds__(256) void k_step_upload(uint4 *dst, const uint4 *src, int32_t n16,
                                                     SetEntries a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
  if (blockIdx.x == 0 && (int)threadIdx.x < a.n) a.base[a.index[threadIdx.x]] = a.value[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t *dst, int32_t value, int32_t n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = value;
}

// Fork: the first pt_blocks workgroups copy the page-table row and set its
// tail entry, the others (one per layer and head) copy the tail page.
template <int D, class E>
__global__ __launch_bounds__(256) void k_fork(Pools p, int32_t *dst, const int32_t *src, int32_t n,
                                              int32_t src_tail, int32_t tail_page, int32_t pt_blocks) {
  if ((int)blockIdx.x < pt_blocks) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
    if (i == n && tail_page >= 0) dst[n] = tail_page;
    return;
  }
  constexpr int U = P * D * (int)sizeof(E) / 16;
  const int lh = blockIdx.x - pt_blocks;
  const int layer = lh / p.hkv;
  const int head = lh % p.hkv;
  const uint4 *ks = reinterpret_cast<const uint4 *>(chunk_of<E>(p.k, p, layer, src_tail, head));
  const uint4 *vs = reinterpret_cast<const uint4 *>(chunk_of<E>(p.v, p, layer, src_tail, head));
  uint4 *kd = reinterpret_cast<uint4 *>(chunk_of<E>(p.k, p, layer, tail_page, head));
  uint4 *vd = reinterpret_cast<uint4 *>(chunk_of<E>(p.v, p, layer, tail_page, head));
  for (int u = threadIdx.x; u < U; u += blockDim.x) {
    kd[u] = ks[u];
    vd[u] = vs[u];
  }
  if (lh == 0 && threadIdx.x < P)
    p.pos[(int64_t)tail_page * P + threadIdx.x] = p.pos[(int64_t)src_tail * P + threadIdx.x];
}

// ---------------------------------------------------------------------------
// Eviction index.  keep[i] = 0 iff token i lies in one of the evicted spans;
// dst = exclusive prefix sum of keep; src_of[dst[i]] = i for kept i.  The
// keep mask is a union of sorted spans, so its prefix sum at i is
// i - (evicted tokens before i): the span-level exclusive prefix sums of the
// span lengths (spans[k][2]) plus the part of the span that contains i.
// Every token is independent, so one pass over the tokens suffices.
constexpr int kPerThread = kScanBlock / kScanThreads; // 8

__device__ inline int span_search(const int32_t *spans, int n_spans, int i) {
  // index of the last span whose start <= i, or -1
  int lo = 0, hi = n_spans - 1, ans = -1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    if (spans[3 * mid] <= i) {
      ans = mid;
      lo = mid + 1;
    } else {
      hi = mid - 1;
    }
  }
  return ans;
}

// The span list where a workgroup reads it: copied to LDS (lsp, 3 *
// kInlineSpans ints) from the kernel arguments when it travels there, else
// the device copy.  Every thread of the workgroup must call it.
__device__ inline const int32_t *stage_spans(const EvictArgs &a, int32_t *lsp) {
  const bool inl = a.n_spans <= kInlineSpans;
  if (inl)
    for (int i = threadIdx.x; i < 3 * a.n_spans; i += blockDim.x) lsp[i] = a.inl[i];
  __syncthreads();
  return inl ? lsp : a.spans;
}

// The old index of the kept token that lands at new index d: the last span k
// whose start lies at or before d once the tokens evicted before it are
// taken out (start_k - before_k <= d; non-decreasing in k) has every span up
// to it evicted before that token, so it is d + before_k + (end_k - start_k);
// with no such span it is d.
__device__ inline int source_of(const int32_t *spans, int n_spans, int d) {
  int lo = 0, hi = n_spans - 1, k = -1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    if (spans[3 * mid] - spans[3 * mid + 2] <= d) {
      k = mid;
      lo = mid + 1;
    } else {
      hi = mid - 1;
    }
  }
  return k < 0 ? d : d + spans[3 * k + 2] + (spans[3 * k + 1] - spans[3 * k]);
}

// Block blk (kScanBlock tokens) of the eviction index, by a workgroup of
// kScanThreads threads (the gather's too).
static_assert(kScanThreads == 256, "gather workgroups also run index blocks");
__device__ inline void evict_index_block(const EvictArgs &a, const int32_t *spans, int blk) {
  const int base = blk * kScanBlock + threadIdx.x * kPerThread;
  if (base >= a.n_tokens) return;
  int s = span_search(spans, a.n_spans, base);
  for (int e = 0; e < kPerThread; ++e) {
    const int i = base + e;
    if (i >= a.n_tokens) break;
    while (s + 1 < a.n_spans && spans[3 * (s + 1)] <= i) ++s;
    int before = 0; // evicted tokens before i
    bool inside = false;
    if (s >= 0) {
      const int st = spans[3 * s], en = spans[3 * s + 1];
      inside = i < en;
      before = spans[3 * s + 2] + (inside ? i - st : en - st);
    }
    const int d = i - before;
    a.keep[i] = inside ? 0 : 1;
    a.dst[i] = d;
    if (!inside) a.src_of[d] = i;
  }
}

__global__ __launch_bounds__(kScanThreads) void k_evict_index(EvictArgs a) {
  __shared__ int32_t lsp[3 * kInlineSpans];
  evict_index_block(a, stage_spans(a, lsp), blockIdx.x);
}

// Fresh page id number i of an eviction.
__device__ inline int32_t new_page_id(const NewIds &ids, int i) {
  if (ids.list) return ids.list[i];
  int r = 0;
  while (r + 1 < ids.n_runs && ids.before[r + 1] <= i) ++r;
  return ids.first[r] + (i - ids.before[r]);
}

// dst[i] = fresh id i: the page-table row takes the fresh ids after the gather.
__global__ __launch_bounds__(256) void k_write_ids(int32_t *dst, NewIds ids, int32_t n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = new_page_id(ids, i);
}

// ---------------------------------------------------------------------------
// The move of one destination page of one or more KV rows (row = layer * Hkv
// + head; the rows of a pool are head_stride apart).
//
// Where spans and the stretches between them are long, almost every page of a
// compacted tail is a run: its P kept tokens are P consecutive old tokens.
// They lie in slots [slot0, P) of one old page and [0, slot0) of the next,
// so the destination's K is P * D consecutive elements of the two, and a
// 16-byte unit of its V^T is 16 bytes of two neighbouring units of a
// channel's row, put together by a funnel shift that is the same for the
// whole workgroup.  Nothing passes through LDS and nothing waits but the
// stores for the loads: one unit of K and one of V per thread.  Bound by HBM:
// 20K tokens of 6 layers moved (8 heads of 128, 0.98 GB read and written)
// 216 -> 181 us a call (with two units per thread 194, with four 203), 36K
// tokens of 4 layers of an 8-bit store 207 -> 97 us, both against staging the
// source pages' V^T in LDS and putting each element together from there.
template <int D, class E> constexpr int kPageUnits = P * D * (int)sizeof(E) / 16;
template <int D, class E> constexpr int kGatherRows = 256 / kPageUnits<D, E>; // rows per workgroup

// Bytes [sh, sh + 16) of lo | hi (sh < 16, uniform).
__device__ inline uint4 funnel16(uint4 lo, uint4 hi, int sh) {
  const int b = sh & 3;
  auto pick = [&](uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t w4) {
    return make_uint4(__builtin_amdgcn_alignbyte(w1, w0, b), __builtin_amdgcn_alignbyte(w2, w1, b),
                      __builtin_amdgcn_alignbyte(w3, w2, b), __builtin_amdgcn_alignbyte(w4, w3, b));
  };
  switch (sh >> 2) {
  case 0: return pick(lo.x, lo.y, lo.z, lo.w, hi.x);
  case 1: return pick(lo.y, lo.z, lo.w, hi.x, hi.y);
  case 2: return pick(lo.z, lo.w, hi.x, hi.y, hi.z);
  default: return pick(lo.w, hi.x, hi.y, hi.z, hi.w);
  }
}

// Rows [row0, min(row0 + kGatherRows, nl * hkv)) of a run: old pages page_a
// (slots from slot0 on) and page_b (read only when slot0 > 0) -> dst.  With
// SYNC every load of the workgroup lands before its first store, since dst
// may be one of the sources.
template <int D, class E, bool SYNC>
__device__ inline void move_run(const Pools &p, int row0, int page_a, int page_b, int slot0, int dst) {
  constexpr int VU = kPageUnits<D, E>;
  constexpr int U = VU / P;                 // units per K row
  constexpr int EPU = 16 / (int)sizeof(E);  // V^T elements per unit
  constexpr int UPC = P / EPU;              // units per channel's row
  const int un = threadIdx.x % VU, row = row0 + threadIdx.x / VU;
  const bool in = row < p.nl * p.hkv;
  const int sk = un + slot0 * U;
  const int x = un % UPC * EPU + slot0;     // first element of the V^T unit, from page_a's row on
  const int u0 = x / EPU, u1 = u0 + 1, sh = slot0 % EPU * (int)sizeof(E);
  auto unit = [&](uint16_t *pool, int page, int u) {
    return reinterpret_cast<uint4 *>(reinterpret_cast<E *>(pool) + row * p.head_stride +
                                     (int64_t)page * p.page_stride) + u;
  };
  auto v_unit = [&](int u) { return *unit(p.v, u < UPC ? page_a : page_b, un / UPC * UPC + u % UPC); };
  uint4 k{}, v0{}, v1{};
  if (in) {
    k = *unit(p.k, sk < VU ? page_a : page_b, sk % VU);
    v0 = v_unit(u0);
    if (sh != 0) v1 = v_unit(u1);
  }
  if constexpr (SYNC) {
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  if (in) {
    store_nt(unit(p.k, dst, un), k);
    store_nt(unit(p.v, dst, un), funnel16(v0, v1, sh));
  }
}

// A page of a few runs (spans end or begin inside it, or it is the last and
// not full): run r is the old tokens [src[r], ..) for slots [at[r], at[r + 1])
// of the page (the last run ends at nv), its first token in old page page_a[r]
// and its last in page_b[r].
constexpr int kFewRuns = 4;
struct FewRuns {
  int n;
  int at[kFewRuns], src[kFewRuns], last[kFewRuns], page_a[kFewRuns], page_b[kFewRuns];
};

// w with the bytes from n on (n <= 0: all, n >= 4: none) replaced by x's.
__device__ inline uint32_t bytes_from(uint32_t w, uint32_t x, int n) {
  const uint32_t m = n <= 0 ? ~0u : n >= 4 ? 0u : ~0u << (8 * n);
  return (w & ~m) | (x & m);
}

// Such a page, moved as a page of one run is: a V^T unit is put together from
// one funnel shift per run that reaches into it, the shift uniform for each
// run, later runs over earlier ones, with every load in flight at once.
// Of 16K tokens of 24 layers (8 heads of 128) 8 in every 10 kept: 579 us a
// call, against 708 with each element from its own page, as pages of more
// runs are moved, and 645 with the source pages staged in LDS; 8 in every 16:
// 398, 465 and 424.  Not for an in-place eviction: its pages of one run got
// slower by the registers (16K tokens of 24 layers of 64 channels, 400 of 700
// kept: 463 -> 475 us with the appends).
template <int D, class E>
__device__ inline void move_few(const Pools &p, int row0, int nv, const FewRuns &f, int dst) {
  constexpr int VU = kPageUnits<D, E>;
  constexpr int U = VU / P;                // units per K row
  constexpr int EPU = 16 / (int)sizeof(E); // V^T elements per unit
  constexpr int UPC = P / EPU;             // units per channel's row
  const int un = threadIdx.x % VU, row = row0 + threadIdx.x / VU;
  const bool in = row < p.nl * p.hkv;
  const int j = un / U, c = un % UPC;
  auto unit = [&](uint16_t *pool, int page, int u) {
    return reinterpret_cast<uint4 *>(reinterpret_cast<E *>(pool) + row * p.head_stride +
                                     (int64_t)page * p.page_stride) + u;
  };
  uint4 k{}, v0[kFewRuns], v1[kFewRuns];
  if (in) {
    int src = f.src[0] + j, page = 0; // old token of K row j, and its page
#pragma unroll
    for (int r = 0; r < kFewRuns; ++r)
      if (r < f.n && j >= f.at[r]) {
        src = f.src[r] + j - f.at[r];
        page = src / P == f.src[r] / P ? f.page_a[r] : f.page_b[r];
      }
    if (j < nv) k = *unit(p.k, page, src % P * U + un % U);
  }
#pragma unroll
  for (int r = 0; r < kFewRuns; ++r) {
    v0[r] = v1[r] = uint4{};
    if (r >= f.n) continue;
    const int len = f.last[r] - f.src[r] + 1;
    // the old index that goes with the unit's first slot (no token moves
    // up, so src >= at), its unit and the next, within those of the run
    const int x = f.src[r] - f.at[r] + c * EPU, u0 = x / EPU;
    const int lo = f.src[r] / EPU, hi = f.last[r] / EPU;
    auto v_unit = [&](int u) {
      return *unit(p.v, u / UPC == f.src[r] / P ? f.page_a[r] : f.page_b[r], un / UPC * UPC + u % UPC);
    };
    if (in && f.at[r] < (c + 1) * EPU && f.at[r] + len > c * EPU) {
      if (u0 >= lo) v0[r] = v_unit(u0);
      if (x % EPU != 0 && u0 < hi) v1[r] = v_unit(u0 + 1);
    }
  }
  uint4 v{};
#pragma unroll
  for (int r = 0; r < kFewRuns; ++r) {
    if (r >= f.n) continue;
    const uint4 x = funnel16(v0[r], v1[r], (f.src[r] - f.at[r]) % EPU * (int)sizeof(E));
    const int from = (f.at[r] - c * EPU) * (int)sizeof(E);
    v = make_uint4(bytes_from(v.x, x.x, from), bytes_from(v.y, x.y, from - 4), bytes_from(v.z, x.z, from - 8),
                   bytes_from(v.w, x.w, from - 12));
  }
  const int end = (nv - c * EPU) * (int)sizeof(E); // slots past the tokens: zero
  v = make_uint4(bytes_from(v.x, 0u, end), bytes_from(v.y, 0u, end - 4), bytes_from(v.z, 0u, end - 8),
                 bytes_from(v.w, 0u, end - 12));
  if (in) {
    if (j < nv) store_nt(unit(p.k, dst, un), k);
    store_nt(unit(p.v, dst, un), v);
  }
}

// Any other page: the same rows and units, each slot from its own old page,
// the elements of a V^T unit one by one (they share their source's lines).
// spage and sslot (LDS) hold the page id and slot of each of the nv sources.
template <int D, class E, bool SYNC>
__device__ inline void move_mixed(const Pools &p, int row0, int nv, const int *spage, const int *sslot,
                                  int dst) {
  constexpr int VU = kPageUnits<D, E>;
  constexpr int U = VU / P;                // units per K row
  constexpr int EPU = 16 / (int)sizeof(E); // V^T elements per unit
  constexpr int UPC = P / EPU;             // units per channel's row
  const int un = threadIdx.x % VU, row = row0 + threadIdx.x / VU;
  const bool in = row < p.nl * p.hkv;
  const int j = un / U, d = un / UPC, c = un % UPC;
  auto chunk = [&](uint16_t *pool, int page) {
    return reinterpret_cast<E *>(pool) + row * p.head_stride + (int64_t)page * p.page_stride;
  };
  uint4 k{}, v{};
  if (in) {
    if (j < nv) k = reinterpret_cast<const uint4 *>(chunk(p.k, spage[j]) + sslot[j] * D)[un % U];
    E out[EPU];
#pragma unroll
    for (int e = 0; e < EPU; ++e) {
      const int jv = c * EPU + e;
      out[e] = jv < nv ? chunk(p.v, spage[jv])[d * P + sslot[jv]] : (E)0;
    }
    __builtin_memcpy(&v, out, 16);
  }
  if constexpr (SYNC) {
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  if (in) {
    if (j < nv) store_nt(reinterpret_cast<uint4 *>(chunk(p.k, dst)) + un, k);
    store_nt(reinterpret_cast<uint4 *>(chunk(p.v, dst)) + un, v);
  }
}

// One destination page, tokens [t0, t0 + nv) of the compacted sequence, rows
// from row0 on, and (with row 0) its positions: src_of gives a token's old
// index (s0 and s1 the first and last, which are P - 1 apart in a whole page
// exactly if it is a run), pt_row the old pages.
template <int D, class E, bool SYNC, class SRC>
__device__ inline void move_page(const Pools &p, int row0, int t0, int nv, int s0, int s1,
                                 const SRC &src_of, const int32_t *pt_row, int dst, int *spage,
                                 int *sslot) {
  const int t = threadIdx.x;
  const bool run = nv == P && s1 - s0 == P - 1;
  const bool with_pos = row0 == 0 && t < nv;
  int32_t pos = 0;
  if (run) {
    const int page_a = pt_row[s0 / P], page_b = pt_row[s1 / P]; // the same page when s0 % P = 0
    if (with_pos) pos = p.pos[(int64_t)(s0 % P + t < P ? page_a : page_b) * P + (s0 + t) % P];
    move_run<D, E, SYNC>(p, row0, page_a, page_b, s0 % P, dst);
  } else {
    FewRuns f;
    f.n = kFewRuns + 1;
    int src = 0;
    if constexpr (SYNC) {
      if (t < nv) src = src_of(t0 + t);
    } else { // every wave finds the page's runs for itself, all of them the same
      const int lane = t & 63;
      if (lane < nv) src = src_of(t0 + lane);
      const int before = __shfl_up(src, 1);
      uint64_t starts = __ballot(lane < nv && (lane == 0 || src != before + 1));
      f.n = __popcll(starts);
#pragma unroll
      for (int r = 0; r < kFewRuns; ++r) {
        if (r >= f.n || f.n > kFewRuns) continue;
        f.at[r] = __builtin_ctzll(starts);
        starts &= starts - 1;
        const int next = starts ? __builtin_ctzll(starts) : nv;
        f.src[r] = __builtin_amdgcn_readlane(src, f.at[r]);
        f.last[r] = f.src[r] + next - f.at[r] - 1;
        f.page_a[r] = pt_row[f.src[r] / P];
        f.page_b[r] = pt_row[f.last[r] / P];
      }
    }
    if (f.n <= kFewRuns) {
      if (with_pos) pos = p.pos[(int64_t)pt_row[src / P] * P + src % P];
      move_few<D, E>(p, row0, nv, f, dst);
    } else {
      if (t < nv) {
        spage[t] = pt_row[src / P];
        sslot[t] = src % P;
      }
      __syncthreads();
      if (with_pos) pos = p.pos[(int64_t)spage[t] * P + sslot[t]];
      move_mixed<D, E, SYNC>(p, row0, nv, spage, sslot, dst);
      if constexpr (SYNC) __syncthreads(); // the next page reuses the LDS
    }
  }
  if (with_pos) p.pos[(int64_t)dst * P + t] = pos;
}

// ---------------------------------------------------------------------------
// Gather: a workgroup per (fresh page pi0 + b, kGatherRows rows) fills
// destination page fp + pi0 + b with the kept tokens (fp + pi0 + b) * P + j,
// j < P, j below L'.  Kept token t comes from old token source_of(t) of the
// old pages, whose ids the page-table row still holds (the new ids are
// written there after the last gather).  When the spans travel in the kernel
// arguments, the first launch of an eviction also writes the eviction index
// (keep, dst, src_of) in its first index_blocks workgroups, alongside the
// copies, and takes the sources from the span list so that it does not wait
// for the index; later launches of a chunked eviction, and every launch after
// a separate index kernel, read src_of.  A fresh page is never a page this or
// a later gather reads: it is either a page nothing held or an old page whose
// tokens earlier gathers have all moved, so nothing is read after being
// written.
template <int D, class E>
__global__ __launch_bounds__(256) void k_evict_gather(Pools p, GatherArgs a) {
  __shared__ int spage[P], sslot[P];
  __shared__ int32_t lsp[3 * kInlineSpans];
  const int n = a.n_new;
  const int lin = blockIdx.x + blockIdx.y * gridDim.x;
  // the launch that writes the index takes the sources from the spans; later
  // launches of a chunked eviction read them from src_of (one round of loads)
  const bool from_spans = a.index_blocks > 0;
  const int32_t *spans = from_spans ? stage_spans(a.ev, lsp) : nullptr;
  if (lin < a.index_blocks) {
    evict_index_block(a.ev, spans, lin);
    return;
  }
  // Work item w = (group of rows, tail page pl), page fastest.  Workgroups are
  // dealt to the 8 XCDs in turn, so each XCD takes a contiguous range of
  // w: neighbouring destination pages, which share source pages, then hit
  // the same L2.  (Workgroups past the last item, which round the grid up
  // to whole rows, have nothing to do.)
  const int groups = (p.nl * p.hkv + kGatherRows<D, E> - 1) / kGatherRows<D, E>;
  const int total = n * groups;
  const int gl = lin - a.index_blocks;
  if (gl >= total) return;
  const int x = gl % 8, q = total / 8, r = total % 8;
  const int w = x * q + min(x, r) + gl / 8;
  const int pl = w % n;
  const int row0 = w / n * kGatherRows<D, E>;
  const int t0 = (a.fp + a.pi0 + pl) * P;
  const int nv = min(P, a.new_len - t0);
  const int ns = a.ev.n_spans;
  auto src_of = [&](int t) { return from_spans ? source_of(spans, ns, t) : a.ev.src_of[t]; };
  const int s0 = __builtin_amdgcn_readfirstlane(src_of(t0));
  const int s1 = __builtin_amdgcn_readfirstlane(src_of(t0 + nv - 1));
  if (a.remap && nv == P && s0 % P == 0 && s1 - s0 == P - 1) return; // remapped, not copied
  move_page<D, E, false>(p, row0, t0, nv, s0, s1, src_of, a.pt_row, new_page_id(a.ids, pl), spage, sslot);
}

// ---------------------------------------------------------------------------
// In-place eviction: tail page k of the compacted sequence is written to
// ids(k), normally the old page at list index fp + k itself.  Its kept
// tokens come from old list indices >= fp + k, so a page is never read after
// a page before it in the tail has been rewritten, as long as the pages of
// one launch read no page of the launch but their own: the host cuts the
// tail into such runs (round mode, a workgroup per page and kGatherRows rows,
// like the gather), or hands a run of short ones to sweep mode, where one
// workgroup per kGatherRows rows takes the pages in order.  Either way a
// workgroup has loaded everything a page of its rows needs before it writes
// the page, which may be one of its own sources.
template <int D, class E>
__global__ __launch_bounds__(256) void k_evict_inplace(Pools p, InplaceArgs a) {
  __shared__ int spage[P], sslot[P];
  int pl0, pl1, row0;
  if (a.sweep) {
    pl0 = 0;
    pl1 = a.n_pages;
    row0 = blockIdx.x * kGatherRows<D, E>;
  } else {
    // consecutive pages of one group of rows to one XCD, as in the gather
    const int n = gridDim.x;
    const int total = n * gridDim.y;
    const int lin = blockIdx.x + blockIdx.y * n;
    const int x = lin % 8, q = total / 8, r = total % 8;
    const int w = x * q + min(x, r) + lin / 8;
    pl0 = w % n;
    pl1 = pl0 + 1;
    row0 = w / n * kGatherRows<D, E>;
  }
  auto src_of = [&](int t) { return a.src_of[t]; };
  for (int pl = pl0; pl < pl1; ++pl) {
    const int k = a.k0 + pl;
    const int t0 = (a.fp + k) * P;
    const int nv = min(P, a.new_len - t0);
    const int s0 = __builtin_amdgcn_readfirstlane(src_of(t0));
    const int s1 = __builtin_amdgcn_readfirstlane(src_of(t0 + nv - 1));
    move_page<D, E, true>(p, row0, t0, nv, s0, s1, src_of, a.pt_row, new_page_id(a.ids, k), spage, sslot);
  }
}

} // namespace

// ---------------------------------------------------------------------------
namespace {
constexpr int64_t kMemSideCache = 256ll << 20;

template <int D, class E>
hipError_t append_dispatch(const Pools &p, const AppendArgs &a, const uint16_t *kn,
                           const uint16_t *vn, hipStream_t s) {
  const dim3 grid((a.n_pages + kAppendGroup<D> - 1) / kAppendGroup<D>, p.nl * p.hkv), block(256);
  const int64_t elems = 2ll * p.nl * a.n_total * p.hkv * D; // K and V
  if (elems * 2 > kMemSideCache)
    hipLaunchKernelGGL((k_append<D, E, 2>), grid, block, 0, s, p, a, kn, vn);
  else if (elems * (int64_t)(2 + sizeof(E)) > kMemSideCache)
    hipLaunchKernelGGL((k_append<D, E, 1>), grid, block, 0, s, p, a, kn, vn);
  else
    hipLaunchKernelGGL((k_append<D, E, 0>), grid, block, 0, s, p, a, kn, vn);
  return hipGetLastError();
}
} // namespace

hipError_t launch_append(const Pools &p, const AppendArgs &a, const void *k_new,
                         const void *v_new, hipStream_t s) {
  const auto *kn = static_cast<const uint16_t *>(k_new);
  const auto *vn = static_cast<const uint16_t *>(v_new);
  if (p.kv8)
    return p.d == 128 ? append_dispatch<128, uint8_t>(p, a, kn, vn, s)
                      : append_dispatch<64, uint8_t>(p, a, kn, vn, s);
  return p.d == 128 ? append_dispatch<128, uint16_t>(p, a, kn, vn, s)
                    : append_dispatch<64, uint16_t>(p, a, kn, vn, s);
}

hipError_t launch_append_batch(const Pools &p, const AppendBatchArgs &a, const void *k_new,
                               const void *v_new, hipStream_t s) {
  dim3 grid(a.n, p.nl * p.hkv);
  const auto *kn = static_cast<const uint16_t *>(k_new);
  const auto *vn = static_cast<const uint16_t *>(v_new);
  if (p.kv8) {
    if (p.d == 128)
      hipLaunchKernelGGL(k_append_batch8<128>, grid, dim3(64), 0, s, p, a, kn, vn);
    else
      hipLaunchKernelGGL(k_append_batch8<64>, grid, dim3(64), 0, s, p, a, kn, vn);
  } else if (p.d == 128)
    hipLaunchKernelGGL(k_append_batch<128>, grid, dim3(64), 0, s, p, a, kn, vn);
  else
    hipLaunchKernelGGL(k_append_batch<64>, grid, dim3(64), 0, s, p, a, kn, vn);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *dst, int32_t value, int32_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, s, dst, value, n);
  return hipGetLastError();
}

hipError_t launch_step_upload(void *dst, const void *src, int64_t bytes, const SetEntries &a,
                              hipStream_t s) {
  if (a.n > kMaxBatch || bytes % 16 != 0) return hipErrorInvalidValue;
  const int32_t n16 = (int32_t)(bytes / 16);
  hipLaunchKernelGGL(k_step_upload, dim3((n16 + 255) / 256), dim3(256), 0, s, static_cast<uint4 *>(dst),
                     static_cast<const uint4 *>(src), n16, a);
  return hipGetLastError();
}

hipError_t launch_fork(const Pools &p, int32_t *dst, const int32_t *src, int32_t n, int32_t src_tail,
                       int32_t tail_page, hipStream_t s) {
  const int32_t ptb = (n + 1 + 255) / 256;
  const dim3 grid(ptb + (tail_page >= 0 ? p.nl * p.hkv : 0)), block(256);
  if (p.kv8) {
    if (p.d == 128)
      hipLaunchKernelGGL((k_fork<128, uint8_t>), grid, block, 0, s, p, dst, src, n, src_tail, tail_page, ptb);
    else
      hipLaunchKernelGGL((k_fork<64, uint8_t>), grid, block, 0, s, p, dst, src, n, src_tail, tail_page, ptb);
  } else if (p.d == 128)
    hipLaunchKernelGGL((k_fork<128, uint16_t>), grid, block, 0, s, p, dst, src, n, src_tail, tail_page, ptb);
  else
    hipLaunchKernelGGL((k_fork<64, uint16_t>), grid, block, 0, s, p, dst, src, n, src_tail, tail_page, ptb);
  return hipGetLastError();
}

hipError_t launch_evict_index(const EvictArgs &a, hipStream_t s) {
  const int nblk = (a.n_tokens + kScanBlock - 1) / kScanBlock;
  if (nblk == 0) return hipSuccess;
  hipLaunchKernelGGL(k_evict_index, dim3(nblk), dim3(kScanThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_write_ids(int32_t *dst, const NewIds &ids, int32_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_write_ids, dim3((n + 255) / 256), dim3(256), 0, s, dst, ids, n);
  return hipGetLastError();
}

// Groups of rows that a workgroup of the gather takes.
static int gather_groups(const Pools &p) {
  const int rows = p.nl * p.hkv;
  const int per = p.kv8 ? (p.d == 128 ? kGatherRows<128, uint8_t> : kGatherRows<64, uint8_t>)
                        : (p.d == 128 ? kGatherRows<128, uint16_t> : kGatherRows<64, uint16_t>);
  return (rows + per - 1) / per;
}

hipError_t launch_evict_inplace(const Pools &p, const InplaceArgs &a, hipStream_t s) {
  if (a.n_pages <= 0) return hipSuccess;
  const int groups = gather_groups(p);
  const dim3 grid = a.sweep ? dim3(groups) : dim3(a.n_pages, groups);
  if (p.kv8) {
    if (p.d == 128)
      hipLaunchKernelGGL((k_evict_inplace<128, uint8_t>), grid, dim3(256), 0, s, p, a);
    else
      hipLaunchKernelGGL((k_evict_inplace<64, uint8_t>), grid, dim3(256), 0, s, p, a);
  } else if (p.d == 128)
    hipLaunchKernelGGL((k_evict_inplace<128, uint16_t>), grid, dim3(256), 0, s, p, a);
  else
    hipLaunchKernelGGL((k_evict_inplace<64, uint16_t>), grid, dim3(256), 0, s, p, a);
  return hipGetLastError();
}

hipError_t launch_evict_gather(const Pools &p, const GatherArgs &a, hipStream_t s) {
  if (a.n_new == 0) return hipSuccess;
  // rows of n_new workgroups: the copies' groups of (layer, head) rows, then
  // enough for the index blocks
  const int rows = gather_groups(p) + (a.index_blocks + a.n_new - 1) / a.n_new;
  dim3 grid(a.n_new, rows);
  if (p.kv8) {
    if (p.d == 128)
      hipLaunchKernelGGL((k_evict_gather<128, uint8_t>), grid, dim3(256), 0, s, p, a);
    else
      hipLaunchKernelGGL((k_evict_gather<64, uint8_t>), grid, dim3(256), 0, s, p, a);
  } else if (p.d == 128)
    hipLaunchKernelGGL((k_evict_gather<128, uint16_t>), grid, dim3(256), 0, s, p, a);
  else
    hipLaunchKernelGGL((k_evict_gather<64, uint16_t>), grid, dim3(256), 0, s, p, a);
  return hipGetLastError();
}

} // namespace sq
