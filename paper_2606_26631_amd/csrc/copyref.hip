// Reference copy kernels for the bandwidth measurement (not part of the PRCR
// path): what a plain device copy attains on this GPU, and what a copy with
// exactly the rebinding kernel's addresses attains.
//
//   prcr_copyref_stream   src -> dst, each workgroup owning one contiguous chunk:
//                         the attainable read + write rate of the GPU.
//   prcr_copyref_decode_read  decode attention's reads with no arithmetic: every K and
//                         V row of one layer's attended slots, with the bf16
//                         decode kernel's tiles, lane layouts, loads in flight and
//                         order of workgroups (four waves each), each sequence split
//                         evenly over as many workgroups as the caller says.
//   prcr_copyref_prefill  prefill capture's access pattern with no arithmetic: one
//                         layer's raw K/V rows of every prompt token to the
//                         contiguous cache at slot s, and visual tokens' rows to the
//                         memory, with the prefill kernel's wave mapping (8
//                         consecutive (token, head) rows per wave, lane layout as
//                         in the rebind).
//   prcr_copyref_pattern  the rebind's own access pattern with no arithmetic and no
//                         metadata: per selected token, its (layer, head) rows are
//                         read from one contiguous run of the memory and written to
//                         the cache rows of its slot, with the rebinding kernel's
//                         wave structure (one wave per token x run of rows, four
//                         waves per workgroup, 16-row load batches with the next
//                         batch in flight) and dispatch order (token fastest, then
//                         row group, then the key array before the value array).
//
// They use 16-byte non-temporal loads and stores, as the kernels do.  Offsets
// are byte offsets computed by the caller, who checks them against the arrays.
#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 ld(const char *p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
}
__device__ __forceinline__ void st(char *p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(p));
}

constexpr int kThreads = 256;
constexpr int kStreamUnroll = 4;     // 16-byte chunks per thread per pass: 16 KB per workgroup

__global__ __launch_bounds__(kThreads) void stream_kernel(const char *src, char *dst, int64_t bytes,
                                                          int64_t chunk) {
  const int64_t base = static_cast<int64_t>(blockIdx.x) * chunk;
  const int64_t end = base + chunk < bytes ? base + chunk : bytes;
  for (int64_t i = base + threadIdx.x * 16; i < end; i += kStreamUnroll * kThreads * 16) {
    u32x4 v[kStreamUnroll];
#pragma unroll
    for (int u = 0; u < kStreamUnroll; ++u) {
      const int64_t j = i + static_cast<int64_t>(u) * kThreads * 16;
      if (j < end) v[u] = ld(src + j);
    }
#pragma unroll
    for (int u = 0; u < kStreamUnroll; ++u) {
      const int64_t j = i + static_cast<int64_t>(u) * kThreads * 16;
      if (j < end) st(dst + j, v[u]);
    }
  }
}

struct PatternParams {
  const char *src[2];          // key memory, value memory
  char *dst[2];                // key cache, value cache
  const int64_t *src_tok;      // [n_tok] byte offset of token g's first row in the memory
  const int64_t *dst_tok;      // [n_tok] byte offset of token g's row 0 in the cache
  int64_t group_stride;        // cache byte distance between consecutive row groups of G rows
  int32_t n_tok, rows_total, rows_per_wave, n_row_groups, group_log2;
};

// Row r of a token goes from src_tok + r * 256 to
// dst_tok + (r >> group_log2) * group_stride + (r & (2^group_log2 - 1)) * 256:
// contiguous caches use group_log2 = 0 and the cache's row stride, paged caches
// the KV-head count and the layer stride of the block pool.  Rows are 256 bytes
// (head_dim 128, bf16).  As in the rebinding kernel, a lane holds one 16-byte
// chunk of the first half of a row and the same chunk of the second half (8
// lanes per row, 8 rows per pass), two passes per batch of loads.
__global__ __launch_bounds__(kThreads) void pattern_kernel(const PatternParams p) {
  constexpr int kRowBytes = 256, kHalf = 128, kLanesPerRow = 8, kRowsPerPass = 8, kUnroll = 2;
  constexpr int kStep = kRowsPerPass * kUnroll;        // 16 rows per batch of loads
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n_tblk = (static_cast<int64_t>(p.n_tok) + 3) / 4;
  const int64_t L = blockIdx.x;
  const int64_t tblk = L % n_tblk;
  const int grp = static_cast<int>((L / n_tblk) % p.n_row_groups);
  const int arr = L < n_tblk * p.n_row_groups ? 0 : 1;
  const int64_t g = tblk * 4 + wave;
  if (g >= p.n_tok) return;
  const int r = lane / kLanesPerRow, c = lane % kLanesPerRow;
  const int row0 = grp * p.rows_per_wave;
  const int row_end = min(p.rows_total, row0 + p.rows_per_wave);
  const int gmask = (1 << p.group_log2) - 1;
  const char *s = p.src[arr] + p.src_tok[g] + c * 16;
  char *d = p.dst[arr] + p.dst_tok[g] + c * 16;
  auto dst_off = [&](int row) -> int64_t {
    return static_cast<int64_t>(row >> p.group_log2) * p.group_stride +
           static_cast<int64_t>(row & gmask) * kRowBytes;
  };
  u32x4 lo[kUnroll], hi[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const int64_t o = static_cast<int64_t>(min(row0 + u * kRowsPerPass + r, row_end - 1)) * kRowBytes;
    lo[u] = ld(s + o);
    hi[u] = ld(s + o + kHalf);
  }
  int rb = row0;
  for (; rb + kStep < row_end; rb += kStep) {
    u32x4 nlo[kUnroll], nhi[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t o =
          static_cast<int64_t>(min(rb + kStep + u * kRowsPerPass + r, row_end - 1)) * kRowBytes;
      nlo[u] = ld(s + o);
      nhi[u] = ld(s + o + kHalf);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t o = dst_off(rb + u * kRowsPerPass + r);
      st(d + o, lo[u]);
      st(d + o + kHalf, hi[u]);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      lo[u] = nlo[u];
      hi[u] = nhi[u];
    }
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const int row = rb + u * kRowsPerPass + r;
    if (row < row_end) {
      const int64_t o = dst_off(row);
      st(d + o, lo[u]);
      st(d + o + kHalf, hi[u]);
    }
  }
}

struct DecodeReadParams {
  const char *k;               // cache keys
  const char *v;               // cache values
  const int32_t *block_table;  // paged: [batch][max_blocks]
  const int32_t *len;          // [batch] attended slots
  uint32_t *out;               // [batch][n_kv_heads][n_split] one word per workgroup
  int32_t n_layers, n_kv_heads, layer, s_max, block_size, max_blocks, n_blocks, n_split, paged;
};

// One workgroup of four waves per (KV head, sequence, split), splits outermost, with the
// bf16 decode kernel's accesses.  Rows are 256 bytes (head_dim 128, bf16).  At most 64
// sequences are taken longest first, in reverse in every second round of 256 workgroups.
// The sequence's keys are split in whole rounds of 128 keys; a wave takes tiles of 32
// keys 128 keys apart.  Key loads take whole cache lines of 8 rows, value loads 4 whole
// rows; one buffer of each, the next tile's keys loaded once this tile's keys are used and
// its values once this tile's values are.  Paged caches read a block-table entry per key, two
// tiles ahead: one base per 16 keys where the block size is a multiple of 16, else a row
// per key.  Keys past the chunk (or in a block outside the pool) read a row that exists and
// are left out of the result: the exclusive or of the words read, one value per workgroup.
template <bool kPaged, bool kHalfBlocks>
__global__ __launch_bounds__(kThreads) void decode_read_kernel(const DecodeReadParams p) {
  constexpr int kRowBytes = 256, kTile = 32, KPB = 128, kUnits = 256;
  const int split = blockIdx.z, kvh = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n16 = lane % 16, kj = lane / 16;
  const int nb = static_cast<int>(gridDim.y);
  const uint32_t before = static_cast<uint32_t>(split) * gridDim.x * gridDim.y;
  int b = (before / kUnits) & 1 ? nb - 1 - static_cast<int>(blockIdx.y) : static_cast<int>(blockIdx.y);
  if (nb <= 64) {
    const int mine = lane < nb ? max(p.len[lane], 0) : -1;
    int rank = 0;
    for (int i = 0; i < nb; ++i) {
      const int other = __builtin_amdgcn_readlane(mine, i);
      rank += (other > mine) || (other == mine && i < lane);
    }
    const unsigned long long hit = __ballot(lane < nb && rank == b);
    b = hit ? __ffsll(static_cast<long long>(hit)) - 1 : b;
  }
  // Lengths clamped to the capacity: every access stays inside the arrays whatever the inputs.
  const int64_t cap = kPaged ? static_cast<int64_t>(p.max_blocks) * p.block_size : p.s_max;
  const int len = static_cast<int>(min(max(static_cast<int64_t>(p.len[b]), int64_t{0}), cap));
  const int per = (len + p.n_split - 1) / p.n_split;
  const int64_t chunk = (static_cast<int64_t>(per) + KPB - 1) / KPB * KPB;
  const int j0 = static_cast<int>(min(static_cast<int64_t>(len), split * chunk));
  const int j1 = static_cast<int>(min(static_cast<int64_t>(len), j0 + chunk));
  uint32_t *const out = p.out + (static_cast<int64_t>(b) * p.n_kv_heads + kvh) * p.n_split + split;
  if (j0 >= j1) {
    if (threadIdx.x == 0) *out = 0;
    return;
  }
  const int64_t row_layer = static_cast<int64_t>(p.layer) * p.n_blocks * p.block_size;   // paged
  const int64_t row_any = kPaged ? row_layer * p.n_kv_heads + kvh
                                 : ((static_cast<int64_t>(b) * p.n_layers + p.layer) * p.n_kv_heads + kvh) * p.s_max;
  // Slot in the pool of key lane % 32 of the tile at tb, or -1.
  auto slot_of = [&](int tb) -> int64_t {
    if constexpr (!kPaged) return 0;
    const int j = tb + lane % kTile, js = j < j1 ? j : 0, lb = js / p.block_size;
    const int32_t blk = p.block_table[static_cast<int64_t>(b) * p.max_blocks + lb];
    return j < j1 && blk >= 0 && blk < p.n_blocks
               ? static_cast<int64_t>(blk) * p.block_size + (js - lb * p.block_size) : -1;
  };
  struct Rows {
    int64_t base[2];
    int last[2];
    int slot;
    uint32_t live;
  };
  auto rows_of = [&](int tb, int64_t slot) -> Rows {
    Rows t{};
    const int n_in = min(max(j1 - tb, 0), kTile);
    t.live = n_in >= kTile ? ~0u : (1u << n_in) - 1u;
    if constexpr (!kPaged) {
      const int tc = min(tb, j1 - 1);
      t.base[0] = row_any + tc;
      t.last[0] = j1 - 1 - tc;
    } else {
      t.live = static_cast<uint32_t>(__ballot(slot >= 0));   // lanes t and t + 32 agree
      if constexpr (kHalfBlocks) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t lh = (t.live >> (16 * h)) & 0xFFFFu;
          const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(slot), 16 * h);
          const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(slot >> 32), 16 * h);
          const int64_t first = static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
          t.base[h] = lh != 0 ? (row_layer + first) * p.n_kv_heads + kvh : row_any;
          t.last[h] = lh != 0 ? __popc(lh) - 1 : 0;
        }
      } else {
        t.slot = slot >= 0 ? static_cast<int>(slot) : 0;
      }
    }
    return t;
  };
  const uint32_t step = kPaged ? static_cast<uint32_t>(p.n_kv_heads) * kRowBytes : kRowBytes;
  auto offset = [&](const Rows &t, int key, int half) -> int64_t {
    if constexpr (!kPaged)
      return t.base[0] * kRowBytes + static_cast<uint32_t>(min(key, t.last[0])) * step;
    else if constexpr (kHalfBlocks)
      return t.base[half] * kRowBytes + static_cast<uint32_t>(min(key - 16 * half, t.last[half])) * step;
    else
      return (row_layer + static_cast<int64_t>(static_cast<uint32_t>(__shfl(t.slot, key)))) * step +
             static_cast<int64_t>(kvh) * kRowBytes;
  };
  // Key of load (st, kk): line kk / 2 of the rows of product columns 0..7 (kk even) or 8..15.
  auto key_of = [&](int st, int kk) -> int { return 8 * (n16 % 8 / 4) + n16 % 4 + 4 * st + 16 * (kk % 2); };
  auto load_k = [&](const Rows &t, u32x4 (&kd)[2][4]) {
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        kd[st][kk] = ld(p.k + offset(t, key_of(st, kk), kk % 2) + (n16 / 8) * 64 + kj * 16 + kk / 2 * 128);
  };
  auto load_v = [&](const Rows &t, u32x4 (&vd)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u) vd[u] = ld(p.v + offset(t, 4 * u + kj, u / 4) + n16 * 16);
  };
  uint32_t acc = 0;
  auto fold = [&](u32x4 w, bool in) { acc ^= in ? w.x ^ w.y ^ w.z ^ w.w : 0u; };
  const int jw = j0 + wave * kTile;
  u32x4 kr[2][4], vv[8];
  const int64_t s0 = slot_of(jw);
  int64_t s_next = slot_of(jw + KPB);
  Rows t = rows_of(jw, s0);
  load_k(t, kr);
  load_v(t, vv);
  for (int jt = jw; jt < j1; jt += KPB) {
    const uint32_t live = t.live;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) fold(kr[st][kk], (live >> key_of(st, kk)) & 1u);
    t = rows_of(jt + KPB, s_next);
    s_next = slot_of(jt + 2 * KPB);
    load_k(t, kr);
#pragma unroll
    for (int u = 0; u < 8; ++u) fold(vv[u], (live >> (4 * u + kj)) & 1u);
    load_v(t, vv);
  }
  for (int o = 32; o > 0; o >>= 1) acc ^= __shfl_xor(acc, o);
  __shared__ uint32_t s_acc[kThreads / 64];
  if (lane == 0) s_acc[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t a = 0;
    for (int w = 0; w < kThreads / 64; ++w) a ^= s_acc[w];
    *out = a;
  }
}

struct PrefillPatternParams {
  const char *raw_k, *raw_v;   // [batch][s_src][H][128] bf16 rows
  const int32_t *vis_index;    // [batch][s_src]: visual index or -1
  const int32_t *n_tokens;     // [batch]
  char *cache_k, *cache_v;     // contiguous [batch][n_layers][H][s_max][128]
  char *mem_k, *mem_v;         // [batch][max_visual][n_layers][H][128]
  int32_t batch, s_src, n_kv_heads, n_layers, layer, s_max, max_visual;
};

// Rows are 256 bytes (head_dim 128, bf16); row R = (b * s_src + s) * H + h.
__global__ __launch_bounds__(kThreads) void prefill_pattern_kernel(const PrefillPatternParams p) {
  constexpr int kRowBytes = 256, kHalf = 128, kLanesPerRow = 8, kRowsPerWave = 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int H = p.n_kv_heads;
  const int64_t rows_all = static_cast<int64_t>(p.batch) * p.s_src * H;
  const int64_t R = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * kRowsPerWave + lane / kLanesPerRow;
  if (R >= rows_all) return;
  const int c = lane % kLanesPerRow;
  const int b = static_cast<int>(R / (static_cast<int64_t>(p.s_src) * H));
  const int64_t rem = R - static_cast<int64_t>(b) * p.s_src * H;
  const int s = static_cast<int>(rem / H), h = static_cast<int>(rem - static_cast<int64_t>(s) * H);
  const int nt = p.n_tokens[b];
  const int m = p.vis_index[static_cast<int64_t>(b) * p.s_src + s];
  if (s >= nt || s >= p.s_max) return;
  const int64_t o = R * kRowBytes + c * 16;
  const u32x4 kl = ld(p.raw_k + o), kh = ld(p.raw_k + o + kHalf);
  const u32x4 vl = ld(p.raw_v + o), vh = ld(p.raw_v + o + kHalf);
  const int64_t d = ((((static_cast<int64_t>(b) * p.n_layers + p.layer) * H + h) * p.s_max) + s) * kRowBytes + c * 16;
  st(p.cache_k + d, kl);
  st(p.cache_k + d + kHalf, kh);
  st(p.cache_v + d, vl);
  st(p.cache_v + d + kHalf, vh);
  if (m >= 0 && m < p.max_visual) {
    const int64_t mo = (((static_cast<int64_t>(b) * p.max_visual + m) * p.n_layers + p.layer) * H + h) * kRowBytes +
                       c * 16;
    st(p.mem_k + mo, kl);
    st(p.mem_k + mo + kHalf, kh);
    st(p.mem_v + mo, vl);
    st(p.mem_v + mo + kHalf, vh);
  }
}

}  // namespace

extern "C" {

// Copies `bytes` (a multiple of 16) from src to dst, `chunk` bytes per workgroup.
int prcr_copyref_stream(const void *src, void *dst, int64_t bytes, int64_t chunk,
                        hipStream_t stream) {
  if (src == nullptr || dst == nullptr || bytes <= 0 || bytes % 16 != 0 || chunk <= 0 ||
      chunk % 16 != 0)
    return 1;
  const int64_t grid = (bytes + chunk - 1) / chunk;
  if (grid > 0x7FFFFFFF / kThreads) return 2;
  stream_kernel<<<dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, stream>>>(
      static_cast<const char *>(src), static_cast<char *>(dst), bytes, chunk);
  return hipGetLastError() == hipSuccess ? 0 : 3;
}

// The rebind's access pattern over two arrays (keys, then values); see above.
int prcr_copyref_pattern(const void *src_k, const void *src_v, void *dst_k, void *dst_v,
                         const int64_t *src_tok, const int64_t *dst_tok, int32_t n_tok,
                         int32_t rows_total, int32_t rows_per_wave, int32_t group_log2,
                         int64_t group_stride, hipStream_t stream) {
  if (src_k == nullptr || src_v == nullptr || dst_k == nullptr || dst_v == nullptr ||
      src_tok == nullptr || dst_tok == nullptr || n_tok < 1 || rows_total < 1 ||
      rows_per_wave < 1 || group_log2 < 0 || group_log2 > 8)
    return 1;
  PatternParams p{};
  p.src[0] = static_cast<const char *>(src_k);
  p.src[1] = static_cast<const char *>(src_v);
  p.dst[0] = static_cast<char *>(dst_k);
  p.dst[1] = static_cast<char *>(dst_v);
  p.src_tok = src_tok;
  p.dst_tok = dst_tok;
  p.group_stride = group_stride;
  p.n_tok = n_tok;
  p.rows_total = rows_total;
  p.rows_per_wave = rows_per_wave;
  p.n_row_groups = (rows_total + rows_per_wave - 1) / rows_per_wave;
  p.group_log2 = group_log2;
  const int64_t grid = (static_cast<int64_t>(n_tok) + 3) / 4 * p.n_row_groups * 2;
  if (grid > 0x7FFFFFFF / kThreads) return 2;
  pattern_kernel<<<dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, stream>>>(p);
  return hipGetLastError() == hipSuccess ? 0 : 3;
}

// Decode attention's reads of one layer (see above): n_split workgroups per
// (sequence, KV head); out holds batch * n_kv_heads * n_split words.  Capacities are below
// 2^30 slots and a pool below 2^31, as decode attention's own.
int prcr_copyref_decode_read(const void *k, const void *v, const int32_t *block_table,
                             const int32_t *len, uint32_t *out, int32_t batch, int32_t n_layers,
                             int32_t n_kv_heads, int32_t layer, int32_t s_max, int32_t block_size,
                             int32_t max_blocks, int32_t n_blocks, int32_t n_split, int32_t paged,
                             hipStream_t stream) {
  if (k == nullptr || v == nullptr || len == nullptr || out == nullptr || batch < 1 ||
      batch > 65535 || n_kv_heads < 1 || n_kv_heads > 65535 || n_split < 1 || n_split > 65535 ||
      layer < 0 || layer >= n_layers || (paged && (block_table == nullptr || block_size < 1 ||
                                                   max_blocks < 1 || n_blocks < 1)) || (!paged && s_max < 1))
    return 1;
  constexpr int64_t kMostSlots = int64_t{1} << 30;
  if ((paged ? static_cast<int64_t>(max_blocks) * block_size : s_max) >= kMostSlots ||
      (paged && static_cast<int64_t>(n_blocks) * block_size >= 2 * kMostSlots))
    return 1;
  DecodeReadParams p{};
  p.k = static_cast<const char *>(k);
  p.v = static_cast<const char *>(v);
  p.block_table = block_table;
  p.len = len;
  p.out = out;
  p.n_layers = n_layers;
  p.n_kv_heads = n_kv_heads;
  p.layer = layer;
  p.s_max = s_max;
  p.block_size = block_size;
  p.max_blocks = max_blocks;
  p.n_blocks = n_blocks;
  p.n_split = n_split;
  p.paged = paged;
  const dim3 grid(n_kv_heads, batch, n_split);
  if (!paged)
    decode_read_kernel<false, false><<<grid, dim3(kThreads), 0, stream>>>(p);
  else if (block_size % 16 == 0)
    decode_read_kernel<true, true><<<grid, dim3(kThreads), 0, stream>>>(p);
  else
    decode_read_kernel<true, false><<<grid, dim3(kThreads), 0, stream>>>(p);
  return hipGetLastError() == hipSuccess ? 0 : 3;
}

// Prefill capture's access pattern for one layer (see above).
int prcr_copyref_prefill(const void *raw_k, const void *raw_v, const int32_t *vis_index,
                         const int32_t *n_tokens, void *cache_k, void *cache_v, void *mem_k,
                         void *mem_v, int32_t batch, int32_t s_src, int32_t n_kv_heads,
                         int32_t n_layers, int32_t layer, int32_t s_max, int32_t max_visual,
                         hipStream_t stream) {
  if (raw_k == nullptr || raw_v == nullptr || vis_index == nullptr || n_tokens == nullptr ||
      cache_k == nullptr || cache_v == nullptr || mem_k == nullptr || mem_v == nullptr ||
      batch < 1 || s_src < 1 || n_kv_heads < 1 || layer < 0 || layer >= n_layers || s_max < 1 ||
      max_visual < 1)
    return 1;
  PrefillPatternParams p{};
  p.raw_k = static_cast<const char *>(raw_k);
  p.raw_v = static_cast<const char *>(raw_v);
  p.vis_index = vis_index;
  p.n_tokens = n_tokens;
  p.cache_k = static_cast<char *>(cache_k);
  p.cache_v = static_cast<char *>(cache_v);
  p.mem_k = static_cast<char *>(mem_k);
  p.mem_v = static_cast<char *>(mem_v);
  p.batch = batch;
  p.s_src = s_src;
  p.n_kv_heads = n_kv_heads;
  p.n_layers = n_layers;
  p.layer = layer;
  p.s_max = s_max;
  p.max_visual = max_visual;
  const int64_t rows = static_cast<int64_t>(batch) * s_src * n_kv_heads;
  const int64_t grid = (rows + 31) / 32;
  if (grid > 0x7FFFFFFF / kThreads) return 2;
  prefill_pattern_kernel<<<dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, stream>>>(p);
  return hipGetLastError() == hipSuccess ? 0 : 3;
}

}  // extern "C"
