// Decode attention over the active cache (Eq. (14)): for each sequence and query
// head, softmax(RoPE(q, p_next) K^T * scale) V over the cache_len[b] keys of one
// layer, with grouped-query attention (n_q_heads = G * n_kv_heads, query head
// qh reads KV head qh / G).  The query is a text token, so its three M-RoPE
// positions are equal and the rotation is the 1-D one at p_next.
//
// Split-K flash decoding.  Kernel 1: one workgroup per (key chunk, KV head,
// sequence) streams its keys and values once for all G query heads of the
// group, and the sequence's keys are split evenly over its workgroups (plan_splits;
// with at most 64 sequences, the grid's sequence rows take the sequences longest
// first).  bf16 caches run both
// contractions on the matrix cores, 32 keys at a time (decode_partial_bf16_kernel);
// float32 caches take a 16-byte chunk of a key row per lane with scores reduced
// across the lanes of a row by DPP lane permutations (decode_partial_kernel).
// Both keep an online softmax in float32 that rescales only when a running
// maximum rose.  The workgroup's waves are merged in LDS and one (max, sum,
// weighted V) partial per query head and chunk is written to the caller's
// workspace.  Kernel 2 merges the chunks.
#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>
#include <type_traits>

#include "prcr_internal.h"
#include "rotary.h"

namespace prcr {
namespace {

constexpr int kWaves = 4;    // per workgroup, of the float32 kernel and the merge
constexpr int kIters = 2;    // float32 kernel: key rows per lane group in flight
constexpr int kUnits = 256;  // compute units of the chip

__device__ __forceinline__ void unpack(u32x4 w, float *x) {
#pragma unroll
  for (int q = 0; q < 4; ++q) x[q] = __uint_as_float(w[q]);
}

// Scores are kept in base-2 units (the query carries log2(e)), so every
// softmax weight is one hardware exp2.
constexpr double kLog2e = 1.4426950408889634;
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Lane permutation within a 16-lane DPP row (no LDS round trip).
template <int kCtrl>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xF, 0xF, false));
}

// Sum over the LPK consecutive lanes that hold one key row.  Every lane of the
// group ends with the same total: partners add the same two values at each step.
template <int LPK>
__device__ __forceinline__ float group_sum(float s) {
  static_assert(LPK == 16 || LPK == 32, "unsupported lane group");
  s += dpp<0xB1>(s);                               // quad permutation 1,0,3,2: lane ^ 1
  s += dpp<0x4E>(s);                               // quad permutation 2,3,0,1: lane ^ 2
  s += dpp<0x141>(s);                              // mirror in 8-lane halves: the other quad
  s += dpp<0x140>(s);                              // mirror in the 16-lane row: the other half
  if constexpr (LPK >= 32) s += __shfl_xor(s, 16);
  return s;
}

// Workgroup barrier that orders LDS accesses only: loads from memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sequence taken by workgroup row z, and its length entry.  With at most 64 sequences
// (lane l reads length l), the rows go to the sequences in order of decreasing length,
// ties by index.  Workgroups are dealt to the compute units in turn, so that each unit
// then holds chunks of long and of short sequences rather than a random mix: on a
// paged batch of 2,918-6,424 keys this measured 6 % faster.  Results do not depend
// on the order (each sequence is computed the same way by whichever row takes it).
//
// Every workgroup does this before its first key, so its waves share the work: a lane's
// rank is the number of keys (length, then lower index) above its own, and wave w counts
// among sequences 16 w to 16 w + 15.  With 64 sequences every wave counting all of them
// took 2.7 us (two compares each) or 1.1 us (one); the shared count takes 0.6.
template <int kWaves>
__device__ __forceinline__ int sequence_of_row(const DecodeParams &p, int lane, int z, int *len) {
  if (p.batch > kWave) {
    *len = p.cache_len[z];
    return z;
  }
  constexpr int kShare = kWave / kWaves;     // sequences a wave counts
  const int raw = lane < p.batch ? p.cache_len[lane] : 0;
  if (p.batch == 1) {
    *len = __builtin_amdgcn_readfirstlane(raw);
    return 0;
  }
  // Order of the lengths as one number: those above 2^25 - 1 count as equal.
  const uint32_t mine = lane < p.batch ? (static_cast<uint32_t>(min(max(raw, 0), (1 << 25) - 1)) << 6 | (63 - lane)) + 1 : 0;
  auto above = [&](int i0, int n) -> int {
    int count = 0;
#pragma unroll
    for (int i = 0; i < n; ++i)
      count += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine), i0 + i)) > mine ? 1 : 0;
    return count;
  };
  int rank = 0;
  if (p.batch <= kShare) {
    for (int i0 = 0; i0 < p.batch; i0 += 4) rank += above(i0, 4);
  } else {
    __shared__ int s_rank[kWaves][kWave];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    s_rank[wave][lane] = above(wave * kShare, kShare);
    lds_barrier();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) rank += s_rank[w][lane];
  }
  const unsigned long long hit = __ballot(lane < p.batch && rank == z);
  const int b = __builtin_amdgcn_readfirstlane(hit ? __ffsll(static_cast<long long>(hit)) - 1 : z);
  *len = __builtin_amdgcn_readlane(raw, b);
  return b;
}

// The bf16 kernel's grid is (KV head, row, split): the first workgroups to be placed are the
// first chunks of all sequences, and the ones without keys come last.  (With the splits
// innermost, the workgroups with keys of a sequence of 4,000 in a cache of 63 splits shared
// every second compute unit: 11.1 us a layer, now 9.3.)  Every second round of workgroups over
// the chip takes the rows in reverse, so that a compute unit's second workgroup
// is short where its first is long: two layers of 64 paged sequences of 2,912-6,512 keys
// in two splits took 230.0 us with the splits innermost, 243.2 with the rows in the same
// order in both splits and 215.7 this way.  The float32 kernel has three rounds, and is
// faster with the splits innermost (238.8 against 257.3 us, 32 such sequences, 4 heads).
__device__ __forceinline__ int row_of(const DecodeParams &p, int split) {
  const int y = static_cast<int>(blockIdx.y);
  const uint32_t before = static_cast<uint32_t>(split) * gridDim.x * gridDim.y;   // workgroups of earlier splits
  return before / kUnits & 1 ? p.batch - 1 - y : y;
}

// Keys per workgroup of a sequence of len keys: an even share of its n_split workgroups,
// in whole rounds of p.round keys, so that no workgroup of a sequence waits on a longer
// one; no fewer than p.min_keys where p.fill workgroups would do (plan_splits).
// Workgroups past the sequence's last key have nothing to do and write nothing (with
// p.all_splits: an empty partial).
__device__ __forceinline__ int chunk_keys(const DecodeParams &p, int len) {
  // ceil(len / n) by the launcher's ceil(2^32 / n): one too many at most (len < 2^30).
  auto share = [&](int n, uint32_t inverse) -> int {
    return n == 1 ? len : static_cast<int>(__umulhi(static_cast<uint32_t>(len + n - 1), inverse));
  };
  int per = share(p.n_split, p.split_inverse);
  if (p.n_split > p.fill && per < p.min_keys) per = share(p.fill, p.fill_inverse);
  return (per + p.round - 1) & -p.round;   // (a power of two)
}

// Length of a sequence as the kernels use it: within [0, capacity].
__device__ __forceinline__ int clamp_len(const DecodeParams &p, bool paged, int len) {
  const int64_t cap = paged ? static_cast<int64_t>(p.max_blocks) * p.block_size : p.s_max;
  return static_cast<int>(min(max(static_cast<int64_t>(len), int64_t{0}), cap));
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // at any float

// Ends a workgroup's chunk: merges its waves' running maxima, sums of weights and weighted
// values (a head's value is the sum of kParts rows, kStep rows apart) and writes them to the
// workspace for decode_combine_kernel, or, where every sequence is one chunk (p.direct), to
// the output at once.  Four features of one head per thread, every LDS read issued before
// the first use; a feature at a time this took 0.6 us of the 4 us that a short chunk takes.
template <int kWaves, int D, int GT, int kParts, int kStep, int kRows>
__device__ __forceinline__ void finish_split(const DecodeParams &p, int b, int kvh, int G, int split,
                                             const float (&s_m)[kWaves][GT], const float (&s_l)[kWaves][GT],
                                             const float (&s_o)[kWaves][kRows][D]) {
  const int64_t head0 = static_cast<int64_t>(b) * p.n_q_heads + kvh * G;
#pragma unroll
  for (int u = 0; u < (GT * D / 4 + kWaves * kWave - 1) / (kWaves * kWave); ++u) {
    const int idx = u * kWaves * kWave + threadIdx.x;
    const int g = idx / (D / 4), d = idx % (D / 4) * 4;
    if (g >= G) break;
    float m[kWaves], l[kWaves];
    f32x4 o[kWaves][kParts];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      m[w] = s_m[w][g];
      l[w] = s_l[w][g];
#pragma unroll
      for (int q = 0; q < kParts; ++q) o[w][q] = *reinterpret_cast<const f32x4 *>(&s_o[w][q * kStep + g][d]);
    }
    float M = -FLT_MAX, L = 0.f;
    f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, m[w]);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float wt = exp2_fast(m[w] - M);
      L += l[w] * wt;
      f32x4 v = o[w][0];
#pragma unroll
      for (int q = 1; q < kParts; ++q) v += o[w][q];
      O += v * wt;
    }
    if (p.direct) {
#pragma unroll
      for (int e = 0; e < 4; ++e) O[e] = L != 0.f ? O[e] / L : 0.f;   // (a NaN stays one)
      *reinterpret_cast<f32x4_any *>(p.out + (head0 + g) * D + d) = O;
    } else {
      float *ws = p.ws + ((head0 + g) * p.n_split + split) * (D + 2);
      *reinterpret_cast<f32x4_any *>(ws + d) = O;
      if (d == 0) {
        ws[D] = M;
        ws[D + 1] = L;
      }
    }
  }
}

template <int D, int GT, bool kPaged>
__global__ __launch_bounds__(kWaves * kWave) void decode_partial_kernel(const DecodeParams p) {
  constexpr int EPL = 4;                     // elements per lane (one 16-byte chunk)
  constexpr int LPK = D / EPL;               // lanes per key row
  constexpr int KPW = kWave / LPK;           // key rows per wave per iteration
  constexpr int KPB = kWaves * KPW;          // key rows per workgroup per iteration
  constexpr int kRowBytes = D * static_cast<int>(sizeof(float));
  constexpr int P = D / 2;
  static_assert(LPK >= 2 && kWave % LPK == 0, "unsupported head_dim");
  __shared__ float s_m[kWaves][GT];
  __shared__ float s_l[kWaves][GT];
  __shared__ __align__(16) float s_o[kWaves][GT][D];

  const int split = blockIdx.x, kvh = blockIdx.y;
  const int lane = threadIdx.x & (kWave - 1);
  int len_in;
  const int b = sequence_of_row<kWaves>(p, lane, blockIdx.z, &len_in);
  const int wave = threadIdx.x / kWave;
  const int kg = lane / LPK;                 // key row slot within the wave
  const int c = lane % LPK;                  // 16-byte chunk of the row
  const int grp = wave * KPW + kg;           // key row slot within the workgroup
  const int G = p.group;

  const int len = clamp_len(p, kPaged, len_in);
  if (len != len_in && split == 0 && kvh == 0 && threadIdx.x == 0 && p.err != nullptr)
    atomicOr(p.err, PRCR_DERR_CAPACITY);
  const int chunk = chunk_keys(p, len);
  const int j0 = static_cast<int>(min(static_cast<int64_t>(len), static_cast<int64_t>(split) * chunk));
  const int j1 = static_cast<int>(min(static_cast<int64_t>(len), static_cast<int64_t>(j0) + chunk));
  if (j0 >= j1 && split > 0 && !p.all_splits) return;

  // Rotated, scaled query chunk of every head of the group: the lane's elements
  // e = c*EPL .. c*EPL+EPL-1 pair with e +/- D/2, which sits in chunk c +/- LPK/2.
  float qv[GT][EPL];
  {
    const double pq = static_cast<double>(p.q_pos[b]);
    const bool first = c < LPK / 2;
    const int cp = first ? c + LPK / 2 : c - LPK / 2;
    double cs[EPL], sn[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const int i = (c * EPL + e) % P;
      sincos(pq * p.inv_freq[i], &sn[e], &cs[e]);
    }
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      const int qh = kvh * G + (g < G ? g : 0);
      const char *qrow = static_cast<const char *>(p.q) + (static_cast<int64_t>(b) * p.n_q_heads + qh) * kRowBytes;
      float x[EPL], xp[EPL];
      unpack(*reinterpret_cast<const u32x4 *>(qrow + c * 16), x);
      unpack(*reinterpret_cast<const u32x4 *>(qrow + cp * 16), xp);
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const double y = first ? static_cast<double>(x[e]) * cs[e] - static_cast<double>(xp[e]) * sn[e]
                               : static_cast<double>(x[e]) * cs[e] + static_cast<double>(xp[e]) * sn[e];
        qv[g][e] = static_cast<float>(y * (p.scale * kLog2e));
      }
    }
  }

  float m[GT], l[GT], o[GT][EPL];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    m[g] = -FLT_MAX;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[g][e] = 0.f;
  }

  const int64_t row_base = kPaged ? 0
                                  : ((static_cast<int64_t>(b) * p.n_layers + p.layer) * p.n_kv_heads + kvh) * p.s_max;
  int bad_block = 0;
  // Loads of the next batch of key rows are issued before the current batch is
  // scored, so one batch is always in flight.
  u32x4 kc[kIters], vc[kIters];
  bool live[kIters];
  // Slot 0 of this head's first row of the layer: present in every cache.
  const int64_t row_any = kPaged ? static_cast<int64_t>(p.layer) * p.n_blocks * p.block_size * p.n_kv_heads + kvh
                                 : row_base;
  auto load_batch = [&](int jb, u32x4 *kd, u32x4 *vd, bool *lv) {
    int32_t blk[kIters], in[kIters];
    if constexpr (kPaged) {
      // Every block-table entry of the batch is read before any row load is
      // issued: a wait for a table entry also waits for every load issued before
      // it, so reading them row by row would serialise the batch's row loads.
      // Rows past the chunk read the sequence's first entry (always present).
#pragma unroll
      for (int u = 0; u < kIters; ++u) {
        const int j = jb + u * KPB + grp;
        const int js = j < j1 ? j : 0;
        // Block and offset of slot js: a shift and a mask for power-of-two block
        // sizes (the common case), else one integer division.
        const int lb = p.block_shift >= 0 ? (js >> p.block_shift) : js / p.block_size;
        in[u] = js - lb * p.block_size;
        blk[u] = p.block_table[static_cast<int64_t>(b) * p.max_blocks + lb];
      }
    }
#pragma unroll
    for (int u = 0; u < kIters; ++u) {
      const int j = jb + u * KPB + grp;
      lv[u] = j < j1;
      int64_t row;
      if constexpr (kPaged) {
        if (lv[u] && (blk[u] < 0 || blk[u] >= p.n_blocks)) {
          lv[u] = false;
          bad_block = 1;
        }
        row = ((static_cast<int64_t>(p.layer) * p.n_blocks + blk[u]) * p.block_size + in[u]) *
                  p.n_kv_heads + kvh;
      } else {
        row = row_base + j;
      }
      // Rows past the chunk (or in a block outside the pool) read a row that
      // always exists, so that every load is issued unconditionally; they get
      // zero weight, and their values are taken as zero when scored.
      row = lv[u] ? row : row_any;
      kd[u] = load_nt(static_cast<const char *>(p.cache_k) + row * kRowBytes + c * 16);
      vd[u] = load_nt(static_cast<const char *>(p.cache_v) + row * kRowBytes + c * 16);
    }
  };
  load_batch(j0, kc, vc, live);
  for (int jb = j0; jb < j1; jb += KPB * kIters) {
    u32x4 nk[kIters], nv[kIters];
    bool nl[kIters];
    load_batch(jb + KPB * kIters, nk, nv, nl);
    // Scores of the batch's rows for every head of the group, then one rescale
    // of the running sums per head and batch.
    float sc[kIters][GT];
#pragma unroll
    for (int u = 0; u < kIters; ++u) {
      float k[EPL];
      unpack(kc[u], k);
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) s = fmaf(qv[g][e], k[e], s);
        sc[u][g] = group_sum<LPK>(s);
      }
    }
    // A zero weight times a value read from another row could make a NaN:
    // values of rows without weight are taken as zero.
    float v[kIters][EPL];
#pragma unroll
    for (int u = 0; u < kIters; ++u) unpack(live[u] ? vc[u] : u32x4{0u, 0u, 0u, 0u}, v[u]);
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      float mn = m[g];
#pragma unroll
      for (int u = 0; u < kIters; ++u) mn = live[u] ? fmaxf(mn, sc[u][g]) : mn;
      // Rescale only when some lane's running maximum rose (rarely, after the
      // first rows): for every other lane the factor is exactly 1.
      if (__any(mn > m[g])) {
        const float corr = exp2_fast(m[g] - mn);
        l[g] *= corr;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[g][e] *= corr;
        m[g] = mn;
      }
#pragma unroll
      for (int u = 0; u < kIters; ++u) {
        const float pj = live[u] ? exp2_fast(sc[u][g] - mn) : 0.f;
        l[g] += pj;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[g][e] = fmaf(pj, v[u][e], o[g][e]);
      }
    }
#pragma unroll
    for (int u = 0; u < kIters; ++u) {
      kc[u] = nk[u];
      vc[u] = nv[u];
      live[u] = nl[u];
    }
  }
  if (bad_block && p.err != nullptr && c == 0) atomicOr(p.err, PRCR_DERR_BLOCK);

  // Merge the wave's key-row slots (lanes LPK apart hold the same elements of
  // different slots), then the workgroup's waves in LDS, and write this chunk's
  // partials.  Empty slots carry l = 0 and o = 0, so their weight is harmless.
#pragma unroll
  for (int off = LPK; off < kWave; off <<= 1) {
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      const float m2 = __shfl_xor(m[g], off);
      const float l2 = __shfl_xor(l[g], off);
      const float mx = fmaxf(m[g], m2);
      const float w1 = exp2_fast(m[g] - mx), w2 = exp2_fast(m2 - mx);
      l[g] = l[g] * w1 + l2 * w2;
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[g][e] = o[g][e] * w1 + __shfl_xor(o[g][e], off) * w2;
      m[g] = mx;
    }
  }
  if (kg == 0) {
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      if (c == 0) {
        s_m[wave][g] = m[g];
        s_l[wave][g] = l[g];
      }
#pragma unroll
      for (int e = 0; e < EPL; ++e) s_o[wave][g][c * EPL + e] = o[g][e];
    }
  }
  __syncthreads();
  finish_split<kWaves, D, GT, 1, 1>(p, b, kvh, G, split, s_m, s_l, s_o);
}

// ---------------------------------------------------------------------------
// bf16 caches: both contractions of a tile of 32 keys run on the matrix cores,
// with float32 accumulation and no precision given up to the 16-bit operands.
//
//   scores   K(16 keys) x Q^T: the float32 query of each head is split into three
//            bf16 parts (the leading 8 significant bits, the next 8 of what is
//            left, then the rest) whose sum is exactly the float32 value.  Row
//            4 h + part of the query operand is part `part` of head h, so that a
//            lane ends with the three part scores of one (head, key) in its own
//            accumulators and adds them: a float32 dot product's accuracy.
//   values   P x V: the float32 weights are split into three bf16 parts in the
//            same way and are rows of the product, so that each output feature is
//            the sum of three rows, again exact products with float32 sums.
//
// The vector ALU is left with the softmax (one exponential per head and key,
// spread over all 64 lanes) and the transpose of the value rows (one byte
// permutation per two elements, in registers), at the same cost for 1 to 4 and for
// 5 to 8 query heads per KV head.  What bounds the kernel is reading the cache.
// With the weighted value sum on the vector ALU (a multiply-add per element and
// head, 16-key tiles) a layer of 64 paged sequences of 2,912-6,512 keys, 4 KV heads
// and 7 query heads each took 169.6 us, on the matrix cores 123.5, and 105.6 now, with whole
// cache lines per key load and fewer workgroups (619 MB, 5.9 TB/s); 32 contiguous sequences
// of 2,756-4,256 keys, 8 KV heads and 4 query heads each 81.7, 79.7 and 71.7 (458 MB, 6.4 TB/s).

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma_16x16x32(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Orders this wave's LDS writes before its later LDS reads (LDS operations of a
// wave complete in issue order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Part `part` (0, 1, 2) of the three-way bf16 split of x, as bf16 bits in the
// upper half of a word.  Each part is the truncation of what the previous parts
// left, and every difference is exact in float32, so the parts sum to x.
__device__ __forceinline__ uint32_t split_part(float x, int part) {
  const uint32_t hi = __float_as_uint(x) & 0xFFFF0000u;
  const float r1 = x - __uint_as_float(hi);
  const uint32_t mid = __float_as_uint(r1) & 0xFFFF0000u;
  const float r2 = r1 - __uint_as_float(mid);
  return part == 0 ? hi : (part == 1 ? mid : __float_as_uint(r2));
}

// Maximum over the 16 lanes of a DPP row; every lane of the row ends with it.
__device__ __forceinline__ float row_max16(float s) {
  s = fmaxf(s, dpp<0xB1>(s));
  s = fmaxf(s, dpp<0x4E>(s));
  s = fmaxf(s, dpp<0x141>(s));
  s = fmaxf(s, dpp<0x140>(s));
  return s;
}

// Upper halves of two words (a's in the low half of the result), and lower halves.
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, 0x07060302u);
}
__device__ __forceinline__ uint32_t pack_lo(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, 0x05040100u);
}

// A lane's share of one value row: 16 bytes (head_dim 128) or 8 (head_dim 64).
template <int kWords>
struct Words;
template <>
struct Words<4> {
  typedef uint32_t type __attribute__((ext_vector_type(4)));
};
template <>
struct Words<2> {
  typedef uint32_t type __attribute__((ext_vector_type(2)));
};

// Exchanges lanes 8..15 of each row of 16 in a with lanes 0..7 of the row in b.
__device__ __forceinline__ void swap_rows8(u32x4 &a, u32x4 &b) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int x = static_cast<int>(a[w]), y = static_cast<int>(b[w]);
    a[w] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(x, y, 0x128, 0xF, 0xC, false));
    b[w] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(y, x, 0x128, 0xF, 0x3, false));
  }
}

constexpr int kTile = 32;   // keys per wave and tile: the value product's contraction length

// GT: query heads per KV head the kernel has room for (4 or 8; smaller groups
// repeat their first head).  kHalfBlocks (paged only): block_size is a multiple of
// 16, so that each half of a tile (tiles start at multiples of 32) lies in one
// block; other block sizes look every key up.
// kWaves: waves per workgroup, 4, or 2 where the whole cache is few chunks (plan_splits).
template <int D, int GT, bool kPaged, bool kHalfBlocks, int kWaves>
__global__ __launch_bounds__(kWaves * kWave, GT == 8 && D == 128 ? 2 : 3) void decode_partial_bf16_kernel(const DecodeParams p) {
  constexpr int KK = D / 32;                 // products over the head dim per 16 keys
  constexpr int kA = GT / 4;                 // query operands: 4 heads x (3 parts + 1 unused row)
  constexpr int kPT = GT / 4;                // weight operands of 16 rows (below)
  constexpr int kPRows = 3 * GT + (GT == 4 ? 4 : 0);   // weight rows in LDS
  constexpr int kDL = D / 16;                // value elements per lane and row
  constexpr int kVW = kDL / 2;               // 32-bit words of them
  constexpr int kVL = kTile / 4;             // value loads per lane and tile (4 rows each)
  constexpr int kRowBytes = D * 2;
  constexpr int KPB = kWaves * kTile;        // keys per workgroup per round of tiles
  constexpr int P = D / 2;
  constexpr int kQ = (GT * P + kWaves * kWave - 1) / (kWaves * kWave);   // query pairs per thread
  // Weight rows: the three parts of head h are rows h, 4 + h and 8 + h (4 heads; rows
  // 12..15 are not used), or h, 8 + h and 16 + h (8 heads: the first operand holds rows
  // 0..15, the second adds rows 16..23 to the first eight rows' sums).
  // Rows in LDS: 32 keys of bf16, padded so that the 16 rows an operand
  // read touches at once fall on different banks.
  constexpr int kPS = kTile / 2 + 4;         // words per row
  typedef typename Words<kVW>::type vrow;
  static_assert(GT == 4 || GT == 8, "unsupported group");
  static_assert(D == 64 || D == 128, "unsupported head_dim");
  __shared__ __align__(16) uint16_t s_q[3 * GT][D + 8];   // padded as the weight rows are
  __shared__ __align__(16) uint32_t s_p[kWaves][kPRows][kPS];
  __shared__ float s_m[kWaves][GT];
  __shared__ float s_l[kWaves][GT];
  __shared__ __align__(16) float s_o[kWaves][16][D];

  const int split = blockIdx.z, kvh = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const double inv = p.inv_freq[threadIdx.x % P];
  int len_in;
  const int b = sequence_of_row<kWaves>(p, lane, row_of(p, split), &len_in);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n16 = lane % 16;                 // product column; operand row
  const int kj = lane / 16;                  // k group of the operands; head of the lane's scores
  const int G = p.group;

  const int len = clamp_len(p, kPaged, len_in);
  if (len != len_in && split == 0 && kvh == 0 && threadIdx.x == 0 && p.err != nullptr)
    atomicOr(p.err, PRCR_DERR_CAPACITY);
  const int chunk = chunk_keys(p, len);
  const int j0 = static_cast<int>(min(static_cast<int64_t>(len), static_cast<int64_t>(split) * chunk));
  const int j1 = static_cast<int>(min(static_cast<int64_t>(len), static_cast<int64_t>(j0) + chunk));
  if (j0 >= j1 && split > 0 && !p.all_splits) return;

  // What a short sequence pays for is the chain of dependent loads and the query's set-up.
  // The lengths are read once for the order and the length; then the query's rows, then
  // the first tile's: a wait for one load also waits for those issued before it, and the
  // tile's rows are to stay in flight while the query is prepared.  The query's parts are
  // formed once, by the thread that rotates the pair, and read as operands: as a choice of
  // part per operand element the set-up was 32 LDS reads each behind a branch.  One
  // sequence of 1,152 keys (8 KV heads): 10.7 us a layer before, 8.4 so, with the merge.
  const int32_t q_pos = p.q_pos[b];
  uint32_t q_lo[kQ], q_hi[kQ];
#pragma unroll
  for (int u = 0; u < kQ; ++u) {
    const int g = u * (kWaves * kWave / P) + threadIdx.x / P;
    const int qh = kvh * G + (g < G ? g : 0);
    const uint16_t *qrow = static_cast<const uint16_t *>(p.q) + (static_cast<int64_t>(b) * p.n_q_heads + qh) * D;
    q_lo[u] = qrow[threadIdx.x % P];
    q_hi[u] = qrow[threadIdx.x % P + P];
  }

  // Keys of a tile.  Column n16 of score product st is key 8 (n16/4) + 4 st + n16%4,
  // value load u holds key 4 u + kj: both put key t at position (t % 4) * 8 + t / 4
  // of the value product's contraction, with a lane's two scores in one word.
  const int kt0 = 8 * (n16 / 4) + n16 % 4;
  const int64_t row_layer = static_cast<int64_t>(p.layer) * p.n_blocks * p.block_size;   // paged
  const int64_t row_any = kPaged ? row_layer * p.n_kv_heads + kvh
                                 : ((static_cast<int64_t>(b) * p.n_layers + p.layer) * p.n_kv_heads + kvh) * p.s_max;
  const char *const cache_k = static_cast<const char *>(p.cache_k);
  const char *const cache_v = static_cast<const char *>(p.cache_v);
  int bad_block = 0;

  // Block-table entry of key `lane % 32` of the tile at tb (the sequence's first
  // entry past the chunk), and that key's offset in its block.  Entries are read
  // two tiles ahead, so that the loads that need one never wait for it.
  struct Entry {
    int32_t blk, off;
  };
  auto entry_of = [&](int tb) -> Entry {
    Entry e{0, 0};
    if constexpr (kPaged) {
      const int j = tb + lane % kTile;
      const int js = j < j1 ? j : 0;
      const int lb = p.block_shift >= 0 ? (js >> p.block_shift) : js / p.block_size;
      e.blk = p.block_table[static_cast<int64_t>(b) * p.max_blocks + lb];
      e.off = js - lb * p.block_size;
    }
    return e;
  };
  // Rows of a tile.  Every load is issued unconditionally: keys past the chunk, or
  // in a block outside the pool, read a row that exists and are left out of `live`
  // (bit t: key t); they get no weight, and their values are taken as zero.
  //   contiguous     one base; key t is row min(t, last)
  //   half blocks    one base per half; key t is row min(t % 16, last[t / 16])
  //   other blocks   lane t holds key t's slot in the layer's pool (below 2^32: a
  //                  pool's slots are at least 128 bytes each)
  struct TileRows {
    int64_t base[2];
    int last[2];
    uint32_t slot;
    uint32_t live;
  };
  auto rows_of = [&](int tb, Entry e) -> TileRows {
    TileRows t{};
    const int n_in = min(max(j1 - tb, 0), kTile);
    t.live = n_in >= kTile ? ~0u : (1u << n_in) - 1u;
    if constexpr (!kPaged) {
      const int tc = max(min(tb, j1 - 1), 0);
      t.base[0] = row_any + tc;
      t.last[0] = max(j1 - 1 - tc, 0);
    } else {
      const bool in = (t.live >> (lane % kTile)) & 1u;
      const bool ok = in && e.blk >= 0 && e.blk < p.n_blocks;
      const uint32_t live = static_cast<uint32_t>(__ballot(ok));   // lanes t and t + 32 agree
      bad_block |= live != t.live;
      t.live = live;
      const int64_t slot = static_cast<int64_t>(e.blk) * p.block_size + e.off;
      if constexpr (kHalfBlocks) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t lh = (live >> (16 * h)) & 0xFFFFu;
          const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(slot), 16 * h);
          const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(slot >> 32), 16 * h);
          const int64_t s = static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
          t.base[h] = lh != 0 ? (row_layer + s) * p.n_kv_heads + kvh : row_any;
          t.last[h] = lh != 0 ? __popc(lh) - 1 : 0;
        }
      } else {
        t.slot = ok ? static_cast<uint32_t>(slot) : 0u;
      }
    }
    return t;
  };
  const uint32_t row_step = kPaged ? static_cast<uint32_t>(p.n_kv_heads) * kRowBytes : kRowBytes;
  // Byte offset of key t (t / 16 == half).
  auto key_offset = [&](const TileRows &tr, int t, int half) -> int64_t {
    if constexpr (!kPaged)
      return tr.base[0] * kRowBytes + static_cast<uint32_t>(min(t, tr.last[0])) * row_step;
    else if constexpr (kHalfBlocks)
      return tr.base[half] * kRowBytes + static_cast<uint32_t>(min(t - 16 * half, tr.last[half])) * row_step;
    else
      return (row_layer + static_cast<int64_t>(static_cast<uint32_t>(__shfl(static_cast<int>(tr.slot), t)))) *
                 row_step + static_cast<int64_t>(kvh) * kRowBytes;
  };
  // Key rows.  The product's operand layout would read a half of each of 16 rows' cache
  // lines per load, and the other halves with the next one, through the caches.  So a load
  // reads whole lines of 8 rows, once, past the caches: line q of the keys of columns 0..7
  // by load 2 q, of columns 8..15 by load 2 q + 1, one half of a line in the lanes of its
  // own column and the other 8 lanes away (swap_rows8 brings it over).  Two layers of 64
  // paged sequences of 2,912-6,512 keys (7 heads): 240.4 us in half lines, 224.4 in whole
  // ones; 32 contiguous ones of 2,756-4,256 keys (4 heads): 155.6 and 151.7.  The counters do
  // not say why: in half lines the L1 asks the L2 for 0.6 and 1.0 % more lines, and the bytes
  // from memory are the same.
  const int ka = 8 * (n16 % 8 / 4) + n16 % 4;
  auto load_k = [&](const TileRows &tr, u32x4 (&kd)[2][KK]) {
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const char *kp[2] = {cache_k + key_offset(tr, ka + 4 * st, 0), cache_k + key_offset(tr, ka + 4 * st + 16, 1)};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kd[st][kk] = load_nt(kp[kk % 2] + (n16 / 8) * 64 + kj * 16 + kk / 2 * 128);
    }
  };
  // Value rows, 16 lanes to a row.
  auto load_v = [&](const TileRows &tr, vrow (&vd)[kVL]) {
#pragma unroll
    for (int u = 0; u < kVL; ++u) {
      const int64_t o = key_offset(tr, 4 * u + kj, u / 4);
      vd[u] = __builtin_nontemporal_load(reinterpret_cast<const vrow *>(cache_v + o + n16 * (kDL * 2)));
    }
  };

  // The wave's tiles start at jw + n * KPB.  One buffer per operand, software
  // pipelined: the next tile's key rows are loaded once this tile's products have
  // read them, and its value rows once the value product has; each load's latency
  // hides behind the other half of a tile's work.
  const int jw = j0 + wave * kTile;
  u32x4 kr[2][KK];
  vrow vv[kVL];
  Entry e_next;
  TileRows tr;
  // (Unconditionally: behind a branch, the waits below would have to allow for these
  // loads not being there, and so wait for them.)
  {
    const Entry e0 = entry_of(jw);
    e_next = entry_of(jw + KPB);
    tr = rows_of(jw, e0);
    load_k(tr, kr);
    load_v(tr, vv);
  }

  // Rotated, scaled query of every head of the group (pair i with i + D/2, the
  // 1-D rotation at p_next), in float32, as three bf16 parts in LDS.
  {
    const double qs = static_cast<double>(p.scale) * kLog2e;
    const int i = threadIdx.x % P;
    double sn, cs;
    sincos(static_cast<double>(q_pos) * inv, &sn, &cs);
#pragma unroll
    for (int u = 0; u < kQ; ++u) {
      const int g = u * (kWaves * kWave / P) + threadIdx.x / P;
      if (g < GT) {
        const double x = __uint_as_float(q_lo[u] << 16), xp = __uint_as_float(q_hi[u] << 16);
        const float y = static_cast<float>((x * cs - xp * sn) * qs);
        const float yp = static_cast<float>((xp * cs + x * sn) * qs);
#pragma unroll
        for (int part = 0; part < 3; ++part) {
          s_q[3 * g + part][i] = static_cast<uint16_t>(split_part(y, part) >> 16);
          s_q[3 * g + part][i + P] = static_cast<uint16_t>(split_part(yp, part) >> 16);
        }
      }
    }
  }
  lds_barrier();
  // Query operands: row n16 of operand a is part n16 % 4 of head 4 a + n16 / 4 (the
  // fourth row repeats the third; its scores are not used); the lane's 8 elements of
  // product kk are those of row chunk 4 kk + kj, the same chunk as the key operand.
  u32x4 qa[kA][KK];
#pragma unroll
  for (int a = 0; a < kA; ++a) {
    const uint16_t *row = s_q[3 * (4 * a + n16 / 4) + min(n16 % 4, 2)];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qa[a][kk] = *reinterpret_cast<const u32x4 *>(row + 8 * (4 * kk + kj));
  }

  f32x4 acc[kDL];                            // rows 4 kj + r, features kDL * n16 + dt
#pragma unroll
  for (int dt = 0; dt < kDL; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mrun[kA], lsum[kA];                  // head 4 a + kj; lsum over the lane's own keys
#pragma unroll
  for (int a = 0; a < kA; ++a) {
    mrun[a] = -FLT_MAX;
    lsum[a] = 0.f;
  }

  for (int jt = jw; jt < j1; jt += KPB) {
    const uint32_t live = tr.live;
    f32x4 sa[kA][2];
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int kk = 0; kk < KK; kk += 2) swap_rows8(kr[st][kk], kr[st][kk + 1]);
#pragma unroll
    for (int a = 0; a < kA; ++a) {
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        sa[a][st] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) sa[a][st] = mfma_16x16x32(qa[a][kk], kr[st][kk], sa[a][st]);
      }
    }
    // (A tile past the chunk re-reads one row.)
    tr = rows_of(jt + KPB, e_next);
    e_next = entry_of(jt + 2 * KPB);
    load_k(tr, kr);

    const bool live0 = (live >> kt0) & 1u, live1 = (live >> (kt0 + 4)) & 1u;
    float sc[kA][2];
    bool rise = false;
#pragma unroll
    for (int a = 0; a < kA; ++a) {
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        const float s = (sa[a][st][0] + sa[a][st][1]) + sa[a][st][2];
        sc[a][st] = (st == 0 ? live0 : live1) ? s : -FLT_MAX;
        rise = rise || sc[a][st] > mrun[a];
      }
    }
    // The tile's maxima are needed only when some score rose above the running
    // maximum of its head (rarely, after the first tiles).
    if (__any(rise)) {
      float corr[kA];
#pragma unroll
      for (int a = 0; a < kA; ++a) {
        const float mnew = fmaxf(mrun[a], row_max16(fmaxf(sc[a][0], sc[a][1])));
        corr[a] = exp2_fast(mrun[a] - mnew);
        lsum[a] *= corr[a];
        mrun[a] = mnew;
      }
      // Accumulator row 4 kj + r belongs to head r (4 heads), or to head
      // 4 (kj % 2) + r (8 heads); head h's factor is in lanes 16 (h % 4)...
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(corr[0]), 16 * r));
        if constexpr (kA == 2) {
          const float c1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(corr[kA - 1]), 16 * r));
          c = (kj & 1) ? c1 : c;
        }
#pragma unroll
        for (int dt = 0; dt < kDL; ++dt) acc[dt][r] *= c;
      }
    }
    // Weights and their three bf16 parts, two keys to a word.  A part that is zero
    // is raised to the smallest normal bf16 when the weight is not (2^-126, where the
    // chunk's largest weight is 1): a zero part times an infinite value would make a NaN where
    // weight times value is infinite.
#pragma unroll
    for (int a = 0; a < kA; ++a) {
      uint32_t part[3][2];
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        const float w = (st == 0 ? live0 : live1) ? exp2_fast(sc[a][st] - mrun[a]) : 0.f;
        lsum[a] += w;
        const uint32_t tiny = w > 0.f ? 0x00800000u : 0u;
#pragma unroll
        for (int q = 0; q < 3; ++q) part[q][st] = max(split_part(w, q), tiny);
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int row = GT == 4 ? 4 * q + kj : 8 * q + 4 * a + kj;
        s_p[wave][row][(n16 % 4) * 4 + n16 / 4] = pack_hi(part[q][0], part[q][1]);
      }
    }
    wave_lds_sync();
    u32x4 pa[kPT];
    pa[0] = *reinterpret_cast<const u32x4 *>(&s_p[wave][n16][4 * kj]);
    if constexpr (kPT == 2) {
      // The second operand's other eight rows add to the middle parts' sums: they
      // repeat its weights cut to the smallest normal value (for the reason above).
      pa[kPT - 1] = *reinterpret_cast<const u32x4 *>(&s_p[wave][16 + n16 % 8][4 * kj]);
      const u16x2 most = __builtin_bit_cast(u16x2, n16 < 8 ? 0xFFFFFFFFu : 0x00800080u);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t two = pa[kPT - 1][w];   // (a bit cast of the element itself takes element 0)
        pa[kPT - 1][w] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, two), most));
      }
    }
    // A zero weight times a value read from another row could make a NaN: values
    // of keys without weight are taken as zero.
    if (live != ~0u) {
#pragma unroll
      for (int u = 0; u < kVL; ++u) {
        const uint32_t keep = (live >> (4 * u + kj)) & 1u ? ~0u : 0u;
#pragma unroll
        for (int w = 0; w < kVW; ++w) vv[u][w] &= keep;
      }
    }
    // Transposed value operand: feature kDL * n16 + dt of the lane's 8 keys.
#pragma unroll
    for (int dt = 0; dt < kDL; ++dt) {
      u32x4 vb;
#pragma unroll
      for (int w = 0; w < 4; ++w)
        vb[w] = dt % 2 == 0 ? pack_lo(vv[2 * w][dt / 2], vv[2 * w + 1][dt / 2])
                            : pack_hi(vv[2 * w][dt / 2], vv[2 * w + 1][dt / 2]);
#pragma unroll
      for (int q = 0; q < kPT; ++q) acc[dt] = mfma_16x16x32(pa[q], vb, acc[dt]);
    }
    load_v(tr, vv);
  }
  if (bad_block && lane == 0 && p.err != nullptr) atomicOr(p.err, PRCR_DERR_BLOCK);

  // The lanes of a row of 16 hold different keys of one head.
#pragma unroll
  for (int a = 0; a < kA; ++a) {
    lsum[a] = group_sum<16>(lsum[a]);
    if (n16 == 0) {
      s_m[wave][4 * a + kj] = mrun[a];
      s_l[wave][4 * a + kj] = lsum[a];
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int c = 0; c < kDL / 4; ++c)
      *reinterpret_cast<f32x4 *>(&s_o[wave][4 * kj + r][kDL * n16 + 4 * c]) =
          f32x4{acc[4 * c][r], acc[4 * c + 1][r], acc[4 * c + 2][r], acc[4 * c + 3][r]};
  }
  __syncthreads();
  finish_split<kWaves, D, GT, GT == 4 ? 3 : 2, GT>(p, b, kvh, G, split, s_m, s_l, s_o);
}

// Over the wave's four rows of 16 lanes (the same value in every lane): register lane
// permutations and reads, where a shuffle is a round trip through the LDS unit per step.
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
__device__ __forceinline__ float wave_max(float x) {
  x = row_max16(x);
  return fmaxf(fmaxf(lane_value(x, 0), lane_value(x, 16)), fmaxf(lane_value(x, 32), lane_value(x, 48)));
}
__device__ __forceinline__ float wave_sum(float x) {
  x = group_sum<16>(x);
  return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

// Merge of one query head's split partials, by kHeadWaves waves (each takes every
// kHeadWaves-th split).  What it costs is one launch and its dependent rounds of loads, so
// everything the first kPre splits need goes out in one round: the length (which gives
// the splits that have keys; the others' words hold anything), the (max, sum) pairs, one
// split per lane, and the features, which do not depend on the weights.  With up to kPre
// splits a wave needs neither a second round nor a barrier; with more, 4 or 16 waves share
// a head and meet once in LDS: 16 where 4 would need more than two rounds (125 splits of
// one sequence of 16,000 keys: 3.4 us with 4 waves, 3.0 with 16).  Against one thread per
// feature, with the weights through LDS, a layer took 22.7 us and takes 19.7 (one sequence
// of 16,000 keys, 8 KV heads of 8 query heads, 64 splits), 14.0 and 13.1 (four of
// 1,500-3,000 keys, 4 KV heads of 7, 32 splits), and the same with 3 splits, where launch
// and one round are all.
constexpr int kPre = 8;
constexpr int kMostSplits = 768;             // of any call (decode_splits)
static_assert(kMostSplits <= 16 * kWave, "the merge has a lane for every split of a wave");
template <int D, bool kPaged, int kHeadWaves>
__global__ __launch_bounds__((kHeadWaves > kWaves ? kHeadWaves : kWaves) * kWave) void decode_combine_kernel(
    const DecodeParams p) {
  constexpr int F = D / kWave;               // features per lane: F * lane + f
  constexpr int kBlockWaves = kHeadWaves > kWaves ? kHeadWaves : kWaves;
  typedef float feat __attribute__((ext_vector_type(F), aligned(4)));
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int part = wave % kHeadWaves;        // this wave's splits: part, part + kHeadWaves, ...
  const int b = blockIdx.y;
  const int qh = static_cast<int>(blockIdx.x) * (kBlockWaves / kHeadWaves) + wave / kHeadWaves;
  if (qh >= p.n_q_heads) return;             // (whole workgroups only where waves share a head)
  const int64_t head = static_cast<int64_t>(b) * p.n_q_heads + qh;
  const float *ws = p.ws + head * p.n_split * (D + 2);
  auto split_row = [&](int i) -> const float * {   // the wave's i-th split (clamped: always in the array)
    return ws + static_cast<int64_t>(min(i * kHeadWaves + part, p.n_split - 1)) * (D + 2);
  };
  const int len_in = p.cache_len[b];
  const float m = split_row(lane)[D], l = split_row(lane)[D + 1];   // (at most kWave splits a wave)
  feat o[kPre];
#pragma unroll
  for (int k = 0; k < kPre; ++k) o[k] = *reinterpret_cast<const feat *>(split_row(k) + F * lane);

  const int len = clamp_len(p, kPaged, len_in), chunk = chunk_keys(p, len);
  // Whether the wave's i-th split has keys (an empty sequence writes one empty split).  With
  // p.all_splits the length is not used: its bytes may already be another workgroup's output.
  auto written = [&](int i) -> bool {
    const int split = i * kHeadWaves + part;
    return split < p.n_split && (split == 0 || p.all_splits || static_cast<int64_t>(split) * chunk < len);
  };
  const bool in = written(lane);
  const int n = __popcll(__ballot(in));
  const bool valid = in && l != 0.f;         // (a split with a NaN key counts: its NaN reaches L)
  float M = wave_max(valid ? m : -FLT_MAX);
  const float w = valid ? exp2_fast(m - M) : 0.f;
  float L = wave_sum(valid ? l * w : 0.f);
  feat O = {};
  for (int k0 = 0; k0 < n; k0 += kPre) {
    if (k0 > 0) {
#pragma unroll
      for (int k = 0; k < kPre; ++k) o[k] = *reinterpret_cast<const feat *>(split_row(k0 + k) + F * lane);
      // All loads before the first use.  Below the breaks, where they sink without this, they
      // go one by one: 63 splits of 64 keys, 4 KV heads of 7 heads, 11.2 us a layer and not 9.7.
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
      if (k0 + k >= n) break;
      const float wk = lane_value(w, k0 + k);
#pragma unroll
      for (int f = 0; f < F; ++f) O[f] = fmaf(o[k][f], wk, O[f]);
    }
  }
  if constexpr (kHeadWaves > 1) {
    static_assert(kHeadWaves == kBlockWaves, "a workgroup's waves share one head");
    __shared__ float s_m[kBlockWaves], s_l[kBlockWaves], s_o[kBlockWaves][D];
    if (lane == 0) {
      s_m[wave] = M;
      s_l[wave] = L;
    }
#pragma unroll
    for (int f = 0; f < F; ++f) s_o[wave][F * lane + f] = O[f];
    __syncthreads();
    if (threadIdx.x >= D) return;
    float ms[kBlockWaves], ls[kBlockWaves], os[kBlockWaves];
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) {
      ms[w] = s_m[w];
      ls[w] = s_l[w];
      os[w] = s_o[w][threadIdx.x];
    }
    M = -FLT_MAX;
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) M = fmaxf(M, ms[w]);
    float Ls = 0.f, Os = 0.f;
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) {
      const float wt = exp2_fast(ms[w] - M);
      Ls = fmaf(ls[w], wt, Ls);
      Os = fmaf(os[w], wt, Os);
    }
    p.out[head * D + threadIdx.x] = Ls != 0.f ? Os / Ls : 0.f;
  } else {
#pragma unroll
    for (int f = 0; f < F; ++f) O[f] = L != 0.f ? O[f] / L : 0.f;
    *reinterpret_cast<feat *>(p.out + head * D + F * lane) = O;
  }
}

template <int D, int GT, bool kPaged, int kW>
void launch_bf16(const DecodeParams &p, hipStream_t stream) {
  const dim3 grid(p.n_kv_heads, p.batch, p.n_split), block(kW * kWave);
  if constexpr (kPaged) {
    if (p.block_size % 16 == 0)
      decode_partial_bf16_kernel<D, GT, true, true, kW><<<grid, block, 0, stream>>>(p);
    else
      decode_partial_bf16_kernel<D, GT, true, false, kW><<<grid, block, 0, stream>>>(p);
  } else {
    decode_partial_bf16_kernel<D, GT, false, false, kW><<<grid, block, 0, stream>>>(p);
  }
}

template <typename T, int D, int GT, bool kPaged>
hipError_t launch_split(const DecodeParams &in, hipStream_t stream) {
  DecodeParams p = in;
  // Keys a workgroup's waves take at once: a tile each, or kWave / (D / 4) rows each.
  if constexpr (std::is_same_v<T, uint16_t>) {
    p.round = p.waves * kTile;
    if (p.waves == 2)
      launch_bf16<D, GT, kPaged, 2>(p, stream);
    else
      launch_bf16<D, GT, kPaged, 4>(p, stream);
  } else {
    p.round = kWaves * (kWave / (D / 4));
    decode_partial_kernel<D, GT, kPaged>
        <<<dim3(p.n_split, p.n_kv_heads, p.batch), kWaves * kWave, 0, stream>>>(p);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.direct) return e;
  const unsigned heads = static_cast<unsigned>(p.n_q_heads), rows = static_cast<unsigned>(p.batch);
  if (p.n_split <= kPre)
    decode_combine_kernel<D, kPaged, 1><<<dim3((heads + kWaves - 1) / kWaves, rows), kWaves * kWave, 0, stream>>>(p);
  else if (p.n_split <= 2 * kPre * kWaves)
    decode_combine_kernel<D, kPaged, kWaves><<<dim3(heads, rows), kWaves * kWave, 0, stream>>>(p);
  else
    decode_combine_kernel<D, kPaged, 16><<<dim3(heads, rows), 16 * kWave, 0, stream>>>(p);
  return hipGetLastError();
}

template <typename T, int D, bool kPaged>
hipError_t dispatch_group(const DecodeParams &p, int G, hipStream_t stream) {
  // (The bf16 kernel's products have room for 4 or 8 heads at the same cost as fewer.)
  if constexpr (!std::is_same_v<T, uint16_t>) {
    if (G <= 1) return launch_split<T, D, 1, kPaged>(p, stream);
    if (G <= 2) return launch_split<T, D, 2, kPaged>(p, stream);
  }
  if (G <= 4) return launch_split<T, D, 4, kPaged>(p, stream);
  return launch_split<T, D, 8, kPaged>(p, stream);
}

template <typename T, bool kPaged>
hipError_t dispatch_dim(const DecodeParams &p, int head_dim, int G, hipStream_t stream) {
  if (head_dim == 64) return dispatch_group<T, 64, kPaged>(p, G, stream);
  if (head_dim == 128) return dispatch_group<T, 128, kPaged>(p, G, stream);
  return hipErrorInvalidValue;
}

}  // namespace

int decode_splits(int64_t capacity, int batch, int n_kv_heads, int group) {
  // Partials that a call has room for.  As many workgroups as the chip holds at once:
  // 256 compute units with 3 workgroups each (2 with 8 query heads per KV head, whose
  // bf16 kernel holds more registers).  No split of fewer than 64 keys at full capacity.
  const int64_t target = group > 4 ? 512 : kMostSplits;
  const int64_t pairs = static_cast<int64_t>(batch) * n_kv_heads;
  int64_t ns = (target + pairs - 1) / pairs;
  const int64_t most = (capacity + 63) / 64;
  if (ns > most) ns = most;
  if (ns < 1) ns = 1;
  return static_cast<int>(ns);
}

namespace {

bool overlap(const void *a, double na, const void *b, double nb) {
  const double x = static_cast<double>(reinterpret_cast<uintptr_t>(a));
  const double y = static_cast<double>(reinterpret_cast<uintptr_t>(b));
  return a != nullptr && b != nullptr && x < y + nb && y < x + na;
}

// How a call is split, within the room for decode_splits' partials (p->n_split on entry).
// Only the sequence's length and the call's shape enter, so that a sequence's result does
// not depend on the others'.
//
// float32: all of them.  That kernel is bound by its arithmetic and wants every wave slot.
//
// bf16.  One workgroup per compute unit reads the cache as fast as more do (two layers of 64
// sequences of 4,712 keys, 4 KV heads: 197 us with 256 workgroups and no merge, 206 with 512,
// 208 with 768), so short chunks are merged for nothing: a layer of sequences of 500-800 keys
// takes 18.9 us in one chunk and 23 in two.  But sequences of different lengths are shared
// out better in more (2,912-6,512 keys: 236 us in one, 216 in two), so where every chunk
// keeps 512 keys there are two to four rounds of workgroups over the chip (64 sequences of
// 2,912-6,512 keys, 2 KV heads: 128 us where chunks had to keep 1,024, 115 with 512).  With one
// or two heads per KV head a chunk takes as long and a merge less, and 256 do: the longest of
// 16 sequences (2,007 keys, the others 250; 8 KV heads of one head, D = 64) decides the layer,
// 15.0 us in the two chunks that 512 allow and 12.4 in four; all of 1,003 keys, 12.0 and 12.9.
// Either way the count that fills its last round best is taken.  A cache that is at most 256 chunks of
// 64 keys is read by workgroups of two waves, so that twice as many compute units take part
// (one sequence of 1,152 keys: 8.4 us a layer with four waves, 7.9 with two; 300 keys: 7.3
// and 6.7).  The launcher does not know the lengths, so it is the capacity that decides: the
// same sequence takes 7.1 us in a cache of up to 2,048 slots and 7.7 in a larger one, whose
// workgroups take four waves' tiles each.
void plan_splits(DecodeParams *p, prcr_dtype dtype, bool paged) {
  const int64_t room = p->n_split, pairs = static_cast<int64_t>(p->batch) * p->n_kv_heads;
  const int64_t capacity = paged ? static_cast<int64_t>(p->max_blocks) * p->block_size : p->s_max;
  constexpr int kMinKeys = 512;
  p->waves = 4;
  p->fill = p->n_split;
  p->min_keys = 0;
  if (dtype == PRCR_F32) return;
  auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  // The first splits for lo to hi workgroups that come within 3 % of whole rounds over the
  // chip, or else the nearest (a search of at most some tens of steps, on every call).
  auto rounds = [&](int64_t lo, int64_t hi) {
    int64_t best = ceil_div(lo, pairs);
    double share = 0;
    for (int64_t n = best; n <= std::min(ceil_div(hi, pairs), room) && share < 0.97; ++n) {
      const double s = static_cast<double>(pairs * n) / static_cast<double>(ceil_div(pairs * n, kUnits) * kUnits);
      if (s > share + 1e-9) {
        share = s;
        best = n;
      }
    }
    return std::min(best, room);
  };
  const int64_t fill = pairs >= 3 * kUnits / 4 ? 1 : rounds(3 * kUnits / 4, 2 * kUnits);
  const int64_t most = capacity / kMinKeys;
  const int64_t more = most >= std::min(ceil_div(2 * kUnits, pairs), room) ? rounds(2 * kUnits, 4 * kUnits) : fill;
  p->fill = static_cast<int32_t>(fill);
  p->n_split = static_cast<int32_t>(most >= more ? std::max(fill, more) : fill);
  p->min_keys = p->n_q_heads <= 2 * p->n_kv_heads ? kMinKeys / 2 : kMinKeys;
  if (pairs * ceil_div(capacity, 64) <= kUnits) p->waves = 2;
}

// Whether the partial kernel may write the outputs itself: every sequence is one chunk,
// and no workgroup's output rows are bytes that another one still reads.  96 sequences of
// 500-2,500 keys (8 KV heads, 4 query heads each, paged, two layers): 263 us with the merge
// launch, 251 without.
bool writes_direct(const DecodeParams &p, int elem_bytes, int head_dim, bool paged) {
  if (p.n_split != 1) return false;
  const double rows = static_cast<double>(p.batch) * p.n_q_heads * head_dim;
  const double out = rows * 4;
  const double slots = paged ? static_cast<double>(p.n_blocks) * p.block_size : static_cast<double>(p.batch) * p.s_max;
  const double cache = slots * p.n_layers * p.n_kv_heads * head_dim * elem_bytes;
  return !overlap(p.out, out, p.q, rows * elem_bytes) && !overlap(p.out, out, p.q_pos, 4.0 * p.batch) &&
         !overlap(p.out, out, p.cache_len, 4.0 * p.batch) &&
         !(paged && overlap(p.out, out, p.block_table, 4.0 * p.batch * p.max_blocks)) &&
         !overlap(p.out, out, p.cache_k, cache) && !overlap(p.out, out, p.cache_v, cache);
}

}  // namespace

hipError_t launch_decode(const DecodeParams &in, prcr_dtype dtype, int head_dim, bool paged,
                         hipStream_t stream) {
  DecodeParams p = in;
  const int G = p.n_q_heads / p.n_kv_heads;
  plan_splits(&p, dtype, paged);
  auto inverse = [](int64_t n) { return n > 1 ? static_cast<uint32_t>(((int64_t{1} << 32) + n - 1) / n) : 0u; };
  p.split_inverse = inverse(p.n_split);
  p.fill_inverse = inverse(p.fill);
  p.group = G;
  p.direct = writes_direct(p, dtype == PRCR_F32 ? 4 : 2, head_dim, paged);
  p.all_splits = overlap(p.out, 4.0 * p.batch * p.n_q_heads * head_dim, p.cache_len, 4.0 * p.batch);
  if (dtype == PRCR_F32)
    return paged ? dispatch_dim<float, true>(p, head_dim, G, stream)
                 : dispatch_dim<float, false>(p, head_dim, G, stream);
  return paged ? dispatch_dim<uint16_t, true>(p, head_dim, G, stream)
               : dispatch_dim<uint16_t, false>(p, head_dim, G, stream);
}

}  // namespace prcr
