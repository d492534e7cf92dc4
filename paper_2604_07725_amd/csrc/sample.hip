// Fused full-vocabulary log-softmax + Gumbel-max sampling.
//
// Pass 1: one 256-thread workgroup per (vocab chunk, candidate); a chunk is
// one or more 4096-entry tiles, each with a partial of its own (how many tiles a
// workgroup walks depends on the number of rows; the order of no sum does).
// Thread t owns the 4-entry groups 1024 r + 4 t
// (r < 4) of a tile, each one Philox4x32-10 counter and one 16-byte load; it
// computes z = logit / T, the running max and sum of exp(z - max) (reduced
// over the wave in registers, then through LDS), and the best perturbed value
// z + G (ties -> lowest index).  The
// temperature mode (T = 0, T = 1, other) is a template parameter, so greedy
// sampling carries no noise or division code.  Pass 2: one workgroup per
// candidate merges its tiles in a fixed order and writes the token id and
// log-probability z_id - logsumexp(z).
//
// Optionally (conf_k > 0) the same passes produce the per-token confidence of
// the group-confidence fitness signal (Eq. 1): c = logsumexp(x) - mean of the
// conf_k largest logits x, i.e. minus the mean of the top-conf_k
// log-probabilities under the model's own distribution (T = 1).  Pass 1 keeps
// each chunk's conf_k largest logits (per wave by a threshold and a bitonic
// sort, then a bitonic merge of the four waves' lists), pass 2 merges the
// chunks' lists the same way.  Cross-lane steps are DPP and permlane swaps.
//
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): 10 rounds; round r uses
// key + r * (0x9E3779B9, 0xBB67AE85); multipliers 0xD2511F53, 0xCD9E8D57.
// Counter (v >> 2, position, uid lo, uid hi), key (seed lo, seed hi), word v & 3.
// u = ((w >> 9) + 0.5) 2^-23 (exact in fp32), G = -log(-log u).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sevo {

__device__ __forceinline__ u32x4 philox4x32_10(u32x4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t lo0 = 0xD2511F53u * c.x;
    const uint32_t hi0 = __umulhi(0xD2511F53u, c.x);
    const uint32_t lo1 = 0xCD9E8D57u * c.z;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z);
    c = u32x4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
  }
  return c;
}

__device__ __forceinline__ float gumbel_from_bits(uint32_t w) {
  const float u = ((float)(w >> 9) + 0.5f) * 1.1920928955078125e-07f;  // 2^-23
  return -logf(-logf(u));
}

struct SamplePartial {
  float m;     // max z in the tile
  float s;     // sum exp(z - m)
  float best;  // best perturbed value of the chunk (in its first tile; else -inf)
  int idx;     // its vocab index
  float m1;    // max and sum exp of the raw logits (T = 1), for the confidence
  float s1;
};

constexpr int kConfMaxK = 32;     // largest supported top-K of the confidence
constexpr int kConfMergeNV = 24;  // list entries per lane in the chunk merge

constexpr float kLog2e = 1.4426950408889634f;

// e^d for d <= 0 (or -inf) on the hardware exp2: one rounding of d log2(e),
// then v_exp_f32 (results below 2^-126 may flush to zero; they only ever add
// to sums whose largest term is 1).  In the truncated sampler's confidence,
// against expf: rms error to 64 bits over normal logits of deviation 0.5 / 2 / 5,
// 64 entries 2.67 / 2.74 / 5.59e-7 (expf 2.61 / 2.73 / 5.59), 32000 6.35 / 6.48 /
// 14.4 (6.37 / 6.63 / 14.4), 152K 7.16 / 7.28 / 16.5 (7.14 / 7.25 / 16.5): the same;
// 128 rows of 152K 42.9 us, with expf 46.8
__device__ __forceinline__ float exp_le0(float d) { return __builtin_amdgcn_exp2f(d * kLog2e); }

__device__ __forceinline__ void lse_merge(float& m, float& s, float om, float os) {
  const float M = fmaxf(m, om);
  s = (m == -INFINITY ? 0.f : s * exp_le0(m - M)) + (om == -INFINITY ? 0.f : os * exp_le0(om - M));
  m = M;
}

// ---- top-K lists.  An entry is a logit (the confidence) or a 64-bit key of a
// (logit, vocab index) pair (truncated sampling); both sort descending.  All
// cross-lane steps stay in registers (lane_xor): with shuffles through the
// LDS crossbar the sorts and merges were most of the kernels' time.

// Key of a (value, index) pair: larger value first, then lower index (value
// bits made order-preserving as an unsigned word, -0 as +0, index inverted).
typedef uint64_t pair_key;
__device__ __forceinline__ pair_key make_key(float v, int idx) {
  const uint32_t b = __float_as_uint(v + 0.f);
  const uint32_t o = (b >> 31) ? ~b : b | 0x80000000u;
  return ((pair_key)o << 32) | (uint32_t)~idx;
}
__device__ __forceinline__ float key_value(pair_key k) {
  const uint32_t o = (uint32_t)(k >> 32);
  return __uint_as_float((o >> 31) ? o & 0x7FFFFFFFu : ~o);
}
__device__ __forceinline__ int key_index(pair_key k) { return (int)~(uint32_t)k; }
constexpr int kNoIndex = 0x7FFFFFFF;

template <int J>
__device__ __forceinline__ pair_key lane_xor(pair_key v) {
  return ((pair_key)lane_xor<J>((uint32_t)(v >> 32)) << 32) | lane_xor<J>((uint32_t)v);
}
__device__ __forceinline__ float larger(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ float smaller(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ pair_key larger(pair_key a, pair_key b) { return a > b ? a : b; }
__device__ __forceinline__ pair_key smaller(pair_key a, pair_key b) { return a > b ? b : a; }
template <typename T>
__device__ __forceinline__ T empty_entry();
template <>
__device__ __forceinline__ float empty_entry<float>() { return -INFINITY; }
template <>
__device__ __forceinline__ pair_key empty_entry<pair_key>() { return make_key(-INFINITY, kNoIndex); }
__device__ __forceinline__ float entry_value(float v) { return v; }
__device__ __forceinline__ float entry_value(pair_key k) { return key_value(k); }
// the smallest entry of a value >= L that is not empty: one compare then tests
// both (a NaN logit fails it)
__device__ __forceinline__ float lowest_at(float L, float) { return fmaxf(L, -3.402823466e38f); }
__device__ __forceinline__ pair_key lowest_at(float L, pair_key none) {
  return larger(make_key(L, -1), none + 1);
}

// Descending bitonic sort of one entry per lane (21 compare-exchange steps);
// from K = 64 on only the last merge: a bitonic sequence into order (6 steps).
template <int K, int J, typename T>
__device__ __forceinline__ void sort_steps(T& v) {
  const int lane = threadIdx.x & 63;
  const T o = lane_xor<J>(v);
  v = (((lane & K) == 0) == ((lane & J) == 0)) ? larger(v, o) : smaller(v, o);
  if constexpr (J > 1) sort_steps<K, J / 2>(v);
  else if constexpr (K < kWave) sort_steps<2 * K, K>(v);
}
template <typename T>
__device__ __forceinline__ T wave_sort_desc(T v) {
  sort_steps<2, 1>(v);
  return v;
}
template <typename T>
__device__ __forceinline__ T wave_merge_desc(T v) {
  sort_steps<kWave, kWave / 2>(v);
  return v;
}

// lane i gets the entry of lane 63 - i
template <typename T>
__device__ __forceinline__ T lane_reverse(T v) {
  v = lane_xor<32>(v);
  v = lane_xor<16>(v);
  v = lane_xor<8>(v);
  v = lane_xor<4>(v);
  v = lane_xor<2>(v);
  return lane_xor<1>(v);
}

// The K <= 32 largest of the entries a wave sees, NV per lane at a time.  The
// entries that may belong to them wait in cand (64 entries of LDS): with L a
// lower bound of the K-th largest value, those >= L.  First bound: the K-th
// largest of the 64 lane maxima of the first batch (the K largest lane maxima
// are K values >= it), which leaves K to 2 K candidates of ordinary logits;
// when the waiting ones fill up, they are sorted, the first K stay and the
// last of these is the next bound.  A batch with more candidates than there is
// room for (many equal values) is sorted and merged slot by slot.  K rounds of
// a wave arg-max through LDS shuffles were latency-bound: 45 + 55 us for top-k
// 20 over 16 x 151936 logits, 11 + 9 us so; a step's final merge with the
// confidence at a vocabulary of 4096 26.6 -> 5.2 us.
// NaN logits are empty entries, and those are never taken.
template <typename T>
struct TopList {
  T* cand;
  int K;
  int n = 0;
  float L = -INFINITY;

  // candidates in order, the first K of the wave's n kept (w: more candidates,
  // descending, one per lane)
  __device__ __forceinline__ T sorted(T w) {
    const int lane = threadIdx.x & 63;
    const T b = wave_sort_desc(lane < n ? cand[lane] : empty_entry<T>());
    return wave_merge_desc(larger(b, lane_reverse(w)));
  }
  __device__ __forceinline__ T sorted() {
    const int lane = threadIdx.x & 63;
    return wave_sort_desc(lane < n ? cand[lane] : empty_entry<T>());
  }
  __device__ __forceinline__ void keep(T v) {
    const int lane = threadIdx.x & 63;
    if (lane < K) cand[lane] = v;
    n = __popcll(__ballot(lane < K && v > empty_entry<T>()));
    if (n == K) L = fmaxf(L, __shfl(entry_value(v), K - 1, kWave));
    lds_order();
  }
  // the wave's LDS accesses in program order (the hardware keeps it; this
  // holds the compiler to it)
  __device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // lm: the largest of the lane's values
  template <int NV>
  __device__ __forceinline__ void add(const T (&x)[NV], float lm, bool first) {
    const T none = empty_entry<T>();
    if (first) {
      L = __shfl(wave_sort_desc(lm), K - 1, kWave);
    } else if (!__any(lm >= L)) {
      return;
    } else if (n > kWave / 2) {
      lds_order();
      keep(sorted());
    }
    const int n0 = n;
    const T low = lowest_at(L, none);
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      const bool c = x[e] >= low;
      const uint64_t m = __builtin_amdgcn_ballot_w64(c);
      if (m) {
        const int pos = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if (c && pos < kWave) cand[pos] = x[e];
        n += __popcll(m);
      }
    }
    if (n > kWave) {
      // no room: the batch is merged into the n0 earlier candidates slot by slot
      n = n0;
#pragma unroll 1
      for (int e = 0; e < NV; ++e) {
        T v = none;
#pragma unroll
        for (int j = 0; j < NV; ++j)
          if (j == e) v = larger(x[j], none);
        lds_order();
        keep(sorted(wave_sort_desc(v)));
      }
    }
  }
  // the K largest, descending, to out[0..K) (empty past the last real one)
  __device__ __forceinline__ void finish(T* out) {
    lds_order();
    const T v = sorted();
    if ((threadIdx.x & 63) < K) out[threadIdx.x & 63] = v;
  }
};

// Merges four descending lists of K <= 32 entries (list w at lists[w * 32])
// into their K largest, descending, returned in lanes 0..K-1 (one wave).
template <typename T>
__device__ __forceinline__ T merge4_desc(const T* lists, int K) {
  const int lane = threadIdx.x & 63;
  const T none = empty_entry<T>();
  auto get = [&](int w, int r) { return r < K ? lists[w * kConfMaxK + r] : none; };
  // a list descending then the next ascending: a bitonic sequence
  const T a = wave_merge_desc(lane < 32 ? get(0, lane) : get(1, 63 - lane));
  const T b = wave_merge_desc(lane < 32 ? get(2, lane) : get(3, 63 - lane));
  const T r = lane_reverse(b);  // (by all lanes) lanes 32..63: b[31..0], ascending
  return wave_merge_desc(lane < 32 ? a : r);
}

// sum in order of the first n <= 64 lanes' values (uniform result)
__device__ __forceinline__ float lanes_sum(float v, int n) {
  float s = 0.f;
  for (int r = 0; r < n; ++r)
    s += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), r));
  return s;
}

__device__ __forceinline__ bool better(float a, int ia, float b, int ib) {
  return a > b || (a == b && ia < ib);
}

// (m, s) over a wave: the maximum is found first, so each lane rescales once
__device__ __forceinline__ void wave_lse(float& m, float& s) {
  const float M = wave_max(m);
  s = wave_sum(m == -INFINITY ? 0.f : s * exp_le0(m - M));
  m = M;
}

// RAW: the raw-logit statistics (m1, s1) differ from z's and are merged too;
// otherwise they are set equal to the merged (m, s).
template <int NW, bool RAW = true>
__device__ __forceinline__ SamplePartial block_merge(SamplePartial p, SamplePartial* red) {
  wave_lse(p.m, p.s);
  if constexpr (RAW) wave_lse(p.m1, p.s1);
  const float B = wave_max(p.best);
  p.idx = wave_min(p.best == B ? p.idx : kNoIndex);
  p.best = B;
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = p;
  __syncthreads();
  SamplePartial r = red[0];
#pragma unroll
  for (int k = 1; k < NW; ++k) {
    const SamplePartial o = red[k];
    lse_merge(r.m, r.s, o.m, o.s);
    if constexpr (RAW) lse_merge(r.m1, r.s1, o.m1, o.s1);
    if (better(o.best, o.idx, r.best, r.idx)) {
      r.best = o.best;
      r.idx = o.idx;
    }
  }
  if constexpr (!RAW) {
    r.m1 = r.m;
    r.s1 = r.s;
  }
  return r;
}

// The 16 logits of this thread in the 4096-entry tile at `base` (past the
// vocabulary: -inf).  The four 16-byte loads are issued without a branch
// between them: with the guarded scalar loads of the vocabulary's end in the
// way, each waited for the one before it (scored rows of 152K logits with the
// confidence: 2.8 TB/s).  A group past the end reads the row's first one.
__device__ __forceinline__ void load_tile(const float* row, int base, int vocab, float (&x)[16]) {
  const int v0 = base + threadIdx.x * 4;
  if (base + kSampleChunk <= vocab) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float4 lv = *reinterpret_cast<const float4*>(row + v0 + 1024 * r);
      x[4 * r] = lv.x, x[4 * r + 1] = lv.y, x[4 * r + 2] = lv.z, x[4 * r + 3] = lv.w;
    }
    return;
  }
  if (vocab >= 4) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int v = v0 + 1024 * r;
      const float4 lv = *reinterpret_cast<const float4*>(row + (v + 3 < vocab ? v : 0));
      x[4 * r] = lv.x, x[4 * r + 1] = lv.y, x[4 * r + 2] = lv.z, x[4 * r + 3] = lv.w;
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int v = v0 + 1024 * r;
    if (v + 3 < vocab) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * r + e] = v + e < vocab ? row[v + e] : -INFINITY;
  }
}

__device__ __forceinline__ float max16(const float (&x)[16]) {
  float t = -INFINITY;
#pragma unroll
  for (int e = 0; e < 16; ++e) t = fmaxf(t, x[e]);
  return t;
}

// max and sum of exp(x - max) of 16 values, t their largest; values without a
// comparable one among them (all -inf or NaN) give an empty sum
__device__ __forceinline__ float2 lse16(const float (&x)[16], float t) {
  if (t == -INFINITY) return float2{-INFINITY, 0.f};
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) s += exp_le0(x[e] - t);  // exp(-inf) = 0
  return float2{t, s};
}

// The waves' (m, s) of each tile that a workgroup walks (and of the raw logits).
// A tile is merged over the lanes, then over the four waves, whatever else the
// workgroup holds; carried over its tiles instead, the last bits of the
// log-probabilities and confidences followed the number of rows (greedy with the
// confidence over 152K logits, us, carried / per tile: 1121 rows 163 / 169, 1927
// 266 / 266, 4096 513 / 504).
constexpr int kMaxTiles = kWave;
template <bool RAW, int MAX = kMaxTiles>
struct TileSums {
  float2 z[MAX][4];
  float2 raw[RAW ? MAX : 1][4];
  float best[4];
  int idx[4];

  __device__ __forceinline__ void put(float2 (&to)[4], float2 v) {
    wave_lse(v.x, v.y);
    if ((threadIdx.x & 63) == 0) to[threadIdx.x >> 6] = v;
  }
  __device__ __forceinline__ void put_best(float b, int i) {
    const float B = wave_max(b);
    i = wave_min(b == B ? i : kNoIndex);
    if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = B, idx[threadIdx.x >> 6] = i;
  }
  static __device__ __forceinline__ float2 merged(const float2 (&w)[4]) {
    float2 r = w[0];
#pragma unroll
    for (int k = 1; k < 4; ++k) lse_merge(r.x, r.y, w[k].x, w[k].y);
    return r;
  }
  // after a barrier, by one wave: the partials of the chunk's n tiles
  __device__ __forceinline__ void store(SamplePartial* out, int n) {
    const int t = threadIdx.x & 63;
    if (t >= n) return;
    const float2 zs = merged(z[t]);
    const float2 rs = RAW ? merged(raw[t]) : zs;
    SamplePartial p{zs.x, zs.y, -INFINITY, kNoIndex, rs.x, rs.y};
    if (t == 0)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (better(best[k], idx[k], p.best, p.idx)) p.best = best[k], p.idx = idx[k];
    out[t] = p;
  }
};

// Pass 1.  MODE 0: T = 0 (greedy, no noise, z = x); 1: T = 1 (z = x); 2: any
// other T (z = x / T).  CONF: also the chunk's conf_k largest raw logits (only
// then a chunk may be several tiles).
template <int MODE, bool CONF>
__global__ __launch_bounds__(256) void sample_partial_kernel(
    const float* __restrict__ logits, int vocab, int64_t ld, int row_tiles, int tiles, float temp,
    uint64_t seed, const uint64_t* __restrict__ uid, const int32_t* __restrict__ positions,
    SamplePartial* __restrict__ part, int conf_k, float* __restrict__ topk) {
  // for MODE 2 with the confidence also the statistics of the raw logits
  // (T = 1), else they are z's
  constexpr bool kRaw = MODE == 2 && CONF;
  __shared__ TileSums<kRaw, CONF ? kMaxTiles : 1> sums;
  __shared__ float wtop[4][kConfMaxK];
  __shared__ float cand[4][kWave];
  const int chunk = blockIdx.x;
  const int i = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float* row = logits + (size_t)i * ld;
  if constexpr (!CONF) tiles = 1;
  uint64_t cu = 0;
  uint32_t pos = 0;
  if constexpr (MODE != 0) {
    cu = uid[i];
    pos = (uint32_t)positions[i];
  }
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  float best = -INFINITY;
  int bidx = kNoIndex;
  TopList<float> list{cand[wave], conf_k};
  int best_base = 0;  // MODE 0: the tile of this lane's first largest value
  float next[16];
  load_tile(row, chunk * tiles * kSampleChunk, vocab, next);
  const int nt = min(tiles, row_tiles - chunk * tiles);
  for (int t = 0; t < nt; ++t) {
    const int base = (chunk * tiles + t) * kSampleChunk;
    float raw[16], z[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) raw[e] = next[e];
    if (t + 1 < nt) load_tile(row, base + kSampleChunk, vocab, next);
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = MODE == 2 ? raw[e] / temp : raw[e];
    const float zmax = max16(z);
    if constexpr (MODE == 0) {
      if (zmax > best) {
        best = zmax;
        best_base = base;
      }
    } else {
      // the best perturbed value z + G; v ascends within a thread, so the
      // strict > keeps the lowest index of a tie
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int v0 = base + (r * 256 + threadIdx.x) * 4;
        float g[4] = {0.f, 0.f, 0.f, 0.f};
        if (v0 < vocab) {
          const u32x4 w = philox4x32_10(
              u32x4{(uint32_t)v0 >> 2, pos, (uint32_t)cu, (uint32_t)(cu >> 32)}, k0, k1);
          g[0] = gumbel_from_bits(w.x);
          g[1] = gumbel_from_bits(w.y);
          g[2] = gumbel_from_bits(w.z);
          g[3] = gumbel_from_bits(w.w);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float pv = z[4 * r + e] + g[e];
          if (v0 + e < vocab && pv > best) {
            best = pv;
            bidx = v0 + e;
          }
        }
      }
    }
    sums.put(sums.z[t], lse16(z, zmax));
    const float rmax = kRaw ? max16(raw) : zmax;
    if constexpr (kRaw) sums.put(sums.raw[t], lse16(raw, rmax));
    if constexpr (CONF) list.add(raw, rmax, t == 0);
  }
  if constexpr (MODE == 0) {
    // the index of the largest value: its first place in the lane's tile
    if (best > -INFINITY) {
      if (tiles > 1) load_tile(row, best_base, vocab, next);
#pragma unroll
      for (int e = 15; e >= 0; --e)
        if (next[e] == best) bidx = best_base + ((e >> 2) * 256 + threadIdx.x) * 4 + (e & 3);
    }
  }
  if constexpr (CONF) list.finish(wtop[wave]);
  sums.put_best(best, bidx);
  __syncthreads();  // orders the sums, the bests and the four lists
  if (wave != 0) return;
  sums.store(part + (size_t)i * row_tiles + chunk * tiles, nt);
  if constexpr (CONF) {
    const float v = merge4_desc(&wtop[0][0], conf_k);
    if (lane < conf_k) topk[((size_t)i * gridDim.x + chunk) * kConfMaxK + lane] = v;
  }
}

// Loads a wave's share of a row's chunk lists (nchunks lists of L entries at
// stride kConfMaxK, flattened; wave w takes a contiguous quarter) and leaves
// the share's L largest in out: NV * 64 entries per wave at most.
template <int NV, typename T, typename Get>
__device__ __forceinline__ void merge_share(int nchunks, int L, Get get, T* out, T* cand) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int total = nchunks * L, per = (total + 3) / 4;
  T x[NV];
#pragma unroll
  for (int e = 0; e < NV; ++e) {
    const int q = wave * per + e * kWave + lane;  // entry of the flattened lists
    const bool ok = e * kWave + lane < per && q < total;
    const int c = ok ? q / L : 0;
    x[e] = ok ? get((size_t)c * kConfMaxK + (q - c * L)) : empty_entry<T>();
  }
  float lm = -INFINITY;
#pragma unroll
  for (int e = 0; e < NV; ++e) lm = fmaxf(lm, entry_value(x[e]));
  TopList<T> list{cand, L};
  list.add(x, lm, true);
  list.finish(out);
}
// up to kConfSmallNV * 256 entries (a 152K vocabulary at L <= 26) take the
// short form: the general one walks 24 mostly empty slots per lane
constexpr int kConfSmallNV = 4;
template <typename T, typename Get>
__device__ __forceinline__ void merge_lists(int nchunks, int L, Get get, T* out, T* cand) {
  if (nchunks * L <= kConfSmallNV * 4 * kWave) merge_share<kConfSmallNV>(nchunks, L, get, out, cand);
  else merge_share<kConfMergeNV>(nchunks, L, get, out, cand);
}

__global__ __launch_bounds__(256) void sample_final_kernel(
    const SamplePartial* __restrict__ part, int row_tiles, int nchunks,
    const float* __restrict__ logits, int vocab, int64_t ld, float temp,
    int32_t* __restrict__ out_tokens, float* __restrict__ out_lp, int conf_k, const float* __restrict__ topk, float* __restrict__ out_conf,
    float* __restrict__ conf_sum) {
  __shared__ SamplePartial red[4];
  __shared__ float wtop[4][kConfMaxK];
  __shared__ float cand[4][kWave];
  const int i = blockIdx.x;
  SamplePartial p{-INFINITY, 0.f, -INFINITY, kNoIndex, -INFINITY, 0.f};
  for (int c = threadIdx.x; c < row_tiles; c += 256) {
    const SamplePartial o = part[(size_t)i * row_tiles + c];
    lse_merge(p.m, p.s, o.m, o.s);
    lse_merge(p.m1, p.s1, o.m1, o.s1);
    if (better(o.best, o.idx, p.best, p.idx)) {
      p.best = o.best;
      p.idx = o.idx;
    }
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (conf_k > 0) {
    // merge the chunks' lists: a quarter per wave, then wave 0 merges the four
    // results (host checks nchunks * conf_k fits)
    const float* src = topk + (size_t)i * nchunks * kConfMaxK;
    merge_lists(nchunks, conf_k, [&](size_t o) { return src[o]; }, wtop[wave], cand[wave]);
  }
  p = block_merge<4>(p, red);  // its barrier also orders the four lists
  if (wave != 0) return;
  if (lane == 0) {
    const int id = p.idx;
    if (id < 0 || id >= vocab) {
      // no perturbed value compared greater than -inf (every logit NaN): no
      // token, and the logits are not read at the missing index
      out_tokens[i] = -1;
      out_lp[i] = __builtin_nanf("");
    } else {
      float zid = logits[(size_t)i * ld + id];
      if (temp != 0.f && temp != 1.f) zid = zid / temp;
      out_tokens[i] = id;
      out_lp[i] = zid - (p.m + logf(p.s));
    }
  }
  if (conf_k > 0) {
    const float sum = lanes_sum(merge4_desc(&wtop[0][0], conf_k), conf_k);
    if (lane == 0) {
      const float c = (p.m1 + logf(p.s1)) - sum / (float)conf_k;
      if (out_conf) out_conf[i] = c;
      if (conf_sum) conf_sum[i] += c;
    }
  }
}

// GC(g) = (1/K) sum over the group's candidates of conf_sum / token count (Eq. 2)
__global__ __launch_bounds__(256) void group_confidence_kernel(
    const float* __restrict__ conf_sum, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ groups, int n_groups, int K, float* __restrict__ out) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n_groups) return;
  float a = 0.f;
  for (int k = 0; k < K; ++k) {
    const int c = groups[(size_t)g * K + k];
    a += conf_sum[c] / (float)counts[c];
  }
  out[g] = a / (float)K;
}

// ---- truncated sampling (top-k, then min-p and top-p inside the top-k set)
//
// The kept set is the top_k logits in (value desc, vocab index asc) order --
// temperature does not change it.  With z = logit / T over that set, min-p
// keeps z_j >= z_0 + log(min_p); top-p keeps, in list order, the entries whose
// preceding cumulative probability (renormalised over the min-p set) is below
// top_p.  The token is the Gumbel-max over the kept entries (same Philox noise
// as the full sampler), lp = z_id - logsumexp(kept z).  T = 0: the first entry,
// with the truncation and lp evaluated at T = 1.
__global__ __launch_bounds__(256) void sample_trunc_partial_kernel(
    const float* __restrict__ logits, int vocab, int64_t ld, int row_tiles, int tiles, int L,
    SamplePartial* __restrict__ part, float* __restrict__ topv, int* __restrict__ topi) {
  __shared__ TileSums<false> sums;
  __shared__ pair_key wtop[4][kConfMaxK];
  __shared__ pair_key cand[4][kWave];
  const int chunk = blockIdx.x;
  const int i = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float* row = logits + (size_t)i * ld;
  TopList<pair_key> list{cand[wave], L};
  float next[16];
  load_tile(row, chunk * tiles * kSampleChunk, vocab, next);
  const int nt = min(tiles, row_tiles - chunk * tiles);
  for (int t = 0; t < nt; ++t) {
    const int base = (chunk * tiles + t) * kSampleChunk;
    float x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = next[e];
    if (t + 1 < nt) load_tile(row, base + kSampleChunk, vocab, next);
    const float xmax = max16(x);
    sums.put(sums.z[t], lse16(x, xmax));
    pair_key key[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      // past the vocabulary or NaN: empty (a -inf logit is an entry)
      const int v = base + ((e >> 2) * 256 + threadIdx.x) * 4 + (e & 3);
      key[e] = v < vocab && x[e] == x[e] ? make_key(x[e], v) : empty_entry<pair_key>();
    }
    list.add(key, xmax, t == 0);
  }
  list.finish(wtop[wave]);
  sums.put_best(-INFINITY, kNoIndex);
  __syncthreads();  // orders the sums and the four lists
  if (wave != 0) return;
  sums.store(part + (size_t)i * row_tiles + chunk * tiles, nt);
  const pair_key k = merge4_desc(&wtop[0][0], L);
  const size_t o = ((size_t)i * gridDim.x + chunk) * kConfMaxK;
  if (lane < L) {
    topv[o + lane] = key_value(k);
    topi[o + lane] = key_index(k);
  }
}

__global__ __launch_bounds__(256) void sample_trunc_final_kernel(
    const SamplePartial* __restrict__ part, int row_tiles, int nchunks, int L,
    const float* __restrict__ topv,
    const int* __restrict__ topi, float temp, int top_k, float top_p, float min_p, uint64_t seed,
    const uint64_t* __restrict__ uid, const int32_t* __restrict__ positions,
    int32_t* __restrict__ out_tokens, float* __restrict__ out_lp, int conf_k,
    float* __restrict__ out_conf, float* __restrict__ conf_sum) {
  __shared__ SamplePartial red[4];
  __shared__ pair_key wtop[4][kConfMaxK];
  __shared__ pair_key cand[4][kWave];
  const int i = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // logsumexp of the raw logits (confidence)
  SamplePartial p{-INFINITY, 0.f, -INFINITY, kNoIndex, -INFINITY, 0.f};
  for (int c = threadIdx.x; c < row_tiles; c += 256) {
    const SamplePartial o = part[(size_t)i * row_tiles + c];
    lse_merge(p.m, p.s, o.m, o.s);
  }
  // merge the chunks' lists: a quarter per wave, then wave 0 merges the four
  const size_t base = (size_t)i * nchunks * kConfMaxK;
  merge_lists(nchunks, L, [&](size_t o) { return make_key(topv[base + o], topi[base + o]); },
              wtop[wave], cand[wave]);
  p = block_merge<4, false>(p, red);  // its barrier also orders the four lists
  if (wave != 0) return;
  // lane j < L holds entry j of the row's list
  const pair_key k = merge4_desc(&wtop[0][0], L);
  const float fv = key_value(k);
  const int fi = key_index(k);
  const float tdiv = temp == 0.f ? 1.f : temp;  // T = 0: truncation and lp at T = 1
  const float z = fv / tdiv;
  const float z0 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(z)));
  // min-p, then top-p in list order over the renormalised min-p set
  const float d = z - z0;
  bool keep = lane < top_k && (!(min_p > 0.f) || d >= logf(min_p));
  const float ez = expf(d);
  const float et = keep ? ez : 0.f;
  if (top_p < 1.f) {
    const float bound = top_p * lanes_sum(et, top_k);
    float cum = 0.f;
    for (int j = 0; j < top_k; ++j) {  // the probability before entry j, in list order
      if (lane == j && !(cum < bound)) keep = false;
      const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(et), j));
      if (cum < bound) cum += w;
    }
  }
  // Gumbel-max over the kept entries
  float pv = -INFINITY;
  int pid = kNoIndex;
  if (keep) {
    float g = 0.f;
    if (temp != 0.f) {
      const uint64_t cu = uid[i];
      const u32x4 w = philox4x32_10(
          u32x4{(uint32_t)(fi >> 2), (uint32_t)positions[i], (uint32_t)cu, (uint32_t)(cu >> 32)},
          (uint32_t)seed, (uint32_t)(seed >> 32));
      const uint32_t word = (fi & 3) == 0 ? w.x : (fi & 3) == 1 ? w.y : (fi & 3) == 2 ? w.z : w.w;
      g = gumbel_from_bits(word);
    }
    pv = z + g;
    pid = fi;
  }
  const float sum_ez = wave_sum(keep ? ez : 0.f);
  const float best = wave_max(pv);
  const int id = wave_min(pv == best ? pid : kNoIndex);
  const bool found = id >= 0 && id != kNoIndex;  // a kept entry won
  if (lane == 0 && !found) {
    out_tokens[i] = -1;
    out_lp[i] = __builtin_nanf("");
  }
  if (found && keep && fi == id) {  // the winner's lane (indices are unique)
    out_tokens[i] = id;
    out_lp[i] = z - (z0 + logf(sum_ez));
  }
  if (conf_k > 0) {
    const float sum = lanes_sum(fv, conf_k);
    if (lane == 0) {
      const float c = (p.m + logf(p.s)) - sum / (float)conf_k;
      if (out_conf) out_conf[i] = c;
      if (conf_sum) conf_sum[i] += c;
    }
  }
}

// 4096-entry tiles per workgroup of a list pass.  A wave's list admits about
// conf_k / t of tile t's entries and is sorted and merged once per chunk, so with
// enough rows chunks are long: as many tiles as leave kTiledGroups workgroups, in
// equal chunks.  Fewer than kLongChunkTiles tiles in all, and every pass without
// lists, run one tile each: a tile's loads then overlap other workgroups' work
// instead of waiting for their own (us, one tile / long chunks, greedy with the
// confidence, T = 0.7 with it, top-k 20: 256 rows of 152K 52 / 69, 108 / 137, 71 /
// 101; 512 rows 95 / 99, 203 / 222, 131 / 133; 1024 rows 177 / 161, 392 / 377, 247 /
// 193; 4096 rows of 32000 165 / 165, 347 / 341, 226 / 201; without lists 256 rows
// greedy 30 / 45, 2048 rows 212 / 252).
constexpr int kTiledGroups = 2048, kLongChunkTiles = 24576;
static int row_tiles_of(int vocab) { return (vocab + kSampleChunk - 1) / kSampleChunk; }
static int sample_tiles(int n, int row_tiles) {
  if ((long long)n * row_tiles < kLongChunkTiles) return 1;
  const int chunks = std::max(std::min(row_tiles, (kTiledGroups + n - 1) / n),
                              (row_tiles + kMaxTiles - 1) / kMaxTiles);
  return (row_tiles + chunks - 1) / chunks;
}

static size_t partial_bytes(int n, int nchunks) {
  return ((size_t)n * nchunks * sizeof(SamplePartial) + 255) / 256 * 256;
}

static size_t list_bytes(int n, int nchunks) {
  return ((size_t)n * nchunks * kConfMaxK * sizeof(float) + 255) / 256 * 256;
}

size_t sample_workspace_bytes(int n, int vocab) {
  const int nchunks = row_tiles_of(vocab);
  return partial_bytes(n, nchunks) + 2 * list_bytes(n, nchunks);
}

bool sample_conf_supported(int vocab, int list_len) {
  const int nchunks = row_tiles_of(vocab);
  return list_len >= 0 && list_len <= kConfMaxK && list_len <= vocab &&
         (size_t)nchunks * list_len <= (size_t)4 * kWave * kConfMergeNV;
}

hipError_t launch_logprob_sample(const float* logits, int n, int vocab, int64_t ld, float temp,
                                 uint64_t seed, const uint64_t* uid, const int32_t* positions,
                                 int32_t* out_tokens, float* out_lp, float* workspace,
                                 int conf_k, float* out_conf, float* conf_sum, hipStream_t st,
                                 int top_k, float top_p, float min_p) {
  if (n == 0) return hipSuccess;
  const int row_tiles = row_tiles_of(vocab);
  const int tiles = conf_k > 0 || top_k > 0 ? sample_tiles(n, row_tiles) : 1;
  const int nchunks = (row_tiles + tiles - 1) / tiles;
  SamplePartial* part = reinterpret_cast<SamplePartial*>(workspace);  // per tile
  char* lists = reinterpret_cast<char*>(workspace) + partial_bytes(n, row_tiles);
  float* topk = reinterpret_cast<float*>(lists);
  int* topi = reinterpret_cast<int*>(lists + list_bytes(n, nchunks));
  if (top_k > 0) {
    const int L = top_k > conf_k ? top_k : conf_k;
    hipLaunchKernelGGL(sample_trunc_partial_kernel, dim3(nchunks, n), dim3(256), 0, st, logits,
                       vocab, ld, row_tiles, tiles, L, part, topk, topi);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sample_trunc_final_kernel, dim3(n), dim3(256), 0, st, part, row_tiles,
                       nchunks, L, topk, topi, temp, top_k, top_p, min_p, seed, uid, positions,
                       out_tokens, out_lp, conf_k, out_conf, conf_sum);
    return hipGetLastError();
  }
  using PartialFn = void (*)(const float*, int, int64_t, int, int, float, uint64_t, const uint64_t*,
                            const int32_t*, SamplePartial*, int, float*);
  static constexpr PartialFn kPartial[3][2] = {
      {sample_partial_kernel<0, false>, sample_partial_kernel<0, true>},
      {sample_partial_kernel<1, false>, sample_partial_kernel<1, true>},
      {sample_partial_kernel<2, false>, sample_partial_kernel<2, true>}};
  const int mode = temp == 0.f ? 0 : temp == 1.f ? 1 : 2;
  hipLaunchKernelGGL(kPartial[mode][conf_k > 0 ? 1 : 0], dim3(nchunks, n), dim3(256), 0, st,
                     logits, vocab, ld, row_tiles, tiles, temp, seed, uid, positions, part, conf_k,
                     topk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sample_final_kernel, dim3(n), dim3(256), 0, st, part, row_tiles, nchunks,
                     logits, vocab, ld, temp, out_tokens, out_lp, conf_k, topk, out_conf, conf_sum);
  return hipGetLastError();
}

// One workgroup per sequence: binary search of its scored rows, then each
// thread sums a contiguous slice in order and the slices are added in thread
// order (a fixed order: the result does not depend on scheduling).
__global__ __launch_bounds__(256) void seq_confidence_kernel(const float* __restrict__ row_conf,
                                                             const int32_t* __restrict__ rows,
                                                             int n_scored,
                                                             const int32_t* __restrict__ seq_starts,
                                                             float* __restrict__ out) {
  __shared__ float part[256];
  const int s = blockIdx.x;
  auto lower = [&](int key) {  // first r with rows[r] >= key
    int lo = 0, hi = n_scored;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (rows[mid] < key) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  const int a = lower(seq_starts[s]), b = lower(seq_starts[s + 1]);
  const int n = b - a;
  const int per = (n + 255) / 256;
  const int r0 = a + threadIdx.x * per, r1 = min(b, r0 + per);
  float acc = 0.f;
  for (int r = r0; r < r1; ++r) acc += row_conf[r];
  part[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
    for (int i = 0; i < 256; ++i) t += part[i];
    out[s] = n > 0 ? t / (float)n : 0.f;
  }
}

hipError_t launch_seq_confidence(const float* row_conf, const int32_t* scored_rows, int n_scored,
                                 const int32_t* seq_starts, int n_seqs, float* out,
                                 hipStream_t st) {
  if (n_seqs == 0) return hipSuccess;
  hipLaunchKernelGGL(seq_confidence_kernel, dim3(n_seqs), dim3(256), 0, st, row_conf, scored_rows,
                     n_scored, seq_starts, out);
  return hipGetLastError();
}

hipError_t launch_group_confidence(const float* conf_sum, const int32_t* counts,
                                   const int32_t* groups, int n_groups, int K, float* out,
                                   hipStream_t st) {
  if (n_groups == 0) return hipSuccess;
  hipLaunchKernelGGL(group_confidence_kernel, dim3((n_groups + 255) / 256), dim3(256), 0, st,
                     conf_sum, counts, groups, n_groups, K, out);
  return hipGetLastError();
}

}  // namespace sevo
