// libtva, device side of draft-tree construction (gfx950): one layer of expansion and the cut of a grown tree to
// its best nodes.  Definitions and argument layout: include/tva_draft.h (paper, "Tree Expansion Phase", "Tree
// Reranking Phase", "Dynamic Expansion Stage").
//
// Kernels:
//   topk_parts_kernel   the HBM-bound part: every row of log-probabilities is cut into pieces of 8192 tokens, one
//                       workgroup of 256 threads per piece holds its 32 tokens per thread in registers (one
//                       coalesced read, nothing read twice) and finds the piece's best K.  Selection without a
//                       sort of the piece: the K-th largest of the 256 thread maxima is a bound that at least K
//                       tokens reach, and almost only the best K do; the few that reach it are gathered and sorted.
//   row_merge_kernel    a wave per row merges the pieces' sorted lists into the row's best K (skipped when a row is one piece).
//   expand_finish_kernel  one workgroup per sequence: adds the rows' scores and orders the sequence's candidates by
//                       counting the better ones.  (expand_finish_small_kernel: both in one launch for sequences of at most 16 rows.)
//   subtree_kernel      one workgroup per tree: rank of every node by (score, index), keep the best, renumber.
//   rank_trees_kernel, rerank_count_kernel   how many nodes the cut keeps: every tree's best scores in order (one
//                       workgroup per tree, by counting), then one workgroup for the batch: the rank-wise means,
//                       their running sums against the cost row, Algorithm 1.
// Everything is compared through one 64-bit key per element: the float mapped to an unsigned integer of the same
// order in the high word, the complement of the index in the low word -- larger key = better, and no two keys of
// one comparison are equal, so every selection below has exactly one answer.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tva.h"
#include "tva_draft.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kPieceThreads = 256, kPerThread = 32, kPiece = kPieceThreads * kPerThread;  // 8192 tokens
constexpr int kMaxK = TVA_EXPAND_MAX_K;
constexpr int kRowCandidates = 512;  // a row's pieces x K candidates, merged by one wave

// float -> unsigned of the same order (-0.0 first made +0.0, so the two compare equal as numbers do)
__device__ __forceinline__ uint32_t ordered(float x) {
  const uint32_t u = __float_as_uint(x + 0.0f);
  return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float unordered(uint32_t o) {
  return __uint_as_float(o ^ ((o >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
__device__ __forceinline__ uint64_t make_key(float x, uint32_t index) { return ((uint64_t)ordered(x) << 32) | (uint32_t)~index; }
__device__ __forceinline__ uint64_t max64(uint64_t a, uint64_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint64_t shfl_xor64(uint64_t v, int mask) {
  const uint32_t lo = __shfl_xor((uint32_t)v, mask), hi = __shfl_xor((uint32_t)(v >> 32), mask);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t wave_max(uint64_t key) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) key = max64(key, shfl_xor64(key, o));
  return key;
}

// ---- the best 16 keys of a wave, in order ----
// Sorting networks on lane exchanges of the vector ALU (data-parallel primitives: no LDS, no waits).  A row of 16 lanes is
// the unit: its 16 keys are sorted in descending order, and two sorted rows a, b give the best 16 of both as
// max(a[j], b[15 - j]), which four more exchanges sort.  K is at most 16, so a sorted row always holds what is wanted.
// (Before, places were found by counting the larger of 64 .. 192 keys in LDS, 0.7 us per 64 keys; a row costs about
// 0.15 us, a merge 0.07.)
template <int CTRL>
__device__ __forceinline__ uint64_t lanes_from(uint64_t v) {
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, true);
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}
template <int CTRL>
__device__ __forceinline__ float lanes_from(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor3 = 0x1B, kXor7 = 0x141, kXor15 = 0x140, kXor8 = 0x128;  // (8: a rotation of the row by 8)
// the pair keeps its larger key in the lane without `bit`
__device__ __forceinline__ uint64_t keep_one(uint64_t v, uint64_t other, int bit) {
  const bool low = (threadIdx.x & bit) == 0;
  return (other > v) == low ? other : v;
}
__device__ __forceinline__ float keep_one(float v, float other, int bit) {
  return (threadIdx.x & bit) == 0 ? fmaxf(v, other) : fminf(v, other);
}
__device__ __forceinline__ float max64(float a, float b) { return fmaxf(a, b); }
// lanes of the two halves of each pair of rows (of 32 lanes): what row 1 (lanes 32 ..) of `m` holds, in row 0 (lanes 0 ..)
template <bool ROWS>
__device__ __forceinline__ uint32_t from_upper(uint32_t m, uint32_t v) {
  return ROWS ? __builtin_amdgcn_permlane16_swap(m, v, false, false)[1] : __builtin_amdgcn_permlane32_swap(m, v, false, false)[1];
}
template <bool ROWS>
__device__ __forceinline__ uint64_t from_upper(uint64_t m, uint64_t v) {
  return ((uint64_t)from_upper<ROWS>((uint32_t)(m >> 32), (uint32_t)(v >> 32)) << 32) | from_upper<ROWS>((uint32_t)m, (uint32_t)v);
}
template <bool ROWS>
__device__ __forceinline__ float from_upper(float m, float v) {
  return __uint_as_float(from_upper<ROWS>(__float_as_uint(m), __float_as_uint(v)));
}
template <class T>
__device__ __forceinline__ T sort_bitonic_row(T v) {
  v = keep_one(v, lanes_from<kXor8>(v), 8);
  v = keep_one(v, lanes_from<kXor3>(lanes_from<kXor7>(v)), 4);
  v = keep_one(v, lanes_from<kXor2>(v), 2);
  return keep_one(v, lanes_from<kXor1>(v), 1);
}
template <class T>
__device__ __forceinline__ T sort_row(T v) {
  v = keep_one(v, lanes_from<kXor1>(v), 1);
  v = keep_one(v, lanes_from<kXor3>(v), 2);
  v = keep_one(v, lanes_from<kXor1>(v), 1);
  v = keep_one(v, lanes_from<kXor7>(v), 4);
  v = keep_one(v, lanes_from<kXor2>(v), 2);
  v = keep_one(v, lanes_from<kXor1>(v), 1);
  v = keep_one(v, lanes_from<kXor15>(v), 8);
  v = keep_one(v, lanes_from<kXor3>(lanes_from<kXor7>(v)), 4);
  v = keep_one(v, lanes_from<kXor2>(v), 2);
  return keep_one(v, lanes_from<kXor1>(v), 1);
}
// the best 16 of two sets of sorted rows, row by row
__device__ __forceinline__ uint64_t merge_sorted(uint64_t a, uint64_t b) { return sort_bitonic_row(max64(a, lanes_from<kXor15>(b))); }
// the best 16 of the wave's four sorted rows, in lanes 0 .. 15
template <class T>
__device__ __forceinline__ T merge_rows(T v) {
  v = sort_bitonic_row(max64(v, from_upper<true>(lanes_from<kXor15>(v), v)));   // rows 1 and 3, reversed, under rows 0 and 2
  return sort_bitonic_row(max64(v, from_upper<false>(lanes_from<kXor15>(v), v)));  // row 2, reversed, under row 0
}
__device__ __forceinline__ uint64_t read_lane64(uint64_t v, int lane) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}
// sum over the four lanes of a quad
__device__ __forceinline__ int quad_sum(int x) {
  x += __builtin_amdgcn_mov_dpp(x, kXor1, 0xf, 0xf, true);
  return x + __builtin_amdgcn_mov_dpp(x, kXor2, 0xf, 0xf, true);
}
// sums, maxima over the lanes below and the lane itself
template <int CTRL, int ROWS>
__device__ __forceinline__ double lanes_below(double x, double none) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(none), __double2loint(x), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(none), __double2hiint(x), CTRL, ROWS, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <class F>
__device__ __forceinline__ double lane_scan(double x, double none, F f) {
  x = f(x, lanes_below<0x111, 0xf>(x, none));  // from 1, 2, 4, 8 lanes below in the row of 16
  x = f(x, lanes_below<0x112, 0xf>(x, none));
  x = f(x, lanes_below<0x114, 0xf>(x, none));
  x = f(x, lanes_below<0x118, 0xf>(x, none));
  x = f(x, lanes_below<0x142, 0xa>(x, none));  // the row below's last lane, to rows 1 and 3
  return f(x, lanes_below<0x143, 0xc>(x, none));  // lane 31, to rows 2 and 3
}
__device__ __forceinline__ double lane_before(double x, double none) { return lanes_below<0x138, 0xf>(x, none); }
__device__ __forceinline__ double last_lane(double x) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63), __builtin_amdgcn_readlane(__double2loint(x), 63));
}

// Between a wave's LDS writes and its own lanes' reads of what other lanes wrote: the wave's LDS operations run in
// order, so no wait is needed, but the compiler must not move one across the other.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- Algorithm 1 on a utility and a cost sequence (Dynamic Expansion Stage, Dynamic Reranking Stage) ----
// What a count needs once the per-rank sums are known; called by ONE wave of a workgroup.  On entry s_u[k] holds, for rank
// k, the scores of that rank added over the samples in index order (LAYER) or their mean (reranking), s_c[k] the cost
// cost[k] / unit; s_p: LDS for N doubles rounded up to 16 (as s_u).  The steps and their order are the host routines'
// (tva_cast_breadth_prune, tva_cast_rerank_count): the running sum over k (LAYER: divided by B afterwards), index j
// valid unless some chord (u_j - u_i) / (c_j - c_i), i < j, is below C.
// One wave, because between barriers of a large workgroup there is little to do: 100 ranks are two per lane (5.8 us for
// the count of one sequence's layer with 1024 threads and six barriers -> 2 us).
struct CountOut {
  int32_t *count;     // [1]
  int32_t *cu_T;      // [B + 1] or NULL: b * count
  double *at;         // [2] or NULL: u and c at the count
  int32_t *err_flag;  // [1] or NULL: 1 when the costs do not increase strictly (count 0)
};

template <bool LAYER>
__device__ __forceinline__ void count_tail(const double *s_u, const double *s_c, double *s_p, int B, int N, double C, const CountOut &out) {
  const int lane = threadIdx.x & 63;
  const int per = (N + 63) / 64, k0 = lane * per < N ? lane * per : N, k1 = k0 + per < N ? k0 + per : N;  // the lane's ranks
  bool bad = false;
  for (int k = k0; k < k1; ++k) bad = bad || (k > 0 && !(s_c[k] > s_c[k - 1]));  // costs must grow with the size
  if (__ballot(bad)) {
    if (lane == 0) {
      if (out.err_flag) atomicCAS(out.err_flag, 0, 1);
      *out.count = 0;
      if (out.at) out.at[0] = out.at[1] = 0.0;
    }
    if (out.cu_T)
      for (int b = lane; b <= B; b += 64) out.cu_T[b] = 0;
    return;
  }
  // The running sum, to s_p.  By definition one addition after the other; where every addition of a sum in parallel is
  // exact (the error of each is computed along: values of float32 precision whose exponents lie close), so is every
  // prefix, and the two agree bit for bit.  Otherwise one lane adds, sixteen values fetched from LDS at a time so that
  // only the additions wait for one another.
  {
    bool exact = true;
    auto add = [&](double x, double y) {
      const double t = x + y, yy = t - x, e = (x - (t - yy)) + (y - yy);
      exact = exact && e == 0.0;  // (false for infinities and NaN too)
      return t;
    };
    double run = 0.0;
    for (int k = k0; k < k1; ++k) run = add(run, s_u[k]);
    run = lane_before(lane_scan(run, 0.0, add), 0.0);
    for (int k = k0; k < k1; ++k) {
      run = add(run, s_u[k]);
      s_p[k] = run;
    }
    if (__ballot(!exact)) {
      wave_lds_fence();
      if (lane == 0) {
        run = 0.0;
        for (int i0 = 0; i0 < N; i0 += 16) {
          double v[16];
#pragma unroll
          for (int e = 0; e < 16; ++e) v[e] = s_u[i0 + e];  // (past N: whatever is there, added to nothing that is kept)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            run += v[e];
            s_p[i0 + e] = run;
          }
        }
      }
    }
    wave_lds_fence();
  }
  // Which indices are valid.  The chord from i into j is too flat when (u_j - u_i) / (c_j - c_i) < C; with c rising that
  // is g_j < g_i for g = u - C c, up to rounding.  So j is valid when g_j exceeds the largest g before it by more than
  // a margin that covers every rounding involved (2^-45 of the largest |u| + |C c|: the quotient then clears C by
  // more than 16 units in the last place), invalid when it falls short of it by that margin (that one chord is too
  // flat), and only an index in between -- equal values, a threshold met exactly -- has its chords divided one by
  // one as the definition has them.
  double a = 0.0, top = -INFINITY;
  for (int k = k0; k < k1; ++k) {
    const double u = LAYER ? s_p[k] / B : s_p[k];  // (Eq. 1 divides the accumulated sums by the number of samples)
    s_p[k] = u;
    a = fmax(a, fabs(u) + fabs(C * s_c[k]));
    top = fmax(top, u - C * s_c[k]);
  }
  wave_lds_fence();  // (the chords read other lanes' u)
  auto larger = [](double x, double y) { return fmax(x, y); };
  const double margin = last_lane(lane_scan(a, 0.0, larger)) * 0x1p-45 + 1e-300;
  double before = lane_before(lane_scan(top, -INFINITY, larger), -INFINITY);  // the largest g of the lanes below
  int keep = 1;  // (index 1 has no chord: always valid)
  for (int k = k0; k < k1; ++k) {
    const double u = s_p[k], c = s_c[k], g = u - C * c, gap = g - before;
    before = fmax(before, g);
    bool valid = k > 0 && gap > margin;
    if (k > 0 && !valid && !(gap < -margin)) {
      bool flat = false;
      for (int i = 0; i < k; ++i) flat = flat | ((u - s_p[i]) / (c - s_c[i]) < C);
      valid = !flat;
    }
    if (valid) keep = k + 1;
  }
  const unsigned long long some = __ballot(keep > 1);
  if (some) keep = __builtin_amdgcn_readlane(keep, 63 - __builtin_clzll(some));
  if (lane == 0) {
    *out.count = keep;
    if (out.at) out.at[0] = s_p[keep - 1], out.at[1] = s_c[keep - 1];
  }
  if (out.cu_T)
    for (int b = lane; b <= B; b += 64) out.cu_T[b] = b * keep;
}

// ---- the best K of every piece of every row ----
// grid (pieces, rows).  part[(row * pieces + piece) * K + j] = key of the piece's j-th best token (0 = none: the
// piece has fewer than K tokens).  A thread holds 32 tokens.  The bound -- the K-th largest of the 256 threads' largest
// values -- comes from a sort per wave and a merge of the four; the tokens that reach it, at least K and few more, go
// to a list per wave in the groups of four they were loaded in (places by ballots, no atomics), which one wave sorts.  On
// values alone ties all pass, and rows masked by a grammar or cut to their best tokens are mostly of one value.  Where a
// wave would list more than 32 groups it takes only the first K of those whose largest token just equals the bound: it
// meets them in the order of their tokens, and any later one has K equal and earlier before it (rows cut to the best 50
// of 128256 tokens: 640 rows 253 -> 60 us, 12 rows 21.6 -> 11.5; before, the selection was made again on keys from memory).
// Where that still leaves more than 32 groups (a few threads hold most of the piece's large values), and where a value is
// no number, it is made again on keys, and where even then too many pass by K searches for the maximum.
// Bound by HBM for many rows (640 rows of 128256 tokens: 63.5 -> 52 us, 6.3 TB/s, with eight
// maxima of groups in place of 32 keys per thread to compare); for one sequence's dozen rows by the chain load -
// select (12 rows: 7.3 -> 4.6 us).
typedef f32x4 f32x4_any __attribute__((aligned(4)));  // rows start anywhere: four-byte alignment is all the loads need
constexpr int kGroups = kPerThread / 4;
__global__ void __launch_bounds__(kPieceThreads) topk_parts_kernel(const float *__restrict__ logp, int64_t ld, int V, int K,
                                                                  uint64_t *__restrict__ part) {
  constexpr int kWaves = kPieceThreads / 64;
  __shared__ uint64_t s_top[kWaves * 16];
  __shared__ __align__(16) uint64_t s_list[kWaves][128];
  __shared__ int s_count[kWaves], s_flag[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int piece = blockIdx.x, row = blockIdx.y;
  const int base = piece * kPiece;
  const float *src = logp + (size_t)row * ld;
  uint64_t *dst = part + ((size_t)row * gridDim.x + piece) * K;
  // 16 bytes per lane and load: thread t holds tokens base + 1024 i + 4 t + e
  const int first = base + 4 * tid;
  auto token_of = [&](int i, int e) { return first + i * (4 * kPieceThreads) + e; };
  f32x4 x[kGroups];
  if (base + kPiece <= V) {
#pragma unroll
    for (int i = 0; i < kGroups; ++i) x[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any *>(src + token_of(i, 0)));
  } else {
    // the row's last piece: a group that reaches past the row's end is fetched element by element
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
      const int v = token_of(i, 0);
      x[i] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      if (v + 4 <= V) {
        x[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any *>(src + v));
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (v + e < V) x[i][e] = src[v + e];
      }
    }
  }
  // the largest of each group and of all (a NaN among them stays)
  auto larger = [](float a, float b) { return __builtin_elementwise_maximum(a, b); };
  float most[kGroups], top = -INFINITY;
#pragma unroll
  for (int i = 0; i < kGroups; ++i) {
    most[i] = larger(larger(x[i][0], x[i][1]), larger(x[i][2], x[i][3]));
    top = larger(top, most[i]);
  }
  bool keys_wanted;
  {
    float *s_value = reinterpret_cast<float *>(s_top);
    const bool no_number = __ballot(top != top) != 0;
    const float best = merge_rows(sort_row(top));
    if (lane < 16) s_value[wave * 16 + lane] = best;
    if (lane == 0) s_flag[wave] = no_number;
    __syncthreads();
    keys_wanted = (s_flag[0] | s_flag[1] | s_flag[2] | s_flag[3]) != 0;
    const float merged = merge_rows(s_value[lane]);
    const float bound = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(merged), K - 1));
    int count = 0;  // groups of four with a token that reaches the bound (the others of a group read as none)
    const uint64_t below = (1ull << lane) - 1ull;
    auto list_group = [&](int i, bool in) {
      const uint64_t votes = __ballot(in);
      if (votes == 0) return;
      const int pos = count + __popcll(votes & below);
      count += __popcll(votes);
      if (in && pos < 32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int v = token_of(i, e);
          s_list[wave][4 * pos + e] = x[i][e] >= bound && v < V ? make_key(x[i][e], (uint32_t)v) : 0ull;
        }
      }
    };
    if (!keys_wanted) {
#pragma unroll
      for (int i = 0; i < kGroups; ++i) list_group(i, most[i] >= bound);
      if (count > 32) {  // (the wave's list again, with K of the groups that only equal the bound)
        count = 0;
        int equal = 0;
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
          const uint64_t level = __ballot(most[i] == bound);
          list_group(i, most[i] > bound || (most[i] == bound && equal + __popcll(level & below) < K));
          equal += __popcll(level);
        }
      }
    }
    if (lane == 0) s_count[wave] = count;
    __syncthreads();
  }
  static_assert(kWaves == 4, "four lists");
  // entry e of the four lists, one after the other, c0 .. c3 long (0 past their end)
  auto entry = [&](int e, int c0, int c1, int c2, int c3) -> uint64_t {
    if (e < c0) return s_list[0][e];
    if ((e -= c0) < c1) return s_list[1][e];
    if ((e -= c1) < c2) return s_list[2][e];
    return (e -= c2) < c3 ? s_list[3][e] : 0ull;
  };
  // the lists' keys in order, by one wave; zeros past the last token of a piece of fewer than K
  {
    const int c0 = 4 * s_count[0], c1 = 4 * s_count[1], c2 = 4 * s_count[2], c3 = 4 * s_count[3];
    if (!keys_wanted && max(max(c0, c1), max(c2, c3)) <= 128) {
      if (wave != 0) return;
      uint64_t key = sort_row(entry(lane, c0, c1, c2, c3));
      for (int e = 64; e < c0 + c1 + c2 + c3; e += 64) key = merge_sorted(key, sort_row(entry(lane + e, c0, c1, c2, c3)));
      key = merge_rows(key);
      if (lane < K) dst[lane] = key;
      return;
    }
  }
  // ---- on keys (read again: what is rare keeps no registers) ----
  auto key_at = [&](int i) {
    const int v = token_of(i / 4, i % 4);
    return v < V ? make_key(src[v], (uint32_t)v) : 0ull;
  };
  uint64_t mine = 0;
  for (int i = 0; i < kPerThread; ++i) mine = max64(mine, key_at(i));
  mine = merge_rows(sort_row(mine));
  __syncthreads();
  if (lane < 16) s_top[wave * 16 + lane] = mine;
  __syncthreads();
  const uint64_t bound = read_lane64(merge_rows(s_top[lane]), K - 1);  // (0 if fewer than K threads hold a token)
  int count = 0;
  for (int i = 0; i < kPerThread; ++i) {
    const uint64_t key = key_at(i);
    const bool in = key >= bound && key != 0ull;
    const uint64_t votes = __ballot(in);
    const int pos = count + __popcll(votes & ((1ull << lane) - 1ull));
    if (in && pos < 64) s_list[wave][pos] = key;
    count += __popcll(votes);
  }
  if (lane == 0) s_count[wave] = count;
  __syncthreads();
  const int c0 = s_count[0], c1 = s_count[1], c2 = s_count[2], c3 = s_count[3];
  if (c0 + c1 + c2 + c3 <= 64) {
    const uint64_t key = merge_rows(sort_row(entry(lane, c0, c1, c2, c3)));
    if (wave == 0 && lane < K) dst[lane] = key;
    return;
  }
  uint64_t before = ~0ull;  // the key found last
  for (int j = 0; j < K; ++j) {
    uint64_t best = 0;
    for (int i = 0; i < kPerThread; ++i) {
      const uint64_t key = key_at(i);
      if (key < before) best = max64(best, key);
    }
    best = wave_max(best);
    __syncthreads();
    if (lane == 0) s_top[wave] = best;
    __syncthreads();
    before = max64(max64(s_top[0], s_top[1]), max64(s_top[2], s_top[3]));
    if (tid == 0) dst[j] = before;
  }
}

// ---- per row: its best K out of its pieces' ----
// One wave merges one row, whose pieces' keys are sorted lists of K (at most 16) already: lane j < K of the result (lanes
// 0 .. 15) is the key of the row's j-th best token.  A row of 16 lanes takes a list, four lists a load.
__device__ __forceinline__ uint64_t merge_row(const uint64_t *__restrict__ src, int pieces, int K) {
  const int j = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
  uint64_t best = 0;
  for (int p0 = 0; p0 < pieces; p0 += 16) {
    uint64_t v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int piece = p0 + 4 * r + q;
      v[r] = piece < pieces && j < K ? src[piece * K + j] : 0ull;
    }
    best = merge_sorted(best, merge_sorted(merge_sorted(v[0], v[1]), merge_sorted(v[2], v[3])));
  }
  return merge_rows(best);
}

// a wave per row, four rows per workgroup; best[row * K + j]
__global__ void __launch_bounds__(256) row_merge_kernel(const uint64_t *__restrict__ part, int pieces, int K, int rows,
                                                        uint64_t *__restrict__ best) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= rows) return;
  const uint64_t key = merge_row(part + (size_t)r * pieces * K, pieces, K);
  if (lane < K) best[(size_t)r * K + lane] = key;
}

// ---- per sequence: the candidates' scores, the candidates in order ----
// s_key[i] = key of candidate i (row i / K of the sequence, its (i % K)-th best token), s_tok[i] its token; complete
// behind a barrier, zeros from total to the next multiple of 32.  A candidate's place in the sequence's order is the
// number of candidates that are better: the four lanes of a quad count a quarter each (144 candidates: 36 reads of LDS
// instead of 144) and write one of its results each.  values: the candidates' values in order, exp(score) in double
// precision rounded to float32, as the breadth decision takes them; to LDS as doubles for a count that follows in the
// launch, or to global memory as floats.
template <class T>
__device__ __forceinline__ void order_candidates(const uint64_t *s_key, const int32_t *s_tok, int total, int K, size_t out0,
                                                 float *__restrict__ cand_score, int32_t *__restrict__ cand_parent,
                                                 int32_t *__restrict__ cand_token, T *values) {
  const int sub = threadIdx.x & 3, step = blockDim.x >> 2;
  for (int i = threadIdx.x >> 2; i < total; i += step) {
    const uint64_t mine = s_key[i];
    int better = 0;
#pragma unroll 8
    for (int j = 0; j < (total + 31) / 32 * 8; ++j) better += s_key[4 * j + sub] > mine;
    const int place = quad_sum(better);
    const float x = unordered((uint32_t)(mine >> 32));
    if (sub == 0) cand_score[out0 + place] = x;
    if (sub == 1) cand_parent[out0 + place] = i / K;
    if (sub == 2) cand_token[out0 + place] = s_tok[i];
    if (sub == 3 && values) values[place] = (T)(float)exp((double)x);
  }
}

__global__ void __launch_bounds__(1024) expand_finish_kernel(const uint64_t *best, int K,
                                                             const int32_t *__restrict__ cu_N, const float *__restrict__ score,
                                                             float *__restrict__ cand_score, int32_t *__restrict__ cand_parent,
                                                             int32_t *__restrict__ cand_token, uint64_t *values, int64_t values_ld) {
  __shared__ uint64_t s_key[TVA_EXPAND_MAX_CANDIDATES];
  __shared__ int32_t s_tok[TVA_EXPAND_MAX_CANDIDATES];
  const int b = blockIdx.x;
  const int r0 = cu_N[b], n = cu_N[b + 1] - r0, total = n * K;
  if (n <= 0 || total > TVA_EXPAND_MAX_CANDIDATES) return;  // (more rows than the caller's max_N said: nothing written)
  for (int i = threadIdx.x; i < (total + 31) / 32 * 32; i += blockDim.x) {
    uint64_t key = 0;
    if (i < total) {
      const uint64_t k = best[(size_t)r0 * K + i];  // (a row has at least K tokens: a real key)
      key = make_key(score[r0 + i / K] + unordered((uint32_t)(k >> 32)), (uint32_t)i);
      s_tok[i] = (int32_t)~(uint32_t)k;
    }
    s_key[i] = key;
  }
  __syncthreads();
  order_candidates(s_key, s_tok, total, K, (size_t)r0 * K, cand_score, cand_parent, cand_token,
                   values && total <= 2 * values_ld ? reinterpret_cast<float *>(values + b * values_ld) : nullptr);
}

// Both steps in one launch for sequences of at most 16 rows of at most 256 piece candidates each (a sequence's rows each
// get a wave of one workgroup of 16): what a draft layer looks like.  Bound by the chain load - merge - rank - store.
// A batch of one sequence that also wants the breadth decision gets it here too, by the first wave on the values that
// are in LDS already.  (One sequence of 12 rows with the count: 13.6 us -> 6.2; 64 sequences of 10 rows: 8.3 us -> 5.2.)
constexpr int kSmallRows = 16, kSmallPerRow = 256;
__global__ void __launch_bounds__(64 * kSmallRows) expand_finish_small_kernel(const uint64_t *part, int pieces, int K,
                                                                             const int32_t *__restrict__ cu_N,
                                                                             const float *__restrict__ score,
                                                                             float *__restrict__ cand_score,
                                                                             int32_t *__restrict__ cand_parent,
                                                                             int32_t *__restrict__ cand_token, uint64_t *values,
                                                                             int64_t values_ld, const double *__restrict__ cost,
                                                                             double unit, double C, CountOut count_out) {
  constexpr int kMost = kSmallRows * kMaxK;
  __shared__ double s_u[kMost], s_c[kMost], s_p[kMost];
  __shared__ uint64_t s_key[kMost];
  __shared__ int32_t s_tok[kMost];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int b = blockIdx.x;
  const int r0 = cu_N[b], n = cu_N[b + 1] - r0, total = n * K;
  if (n <= 0 || n > kSmallRows) return;  // (more rows than the caller's max_N said: nothing written)
  const bool counted = count_out.count != nullptr;
  double cost_k = 0.0;
  if (counted && tid < total) cost_k = cost[tid];  // (fetched with the keys, used behind the merge)
  if (wave < n) {
    const float parent_score = score[r0 + wave];
    const uint64_t key = merge_row(part + (size_t)(r0 + wave) * pieces * K, pieces, K);
    const int i = wave * K + lane;
    if (lane < K) {
      s_key[i] = make_key(parent_score + unordered((uint32_t)(key >> 32)), (uint32_t)i);
      s_tok[i] = (int32_t)~(uint32_t)key;
    }
  }
  if (wave == kSmallRows - 1 && lane < 32 && total + lane < kMost) s_key[total + lane] = 0ull;
  if (counted && tid < total) s_c[tid] = cost_k / unit;
  __syncthreads();
  if (counted)
    order_candidates(s_key, s_tok, total, K, (size_t)r0 * K, cand_score, cand_parent, cand_token, s_u);
  else
    order_candidates(s_key, s_tok, total, K, (size_t)r0 * K, cand_score, cand_parent, cand_token,
                     values && total <= 2 * values_ld ? reinterpret_cast<float *>(values + b * values_ld) : nullptr);
  if (!counted) return;
  __syncthreads();
  if (wave == 0) count_tail<true>(s_u, s_c, s_p, 1, total, C, count_out);
}

// ---- the best nodes of a grown tree, renumbered ----
// Every node's rank by counting the better ones, a quarter of the tree per lane of a quad; the kept nodes' new indexes by
// ballots over the node order.  Bound by the chain of loads around that (offsets - scores - stores).
constexpr int kTreeThreads = 1024;
__global__ void __launch_bounds__(kTreeThreads) subtree_kernel(const float *__restrict__ score, const int32_t *__restrict__ parent,
                                                              const int32_t *__restrict__ cu_M, const int32_t *__restrict__ cu_T,
                                                              int32_t *__restrict__ old_index, int32_t *__restrict__ new_parent,
                                                              int32_t *__restrict__ err_flag) {
  __shared__ uint64_t s_key[TVA_SUBTREE_MAX_NODES + 32];
  __shared__ int16_t s_new[TVA_SUBTREE_MAX_NODES];  // new index of a kept node, -1 of a dropped one
  __shared__ int32_t s_parent[TVA_SUBTREE_MAX_NODES];
  __shared__ int s_kept[TVA_SUBTREE_MAX_NODES / 64];  // kept nodes of each 64
  const int tid = threadIdx.x, b = blockIdx.x;
  const int m0 = cu_M[b], M = cu_M[b + 1] - m0;
  const int t0 = cu_T[b], keep = cu_T[b + 1] - t0;
  if (keep <= 0) return;
  if (keep > M || M > TVA_SUBTREE_MAX_NODES) {
    if (tid == 0 && err_flag) atomicCAS(err_flag, 0, 1 + b);
    return;
  }
  for (int i = tid; i < (M + 31) / 32 * 32; i += kTreeThreads) {
    s_key[i] = i < M ? make_key(score[m0 + i], (uint32_t)i) : 0ull;
    if (i < M) s_parent[i] = parent[m0 + i];
  }
  __syncthreads();
  // a node is kept iff fewer than `keep` nodes are better (keys are unique: the ranks are 0 .. M-1)
  const int sub = tid & 3;
  for (int i = tid >> 2; i < M; i += kTreeThreads / 4) {
    const uint64_t mine = s_key[i];
    int better = 0;
#pragma unroll 8
    for (int j = 0; j < (M + 31) / 32 * 8; ++j) better += s_key[4 * j + sub] > mine;
    better = quad_sum(better);
    if (sub == 0) s_new[i] = better < keep ? 0 : -1;
  }
  __syncthreads();
  // new index = kept nodes before it
  for (int i = tid; i < (M + 63) / 64 * 64; i += kTreeThreads) {
    const unsigned long long kept = __ballot(i < M && s_new[i] >= 0);
    if ((i & 63) == 0) s_kept[i >> 6] = __popcll(kept);
    if (i < M && s_new[i] >= 0) s_new[i] = (int16_t)__popcll(kept & ((1ull << (i & 63)) - 1ull));
  }
  __syncthreads();
  auto new_of = [&](int i) {
    int at = s_new[i];
    for (int w = 0; w < i >> 6; ++w) at += s_kept[w];
    return at;
  };
  for (int i = tid; i < M; i += kTreeThreads) {
    if (s_new[i] < 0) continue;
    const int at = new_of(i), p = s_parent[i];
    old_index[t0 + at] = i;
    int np = -1;
    if (p >= 0) {
      np = (p < i && s_new[p] >= 0) ? new_of(p) : -1;
      if (np < 0 && err_flag) atomicCAS(err_flag, 0, 1 + b);
    }
    new_parent[t0 + at] = np;
  }
}

// ---- how many nodes the cut keeps (Dynamic Reranking Stage) ----
// Two launches.  rank_trees_kernel, one workgroup per tree: the tree's N best scores in descending order (place of a
// score = the scores of its tree that come before it: larger, or equal with a lower index), to best[B, N].
// rerank_count_kernel, one workgroup: the arithmetic of the host routine (tva_cast_rerank_count) in its order -- the
// rank-s scores are added over the samples in index order, divided by B, and accumulated over s by one thread;
// c_k = cost[k] / cost[0]; index j stays valid unless some chord (u_j - u_i) / (c_j - c_i), i < j, is below C.
constexpr int kRerankMaxN = 1024;

__global__ void __launch_bounds__(kTreeThreads) rank_trees_kernel(const float *__restrict__ score, int N_tot, int N, float *__restrict__ best) {
  __shared__ __align__(16) float s_x[TVA_SUBTREE_MAX_NODES + 64];
  const int tid = threadIdx.x, j = blockIdx.x;
  const float *row = score + (size_t)j * N_tot;
  const int padded = (N_tot + 63) / 64 * 64;  // (the tail reads as scores that come before nothing)
  for (int i = tid; i < padded; i += kTreeThreads) s_x[i] = i < N_tot ? row[i] : -INFINITY;
  __syncthreads();
  // (the four lanes of a quad take every fourth group of four scores; no branches: written with | and &, the compares
  // stay arithmetic)
  const int sub = tid & 3;
  for (int idx = tid >> 2; idx < N_tot; idx += kTreeThreads / 4) {
    const float mine = s_x[idx];
    int before = 0;
#pragma unroll 4
    for (int i0 = 4 * sub; i0 < padded; i0 += 16) {
      const f32x4 x = *reinterpret_cast<const f32x4 *>(s_x + i0);
#pragma unroll
      for (int e = 0; e < 4; ++e) before += (int)(x[e] > mine) | ((int)(x[e] == mine) & (int)(i0 + e < idx));
    }
    before = quad_sum(before);
    if (sub == 0 && before < N) best[(size_t)j * N + before] = mine;
  }
}

constexpr int kCountThreads = 1024;
constexpr int kCountStage = 10240;  // floats of LDS for the trees' best scores (64 samples x 144 candidates fit)

// LAYER = true is the per-layer form (Eq. 1 and Eq. 2 as tva_cast_breadth_prune writes them): best = the layer's
// candidates' values, already in order; the column sums are accumulated first and the running sum divided by B;
// c_k = cost[k] / unit with the target's cost of one token passed in; at[0], at[1] receive u and c at the kept count.
// best: sample j's values at best + j * ld.
template <bool LAYER>
__global__ void __launch_bounds__(kCountThreads) rerank_count_kernel(const float *__restrict__ best, int64_t ld, int B,
                                                                     const double *__restrict__ cost, double unit, int N, double C,
                                                                     CountOut out) {
  __shared__ double s_u[kRerankMaxN], s_c[kRerankMaxN];
  __shared__ __align__(8) float s_best[kCountStage];
  static_assert(kCountThreads >= kRerankMaxN && kCountStage * sizeof(float) >= kRerankMaxN * sizeof(double), "a thread per rank");
  const int tid = threadIdx.x, k = tid;
  double cost_k = 0.0, one = 1.0;
  if (k < N) cost_k = cost[k], one = LAYER ? unit : cost[0];
  // the trees' best scores, fetched by all threads at once where they fit (one round trip, not one per sample)
  const bool staged = B * N <= kCountStage;
  if (staged) {
    // (all of a thread's loads before the first store to LDS)
    constexpr int kLoads = kCountStage / kCountThreads;
    float x[kLoads];
    int j = tid / N, at = tid - j * N;  // (sample and rank of this thread's next score)
    const int dj = kCountThreads / N, dat = kCountThreads - dj * N;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      if (tid + i * kCountThreads < B * N) x[i] = best[j * ld + at];
      j += dj, at += dat;
      if (at >= N) at -= N, ++j;
    }
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      if (tid + i * kCountThreads < B * N) s_best[tid + i * kCountThreads] = x[i];
  }
  __syncthreads();
  if (k < N) {
    double col = 0.0;  // (added in the samples' order)
    if (staged) {
#pragma unroll 16
      for (int j = 0; j < B; ++j) col += (double)s_best[j * N + k];
    } else {
#pragma unroll 8
      for (int j = 0; j < B; ++j) col += (double)best[j * ld + k];
    }
    s_u[k] = LAYER ? col : col / B;  // (reranking: the rank-wise batch mean)
    s_c[k] = cost_k / one;
  }
  __syncthreads();  // (the staged scores have been added up: their place holds the running sums from here on)
  if (tid < 64) count_tail<LAYER>(s_u, s_c, reinterpret_cast<double *>(s_best), B, N, C, out);
}

int pieces_of(int V) { return (int)(((int64_t)V + kPiece - 1) / kPiece); }

// TVA_OK, or why the shapes are refused (from host values only)
int expand_shapes(const tva_expand_args *a) {
  if (!a || a->B < 0 || a->V < 1 || a->K < 1 || a->K > a->V || a->sum_N < 0) return TVA_INVALID_ARG;
  if (a->K > kMaxK) return TVA_UNSUPPORTED;
  if ((int64_t)pieces_of(a->V) * a->K > kRowCandidates) return TVA_UNSUPPORTED;  // what one wave merges per row
  if (a->sum_N > 65535) return TVA_UNSUPPORTED;  // rows are the second grid dimension
  return TVA_OK;
}

}  // namespace

extern "C" {

size_t tva_expand_workspace_bytes(const tva_expand_args *a) {
  if (expand_shapes(a) != TVA_OK) return (size_t)-1;
  // the pieces' best K, then the rows' best K
  return (size_t)a->sum_N * (pieces_of(a->V) + 1) * a->K * sizeof(uint64_t);
}

int tva_expand_layer(const tva_expand_args *a, void *stream) {
  if (const int rc = expand_shapes(a)) return rc;
  if (a->max_N < 0 || (int64_t)a->max_N * a->K > TVA_EXPAND_MAX_CANDIDATES) return TVA_UNSUPPORTED;
  if (a->B == 0 || a->sum_N == 0) return TVA_OK;
  if (!a->cu_N || !a->score || !a->logp || !a->cand_score || !a->cand_parent || !a->cand_token || !a->workspace ||
      a->ld_logp < a->V || ((uintptr_t)a->workspace & 7))
    return TVA_INVALID_ARG;
  if (a->workspace_bytes < tva_expand_workspace_bytes(a)) return TVA_WORKSPACE_TOO_SMALL;
  // the breadth decision on the sorted candidates, if asked for: every sequence the same number of rows
  const bool counted = a->count != nullptr;
  const int n_cand = a->max_N * a->K;
  if (counted && (!a->draft_cost_row || !(a->target_cost_one > 0.0) || (int64_t)a->B * a->max_N != a->sum_N)) return TVA_INVALID_ARG;
  if (counted && n_cand > kRerankMaxN) return TVA_UNSUPPORTED;
  const CountOut count_out{a->count, nullptr, a->u_c_at, a->count_err_flag};
  const CountOut no_count{nullptr, nullptr, nullptr, nullptr};
  const int pieces = pieces_of(a->V);
  uint64_t *part = static_cast<uint64_t *>(a->workspace);
  hipStream_t st = (hipStream_t)stream;
  (void)hipGetLastError();  // the status below is these launches'
  hipLaunchKernelGGL(topk_parts_kernel, dim3(pieces, a->sum_N), dim3(kPieceThreads), 0, st, a->logp, a->ld_logp, a->V, a->K, part);
  // A count over several sequences takes the values from the workspace: each sequence's from where its own pieces' keys
  // were (n * K floats; the sequence's workgroup is the only one that reads those, and has).
  const bool several = counted && a->B > 1;
  const int64_t per_sequence = (int64_t)a->max_N * pieces * a->K;
  uint64_t *const values = several || (counted && (pieces == 1 || a->max_N > kSmallRows || pieces * a->K > kSmallPerRow)) ? part : nullptr;
  if (pieces > 1 && a->max_N <= kSmallRows && pieces * a->K <= kSmallPerRow) {
    hipLaunchKernelGGL(expand_finish_small_kernel, dim3(a->B), dim3(64 * kSmallRows), 0, st, part, pieces, a->K, a->cu_N, a->score,
                       a->cand_score, a->cand_parent, a->cand_token, values, per_sequence, a->draft_cost_row, a->target_cost_one, a->C1,
                       counted && !several ? count_out : no_count);  // (a batch of one sequence: the count rides in the same launch)
  } else {
    uint64_t *best = part;
    if (pieces > 1) {
      best = part + (size_t)a->sum_N * pieces * a->K;
      hipLaunchKernelGGL(row_merge_kernel, dim3((a->sum_N + 3) / 4), dim3(256), 0, st, part, pieces, a->K, a->sum_N, best);
    }
    hipLaunchKernelGGL(expand_finish_kernel, dim3(a->B), dim3(1024), 0, st, best, a->K, a->cu_N, a->score, a->cand_score,
                       a->cand_parent, a->cand_token, values, per_sequence);
  }
  if (values)
    hipLaunchKernelGGL(rerank_count_kernel<true>, dim3(1), dim3(kCountThreads), 0, st, reinterpret_cast<const float *>(values),
                       2 * per_sequence, a->B, a->draft_cost_row, a->target_cost_one, n_cand, a->C1, count_out);
  return hipPeekAtLastError() == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

size_t tva_sizeof_expand_args(void) { return sizeof(tva_expand_args); }

int tva_tree_select_subtree(const float *score, const int32_t *parent, const int32_t *cu_M, const int32_t *cu_T, int32_t B,
                            int32_t max_M, int32_t *old_index, int32_t *new_parent, int32_t *err_flag, void *stream) {
  if (B < 0 || max_M < 0) return TVA_INVALID_ARG;
  if (max_M > TVA_SUBTREE_MAX_NODES) return TVA_UNSUPPORTED;
  if (B == 0) return TVA_OK;
  if (!score || !parent || !cu_M || !cu_T || !old_index || !new_parent) return TVA_INVALID_ARG;
  (void)hipGetLastError();
  hipLaunchKernelGGL(subtree_kernel, dim3(B), dim3(kTreeThreads), 0, (hipStream_t)stream, score, parent, cu_M, cu_T, old_index,
                     new_parent, err_flag);
  return hipPeekAtLastError() == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

size_t tva_rerank_workspace_bytes(int32_t B, int32_t N_tot, int32_t m) {
  if (B < 1 || N_tot < 1 || m < 1) return (size_t)-1;
  return (size_t)B * (N_tot < m ? N_tot : m) * sizeof(float);
}

int tva_tree_rerank_count(const float *tree_scores, int32_t B, int32_t N_tot, const double *cost_row, int32_t m, double C3,
                          int32_t *count, int32_t *cu_T, int32_t *err_flag, void *workspace, size_t workspace_bytes, void *stream) {
  if (B < 1 || N_tot < 1 || m < 1 || !tree_scores || !cost_row || !count || !workspace || ((uintptr_t)workspace & 3))
    return TVA_INVALID_ARG;
  const int N = N_tot < m ? N_tot : m;
  if (N_tot > TVA_SUBTREE_MAX_NODES || N > kRerankMaxN || B > 65535) return TVA_UNSUPPORTED;
  if (workspace_bytes < tva_rerank_workspace_bytes(B, N_tot, m)) return TVA_WORKSPACE_TOO_SMALL;
  float *best = static_cast<float *>(workspace);
  (void)hipGetLastError();
  hipLaunchKernelGGL(rank_trees_kernel, dim3(B), dim3(kTreeThreads), 0, (hipStream_t)stream, tree_scores, N_tot, N, best);
  hipLaunchKernelGGL(rerank_count_kernel<false>, dim3(1), dim3(kCountThreads), 0, (hipStream_t)stream, best, (int64_t)N, B, cost_row, 0.0, N, C3,
                     CountOut{count, cu_T, nullptr, err_flag});
  return hipPeekAtLastError() == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

int tva_layer_breadth_count(const float *cand_score, int32_t B, int32_t N, const double *draft_cost_row, double target_cost_one,
                            double C1, int32_t *count, double *u_c_at, int32_t *err_flag, void *stream) {
  if (B < 1 || N < 1 || !cand_score || !draft_cost_row || !count || !(target_cost_one > 0.0)) return TVA_INVALID_ARG;
  if (N > kRerankMaxN) return TVA_UNSUPPORTED;
  (void)hipGetLastError();
  hipLaunchKernelGGL(rerank_count_kernel<true>, dim3(1), dim3(kCountThreads), 0, (hipStream_t)stream, cand_score, (int64_t)N, B, draft_cost_row,
                     target_cost_one, N, C1, CountOut{count, nullptr, u_c_at, err_flag});
  return hipPeekAtLastError() == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

}  // extern "C"
