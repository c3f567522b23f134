// libtva: greedy tree acceptance and commit of the accepted path's K/V rows (gfx950).
// Entry points and their meaning: include/tva_verify.h.
//
//   accept_kernel   one wave per sequence.  The walk from the root is a chain of dependent steps; each
//                   step's search for the matching child is the parallel part: the 64 lanes test 64
//                   candidate nodes at once and a ballot picks the lowest index.  Integer work,
//                   latency-bound (a few L2 round trips per accepted node).
//   commit_kernel   one workgroup per (path position, sequence): a row of K and a row of V, 16 bytes
//                   per lane, straight from the tree tensors to the cache.  HBM-bound in principle
//                   (read + write of 2 * Hkv * D * 2 bytes per accepted node), launch-bound at the
//                   sizes a decode step has.
//   compact_kernel  the same commit when the tree's K/V already sit in the cache behind the committed
//                   tokens: the accepted rows move down in place, one workgroup per sequence.
//   sample_kernel   acceptance by speculative sampling: one workgroup of 1024 threads per sequence.  The walk
//                   and the tests of the children are a chain of dependent steps that every thread takes in
//                   step (they read the same words); the data-parallel part is over the vocabulary: the
//                   sum of a distribution, the residual after a rejection, the draw of the last token --
//                   one streaming pass over V floats each.
//   walk_kernel     the same with a sequence's rows held in registers, shared among up to 16 workgroups.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <type_traits>

#include "tva.h"
#include "tva_verify.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(64) accept_kernel(const int32_t *__restrict__ parent, const int32_t *__restrict__ cu_T,
                                                    const int32_t *__restrict__ draft, const int32_t *__restrict__ target,
                                                    int max_path, int32_t *__restrict__ path,
                                                    int32_t *__restrict__ path_len, int32_t *__restrict__ next_token, int fill) {
  const int b = blockIdx.x, lane = threadIdx.x;
  auto fill_from = [&](int len) {
    if (fill)
      for (int i = len + lane; i < max_path; i += 64) path[(size_t)b * max_path + i] = -1;
  };
  const int t0 = cu_T[b];
  const int T = cu_T[b + 1] - t0;
  if (T <= 0) {
    if (lane == 0) {
      path_len[b] = 0;
      next_token[b] = -1;
    }
    fill_from(0);
    return;
  }
  int cur = 0, len = 1;
  if (lane == 0) path[(size_t)b * max_path] = 0;
  // every accepted node has a larger index than the one before, so at most T - 1 steps
  while (len < max_path) {
    const int want = target[t0 + cur];
    int found = -1;
    for (int base = cur + 1; base < T && found < 0; base += 64) {
      const int c = base + lane;
      const bool hit = c < T && parent[t0 + c] == cur && draft[t0 + c] == want;
      const uint64_t votes = __ballot(hit);
      if (votes) found = base + __builtin_ctzll(votes);
    }
    if (found < 0) break;
    cur = found;
    if (lane == 0) path[(size_t)b * max_path + len] = cur;
    ++len;
  }
  if (lane == 0) {
    path_len[b] = len;
    next_token[b] = target[t0 + cur];
  }
  fill_from(len);
}

// ---- acceptance by speculative sampling ----
struct SampleParams {
  const int32_t *parent, *cu_T, *token;
  const float *p, *q, *u, *u_final;
  float *residual;
  int32_t *path, *path_len, *next_token, *err_flag;
  int V, max_path;
  int fill_path;  // the path's entries past its length are set to -1
  int unit_rows;  // every target row is taken to sum to one: a freshly reached node's normaliser is 1, not summed
};

constexpr int kSampleThreads = 1024, kSampleWaves = kSampleThreads / 64;
constexpr int kSampleTreeLds = 1024;  // nodes of a tree whose parent, token and uniform number are kept in LDS

// One pass over a vocabulary-long row.  Wave w owns the contiguous segment [w * seg, (w + 1) * seg) and its lanes
// take consecutive elements (coalesced; VEC = 4: consecutive groups of four, which needs seg % 4 == 0 and rows
// aligned to 16 bytes); the row is elements lo .. V-1 (a slice of a longer one when several workgroups share a
// row).  load(v) fetches what element (group) v needs, use(v, t, x) handles it (it may store) and
// adds its weight to x; U fetches are issued before the first is used.  wsum[w] receives the segment's sum; the
// return value, the same in every thread, is their sum taken in segment order.
template <int VEC, int U, class L, class C>
__device__ __forceinline__ double segment_pass(int lo, int V, int seg, double *wsum, L load, C use) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int s0 = lo + wave * seg, s1 = s0 + seg < V ? s0 + seg : V;
  constexpr int step = 64 * VEC;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int v = s0 + lane * VEC; v < s1; v += U * step) {
    decltype(load(0)) t[U];
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (v + k * step < s1) t[k] = load(v + k * step);
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (v + k * step < s1) use(v + k * step, t[k], acc[k & 3]);
  }
  double x = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
  __syncthreads();  // (wsum may still be read from the pass before; stores of use() are visible after the next barrier)
  if (lane == 0) wsum[wave] = x;
  __syncthreads();
  double z = 0.0;
  for (int w = 0; w < kSampleWaves; ++w) z += wsum[w];
  return z;
}

struct Float4Pair {
  float4 a, c;
};
struct FloatPair {
  float a, c;
};

// the two passes: the sum of a row, and the residual max(0, from - Z q) written to r (from may be r itself)
template <int VEC>
__device__ __forceinline__ double row_sum(int V, int seg, double *wsum, const float *row) {
  if constexpr (VEC == 4) {
    return segment_pass<4, 8>(
        0, V, seg, wsum, [&](int v) { return *reinterpret_cast<const float4 *>(row + v); },  // (V % 4 == 0: no straddling)
        [&](int, const float4 &t, double &x) { x += ((double)t.x + (double)t.y) + ((double)t.z + (double)t.w); });
  } else {
    return segment_pass<1, 8>(
        0, V, seg, wsum, [&](int v) { return row[v]; }, [&](int, float t, double &x) { x += (double)t; });
  }
}

template <int VEC>
__device__ __forceinline__ double residual_pass(int V, int seg, double *wsum, const float *from, const float *q, double Z,
                                                float *r) {
  auto one = [&](float pv, float qv) {
    const double d = (double)pv - Z * (double)qv;
    return d > 0.0 ? (float)d : 0.f;
  };
  if constexpr (VEC == 4) {
    return segment_pass<4, 4>(
        0, V, seg, wsum,
        [&](int v) {
          return Float4Pair{*reinterpret_cast<const float4 *>(from + v), *reinterpret_cast<const float4 *>(q + v)};
        },
        [&](int v, const Float4Pair &t, double &x) {
          float4 o;
          o.x = one(t.a.x, t.c.x), o.y = one(t.a.y, t.c.y), o.z = one(t.a.z, t.c.z), o.w = one(t.a.w, t.c.w);
          *reinterpret_cast<float4 *>(r + v) = o;
          x += ((double)o.x + (double)o.y) + ((double)o.z + (double)o.w);
        });
  } else {
    return segment_pass<1, 4>(
        0, V, seg, wsum, [&](int v) { return FloatPair{from[v], q[v]}; },
        [&](int v, const FloatPair &t, double &x) {
          const float o = one(t.a, t.c);
          r[v] = o;
          x += (double)o;
        });
  }
}

// The last token, looked for inside [lo, hi): wsum holds the waves' sums of dist over their segments of that range
// (seg elements each), `before` is the weight in front of lo, `none` says that no place claimed the target (u_final
// was not below 1): then, and when rounding keeps the running sum below the target, it is the last token of the range
// that has weight.  A long segment is summed again in parts by all waves and looked for in its part (one wave's steps
// through it would each wait for the one before); the wave whose segment holds a short one walks it 64 elements at a
// time; its lane 0 stores it.
__device__ __forceinline__ void draw_in_range(const float *dist, int lo, int hi, int seg, double *wsum, double before,
                                              double target, bool none, int32_t *out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int wclaim;
  while (true) {
    wclaim = -1;
    int wlast = 0;
    double pre = before;
    for (int i = 0; i < kSampleWaves; ++i) {
      const double nx = pre + wsum[i];
      if (wclaim < 0 && !none && nx > target) wclaim = i, before = pre;
      if (wsum[i] > 0.0) wlast = i;
      pre = nx;
    }
    none = wclaim < 0;
    if (none) wclaim = wlast;
    if (seg <= 512) break;
    lo += wclaim * seg, hi = lo + seg < hi ? lo + seg : hi;
    seg = (hi - lo + kSampleWaves - 1) / kSampleWaves;
    segment_pass<1, 8>(
        lo, hi, seg, wsum, [&](int v) { return dist[v]; }, [&](int, float x, double &a) { a += (double)x; });
  }
  if (wave != wclaim) return;
  const int s0 = lo + wave * seg, s1 = s0 + seg < hi ? s0 + seg : hi;
  double acc = before;
  int tok = -1, last_pos = -1;
  for (int base = s0; base < s1; base += 64) {
    const int v = base + lane;
    const float f = v < s1 ? dist[v] : 0.f;
    double incl = (double)f;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    const unsigned long long heavy = __ballot(f > 0.f);
    if (heavy) last_pos = base + 63 - __builtin_clzll(heavy);
    const unsigned long long over = none ? 0ull : __ballot(acc + incl > target);
    if (over) {
      tok = base + __builtin_ctzll(over);
      break;
    }
    acc += __shfl(incl, 63);
  }
  if (lane == 0) *out = tok >= 0 ? tok : last_pos;
}

template <int VEC>
__global__ void __launch_bounds__(kSampleThreads) sample_kernel(const SampleParams p) {
  __shared__ double wsum[kSampleWaves];
  __shared__ int32_t s_parent[kSampleTreeLds], s_token[kSampleTreeLds];
  __shared__ float s_u[kSampleTreeLds];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  if (p.fill_path)  // (the walk's entries are stored behind a barrier)
    for (int i = tid; i < p.max_path; i += kSampleThreads) p.path[(size_t)b * p.max_path + i] = -1;
  const int t0 = p.cu_T[b];
  const int T = p.cu_T[b + 1] - t0;
  if (T <= 0) {
    if (tid == 0) p.path_len[b] = 0, p.next_token[b] = -1;
    return;
  }
  // the tree's words, read once (the walk is a chain of dependent reads of them); a tree too long for that is
  // walked in global memory
  const int32_t *parent = p.parent + t0, *token = p.token + t0;
  const float *u = p.u + t0;
  if (T <= kSampleTreeLds) {
    for (int i = tid; i < T; i += kSampleThreads) s_parent[i] = parent[i], s_token[i] = token[i], s_u[i] = u[i];
    parent = s_parent, token = s_token, u = s_u;
  }
  __syncthreads();
  const int V = p.V;
  const int seg = ((V + kSampleWaves - 1) / kSampleWaves + VEC - 1) / VEC * VEC;
  float *const r = p.residual + (size_t)b * V;
  int cur = 0, len = 1;
  if (tid == 0) p.path[(size_t)b * p.max_path] = 0;
  const float *dist;  // what the next test or the last draw reads: the current node's target row, or the residual
  double Z;
  bool segments;  // wsum holds the segments' sums of dist (the last draw starts from them)
  auto flag_sequence = [&]() {
    if (tid == 0 && p.err_flag) atomicCAS(p.err_flag, 0, 1 + b);
  };
  // the first child of `of` behind node `after` that carries a token (others are flagged and passed over: never
  // accepted, and they leave the residual alone), or -1; 64 candidates at a time, every wave finds the same one
  auto next_child = [&](int of, int after) -> int {
    for (int base = after + 1; base < T; base += 64) {
      const int i = base + lane;
      unsigned long long kids = __ballot(i < T && parent[i] == of);
      while (kids) {
        const int c = base + __builtin_ctzll(kids);
        kids &= kids - 1;
        const int x = token[c];
        if (x >= 0 && x < V) return c;
        flag_sequence();
      }
    }
    return -1;
  };
  while (true) {
    dist = p.p + (size_t)(t0 + cur) * V;
    const float *q = p.q + (size_t)(t0 + cur) * V;
    // the first child and the two entries its test reads: requested before the row's sum, used after it
    int c = len < p.max_path ? next_child(cur, cur) : -1;
    float rx0 = 0.f, qx = 0.f;
    if (c >= 0) rx0 = dist[token[c]], qx = q[token[c]];
    if (p.unit_rows) Z = 1.0, segments = false;
    else Z = row_sum<VEC>(V, seg, wsum, dist), segments = true;
    double rx = (double)rx0;
    bool accepted = false;
    while (c >= 0) {
      if (rx > 0.0 && (double)u[c] * (double)qx * Z <= rx) {
        cur = c;
        if (tid == 0) p.path[(size_t)b * p.max_path + len] = c;
        ++len;
        accepted = true;
        break;
      }
      // rejected: the residual max(0, r - Z q), unnormalised, and its sum; the next child's entry of the draft's
      // row (which stays as it is) is requested before the pass
      const int cn = next_child(cur, c);
      const int xn = cn >= 0 ? token[cn] : 0;
      if (cn >= 0) qx = q[xn];
      __syncthreads();  // every thread has read what it needs of the row before the residual is overwritten in place
      const double Zn = residual_pass<VEC>(V, seg, wsum, dist, q, Z, r);
      if (!(Zn > 0.0)) {
        // q was not a distribution the child could have been drawn from: flagged; the walk ends here
        flag_sequence();
        if (tid == 0) p.path_len[b] = len, p.next_token[b] = -1;
        return;
      }
      Z = Zn;
      dist = r;
      segments = true;
      c = cn;
      if (c >= 0) rx = (double)r[xn];
    }
    if (!accepted) break;
  }
  if (tid == 0) p.path_len[b] = len;
  // (the last draw divides by the sum of what it draws from: a row that was taken as summing to one is summed here)
  if (!segments) Z = row_sum<VEC>(V, seg, wsum, dist);
  // The last token: the smallest v whose cumulative weight exceeds u_final * Z.  The segments' sums of the pass
  // that produced Z say which segment holds it.
  draw_in_range(dist, 0, V, seg, wsum, 0.0, (double)p.u_final[b] * Z, false, &p.next_token[b]);
}

// ---- the same walk with a sequence's rows held in registers, its vocabulary spread over W workgroups ----
// What bounds a walk is a chain: every test needs the sum of the row or residual before it, and one workgroup streams a
// row at what one compute unit can (about 45 GB/s).  So workgroup w of a sequence's W takes the w-th slice of every
// row, few enough elements that its 512 threads hold them in registers (4 NV each, of the target's row or the
// residual, and up to NV = 16 of the draft's row too): a refusal is then arithmetic on registers, and the memory is
// touched once per node.  Three things keep the chain short:
//  - at the start every node's p and q entries are gathered by a thread each, all at once (a hop of the walk would
//    otherwise read them with a cold, dependent access to a row of its own);
//  - the rows that a walk needs one after the other are guessed: with every row's sum taken as one the accepted nodes
//    are known from the gathered entries alone, so their rows are summed in one pass and one wait, after which the tests
//    are taken again with the true sums (a guess that was wrong costs another pass, nothing else);
//  - a wait is one trip: a workgroup's partial sums travel in words that carry a tag of this launch and this wait, so the
//    others poll the data itself, and nothing has to be zeroed beforehand: no launch leaves a word with a tag behind.  A
//    sequence's part of the workspace starts with a counter, which all W read before the first wait and count up by one
//    each behind the last; the one that completes the W has seen all others leave, and clears what was published (a
//    cleared word matches no tag).  So the memory may be taken away, overwritten in whole or in part, put back and
//    handed to the next launch or replay with any counter: what that launch meets is what others wrote there, which
//    passes for a sum only if it holds the launch's 62 bits of tag by chance.
// (Clearing behind the last wait: the call of one sequence, with a commit of 32 layers, 16.35 -> 16.98 us.)
// Measured, one sequence, V = 128256, 60 nodes: 28 us for two launches before (row sums of all nodes, then the walk with
// counters, residuals in memory) -> 13 us; 64 sequences of 8 nodes with unit rows 49 us and a 5 us launch that cleared the
// counters -> 27 us.
// Waits are bounded: a workgroup that does not see the others within about a second flags the sequence and leaves (the
// launch keeps W x B within what the chip holds at once, so this happens only if something else is wrong); it then
// takes back what it had published and counts itself as having left.
constexpr int kWalkThreads = 512, kWalkWaves = kWalkThreads / 64;  // (256 registers per thread)
constexpr int kWalkMaxW = 16;
constexpr int kWalkSpins = 1 << 20;
constexpr int kWalkChain = 8;                        // rows summed in one pass at most
constexpr int kWalkBox = 2 * (1 + kWalkChain);       // words a workgroup publishes: an entry, then the rows' sums, two words each
constexpr int kWalkWords = 16 + 2 * (kWalkMaxW + 1) * kWalkBox;  // per sequence: the counter (a line), two sets of boxes
constexpr size_t kWalkBytes = (kWalkWords * sizeof(uint64_t) + 511) / 512 * 512;

struct WalkParams {
  SampleParams s;
  int W;
  int arrivals;  // workgroups a wait expects: W (one more in the test of the bound: then no wait ever completes)
  int spins;     // polls after which a wait gives up
  uint64_t *mail;  // [B][kWalkBytes / 8]; unused when W is 1
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void mail_store(uint64_t *at, uint64_t word) {
  __hip_atomic_store(at, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t mail_load(const uint64_t *at) {
  return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Inclusive sums along the lanes, by lane shifts in the vector ALU (a tenth of what the shuffles through LDS take);
// lane 63 ends with the wave's sum.
template <int CTRL, int ROWS>
__device__ __forceinline__ double lanes_add(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, true);
  return x + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_scan(double x) {
  x = lanes_add<0x111, 0xf>(x);  // from 1, 2, 4, 8 lanes below in the row of 16
  x = lanes_add<0x112, 0xf>(x);
  x = lanes_add<0x114, 0xf>(x);
  x = lanes_add<0x118, 0xf>(x);
  x = lanes_add<0x142, 0xa>(x);  // the row below's last lane, to rows 1 and 3
  return lanes_add<0x143, 0xc>(x);  // lane 31, to rows 2 and 3
}
__device__ __forceinline__ double read_lane(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}
__device__ __forceinline__ double wave_sum(double x) { return read_lane(wave_scan(x), 63); }

template <int NV, bool WHOLE>
__global__ void __launch_bounds__(kWalkThreads) walk_kernel(const WalkParams wp) {
  // 256 registers per thread: beyond 16 groups the draft's row is read again at each refusal.  (16 groups of an odd vocabulary
  // are 12 registers too many, and the compiler spills those: 100 sequences, V = 50257, 35 us; with the row read again 42.)
  constexpr bool kHoldQ = NV <= 16;
  constexpr int kRows = NV <= 4 ? 4 : 1;  // rows of a chain loaded at once: about 16 loads of 16 bytes in flight per thread
  const SampleParams &p = wp.s;
  __shared__ double s_sum[kWalkChain][kWalkWaves];      // per row of a pass: the waves' sums of their segments
  __shared__ double s_part[kWalkChain][kWalkMaxW + 1];    // and the workgroups' sums of their slices
  __shared__ double s_entry[2];                           // the residual's entry of the next child's token (two passes in turn)
  __shared__ int s_chain[kWalkChain], s_abort, s_bad;
  __shared__ uint64_t s_launch;  // the counter as this launch found it
  __shared__ int32_t s_parent[kSampleTreeLds], s_token[kSampleTreeLds];
  __shared__ float s_u[kSampleTreeLds], s_px[kSampleTreeLds], s_qx[kSampleTreeLds];
  __shared__ int s_first[kSampleTreeLds];  // a node's first child that carries a token, times 2, plus 1 where a row's sum of one refuses it
  const int W = wp.W;
  const int b = blockIdx.x / W, w = blockIdx.x % W, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (p.fill_path && w == 0)  // (the walk's entries are stored behind a barrier)
    for (int i = tid; i < p.max_path; i += kWalkThreads) p.path[(size_t)b * p.max_path + i] = -1;
  const int t0 = p.cu_T[b];
  const int T = p.cu_T[b + 1] - t0;
  if (T <= 0) {
    if (w == 0 && tid == 0) p.path_len[b] = 0, p.next_token[b] = -1;
    return;
  }
  const int V = p.V;
  uint64_t *const mail = wp.mail + (size_t)b * (kWalkBytes / sizeof(uint64_t));
  if (tid == kWalkThreads - 1) {
    s_abort = 0, s_bad = 0;
    s_launch = W > 1 ? mail_load(mail) : 0;
  }
  // the tree's words and what a node's test as its parent's FIRST tested child reads, once (a tree too long for that is
  // walked in global memory)
  const bool in_lds = T <= kSampleTreeLds;
  if (in_lds)
    for (int i = tid; i < T; i += kWalkThreads) s_parent[i] = p.parent[t0 + i], s_token[i] = p.token[t0 + i], s_u[i] = p.u[t0 + i], s_first[i] = INT_MAX;
  for (int i = tid; i < kWalkChain * (kWalkMaxW + 1); i += kWalkThreads) s_part[0][i] = 0.0;
  __syncthreads();
  if (in_lds)
    for (int i = tid; i < T; i += kWalkThreads) {
      const int par = s_parent[i], x = s_token[i];
      float px = 0.f, qx = 0.f;
      if (par >= 0 && par < i) {
        if (x >= 0 && x < V) {
          px = p.p[(size_t)(t0 + par) * V + x], qx = p.q[(size_t)(t0 + par) * V + x];
          atomicMin(&s_first[par], 2 * i + !(px > 0.f && (double)s_u[i] * (double)qx <= (double)px));
        } else {
          s_bad = 1;
        }
      }
      s_px[i] = px, s_qx[i] = qx;
    }
  auto parent = [&](int i) { return in_lds ? s_parent[i] : p.parent[t0 + i]; };
  auto token = [&](int i) { return in_lds ? s_token[i] : p.token[t0 + i]; };
  __syncthreads();
  const uint64_t tag = s_launch * 0x9E3779B97F4A7C15ull + 0xD1B54A32D192ED03ull;
  const uint32_t tag_a = __builtin_amdgcn_readfirstlane(((uint32_t)tag & 0x3fffffffu) | 0x80000000u);  // (tag_a + epoch is never zero)
  const uint32_t tag_b = __builtin_amdgcn_readfirstlane((uint32_t)(tag >> 32));
  // this workgroup's slice of every row, the waves' segments of it; a thread holds groups of four elements, 256 apart
  const int slice = ((V + W - 1) / W + 3) / 4 * 4;
  const int lo = w * slice < V ? w * slice : V, hi = lo + slice < V ? lo + slice : V;
  const int seg = ((hi - lo + kWalkWaves - 1) / kWalkWaves + 3) / 4 * 4;
  const int s0 = lo + wave * seg < hi ? lo + wave * seg : hi, s1 = s0 + seg < hi ? s0 + seg : hi;
  // Row t of a matrix for this wave: buffer loads whose bound is the segment's end, so that a group past it costs nothing
  // and reads as zeros.  The group that a row's end cuts (V no multiple of 4; in one group of one wave) is fetched element
  // by element.  (The whole offset is the one that the bound is checked against.)
  auto row_of = [&](const float *m, int t) { return m + (size_t)(t0 + __builtin_amdgcn_readfirstlane(t)) * V; };
  const int s1_whole = WHOLE ? s1 : s1 & ~3;
  const int cut_k = !WHOLE && s1 > s1_whole ? (s1 - s0) >> 8 : -1;
  auto load_group = [&](const float *row, int k) -> f32x4 {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(row), 0, s1_whole * 4, 0x00020000);
    f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (s0 + lane * 4) * 4 + k * 1024, 0, 0));
    if (!WHOLE && k == cut_k) {
      const auto to_end = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(row), 0, s1 * 4, 0x00020000);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(to_end, (s0 + lane * 4 + e) * 4 + k * 1024, 0, 0));
    }
    return x;
  };
  auto group_sum = [](const f32x4 &x) { return ((double)x[0] + (double)x[1]) + ((double)x[2] + (double)x[3]); };

  // (a scheduling barrier per group: all groups' conversions at once would not fit the registers)
  auto thread_sum = [&](auto group) -> double {
    double acc = 0.0, acc2 = 0.0;
#pragma unroll
    for (int k = 0; k < NV; k += 2) {
      acc += group_sum(group(k));
      acc2 += group_sum(group(k + 1));
      __builtin_amdgcn_sched_barrier(0);
    }
    return acc + acc2;
  };

  int epoch = 0;
  auto publish = [&](int slot, double x) {
    uint64_t *at = mail + 16 + ((size_t)(epoch & 1) * (kWalkMaxW + 1) + w) * kWalkBox + 2 * slot;
    const uint64_t bits = (uint64_t)__double_as_longlong(x);
    mail_store(at, bits << 32 | (uint32_t)(tag_a + epoch));
    mail_store(at + 1, (bits >> 32) << 32 | (uint32_t)(tag_b + epoch));
  };
  // Called once by every workgroup, behind its last wait (a barrier after the last word it polled): counts it as having
  // left.  The last of the W to do so clears all that they published.  Every word of an earlier wait has been read by all
  // when a later one is complete, and those of the last wait have by then been read by all W, each before it counted
  // itself.  One wave; the others go on with the draw.
  auto leave = [&]() {
    if (W == 1 || wave != kWalkWaves - 1) return;
    bool last_one = false;
    if (lane == 0) last_one = __hip_atomic_fetch_add(mail, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - s_launch == (uint64_t)(W - 1);
    if (__ballot(last_one) == 0) return;
    for (int set = 0; set < 2; ++set)
      for (int i = lane; i < W * kWalkBox; i += 64) mail_store(mail + 16 + (size_t)set * (kWalkMaxW + 1) * kWalkBox + i, 0);
  };
  // The sums of a pass over `n` rows: s_sum is complete behind a barrier.  s_part[i][.] then holds the workgroups' sums of
  // row i and s_entry[epoch & 1] the entry that workgroup x_from published (x_from < 0: none), the same in every
  // workgroup of the sequence.  (epoch has been counted up before the pass.)  False: the others did not arrive.
  auto exchange = [&](int n, int x_from) -> bool {
    if (tid < n) {
      double local = 0.0;
#pragma unroll
      for (int i = 0; i < kWalkWaves; ++i) local += s_sum[tid][i];
      if (W > 1) publish(1 + tid, local);
      else s_part[tid][0] = local;
    }
    if (W > 1) {
      const int from = tid < 8 * (kWalkMaxW + 1) ? tid >> 3 : x_from, i = tid & 7;  // (a thread per workgroup and row, one for the entry)
      const bool sum = tid < 8 * (kWalkMaxW + 1);
      static_assert(kWalkChain == 8, "");
      if (sum ? from < wp.arrivals && i < n : tid == 8 * (kWalkMaxW + 1) && x_from >= 0) {
        const uint64_t *at = mail + 16 + ((size_t)(epoch & 1) * (kWalkMaxW + 1) + from) * kWalkBox + (sum ? 2 * (1 + i) : 0);
        uint64_t a = 0, c = 0;
        int spins = 0;
        while (true) {
          a = mail_load(at), c = mail_load(at + 1);
          if ((uint32_t)a == (uint32_t)(tag_a + epoch) && (uint32_t)c == (uint32_t)(tag_b + epoch)) break;
          if (++spins > wp.spins) {
            s_abort = 1;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
        const double x = __longlong_as_double((long long)((c >> 32) << 32 | a >> 32));
        if (sum) s_part[i][from] = x;
        else s_entry[epoch & 1] = x;
      }
    }
    __syncthreads();
    if (W > 1) {
      if (s_abort != 0) {
        // Taken back by itself: a workgroup that starts after this one has counted itself reads another counter, and
        // then no count need come to W.  (It never comes to W too early: a later start only lowers it.)
        if (tid < kWalkBox)
          for (int set = 0; set < 2; ++set) mail_store(mail + 16 + ((size_t)set * (kWalkMaxW + 1) + w) * kWalkBox + tid, 0);
        leave();
        if (tid == 0 && p.err_flag) atomicCAS(p.err_flag, 0, 1 + b);
        return false;
      }
    }
    return true;
  };
  auto total = [&](int i) -> double {
    double z = 0.0;
#pragma unroll
    for (int k = 0; k < kWalkMaxW; ++k) z += s_part[i][k];  // (zeros past W)
    return z;
  };
  // the first child of `of` behind node `after` that carries a token (others are passed over, and flagged where the walk
  // itself looks), or -1; 64 candidates at a time, every wave finds the same one
  auto next_child = [&](int of, int after, bool flag) -> int {
    for (int base = after + 1; base < T; base += 64) {
      const int i = base + lane;
      unsigned long long kids = __ballot(i < T && parent(i) == of);
      while (kids) {
        const int c = base + __builtin_ctzll(kids);
        kids &= kids - 1;
        const int x = token(c);
        if (x >= 0 && x < V) return c;
        if (flag && tid == 0 && p.err_flag) atomicCAS(p.err_flag, 0, 1 + b);
      }
    }
    return -1;
  };
  auto p_entry = [&](int of, int c) -> float { return in_lds ? s_px[c] : p.p[(size_t)(t0 + of) * V + token(c)]; };
  auto q_entry = [&](int of, int c) -> float { return in_lds ? s_qx[c] : p.q[(size_t)(t0 + of) * V + token(c)]; };
  auto accepts = [&](int c, float qx, double rx, double Z) { return rx > 0.0 && (double)(in_lds ? s_u[c] : p.u[t0 + c]) * (double)qx * Z <= rx; };

  int cur = 0, len = 1, last = 0;   // last: which row of s_sum and s_part belongs to r
  double Z = 1.0;
  if (w == 0 && tid == 0) p.path[(size_t)b * p.max_path] = 0;
  while (true) {
    // ---- the rows ahead, guessed with sums of one ----
    __syncthreads();  // (the chain before this one has been read)
    int n = 0, at = cur, end = -1;  // end: the child that the last node's test is about, or -1
    bool refusal = false;           // the guess: that test refuses
    if (in_lds) {
      while (true) {
        const int f = len + n < p.max_path ? s_first[at] : INT_MAX;
        if (tid == 0) s_chain[n] = at;
        ++n;
        end = f == INT_MAX ? -1 : f >> 1, refusal = f != INT_MAX && (f & 1);
        if (end < 0 || refusal || n == kWalkChain) break;
        at = end;
      }
    } else {
      end = len < p.max_path ? next_child(cur, cur, true) : -1;
      if (tid == 0) s_chain[0] = cur;
      n = 1, refusal = end >= 0 && !accepts(end, q_entry(cur, end), (double)p_entry(cur, end), 1.0);
    }
    __syncthreads();
    // ---- one pass over them; with unit rows the guess is the rule, and only the last node's row is looked at ----
    f32x4 q[kHoldQ ? NV : 1];
    f32x4 r[NV];  // the row or residual that the walk stands on; q: the draft's row under it
    if (kHoldQ && refusal) {
      const auto q_row = row_of(p.q, s_chain[n - 1]);
#pragma unroll
      for (int k = 0; k < NV; ++k) q[kHoldQ ? k : 0] = load_group(q_row, k);
    }
    const int first = p.unit_rows ? n - 1 : 0;
    const bool summed = !p.unit_rows || !refusal;
    for (int i0 = first; i0 < n; i0 += kRows) {
      // (one row at a time is loaded in place: the last one stays)
      f32x4 more[kRows > 1 ? kRows : 1][kRows > 1 ? NV : 1];
      auto part = [&](int j, int k) -> f32x4 & { return kRows > 1 ? more[kRows > 1 ? j : 0][kRows > 1 ? k : 0] : r[k]; };
#pragma unroll
      for (int j = 0; j < kRows; ++j)
        if (i0 + j < n) {
          const auto row = row_of(p.p, s_chain[i0 + j]);
#pragma unroll
          for (int k = 0; k < NV; ++k) part(j, k) = load_group(row, k);
        }
#pragma unroll
      for (int j = 0; j < kRows; ++j)
        if (i0 + j < n) {
          if (summed) {
            const double acc = wave_sum(thread_sum([&](int k) -> const f32x4 & { return part(j, k); }));
            if (lane == 0) s_sum[i0 + j - first][wave] = acc;
          }
          if (kRows > 1 && i0 + j == n - 1) {
#pragma unroll
            for (int k = 0; k < NV; ++k) r[k] = part(j, k);
          }
        }
    }
    last = n - 1 - first;
    if (summed) {
      __syncthreads();
      ++epoch;
      if (!exchange(n - first, -1)) return;
    }
    // ---- the tests, with the true sums: a lane takes one node of the chain ----
    int i, c;  // nodes whose child is accepted; the child that is refused, or -1
    {
      const int k = lane < n ? lane : 0, node = s_chain[k], child = k < n - 1 ? s_chain[k + 1 < kWalkChain ? k + 1 : k] : end;
      const double z = p.unit_rows ? 1.0 : total(k);
      const bool ok = lane < n && child >= 0 && accepts(child, q_entry(node, child), (double)p_entry(node, child), z);
      const unsigned long long taken = __ballot(ok);
      i = __builtin_ctzll(~taken);
      if (w == 0 && tid < i) p.path[(size_t)b * p.max_path + len + tid] = child;
      if (in_lds && s_bad && p.err_flag) {  // (children without a token, passed over at the nodes that were reached)
        for (int bad = tid; bad < T; bad += kWalkThreads) {
          const int par = s_parent[bad], x = s_token[bad];
          if (par < 0 || par >= bad || (x >= 0 && x < V) || bad > s_first[par] >> 1) continue;
          for (int j = 0; j <= i && j < n; ++j)
            if (s_chain[j] == par && len + j < p.max_path) atomicCAS(p.err_flag, 0, 1 + b);
        }
      }
      len += i;
      cur = i < n ? s_chain[i] : end;
      c = i < n ? __builtin_amdgcn_readlane(child, i) : -1;
      Z = read_lane(z, i < n ? i : 0);
    }
    if (i == n) continue;  // (the chain was cut at its longest, or its last guess was a refusal that is none)
    // ---- refused at `cur`: its rows are held already, unless the guess went past it ----
    if (c >= 0 && (i != n - 1 || !refusal)) {
      const auto p_at = row_of(p.p, cur), q_at = row_of(p.q, cur);
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        r[k] = load_group(p_at, k);
        if (kHoldQ) q[kHoldQ ? k : 0] = load_group(q_at, k);
      }
    }
    bool accepted = false;
    if (c >= 0) last = 0;
    else if (p.unit_rows) Z = total(last);  // (nothing to test, which only the chain's last node can be: the draw divides by its row's sum)
    while (c >= 0) {
      // the residual max(0, r - Z q), unnormalised; the entry of the next child's token goes to the others with its sum
      const int cn = next_child(cur, c, true);
      const int xn = cn >= 0 ? token(cn) : -1;
      const int off = xn - s0;
      const int own = xn >= s0 && xn < s1 && (off >> 2 & 63) == lane ? off >> 8 : -1;  // this thread's group that holds it
      const auto q_at = row_of(p.q, cur);
      double acc = 0.0, acc2 = 0.0;
      const auto pass = [&](auto unit_tag) __attribute__((always_inline)) {
      constexpr bool unit = decltype(unit_tag)::value;
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        f32x4 qk = kHoldQ ? q[kHoldQ ? k : 0] : load_group(q_at, k);
        // (opaque, or the conversions to double would be kept from pass to pass, in twice the registers)
        asm volatile("" : "+v"(qk), "+v"(r[k]));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // (a sum of one: the subtraction in float32 is the one in double rounded to float32)
          const float d = unit ? r[k][e] - qk[e] : (float)((double)r[k][e] - Z * (double)qk[e]);
          r[k][e] = fmaxf(d, 0.f);
        }
        if (k & 1) acc2 += group_sum(r[k]);
        else acc += group_sum(r[k]);
        __builtin_amdgcn_sched_barrier(0);
      }
      };
      if (Z == 1.0) pass(std::true_type{});
      else pass(std::false_type{});
      ++epoch;
      if (xn >= s0 && xn < s1) {  // (one wave of one workgroup)
        f32x4 g = r[0];
#pragma unroll
        for (int k = 1; k < NV; ++k)
          if (k == own) g = r[k];
        const double entry = (double)((off & 2) ? (off & 1) ? g[3] : g[2] : (off & 1) ? g[1] : g[0]);
        if (own >= 0) {
          if (W > 1) publish(0, entry);
          else s_entry[epoch & 1] = entry;
        }
      }
      acc = wave_sum(acc + acc2);
      if (lane == 0) s_sum[0][wave] = acc;
      __syncthreads();
      if (!exchange(1, xn >= 0 ? xn / slice : -1)) return;
      Z = total(0);
      if (!(Z > 0.0)) {
        leave();
        // q was not a distribution the child could have been drawn from: flagged; the walk ends here
        if (w == 0 && tid == 0) {
          if (p.err_flag) atomicCAS(p.err_flag, 0, 1 + b);
          p.path_len[b] = len, p.next_token[b] = -1;
        }
        return;
      }
      c = cn;
      if (c >= 0 && accepts(c, q_entry(cur, c), s_entry[epoch & 1], Z)) {
        if (w == 0 && tid == 0) p.path[(size_t)b * p.max_path + len] = c;
        ++len;
        cur = c;
        accepted = true;
        break;
      }
    }
    if (accepted) continue;
    leave();
    if (w == 0 && tid == 0) p.path_len[b] = len;
    // ---- the last token: the smallest v whose cumulative weight exceeds u_final Z ----
    // The slices' sums say which workgroup holds it, the segments' which wave; where no place claims it (u_final was not
    // below 1, or rounding kept the running sum below) it is the last token that has weight.
    const double target = (double)p.u_final[b] * Z;
    double before = 0.0;
    bool none;
    {
      int claim = -1, heavy = 0;
      double pre = 0.0;
#pragma unroll
      for (int k = 0; k < kWalkMaxW; ++k) {
        const double x = s_part[last][k], nx = pre + x;
        if (claim < 0 && nx > target) claim = k, before = pre;
        if (x > 0.0) heavy = k;
        pre = nx;
      }
      none = claim < 0;
      if (none) claim = heavy;
      if (w != claim) return;
      claim = -1, heavy = 0, pre = before;
      for (int k = 0; k < kWalkWaves; ++k) {
        const double x = s_sum[last][k], nx = pre + x;
        if (claim < 0 && !none && nx > target) claim = k, before = pre;
        if (x > 0.0) heavy = k;
        pre = nx;
      }
      none = claim < 0;
      if (none) claim = heavy;
      if (wave != claim) return;
    }
    // this wave's segment: which group of 256 elements, then where in it
    int claim = -1, heavy = 0;
    double pre = before;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const double x = wave_sum(group_sum(r[k])), nx = pre + x;
      if (claim < 0 && !none && nx > target) claim = k, before = pre;
      if (x > 0.0) heavy = k;
      pre = nx;
      if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    none = claim < 0;
    if (none) claim = heavy;
    f32x4 x = r[0];
#pragma unroll
    for (int k = 1; k < NV; ++k)
      if (k == claim) x = r[k];
    const double mine = group_sum(x);
    double run = before + (wave_scan(mine) - mine);
    int tok = -1, weight = -1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int v = s0 + (claim * 64 + lane) * 4 + e;
      run += (double)x[e];
      if (x[e] > 0.f) weight = v;
      if (!none && tok < 0 && x[e] > 0.f && run > target) tok = v;
    }
    const unsigned long long over = __ballot(tok >= 0), some = __ballot(weight >= 0);
    const int drawn = over ? __shfl(tok, __builtin_ctzll(over)) : some ? __shfl(weight, 63 - __builtin_clzll(some)) : -1;
    if (lane == 0) p.next_token[b] = drawn;
    return;
  }
}

// How a call runs: workgroups per sequence, and groups of four elements a thread of walk_kernel holds (0: sample_kernel).
// With a workspace the library takes as many workgroups as keep the launch within one per compute unit (all of them
// resident at once, which the waits rely on), at most 16, a power of two, slices of 4096 tokens or more, and one below
// 16 K tokens.  sample_kernel, one workgroup that keeps its residual in memory, is left for what 512 threads
// cannot hold: more than 64 K tokens and no workspace, or more than 128 sequences.
struct WalkPlan {
  int W, NV;
};
int walk_plan(const tva_sample_args *a, WalkPlan *plan) {
  if (a->workgroups_per_sequence < 0 || a->workgroups_per_sequence > kWalkMaxW) return TVA_INVALID_ARG;
  int W = 1;
  if (a->workspace && a->workgroups_per_sequence != 1) {
    if (((uintptr_t)a->workspace & 7) || a->workspace_bytes < (size_t)a->B * kWalkBytes) return TVA_WORKSPACE_TOO_SMALL;
    while (a->V >= 16384 && 2 * W <= kWalkMaxW && (int64_t)a->B * 2 * W <= 256 && a->V / (2 * W) >= 4096) W *= 2;
    if (a->workgroups_per_sequence > 1) {
      W = a->workgroups_per_sequence;
      if ((int64_t)a->B * W > 256) return TVA_UNSUPPORTED;  // more than the chip holds at once
    }
  }
  auto groups = [&](int n) {  // the groups of four that a thread holds when n workgroups share a row
    const int64_t slice = ((int64_t)a->V + n - 1) / n + 3, seg = (slice + kWalkWaves - 1) / kWalkWaves + 3;
    return (seg + 255) / 256;
  };
  int64_t g = groups(W);
  const int most = a->V % 4 == 0 ? 32 : 16;
  while (g > most && W > 1 && W < kWalkMaxW && (int64_t)a->B * 2 * W <= 256) W *= 2, g = groups(W);  // (a named number too small for the vocabulary)
  if (g > most) W = 1, g = groups(1);
  plan->W = W;
  // (no form for 32 groups of a vocabulary that is no multiple of 4: its registers do not suffice)
  plan->NV = a->V < 4 ? 0 : g <= 4 ? 4 : g <= 8 ? 8 : g <= 16 ? 16 : g <= 32 && a->V % 4 == 0 ? 32 : 0;
  return TVA_OK;
}

struct CommitParams {
  const int32_t *cu_T, *L, *path, *path_len, *cu_L, *page_table;
  const char *k_tree, *v_tree;
  char *k_cache, *v_cache;
  int32_t *L_out, *err_flag;
  int Hkv, D, max_path, page_size, max_pages;
  int64_t stride_page, stride_tok, stride_head;  // elements
  int64_t layer_cache, layer_tree;                // bytes between the tensors of consecutive layers
  int n_layers, layers_per_wg;
};

constexpr int kCommitLayers = 4;  // layers whose pieces a thread has in flight at once
// Bound by a workgroup's chain of reads before it moves a byte.  Everything that only needs the sequence's number and the
// place in its path is requested together, before it is known whether the place holds a node (every address is inside its array
// whatever the path says); a paged cache's entry is the one read behind that.
// MANY: where most places hold none, or a workgroup has more layers than it has in flight at once, the path's length comes first
// and the rest behind it: places without a node are left sooner (256 sequences, paths of 3 of 33 places, 32 layers of 4 heads,
// two layers a workgroup: 35 us instead of 53; four: 24.5 instead of 29.4).
template <bool MANY>
__global__ void __launch_bounds__(256) commit_kernel(const CommitParams p) {
  const int j = blockIdx.x, b = blockIdx.y, layer0 = blockIdx.z * p.layers_per_wg;
  const int n = p.path_len[b], Lb = p.L[b];
  const int32_t *const rows = p.page_table ? p.cu_T : p.cu_L;  // (a paged cache has no rows of its own: the value is not used)
  int node, t0, t1, row0, row1;
  auto look = [&]() __attribute__((always_inline)) {
    node = p.path[(size_t)b * p.max_path + j];
    t0 = p.cu_T[b], t1 = p.cu_T[b + 1];
    row0 = rows[b], row1 = rows[b + 1];
    asm volatile("" ::"s"(n), "s"(Lb), "s"(node), "s"(t0), "s"(t1), "s"(row0), "s"(row1));  // all before the next branch
  };
  if constexpr (!MANY) look();
  if (j == 0 && layer0 == 0 && threadIdx.x == 0 && p.L_out) p.L_out[b] = Lb + (n < p.max_path ? n : p.max_path);
  if (j >= n || Lb < 0) return;
  if constexpr (MANY) look();
  if (node < 0 || node >= t1 - t0) {  // not a node of this tree: nothing is copied
    if (threadIdx.x == 0 && p.err_flag) atomicCAS(p.err_flag, 0, 1 + b);
    return;
  }
  const int64_t src_row = (int64_t)t0 + node;
  const int pos = Lb + j;
  int64_t dst;  // element offset of (position, head 0, d 0)
  bool room;
  if (p.page_table) {
    const int pi = pos / p.page_size;
    room = pi < p.max_pages;
    const int page = room ? p.page_table[(int64_t)b * p.max_pages + pi] : 0;
    dst = (int64_t)page * p.stride_page + (int64_t)(pos - pi * p.page_size) * p.stride_tok;
  } else {
    room = (int64_t)row0 + pos < row1;
    dst = ((int64_t)row0 + pos) * p.stride_tok;
  }
  if (!room) {
    if (threadIdx.x == 0 && p.err_flag) atomicCAS(p.err_flag, 0, 1 + b);
    return;
  }
  // 16-byte pieces: piece q of head g; the tree tensors are packed [node, Hkv, D]
  const int per_head = p.D / 8;
  const int pieces = p.Hkv * per_head;
  const int here = p.n_layers - layer0 < p.layers_per_wg ? p.n_layers - layer0 : p.layers_per_wg;
  static_assert(kCommitLayers == 4, "the layers below are moved by fours, twos and ones");
  for (int q = threadIdx.x; q < 2 * pieces; q += blockDim.x) {
    const bool is_v = q >= pieces;
    const int r = is_v ? q - pieces : q;
    const int g = r / per_head, e = (r - g * per_head) * 8;
    const char *src = (is_v ? p.v_tree : p.k_tree) + ((src_row * p.Hkv + g) * p.D + e) * 2;
    char *out = (is_v ? p.v_cache : p.k_cache) + (dst + (int64_t)g * p.stride_head + e) * 2;
    // (counts known when compiled: behind a branch of its own every load would wait for the one before)
    auto move = [&](auto count, int l) __attribute__((always_inline)) {
      constexpr int N = decltype(count)::value;
      u32x4 x[N];
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = *reinterpret_cast<const u32x4 *>(src + (l + i) * p.layer_tree);
#pragma unroll
      for (int i = 0; i < N; ++i) *reinterpret_cast<u32x4 *>(out + (l + i) * p.layer_cache) = x[i];
    };
    int l = layer0, left = here;
    if constexpr (MANY)
      for (; left > kCommitLayers; left -= kCommitLayers, l += kCommitLayers) move(std::integral_constant<int, kCommitLayers>{}, l);
    if (left == kCommitLayers) {
      move(std::integral_constant<int, kCommitLayers>{}, l);
    } else {
      if (left & 2) move(std::integral_constant<int, 2>{}, l);
      if (left & 1) move(std::integral_constant<int, 1>{}, l + (left & 2));
    }
  }
}

// Tree K/V already in the cache behind the L_b committed tokens (tree node i at position L_b + i):
// the accepted nodes are moved down to positions L_b, L_b + 1, ...  One workgroup per sequence; a
// thread owns the same 16-byte pieces of every row and takes the path in order.  Step j reads
// position L_b + path[j] >= L_b + j and writes L_b + j, so a later step never reads what an earlier
// one wrote, and a read that a later step overwrites comes first in the same thread's program order.
__global__ void __launch_bounds__(256) compact_kernel(const CommitParams p) {
  const int b = blockIdx.x, layer = blockIdx.y;
  const int n = p.path_len[b] < p.max_path ? p.path_len[b] : p.max_path;
  const int Lb = p.L[b];
  const int T = p.cu_T[b + 1] - p.cu_T[b];
  if (layer == 0 && threadIdx.x == 0 && p.L_out) p.L_out[b] = Lb + n;
  if (Lb < 0) return;
  const int per_head = p.D / 8;
  const int pieces = p.Hkv * per_head;
  auto row_offset = [&](int pos) -> int64_t {  // element offset of (position, head 0, d 0)
    if (p.page_table) {
      const int pi = pos / p.page_size;
      const int page = p.page_table[(int64_t)b * p.max_pages + pi];
      return (int64_t)page * p.stride_page + (int64_t)(pos - pi * p.page_size) * p.stride_tok;
    }
    return ((int64_t)p.cu_L[b] + pos) * p.stride_tok;
  };
  for (int j = 0; j < n; ++j) {
    const int node = p.path[(size_t)b * p.max_path + j];
    if (node < j || node >= T || (p.page_table && (Lb + node) / p.page_size >= p.max_pages)) {
      // not a path of this tree (entries rise at least as fast as their position): stop here
      if (threadIdx.x == 0 && p.err_flag) atomicCAS(p.err_flag, 0, 1 + b);
      return;
    }
    if (node == j) continue;  // already in place
    const int64_t src = row_offset(Lb + node), dst = row_offset(Lb + j);
    for (int q = threadIdx.x; q < 2 * pieces; q += blockDim.x) {
      const bool is_v = q >= pieces;
      const int r = is_v ? q - pieces : q;
      const int g = r / per_head, e = (r - g * per_head) * 8;
      char *base = (is_v ? p.v_cache : p.k_cache) + layer * p.layer_cache;
      const int64_t inner = (int64_t)g * p.stride_head + e;
      *reinterpret_cast<u32x4 *>(base + (dst + inner) * 2) = *reinterpret_cast<const u32x4 *>(base + (src + inner) * 2);
    }
  }
}

}  // namespace

extern "C" {

static int accept_greedy_impl(const int32_t *parent, const int32_t *cu_T, const int32_t *draft_token,
                              const int32_t *target_token, int32_t B, int32_t max_path, int32_t *path, int32_t *path_len,
                              int32_t *next_token, void *stream, int fill) {
  if (B < 0 || max_path < 1) return TVA_INVALID_ARG;
  if (B == 0) return TVA_OK;
  if (!parent || !cu_T || !draft_token || !target_token || !path || !path_len || !next_token) return TVA_INVALID_ARG;
  (void)hipGetLastError();  // the status below is this launch's
  hipLaunchKernelGGL(accept_kernel, dim3(B), dim3(64), 0, (hipStream_t)stream, parent, cu_T, draft_token, target_token,
                     max_path, path, path_len, next_token, fill);
  return hipPeekAtLastError() == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

int tva_accept_greedy(const int32_t *parent, const int32_t *cu_T, const int32_t *draft_token,
                      const int32_t *target_token, int32_t B, int32_t max_path, int32_t *path, int32_t *path_len,
                      int32_t *next_token, void *stream) {
  return accept_greedy_impl(parent, cu_T, draft_token, target_token, B, max_path, path, path_len, next_token, stream, 0);
}

int tva_accept_greedy_filled(const int32_t *parent, const int32_t *cu_T, const int32_t *draft_token,
                             const int32_t *target_token, int32_t B, int32_t max_path, int32_t *path, int32_t *path_len,
                             int32_t *next_token, void *stream) {
  return accept_greedy_impl(parent, cu_T, draft_token, target_token, B, max_path, path, path_len, next_token, stream, 1);
}

static int accept_sampling_impl(const tva_sample_args *a, void *stream, int missing_arrivals, int spins, bool fill);

int tva_accept_sampling(const tva_sample_args *a, void *stream) { return accept_sampling_impl(a, stream, 0, kWalkSpins, false); }
int tva_accept_sampling_filled(const tva_sample_args *a, void *stream) { return accept_sampling_impl(a, stream, 0, kWalkSpins, true); }

int tva_accept_sampling_wait_bound_test(const tva_sample_args *a, int32_t spins, void *stream) {
  if (!a || spins < 1 || spins > kWalkSpins || !a->workspace || a->workgroups_per_sequence < 2) return TVA_INVALID_ARG;
  return accept_sampling_impl(a, stream, 1, spins, false);
}

static int accept_sampling_impl(const tva_sample_args *a, void *stream, int missing_arrivals, int spins, bool fill) {
  if (!a || a->B < 0 || a->V < 1 || a->max_path < 1) return TVA_INVALID_ARG;
  if (a->B == 0) return TVA_OK;
  if (!a->parent || !a->cu_T || !a->draft_token || !a->p_target || !a->q_draft || !a->u || !a->u_final || !a->residual ||
      !a->path || !a->path_len || !a->next_token)
    return TVA_INVALID_ARG;
  SampleParams p;
  p.parent = a->parent, p.cu_T = a->cu_T, p.token = a->draft_token;
  p.p = a->p_target, p.q = a->q_draft, p.u = a->u, p.u_final = a->u_final;
  p.residual = a->residual;
  p.path = a->path, p.path_len = a->path_len, p.next_token = a->next_token, p.err_flag = a->err_flag;
  p.V = a->V, p.max_path = a->max_path;
  p.unit_rows = a->unit_rows != 0;
  p.fill_path = fill;
  // groups of four need every row to start on 16 bytes
  const bool vec = a->V % 4 == 0 && (((uintptr_t)a->p_target | (uintptr_t)a->q_draft | (uintptr_t)a->residual) & 15) == 0;
  if (a->sum_T < 0) return TVA_INVALID_ARG;
  WalkPlan plan;
  if (const int rc = walk_plan(a, &plan)) return rc;
  (void)hipGetLastError();  // the status below is this launch's
  hipStream_t st = (hipStream_t)stream;
  if (plan.NV == 0) {
    if (vec) hipLaunchKernelGGL(sample_kernel<4>, dim3(a->B), dim3(kSampleThreads), 0, st, p);
    else hipLaunchKernelGGL(sample_kernel<1>, dim3(a->B), dim3(kSampleThreads), 0, st, p);
  } else {
    WalkParams wp;
    wp.s = p, wp.W = plan.W, wp.arrivals = plan.W + missing_arrivals, wp.spins = spins;
    wp.mail = static_cast<uint64_t *>(a->workspace);
    const dim3 grid(a->B * plan.W), block(kWalkThreads);
    auto launch = [&](auto whole) {
      constexpr bool WHOLE = decltype(whole)::value;
      switch (plan.NV) {
        case 4: hipLaunchKernelGGL((walk_kernel<4, WHOLE>), grid, block, 0, st, wp); break;
        case 8: hipLaunchKernelGGL((walk_kernel<8, WHOLE>), grid, block, 0, st, wp); break;
        case 16: hipLaunchKernelGGL((walk_kernel<16, WHOLE>), grid, block, 0, st, wp); break;
        default:
          if constexpr (WHOLE) hipLaunchKernelGGL((walk_kernel<32, true>), grid, block, 0, st, wp);
          break;
      }
    };
    if (a->V % 4 == 0) launch(std::true_type{});
    else launch(std::false_type{});
  }
  return hipPeekAtLastError() == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

size_t tva_sample_workspace_bytes(int32_t B) { return B < 0 ? (size_t)-1 : (size_t)B * kWalkBytes; }

size_t tva_sample_workspace_bytes_rows(int32_t B, int32_t sum_T, int32_t V) {
  return B < 0 || sum_T < 0 || V < 1 ? (size_t)-1 : tva_sample_workspace_bytes(B);
}

size_t tva_sizeof_sample_args(void) { return sizeof(tva_sample_args); }

int tva_commit_path(const tva_commit_args *a, void *stream) {
  if (!a || a->B < 0 || a->Hkv < 1 || a->D < 8 || a->D % 8 || a->max_path < 1) return TVA_INVALID_ARG;
  if (a->B == 0) return TVA_OK;
  if (!a->cu_T || !a->L || !a->path || !a->path_len || !a->k_cache || !a->v_cache) return TVA_INVALID_ARG;
  if ((a->k_tree == nullptr) != (a->v_tree == nullptr)) return TVA_INVALID_ARG;
  const bool in_cache = a->k_tree == nullptr;
  const bool dense = a->cu_L != nullptr, paged = a->page_table != nullptr;
  if (dense == paged) return TVA_INVALID_ARG;
  if (paged && (a->page_size <= 0 || a->max_pages <= 0)) return TVA_INVALID_ARG;
  if ((a->stride_page | a->stride_tok | a->stride_head) % 8) return TVA_INVALID_ARG;
  if (a->stride_page < 0 || a->stride_tok < 0 || a->stride_head < 0) return TVA_INVALID_ARG;
  if (a->L_out == a->L) return TVA_INVALID_ARG;
  if (a->n_layers < 0 || a->layer_stride_cache < 0 || a->layer_stride_tree < 0 ||
      (a->layer_stride_cache | a->layer_stride_tree) % 8)
    return TVA_INVALID_ARG;
  const int layers = a->n_layers > 0 ? a->n_layers : 1;
  if (a->B > 65535 || layers > 65535) return TVA_UNSUPPORTED;
  CommitParams p;
  p.cu_T = a->cu_T; p.L = a->L; p.path = a->path; p.path_len = a->path_len;
  p.cu_L = a->cu_L; p.page_table = a->page_table;
  p.k_tree = (const char *)a->k_tree; p.v_tree = (const char *)a->v_tree;
  p.k_cache = (char *)a->k_cache; p.v_cache = (char *)a->v_cache;
  p.L_out = a->L_out; p.err_flag = a->err_flag;
  p.Hkv = a->Hkv; p.D = a->D; p.max_path = a->max_path;
  p.page_size = paged ? a->page_size : 1; p.max_pages = a->max_pages;
  p.stride_head = a->stride_head ? a->stride_head : a->D;
  p.stride_tok = a->stride_tok ? a->stride_tok : (int64_t)a->Hkv * a->D;
  p.stride_page = a->stride_page ? a->stride_page : (int64_t)p.page_size * p.stride_tok;
  p.n_layers = layers;
  p.layer_cache = a->layer_stride_cache * 2, p.layer_tree = a->layer_stride_tree * 2;
  (void)hipGetLastError();
  if (in_cache) hipLaunchKernelGGL(compact_kernel, dim3(a->B, layers), dim3(256), 0, (hipStream_t)stream, p);
  else {
    // A workgroup finds its row through a chain of reads before it moves a byte, and most places in most paths hold no node: a
    // launch of many workgroups lasts as long as their dispatch, 0.2 .. 0.4 ns each.  So a workgroup moves the row in
    // several layers: up to as many as it has in flight at once while there are workgroups enough, up to 16 where they are few
    // bytes (fewer where paths are short and more of the places hold a node), eight where the launch is one of tens of
    // thousands even so.  MANY from 32 places on and 1024 workgroups: below them it costs 1 .. 2 % in the mean (up to 10 where most
    // places hold a node), from there on it gains 3 .. 8 (up to 30).  (400 calls of 1 .. 256 sequences, 1 .. 80 layers, 1 .. 40
    // heads of 128.  us with 1 / 2 / 4 / 8 / 16 layers each: 64 sequences, 9 places, paths of 3.3 nodes, 32 layers, 8 heads 15.3 /
    // 12.7 / 13.3 / 14.9 / 15.7; 16, 14, 3.2, 32, 8 7.2 / 5.5 / 5.0 / 5.0 / 5.8; MANY: 32, 72, 3.2, 61, 1 32.7 / 18.2 / 10.9 /
    // 7.6 / 6.5; 201, 72, 2.4, 8, 4 28.1 / 16.0 / 10.3 / 8.8 / 8.7.)
    const int64_t groups = (int64_t)a->max_path * a->B * layers, row_bytes = (int64_t)a->Hkv * a->D * 2;
    const int64_t few_bytes = a->max_path >= 32 ? 8192 : a->max_path >= 10 ? 4096 : 2048;
    int k = 1;
    for (bool more = true; more;) {
      int64_t most;
      if (k < kCommitLayers) most = 2 * k * row_bytes <= 8192 ? 1024 : 4096;
      else if (k < 16 && 2 * k * row_bytes <= few_bytes) most = 4096;
      else most = k < 8 ? 49152 : INT64_MAX;
      more = groups / k > most;
      if (more) k *= 2;
    }
    const bool many = k > kCommitLayers || (a->max_path >= 32 && groups / k > 1024 && row_bytes <= 8192);
    p.layers_per_wg = k;
    const dim3 grid(a->max_path, a->B, (layers + k - 1) / k);
    if (many) hipLaunchKernelGGL(commit_kernel<true>, grid, dim3(256), 0, (hipStream_t)stream, p);
    else hipLaunchKernelGGL(commit_kernel<false>, grid, dim3(256), 0, (hipStream_t)stream, p);
  }
  return hipPeekAtLastError() == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

size_t tva_sizeof_commit_args(void) { return sizeof(tva_commit_args); }

}  // extern "C"
