// libtva: tree-masked verification attention for gfx950 (MI355X).
//
// Kernels
//   anc_mask_kernel   parent arrays -> ancestor-or-self bitmasks (the attention mask of the
//                     linearised subtree; paper, Tree Reranking Phase, last paragraph)
//   attn_kernel       split-KV attention of all tree tokens of one (sequence, KV head)
//                     against one chunk of that sequence's cache (+ the tree's own
//                     keys under the ancestor mask, folded into the last chunk)
//   merge_kernel      merges the KV splits where attn_kernel has not done so at its end
//
// attn_kernel in one paragraph.  The T_b*G query rows that share a KV head
// (row = node*G + head-in-group) form the N side of 32x32x16 bf16 MFMAs; keys
// form the M side, so that S^T = K Q^T comes out with one query row per lane
// (row max / row sum need one cross-half exchange, no LDS) and the
// probabilities are already in the B-operand layout of the second product
// O^T = V^T P^T.  K/V tiles are staged once per workgroup in LDS; the V^T
// operand is fetched with the LDS transpose read (ds_read_b64_tr_b16), so V
// stays in its natural [key][d] layout.  Waves of a workgroup are arranged
// WM x WK: WM groups own different query rows, WK groups own different keys of
// each tile and are merged through LDS at the end (used when few rows share a
// KV head, so that the workgroup still has several waves streaming keys).
//
// Every load on the key path is an LDS-writing load the compiler does not track
// (tiles, page-table entries, the tree's parent array), and every wait on them
// is written by hand as a count of the operations queued behind the one waited
// for: left to the compiler, any register it believes pending costs a
// vmcnt(0), which drains the prefetched tiles.
//
// Variants of the inputs handled by the same kernel: dense or paged cache;
// tree K/V in their own tensors or in the cache behind the committed tokens;
// ancestor sets passed as bitmasks or derived here from the parent array; all
// tree nodes as queries or only the last ones of each tree; K/V stored as bf16
// or as 8-bit floating point (E4M3) bytes, which the wave that loaded them
// widens exactly to bf16 inside LDS before the same arithmetic runs.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/random.h>
#include <time.h>
#include <unistd.h>

#include <algorithm>
#include <cmath>

#include <atomic>
#include <type_traits>
#include <utility>

#include "tva.h"

namespace {

// Instrumented build (-DTVA_TIMELINE, a library of its own): workgroup w of the attention kernel records
// the constant 100 MHz counter at six points of its life (eight where it merges the splits), block w of the merge kernel at two; the
// stamps stay in lanes of one vector register until the end of the kernel and are stored then, so that the kernel's
// own memory operations are disturbed as little as possible.  (The clock's low words.  In scalar registers eight stamps made the deep
// 64-row shape write 15 vector registers to memory: 16 sequences of 512 .. 2048 keys 34 us instead of 27.)
// tva_timeline_read copies them out.
#ifdef TVA_TIMELINE
constexpr int TL_MAX_WG = 8192, TL_SLOTS = 8;
__device__ unsigned long long timeline[TL_MAX_WG * TL_SLOTS];
#define TL_DECL uint32_t tl_t = 0, tl_mark = 0
#define TL_STAMP(i) asm volatile("v_writelane_b32 %0, %1, " #i : "+v"(tl_t) : "s"((uint32_t)__builtin_amdgcn_s_memrealtime()))
#define TL_MARK tl_mark = 1  /* stamps of merge_kernel: bit 63 */
#define TL_STORE(wg, first, n)                                                              \
  if (threadIdx.x < (n) && (wg) < TL_MAX_WG) timeline[(size_t)(wg) * TL_SLOTS + (first) + threadIdx.x] = tl_t | (uint64_t)tl_mark << 63
#else
#define TL_DECL
#define TL_STAMP(i)
#define TL_MARK
#define TL_STORE(wg, first, n)
#endif

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

// Full tiles from which a split of the 256-row shape with D = 64 runs its steady loop.  A shorter one would run little of it, and
// its blocks still move the reference.  Timed with and without it, three head shapes, unsplit and in four splits, geometric
// mean with / without at 8, 12, 16, 20 and 32 full tiles: dense 1.02, 0.98, 0.98, 0.92, 0.88, paged 1.00, 0.98, 0.95, 0.92, 0.87.
constexpr int kSteadyTiles = 11;
constexpr int kShareSplits = 12;  // the most splits that are merged in the attention launch (merged_in_launch)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// A tile takes the low-order P pass when, for some row, (largest probability of the tile) >
// kLoThreshold * (the row's running sum over the keys this wave has seen: both lane halves): then one
// weight can exceed 1/8 of the row's total and its bf16 rounding (2^-8 relative at worst) would be
// visible at the 2e-3 output tolerance.
constexpr float kLoThreshold = 0.125f;
// The reference maximum of a row is only moved (and O, l rescaled) when a tile maximum exceeds it by
// more than 2^kLazy: probabilities then stay below 2^kLazy, harmless in fp32 sums and bf16 operands.
constexpr float kLazy = 8.f, kLazyCap = 256.f;  // (the cap: 2^kLazy)

// ---------------------------------------------------------------------------------------
// ancestor masks
// ---------------------------------------------------------------------------------------
// One workgroup per tree: the parent array is staged in LDS (trees of up to kMaskLds nodes; larger
// ones are walked in global memory), then one thread per node walks its parent chain.  A link that
// does not go strictly downward (or below -1) is reported and ends the walk, so every thread
// finishes in at most T_b steps.
constexpr int kMaskLds = 1024;
__global__ void anc_mask_kernel(const int32_t *__restrict__ parent, const int32_t *__restrict__ cu_T,
                                int B, int W, uint64_t *__restrict__ mask, int32_t *err_flag) {
  __shared__ int32_t spar[kMaskLds];
  const int b = blockIdx.x;
  const int t0 = cu_T[b], T = cu_T[b + 1] - t0;
  const bool in_lds = T <= kMaskLds;
  if (in_lds) {
    for (int i = threadIdx.x; i < T; i += blockDim.x) spar[i] = parent[t0 + i];
    __syncthreads();
  }
  for (int i = threadIdx.x; i < T; i += blockDim.x) {
    uint64_t m[4] = {0, 0, 0, 0};  // W <= 4 handled in registers, larger W goes through memory
    uint64_t *row = mask + (size_t)(t0 + i) * W;
    if (W > 4)
      for (int w = 0; w < W; ++w) row[w] = 0;
    int a = i;
    while (true) {
      if ((a >> 6) < W) {  // a tree larger than the mask row (caller's max_T too small) loses bits, never memory
        if (W <= 4) m[a >> 6] |= 1ull << (a & 63);
        else row[a >> 6] |= 1ull << (a & 63);
      }
      const int p = in_lds ? spar[a] : parent[t0 + a];
      if (p < -1 || p >= a) {
        if (err_flag) {
          // smallest offending global index + 1 (0 = none yet)
          const int code = t0 + a + 1;
          int old = atomicCAS(err_flag, 0, code);
          while (old != 0 && old > code) {
            const int seen = atomicCAS(err_flag, old, code);
            if (seen == old) break;
            old = seen;
          }
        }
        break;
      }
      if (p < 0) break;
      a = p;
    }
    if (W <= 4)
      for (int w = 0; w < W; ++w) row[w] = m[w];
  }
}

// ---------------------------------------------------------------------------------------
// attention
// ---------------------------------------------------------------------------------------
struct AttnParams {
  const __bf16 *q, *k_tree, *v_tree, *k_cache, *v_cache;
  const int32_t *cu_T, *L, *cu_L, *page_table;
  const int32_t *cu_Q;  // null: every tree node is a query; else the last cu_Q[b+1]-cu_Q[b] nodes are
  const uint64_t *mask;
  const int32_t *parent;  // used when mask is null: ancestor masks are derived in the kernel
  float *out, *lse;            // final results
  float *part_out, *part_lse;  // [S, sum_Q, Hq, D], [S, sum_Q, Hq] when S > 1
  int B, Hq, Hkv, G, sum_Q, W;  // sum_Q: query rows of the whole batch (= sum_T without cu_Q)
  uint32_t g_magic, g_bits;     // row / G, rows below 2^30: node_of
  int chunk_keys, n_chunks, n_row_blocks, max_L;
  int pair_slots;          // > 0: sequences are matched to workgroup slots by length: slot j takes the sequence in
  uint32_t slot_seq[16];   // byte j of this array
  int real_splits;         // > 0: the splits that the given lengths fill come first, this many of them: half-word b of
                           // slot_seq is the number of those of sequences 0 .. b
  int page_size, page_shift, max_pages;
  int64_t stride_page, stride_tok, stride_head;
  float scale_log2;  // scale * log2(e) (times the K scale of an fp8 cache)
  float v_scale;     // 1, or the V scale of an fp8 cache
  uint64_t share_tag;  // not 0: a row block's splits are merged in this launch, and this is what tells it from every other
  int share_polls;     // ... looks for the others after which a workgroup stops waiting for them (16 bits; bit 16 + s: split s looks for none)
};

// The node of a query row (row = node * G + head in the group): row / G, exact for rows below 2^30 (g_magic is
// 2^(31 + g_bits) / G rounded up, 2^g_bits >= G).
__device__ __forceinline__ int node_of(const AttnParams &p, int row) { return (int)(__umulhi((uint32_t)row * 2u, p.g_magic) >> p.g_bits); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max over the two 32-lane halves (lanes l and l^32 hold the same query row)
__device__ __forceinline__ float half_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The shapes that can merge a row block's splits in the attention launch (row_groups: their 32-row groups, AttnCfg::WM), for their
// kernels and for the launch alike.  Not the 32-row shape nor D = 64 (merged_in_launch), nor the paged 256-row shape with 8-bit K/V,
// whose loop pays for it: 49 sequences of 557 keys, unsplit, 62.6 -> 64.0 us.
constexpr bool shape_shares(int D, int row_groups, bool paged, bool kv8) { return D == 128 && row_groups > 1 && !(kv8 && paged && row_groups == 8); }

template <int D, int WM, int WK, int RB, bool PAGED, int NST, bool KV8 = false>
struct AttnCfg {
  static constexpr int NW = WM * WK;
  static constexpr int NT = NW * 64;
  static constexpr int KBW = (WK == 1) ? (2) : 1;  // 32-key blocks each wave owns in a tile
  static constexpr int TK = WK * KBW * 32;       // keys per tile
  static constexpr int BM = WM * RB * 32;        // query rows per workgroup
  static constexpr int DC = D / 8;               // 16-byte chunks per K/V row
  static constexpr int ROWB = D * 2;             // bytes per K/V row
  static constexpr int RPI = 64 / DC;            // rows one wave-wide 16-byte-per-lane load covers
  // 8-bit K/V: a row is D bytes, a wave-wide load covers twice the rows
  static constexpr int DC8 = D / 16, RPI8 = 64 / DC8;
  static constexpr int NLDK = KV8 ? TK / RPI8 / NW : TK / RPI / NW;  // such loads per wave per tile, for K (same for V)
  static constexpr int NLD = 2 * NLDK;
  // LDS tile layout: NBLK blocks; block n holds rows n, n+NBLK, n+2*NBLK, ... back to back, and
  // blocks are PAD bytes further apart than their size.  Rows that are read together (16
  // consecutive keys, one per lane, by the K operand load; 4 consecutive keys x 32 bytes by one
  // 16-lane group of the V transpose load) then sit in different blocks, PAD apart in bank
  // position, and every read address is one per-lane base plus a compile-time offset.
  static constexpr int NBLK = DC;                // 16 (D=128) or 8 (D=64)
  // 8-bit K/V (see NL below).  Workgroups of up to four waves widen nothing in LDS: the operand reads
  // take the bytes straight from where they landed (8 bytes per lane for K, the 8-bit LDS transpose read
  // for V) and widen them in registers; the ring is four byte tiles, two workgroups fit a CU.  With one
  // row group (WM = 1) every wave reads only the rows it loaded itself and there is no barrier either.
  // (With two row groups each key is widened twice, with eight waves it would be up to eight times:
  // those widen once, cooperatively, through LDS.)
  static constexpr bool KV8_REG = KV8 && NW <= 4;
  static constexpr int SUBS = TK / NBLK;         // rows per block
  static constexpr int BLKB = SUBS * ROWB;       // 1 KiB (TK=64) or 2 KiB (TK=128)
  static constexpr int IPB = BLKB / 1024;        // load instructions per block (16-bit K/V)
  static constexpr int PK = BLKB + 16;           // block pitch of the K tile
  static constexpr int PV = BLKB + 32;           // block pitch of the V tile
  static constexpr int KTILE = NBLK * PK, VTILE = NBLK * PV;
  static constexpr int STAGE_BYTES = KV8_REG ? 2 * TK * D : (KTILE + VTILE + 1023) / 1024 * 1024;
  // NST = stages of the ring (16-bit K/V): NST - 1 tiles are in flight ahead of the one being computed.
  // Two stages of 64-key tiles keep the footprint small enough for two workgroups per CU.
  // 8-bit K/V: the loads land in per-wave zones of NL landing slots (a tile of bytes each); the wave that
  // loaded a piece widens it to bf16 into one of two tiles of the layout above, one tile ahead of
  // the arithmetic.  NL tiles are in flight or being widened.
  static constexpr int NL = KV8_REG ? 0 : KV8 ? NST : 0;
  static constexpr int LAND_SLOT = KV8 ? 2 * TK * D : 0;
  static constexpr int NSTAGE = KV8_REG ? 4 : KV8 ? 2 : NST;
  // the 256-row shape: its full tiles take consecutive keys per load and, with D = 64, its loop has a steady part of its own (the
  // others' plain loops ran no faster with one: they wait for data)
  static constexpr bool STEADY = WK == 1 && !KV8;
  // Splits of PIPE_TILES full tiles and more run a loop that is a software pipeline over 32-key blocks.  LEAD: tiles that K is
  // fetched further ahead than V; the blocks of the first LO_TILES tiles come with the low-order pass ready.  With / without it,
  // 1 .. 32 sequences unsplit: 256-row shape 0.98 at 6 full tiles, 0.92 at 12 and 16, 0.96 at 32, dense and paged alike; deep
  // 64-row shape dense 1.02 at 12, 0.98 at 15, 0.89 at 32.  128-row shape dense, 1950 drawn calls, split and unsplit: 1.000 at 18
  // and 19 tiles, where one in nine is 2 .. 4 % slower, 0.987 at 20 (one in 22), 0.98 from 22 on, 0.964 beyond 33; of more rows than
  // one workgroup has, where keys are read more than once (PIPE_TILES_ROWS), 1.00 at 16, 0.985 at 18, 0.97, 0.96 and 0.89.  Paged, the
  // two last lost up to 6 % below 27 tiles (K's and V's rows are each looked up, at one block per tile) and gain 2 % at 32: without.
  static constexpr bool PIPED = D == 128 && !KV8 && NST == 4 && (WK == 1 || !PAGED);
  static constexpr int LEAD = KBW == 1 ? 2 : 1, LO_TILES = KBW == 1 ? 6 : 3;
  static constexpr int PIPE_TILES = KBW == 2 ? 5 : WM == 4 ? 22 : 14, PIPE_TILES_ROWS = KBW == 1 && WM == 4 ? 17 : PIPE_TILES;
  // m_use (in the kernel) is kept from block to block, or derived in each from the reference: kept, launches are 0.5 %
  // faster, but 1 % slower where 8-bit tiles are widened through LDS, and the paged 256-row shape with D = 64 has no
  // register for it
  static constexpr bool KEEP_USE = (!KV8 || KV8_REG) && !(D == 64 && PAGED && WK == 1);
  // A block's K operands and V^T operands are read ahead, in one go, and (dense) the loads of the tile to come are queued under
  // its products.  (One sequence of 2048 keys, 60 nodes, 7 splits of five tiles, one wave per SIMD; cycles a tile: queueing 434 -> 102,
  // since a CU takes 64 bytes a cycle and all waves queue at once, the arithmetic with the queueing in it 1541 -> 1621; 13.1 -> 12.6 us.
  // 128 keys, 4 heads, D = 64: 5.47 -> 5.38.  The shapes with a pipelined loop keep their plain one for their short splits.)
  // The rings of three and four stages, 24 drawn calls each, with / without: paged deep 64-row shape 0.964; D = 64 dense, deep 64-row shape
  // 0.985, 128-row shape 0.995, paged 0.996.  Not the paged 128-row shape, 1.008 (two at 1.02 and more; 16 sequences of 3000 keys, 60
  // nodes, two row blocks, 1.05), nor D = 64, paged, in the deep 64-row shape, 1.003 (27 sequences of 1707 keys, 55 nodes, 1.04).
  static constexpr bool AHEAD = WK > 1 && !KV8 && RB == 1 && !PIPED && !(PAGED && (D == 128 ? WM == 4 : NST == 3));
  static constexpr int PD = KV8_REG ? NSTAGE - 1 : KV8 ? NL : NSTAGE - 1;  // tiles in flight ahead of the one being computed (widened)
  static constexpr int WG_PER_CU = KV8 ? (KV8_REG ? 2 : 1) : (NSTAGE == 2 && TK == 64) ? 2 : 1;
  // wavefronts per SIMD that the registers have to leave room for.  (The rings of the eight-wave shapes with D = 64 let two
  // workgroups share a CU, and so do up to 128 registers per lane: with 131, 50 sequences of 200 keys took 21 us instead
  // of 14.5, paged, 256-row shape.  The dense 256-row shape needs four more than that and has one workgroup per CU.  Of the 64-row shape's short ring four
  // fit: with 131 registers 60 paged sequences of 300 keys, 30 nodes, took 23.7 us, with 128 22.2.)
  static constexpr int WAVES_PER_SIMD = NST == 4 && D == 128 && !KV8 ? 2 : D == 64 && ((NW == 8 && (PAGED || WK == 2)) || (NW == 4 && NST == 2)) ? 4 : WG_PER_CU;
  // after the key loop the ring is reused: exchange area of the key-group merge, then (behind it,
  // when the groups are paired; else on top of it, after a barrier) the output transpose patches
  static constexpr bool PAIR = (WK == 2);
  static constexpr int NDW = PAIR ? D / 64 : D / 32;  // 32-wide d blocks of the result each wave writes
  static constexpr int TP = NDW * 32 + 4;             // patch row pitch, floats
  static_assert(WK == 1 || WK == 2, "one key group, or two that are merged pairwise");
  static constexpr int MERGE_BYTES = PAIR ? (2 * WK * WM * RB * 32 * 4 + WM * WK * RB * (D / 64) * 16 * 64 * 4) : 0;
  static constexpr int PATCH_OFF = PAIR ? MERGE_BYTES : 0;
  static constexpr int PATCH_BYTES = (PAIR ? NW : WM) * 32 * TP * 4;
  static constexpr int LAND_OFF = NSTAGE * STAGE_BYTES;
  static constexpr int RING_BYTES = NSTAGE * STAGE_BYTES + NL * LAND_SLOT;
  // paged cache: table entries of the next LOOK tiles, fetched by the same LDS-writing loads as the
  // tiles themselves: [slot][wave][key of the tile], behind the ring.  Entries are needed when their
  // tile is queued, PD tiles ahead; requested LOOK >= PD tiles ahead they are older than every tile still in flight, so
  // that waiting for them drains none.
  static constexpr int LOOK = PD >= 3 ? 3 : 2, PG_SLOTS = LOOK >= 3 ? 4 : 2;
  static constexpr int NPG = PAGED ? 1 : 0;      // table-entry loads per wave and tile: one entry per lane and key
  static constexpr int TILE_OPS = NLD + NPG;     // this wave's memory operations per tile
  static constexpr int PG_SLOT = NW * 256;
  // (the paged 256-row shape with D = 64 has no register for the short form of the addresses outside its steady loop)
  static constexpr bool SMALL_PAGES = PAGED && !(D == 64 && STEADY);
  static constexpr bool PG_BY_KEY = NLDK > 1;
  static constexpr int PG_BYTES = PAGED ? PG_SLOTS * PG_SLOT : 0;
  // parent indices of the sequence's tree (used when no ancestor masks are passed), behind those
  static constexpr int PARENT_OFF = RING_BYTES + PG_BYTES;
  static constexpr int PARENT_BYTES = TVA_MAX_TREE * 4;
  // Splits merged in the launch itself (the end of the kernel): per row its log-sum-exp, its number and where each wave stores it, and
  // a word.  Where the references of the key groups were, or behind the patches.
  static constexpr bool SHARES = shape_shares(D, WM, PAGED, KV8);
  static constexpr int OWN_OFF = PAIR ? 0 : PATCH_BYTES, OWN_BYTES = SHARES ? (2 * WM + NW) * 32 * 4 + 16 : 0;
  static_assert(RB == 1 && (!PAIR || !SHARES || OWN_BYTES <= MERGE_BYTES), "");
  static constexpr int TAIL_BYTES = PAIR ? MERGE_BYTES + PATCH_BYTES : PATCH_BYTES + OWN_BYTES;
  static constexpr int SMEM = PARENT_OFF + PARENT_BYTES > TAIL_BYTES ? PARENT_OFF + PARENT_BYTES : TAIL_BYTES;
  // load instruction n of a tile (n = wave * NLDK + j): the first tile row it covers
  static constexpr int load_row0(int n) { return KV8 ? n * RPI8 : n / IPB + NBLK * ((n % IPB) * RPI); }
  static_assert(SMEM * WG_PER_CU <= 160 * 1024, "LDS of the workgroups that share a CU");
  static_assert(PD <= 3 && TILE_OPS * (PD > 1 ? PD - 1 : 1) < 64 && NPG * LOOK + TILE_OPS < 64, "the wait counter holds 6 bits");
  static_assert(!PAGED || TK == 64, "a tile's table entries are one load of a wave");
  static_assert(TK % ((KV8 ? RPI8 : RPI) * NW) == 0, "tile must divide evenly over the waves");
  static_assert(!KV8 || (D == 128 && NLDK >= 1), "8-bit K/V: head dimension 128");
  static_assert(BLKB % 1024 == 0, "a block is a whole number of wave-wide loads");
};

template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_each(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) { static_for_each<N>(f, std::make_integer_sequence<int, N>{}); }

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
constexpr int vm_cap(int n) { return n > 63 ? 63 : n; }  // the counter holds 6 bits; waiting for less is safe
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | (((n >> 4) & 3) << 14); }

// Cache policy of the K/V tile loads and of the stores of partial results: the non-temporal hint (the `nt` bit
// of the instruction).  A launch streams K and V through once and its partial rows are read next by another
// kernel; without the hint both displace each other and the rest in the L2s (measured: 3 ... 10 % of the step).
constexpr int kLoadOnce = 2;  // cache-policy operand of the LDS-writing loads: bit 1 = nt
#define GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))
typedef __attribute__((address_space(3))) unsigned char lds_byte;

// LDS transpose read of four 16-bit elements per lane (see the V operand comment in attn_kernel),
// issued from inline assembly: the compiler cannot tell these reads apart from the ring stages the
// asynchronous tile loads are still filling and would otherwise drain all outstanding loads
// (vmcnt 0) in front of every one of them.  The matching wait is lds_wait below.
template <int OFF>
__device__ __forceinline__ s16x4 lds_read_tr(uint32_t addr) {
  s16x4 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
// Waits for every outstanding LDS read of this wave; the operands tie the wait to the values.
__device__ __forceinline__ void lds_wait(s16x4 &a, s16x4 &b, s16x4 &c, s16x4 &d) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

// The same into a given register, a 16-byte read of a K operand, and the wait until at most N LDS operations are
// outstanding (they return in order): the pipelined loop's reads are in flight over several matrix instructions.
template <int OFF>
__device__ __forceinline__ void lds_read_v(s16x4 &v, uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void lds_read_k(bf16x8 &v, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
}
template <int N>
__device__ __forceinline__ void lds_wait_n(bf16x8 &a) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "n"(N));
}
template <int N>
__device__ __forceinline__ void lds_wait_n(bf16x8 &a, s16x4 &b, s16x4 &c) {
  asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(a), "+v"(b), "+v"(c) : "n"(N));
}

// 16-byte LDS read from a landing zone of the 8-bit K/V path (inline assembly for the same reason),
// and its wait.
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr));
  return v;
}
__device__ __forceinline__ void lds_wait(u32x4 &a, u32x4 &b) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a), "+v"(b));
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2 lds_read_b64(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64 %0, %1" : "=v"(v) : "v"(addr));
  return v;
}
// LDS transpose read of bytes: the 16 lanes of a group pass the addresses of 8 bytes each, rows
// (lane >> 1) of an 8 x 16 byte matrix, columns 8 * (lane & 1) ...; lane j of the group receives
// column j, rows 0 .. 7.
__device__ __forceinline__ u32x2 lds_read_tr8(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b8 %0, %1" : "=v"(v) : "v"(addr));
  return v;
}
__device__ __forceinline__ void lds_wait(u32x2 &a, u32x2 &b, u32x2 &c, u32x2 &d) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
// E4M3 bytes -> bf16, two to an instruction with the scale of 1 (exact: every E4M3 value, subnormal ones too,
// is a normal bf16 value; a NaN stays one).  By way of fp32 it took twice the instructions, on the chain
// from an operand's arrival to its product: 64 sequences x 512 .. 2048 keys, 8 nodes, 40.4 -> 39.0 us; 16 x
// 1024 .. 4096 paged, 16 nodes, 42.7 -> 39.7; 32 x 2048, 60 nodes (256-row shape, widened through LDS) 85.1 -> 84.4.
__device__ __forceinline__ u32x2 widen_e4m3_word(uint32_t raw) {
  u32x2 out;
  out[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw, 1.f, false));
  out[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw, 1.f, true));
  return out;
}
__device__ __forceinline__ bf16x8 widen_e4m3(const u32x2 raw) {
  const u32x2 a = widen_e4m3_word(raw[0]), b = widen_e4m3_word(raw[1]);
  return __builtin_bit_cast(bf16x8, u32x4{a[0], a[1], b[0], b[1]});
}
__device__ __forceinline__ void widen_e4m3(const u32x4 raw, bf16x8 &lo, bf16x8 &hi) {
  lo = widen_e4m3(u32x2{raw[0], raw[1]});
  hi = widen_e4m3(u32x2{raw[2], raw[3]});
}

// RBS: the 32-row blocks of a wave, below 0 (SHARED) in the kernels that merge the row block's splits at their end.
// They are kernels of their own: with the 10 to 20 KB that only those launches run behind its loops, calls without splits and those whose
// splits a second launch merges took 1 .. 3 % longer in the dense deep 64-row and 128-row shapes below 14 and 22 tiles (8 sequences of 700
// keys, 30 nodes: 16.9 -> 17.3 and 20.9 -> 21.4 us; 36 such calls of three shapes now 0.99 of the time before there was a merge in
// the launch, the 128-row shape's 1.01).  And both are this function, not two that call one: inlined into them, it came out with more
// scalar instructions in the loops of the paged shapes with D = 64 (60 sequences of 1384 keys, 37 nodes, 62 -> 64 us).
template <int D, int WM, int WK, int RBS, bool PAGED, int NST, bool KV8>
__global__ void __launch_bounds__(WM *WK * 64, (AttnCfg<D, WM, WK, RBS < 0 ? -RBS : RBS, PAGED, NST, KV8>::WAVES_PER_SIMD))
    attn_kernel(const AttnParams p_in) {
  constexpr bool SHARED = RBS < 0;
  constexpr int RB = SHARED ? -RBS : RBS;
  using C = AttnCfg<D, WM, WK, RB, PAGED, NST, KV8>;
  static_assert(!SHARED || C::SHARES, "");
  // The arguments the prologue needs, tied together by an empty statement so that they are fetched
  // in one batch at the top rather than one by one, each with its own wait, at their first uses.
  AttnParams p = p_in;
  asm("" : "+s"(p.cu_T), "+s"(p.L), "+s"(p.cu_L), "+s"(p.q), "+s"(p.k_cache), "+s"(p.v_cache), "+s"(p.mask),
      "+s"(p.stride_tok), "+s"(p.stride_head), "+s"(p.G), "+s"(p.g_magic), "+s"(p.g_bits), "+s"(p.Hq), "+s"(p.chunk_keys),
      "+s"(p.n_chunks), "+s"(p.max_L));
  constexpr int TK = C::TK, BM = C::BM, DC = C::DC, ROWB = C::ROWB, RPI = C::RPI, NLDK = C::NLDK, NLD = C::NLD;
  constexpr int KBW = C::KBW, NSTAGE = C::NSTAGE, PD = C::PD, STAGE_BYTES = C::STAGE_BYTES;
  constexpr int NBLK = C::NBLK, IPB = C::IPB, PK = C::PK, PV = C::PV, KTILE = C::KTILE;
  constexpr int NS = D / 16;  // k-steps of the QK product
  constexpr int ND = D / 32;  // 32-wide d blocks of the PV product
  extern __shared__ __align__(1024) unsigned char smem[];
  lds_byte *const lds = (lds_byte *)smem;

  TL_DECL;
  TL_STAMP(0);
  // ---- which (sequence, KV head, row block, chunk) ----
  // grid = (Hkv, row blocks, B * splits): the KV head varies fastest in dispatch order
  const int kvh = blockIdx.x;
  const int rblk = blockIdx.y;
  int b = (int)blockIdx.z / p.n_chunks;
  const int chunk_of_slot = (int)blockIdx.z - b * p.n_chunks;
  if (p.pair_slots > 0) {
    // (a permutation of the sequences, made on the host: see fill_slots; picked with scalar selects, so that the
    // argument block is never indexed by a register)
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) word = (b >> 2) == i ? p.slot_seq[i] : word;
    b = (int)((word >> (8 * (b & 3))) & 0xFFu);
  }
  int split = chunk_of_slot;
  if (C::NW == 8 && p.real_splits > 0) {
    // (a permutation of (sequence, split), made on the host: see fill_slots.  Lane i looks at sequence i: the argument block is
    // never indexed by a register, and none of its words is held past this.  Picked with scalars instead, up to 54 of the
    // kernel's were parked in lanes of vector registers over the whole loop, in every launch of these shapes: 43 paged
    // sequences of 223 keys, 8-bit, 256-row shape 42.3 us instead of 39.9; 63 of 648 keys, D = 64, 128-row shape, which then needed
    // more than 128 registers, 36.5 instead of 27.2.)
    const int z = (int)blockIdx.z, over = z - p.real_splits, i = (int)threadIdx.x & 63;
    uint32_t word = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) word = (i >> 1) == k ? p.slot_seq[k] : word;
    const int filled = (int)((word >> (16 * (i & 1))) & 0xFFFFu);  // of sequences 0 .. i; past them, the unfilled ones
    const int upto = over < 0 ? filled : (i + 1) * p.n_chunks - filled, place = over < 0 ? z : over;
    b = __builtin_popcountll(__builtin_amdgcn_ballot_w64(i < p.B && upto <= place));
    split = place - (b > 0 ? __builtin_amdgcn_readlane(upto, b - 1) : 0);
    // (the unfilled splits of b are its last ones)
    if (over >= 0) split += __builtin_amdgcn_readlane(filled, b) - (b > 0 ? __builtin_amdgcn_readlane(filled, b - 1) : 0);
  }
  const int chunk = split;

  // Arguments that only the last tiles and the end of the workgroup need are read again there: held over the loop, paged, they
  // were the scalars too many (up to 25 parked in lanes of vector registers).
  typedef const __attribute__((address_space(4))) AttnParams *const_args;
  auto late_args = [&]() __attribute__((always_inline)) {
    const_args a = (const_args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return a;
  };
  // every per-sequence scalar is requested before the first one is needed
  // (read through the constant address space: none of these arrays changes while the kernel
  // runs, and saying so keeps the loads scalar wherever they sit)
  typedef const __attribute__((address_space(4))) int32_t const_i32;
  int t0 = ((const_i32 *)(uintptr_t)p.cu_T)[b];
  int t1 = ((const_i32 *)(uintptr_t)p.cu_T)[b + 1];
  int Lb0 = ((const_i32 *)(uintptr_t)p.L)[b];
  int cuL = PAGED ? 0 : ((const_i32 *)(uintptr_t)p.cu_L)[b];
  // (an empty statement that ties them together: keeps the compiler from moving one of the loads
  // down to its first use, where the wave would wait for it alone)
  int q0 = p.cu_Q ? ((const_i32 *)(uintptr_t)p.cu_Q)[b] : 0;
  int q1 = p.cu_Q ? ((const_i32 *)(uintptr_t)p.cu_Q)[b + 1] : 0;
  asm("" : "+s"(t0), "+s"(t1), "+s"(Lb0), "+s"(cuL), "+s"(q0), "+s"(q1));
#ifdef TVA_TIMELINE
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the scalars have arrived
  TL_STAMP(1);
#endif
  const int Tb = t1 - t0;
  // query nodes: all T_b of the tree, or (draft-stage use: one expansion layer attends to the layers
  // before it) only its last Tq; tq0 is the first query row of the sequence in q / out / lse
  const int Tq = p.cu_Q ? (q1 - q0 < Tb ? q1 - q0 : Tb) : Tb;
  const int tq0 = p.cu_Q ? q0 : t0;
  const int node_off = Tb - Tq;
  const int R = Tq * p.G;
  if (rblk * BM >= R) return;
  const int Lb = Lb0 < p.max_L ? Lb0 : p.max_L;
  int nc = (Lb + p.chunk_keys - 1) / p.chunk_keys;
  nc = nc < 1 ? 1 : nc;
  if (chunk >= nc) {
    // this sequence has fewer chunks than the launch provides: mark the slot empty, for the merge's launch
    if constexpr (SHARED) return;
    for (int row = rblk * BM + (int)threadIdx.x; row < R && row < (rblk + 1) * BM; row += blockDim.x) {
      const int t = node_of(p, row), g = row - t * p.G;
      p.part_lse[(size_t)chunk * p.sum_Q * p.Hq + (size_t)(tq0 + t) * p.Hq + kvh * p.G + g] = -INFINITY;
    }
    return;
  }
  const int k0 = chunk * p.chunk_keys;
  const int k1 = (k0 + p.chunk_keys < Lb) ? k0 + p.chunk_keys : Lb;
  const bool has_tree = (chunk == nc - 1);
  const int n_full = (k1 - k0) / TK;               // cache tiles that need no masking
  const int n_ct = (k1 - k0 + TK - 1) / TK;
  const int n_tt = has_tree ? (Tb + TK - 1) / TK : 0;
  const int n_tiles = n_ct + n_tt;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wk = wave / WM;
  const int l32 = lane & 31, hh = lane >> 5;
  // Two key groups: at the end each wave keeps one half of the head dimension and hands the other to its partner.  The kept
  // half's 32-wide blocks come first in the accumulators, whichever it is, so that both run the same instructions.
  const int kept0 = C::PAIR ? wk * (D / 2) : 0, other0 = C::PAIR ? (1 - wk) * (D / 2) : 0;  // first element of each

  const bool wave_has_rows = rblk * BM + wm * RB * 32 < R;  // wave-uniform
  // ---- Q operands (B operand of S^T = K Q^T: lane = query row, 8 consecutive d per k-step) ----
  bf16x8 qreg[RB][NS];
  uint64_t mrow[RB][2];
  bool rvalid[RB];
  int64_t orow[RB];  // (global token * Hq + head) of the lane's row
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const int row = rblk * BM + (wm * RB + r) * 32 + l32;
    rvalid[r] = row < R;
    // rows past the end compute on a copy of the last row (finite data) and are never stored
    const int rowc = rvalid[r] ? row : R - 1;
    const int t = node_of(p, rowc);
    const int g = rowc - t * p.G;
    orow[r] = (int64_t)(tq0 + t) * p.Hq + kvh * p.G + g;
    const __bf16 *qp = p.q + orow[r] * D + 8 * hh;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      qreg[r][s] = *(const __attribute__((address_space(1))) bf16x8 *)(uintptr_t)(qp + 16 * s);
    }
    // mask rows are only requested here (rows past the end read their stand-in's); the first use
    // is in the tree tiles, so nothing waits for them before the key loads have been queued
    mrow[r][0] = mrow[r][1] = 0;
    if (has_tree && p.mask != nullptr) {
      const auto *mp = (const __attribute__((address_space(1))) uint64_t *)(uintptr_t)(p.mask + (size_t)(t0 + node_off + t) * p.W);
      mrow[r][0] = mp[0];
      if (p.W > 1) mrow[r][1] = mp[1];
    }
  }

  // ---- running softmax state (log2 domain; m_run is the reference the exponentials use) ----
  // (m_use: the reference, or 0 while there is none; cap, steady part of the loop only: the largest sum of one lane's
  // probabilities of a block that needs no look at the maximum, -1 while there is no reference)
  float m_run[RB], l_run[RB], m_use[RB], cap[RB];
  f32x16 oacc[RB][ND];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    m_run[r] = -INFINITY, m_use[r] = 0.f;
    l_run[r] = 0.f;
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[r][d][i] = 0.f;
  }

  // ---- tile loads: global -> LDS directly (16 bytes per lane, 1 KiB per wave instruction) ----
  // Instruction n of a tile fills part n%IPB of block n/IPB; lane l lands at sub-row
  // (n%IPB)*RPI + l/DC of that block, chunk l%DC.  Rows past the tile's limit re-read the last
  // valid row (finite data; their scores are masked to -inf), so LDS never holds stale values.
  // (8-bit K/V: a row is D bytes, instruction n covers rows n*RPI8 .. n*RPI8 + RPI8 - 1 of the tile and
  // lands in the wave's own zone of a landing slot, from where the same lanes widen it to bf16 into
  // the layout above.)
  constexpr int EB = KV8 ? 1 : 2;                 // bytes per K/V element
  constexpr int LDC = KV8 ? C::DC8 : DC;          // lanes (16-byte chunks) per row of a wave-wide load
  const int lsub = lane / LDC, lpos = lane % LDC;
  // the lane's row within its load instruction's rows (an expression and not a variable: the register it would be kept in
  // is the one too many for two workgroups of the paged 256-row shape with D = 64 to share a CU, 128 per lane)
#define lrow (KV8 ? lsub : NBLK * lsub)
  // tile row of (load instruction j of this wave, lane 0), and the LDS byte offsets of that
  // instruction's K and V destinations inside a stage (8-bit: inside the wave's zone of a landing
  // slot): wave-uniform.  (Plain expressions: with calls in their place the host pass of the compiler
  // silently drops the kernel's launch stub.)
  auto row0_of = [&](int j) __attribute__((always_inline)) { return C::load_row0(wave * NLDK + j); };
  // A full cache tile's keys may sit in any of its rows (nothing in it is masked, K and V agree): there, the rows one
  // instruction fills take consecutive keys -- one page of a paged cache, neighbouring lines of a dense one, instead of
  // rows 16 keys apart.  (Timed with and without it, 220 calls: the 256-row shape dense with D = 128 0.5 .. 1 % faster, dense with
  // D = 64 1 % slower, paged within 0.5 %; the 128-row shape within 1 % either way, shapes of fewer rows up to 2 % slower.)
  constexpr int LPI = KV8 ? C::RPI8 : RPI;
  auto full_key = [&](int j) __attribute__((always_inline)) { return (wave * NLDK + j) * LPI + lsub; };
  auto row_of = [&](int t, int j) __attribute__((always_inline)) { return C::STEADY && t < n_full ? full_key(j) : row0_of(j) + lrow; };  // what the lane loads of tile t
#define kdst_of(j) (KV8 ? (wave * 2 * NLDK + (j)) * 1024 : ((wave * NLDK + (j)) / IPB) * PK + ((wave * NLDK + (j)) % IPB) * 1024)
#define vdst_of(j) (KV8 ? (wave * 2 * NLDK + NLDK + (j)) * 1024 : KTILE + ((wave * NLDK + (j)) / IPB) * PV + ((wave * NLDK + (j)) % IPB) * 1024)
  const char *const kc_bytes = reinterpret_cast<const char *>(p.k_cache);
  const char *const vc_bytes = reinterpret_cast<const char *>(p.v_cache);
  const char *const kt_bytes = reinterpret_cast<const char *>(p.k_tree);
  const char *const vt_bytes = reinterpret_cast<const char *>(p.v_tree);
  const int64_t cache_base = PAGED ? 0 : (int64_t)cuL * p.stride_tok + (int64_t)kvh * p.stride_head;
  // (8-bit K/V read in place: inside each 1 KiB piece -- 8 rows of 8 chunks -- the lane that lands in
  // slot (row, c) fetches chunk c ^ row ^ (j & 1) of that row, j the piece's index: the 8-byte operand
  // reads and the byte transpose reads then spread over the LDS banks)
  auto chunk_of = [&](int j) __attribute__((always_inline)) { return C::KV8_REG ? (lpos ^ lsub ^ (j & 1)) : lpos; };
  // paged cache: each lane needs the page of the row it loads.  The entries of tile t + LOOK, lane i's that of the tile's
  // key i, are requested right after the loads of tile t have been queued, by an LDS-writing load like the tiles' own, into a
  // ring of slots; the wave's memory operations then come in a fixed order and number per tile (every tile, also a
  // tree tile or the last ones, is followed by a request: past the end it re-reads the entry of the
  // last key), which is what the counted waits below rely on.
  // (Where a wave loads a tile with one instruction the entry is that of the row the lane loads: no register for another index.)
  // STEADY_PART: there are cache keys, and the page size is a power of two.
  lds_byte *const pg_lds = lds + C::RING_BYTES + wave * 256;
  const int32_t *const pages_of_b = PAGED ? p.page_table + (int64_t)b * p.max_pages : nullptr;
  auto request_pages = [&](int t, auto steady_tag) __attribute__((always_inline)) {
    if (!PAGED) return;
    constexpr bool STEADY_PART = decltype(steady_tag)::value == 1, SHIFT = decltype(steady_tag)::value != 0;
    const int row = C::PG_BY_KEY ? lane : row_of(t, 0);
    // a tree tile whose keys live in the cache (no separate tree tensors): positions L_b + node
    const bool tree_in_cache = t >= n_ct && p.k_tree == nullptr;
    int key;
    if constexpr (STEADY_PART) {  // (written so, the 256-row shape with D = 64 has the registers for it)
      key = k0 + t * TK + row;
      key = key < k1 ? key : k1 - 1;
      if (tree_in_cache) key = Lb0 + (t - n_ct) * TK + row, key = key < Lb0 + Tb ? key : Lb0 + Tb - 1;
    } else {
      const int last = tree_in_cache ? Lb0 + Tb - 1 : k1 - 1;
      key = (tree_in_cache ? Lb0 + (t - n_ct) * TK : k0 + t * TK) + row;
      key = key < last ? key : last;
      key = key < 0 ? 0 : key;
    }
    int pidx = SHIFT || p.page_shift >= 0 ? (key >> p.page_shift) : (key / p.page_size);
    pidx = pidx < p.max_pages ? pidx : p.max_pages - 1;  // never past the sequence's row of the table
    const int32_t *src = pages_of_b + pidx;
    __builtin_amdgcn_global_load_lds(GLOBAL_PTR(src), pg_lds + (t & (C::PG_SLOTS - 1)) * C::PG_SLOT, 4, 0, 0);
  };
  // the entry of row `row` of tile t
  auto page_of = [&](int t, int row) __attribute__((always_inline)) {
    return *reinterpret_cast<const __attribute__((address_space(3))) uint32_t *>(pg_lds + (t & (C::PG_SLOTS - 1)) * C::PG_SLOT + (C::PG_BY_KEY ? row : lane) * 4);
  };
  // (pages whose slots and strides fit 32 bits: the row's address is one multiply-add on its page's
  // number; others take 64-bit products and, where the page size is no power of two, a division.  With these addresses in every
  // tile and one load of table entries per tile instead of one per load of rows, from which each row finds its own --
  // bound by the instructions between two tiles' loads, 16 products and eight requests a tile in the two-wave shape:
  // 48 sequences of 500 .. 1300 keys, 6 nodes, 42.1 -> 37.8 us, 8-bit 48 x 1000 35.4 -> 31.7, D = 64 40 x 500 .. 700
  // 20.1 -> 17.1; 64-row shape, 16 x 1024 .. 4096, 8-bit, 40.0 -> 38.4; 128-row shape, 16 x 700 .. 1500, 30 nodes,
  // 36.5 -> 34.1; 256-row shape, 4 x 16 .. 32 K, 48 nodes, 122.5 -> 114 at its power limit.  The strides are held in bytes
  // once, 64 bits wide, and the 32-bit form takes their low words: with a second set the kernels had more scalars than
  // registers.)
  const bool small_pages = PAGED && p.page_shift >= 0 && p.stride_page * EB < (1ll << 31) &&
                           ((int64_t)p.page_size * p.stride_tok + (int64_t)p.Hkv * p.stride_head) * EB < (1ll << 31);
  const int64_t page_bytes = p.stride_page * EB, tok_bytes = p.stride_tok * EB, head_bytes = kvh * p.stride_head * EB;
  auto small_off = [&](uint32_t page, int pos, int j) __attribute__((always_inline)) {
    const uint32_t slot = (uint32_t)pos & ((uint32_t)p.page_size - 1u);
    return (uint64_t)page * (uint32_t)page_bytes + (slot * (uint32_t)tok_bytes + (uint32_t)head_bytes + (uint32_t)chunk_of(j) * 16u);
  };
  auto large_off = [&](uint32_t page, int pos, int j) __attribute__((always_inline)) {
    const int pidx = p.page_shift >= 0 ? (pos >> p.page_shift) : (pos / p.page_size);
    return (uint64_t)((int64_t)(int)page * page_bytes + (int64_t)(pos - pidx * p.page_size) * tok_bytes + head_bytes + chunk_of(j) * 16);
  };
  // full tiles of a dense cache: a wave-uniform row pointer plus one tile-independent lane offset
  const int full_row = C::STEADY ? lsub : lrow;
  const uint32_t lane_off2[2] = {(uint32_t)full_row * (uint32_t)p.stride_tok * (uint32_t)EB + (uint32_t)chunk_of(0) * 16u,
                                 (uint32_t)full_row * (uint32_t)p.stride_tok * (uint32_t)EB + (uint32_t)chunk_of(1) * 16u};
  auto tile_row = [&](int j) __attribute__((always_inline)) { return C::STEADY ? full_key(j) : row0_of(j) + lrow; };
  uint32_t lane_off[NLDK];
#pragma unroll
  for (int j = 0; j < NLDK; ++j) lane_off[j] = (uint32_t)tile_row(j) * (uint32_t)tok_bytes + (uint32_t)chunk_of(j) * 16u;
  auto issue_impl = [&](int t, auto tree_tag) __attribute__((always_inline)) {
    constexpr bool tree = decltype(tree_tag)::value;
    const int base = tree ? (t - n_ct) * TK : k0 + t * TK;
    const int limit = tree ? Tb : k1;
    lds_byte *stage = (KV8 && !C::KV8_REG) ? lds + C::LAND_OFF + (t % (C::NL > 0 ? C::NL : 1)) * C::LAND_SLOT
                                           : lds + (t % NSTAGE) * STAGE_BYTES;
    if (!PAGED && t < n_full) {
#pragma unroll
      for (int j = 0; j < NLDK; ++j) {
        // (an address per load, or, where operands are read ahead, a register per load of a tile: 8-bit K/V 1 % slower with it, the
        // short splits of the dense deep 64-row and 256-row shapes 0.5 %)
        const int row0 = C::AHEAD ? 0 : C::STEADY ? (wave * NLDK + j) * LPI : row0_of(j);
        const int64_t urow = cache_base + (int64_t)(base + row0) * p.stride_tok;
        const uint32_t off = C::AHEAD ? lane_off[j] : lane_off2[j & 1];
        const char *ksrc = kc_bytes + urow * EB + off;
        const char *vsrc = vc_bytes + urow * EB + off;
        __builtin_amdgcn_global_load_lds(GLOBAL_PTR(ksrc), stage + kdst_of(j), 16, 0, kLoadOnce);
        __builtin_amdgcn_global_load_lds(GLOBAL_PTR(vsrc), stage + vdst_of(j), 16, 0, kLoadOnce);
      }
    } else if (PAGED && !(tree && p.k_tree != nullptr)) {
      // (tree keys stored in the cache follow the sequence's L_b committed tokens)
      if (C::SMALL_PAGES && small_pages) {
#pragma unroll
        for (int j = 0; j < NLDK; ++j) {
          const int row = tree ? row0_of(j) + lrow : row_of(t, j);
          int key = base + row;
          key = key < limit ? key : limit - 1;
          const uint64_t off = small_off(page_of(t, row), tree ? Lb0 + key : key, j);
          __builtin_amdgcn_global_load_lds(GLOBAL_PTR(kc_bytes + off), stage + kdst_of(j), 16, 0, kLoadOnce);
          __builtin_amdgcn_global_load_lds(GLOBAL_PTR(vc_bytes + off), stage + vdst_of(j), 16, 0, kLoadOnce);
        }
      } else {
#pragma unroll
        for (int j = 0; j < NLDK; ++j) {
          const int row = tree ? row0_of(j) + lrow : row_of(t, j);
          int key = base + row;
          key = key < limit ? key : limit - 1;
          const uint64_t off = large_off(page_of(t, row), tree ? Lb0 + key : key, j);
          __builtin_amdgcn_global_load_lds(GLOBAL_PTR(kc_bytes + off), stage + kdst_of(j), 16, 0, kLoadOnce);
          __builtin_amdgcn_global_load_lds(GLOBAL_PTR(vc_bytes + off), stage + vdst_of(j), 16, 0, kLoadOnce);
        }
      }
    } else {
#pragma unroll
    for (int j = 0; j < NLDK; ++j) {
      const char *ksrc, *vsrc;
      int key = base + (tree ? row0_of(j) + lrow : row_of(t, j));
      key = key < limit ? key : limit - 1;
      const int eoff = chunk_of(j) * (16 / EB);  // first element of the lane's 16-byte chunk
      if (tree && p.k_tree != nullptr) {
        const int64_t off = ((int64_t)(t0 + key) * p.Hkv + kvh) * D + eoff;
        ksrc = kt_bytes + off * EB;
        vsrc = vt_bytes + off * EB;
      } else {
        const int64_t off = cache_base + (int64_t)(tree ? Lb0 + key : key) * p.stride_tok + eoff;
        ksrc = kc_bytes + off * EB;
        vsrc = vc_bytes + off * EB;
      }
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(ksrc), stage + kdst_of(j), 16, 0, kLoadOnce);
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(vsrc), stage + vdst_of(j), 16, 0, kLoadOnce);
    }
    }
  };

  auto issue_tile = [&](int t) __attribute__((always_inline)) {
    if (t >= n_ct) issue_impl(t, std::true_type{});
    else issue_impl(t, std::false_type{});
    request_pages(t + C::LOOK, std::false_type{});
  };

  // per-lane LDS read bases (row r of a tile: block r % NBLK, sub-row r / NBLK)
  const int L16 = lane & 15, grp1 = (lane >> 4) & 1;
  const int wave_sub = wk * KBW * (32 / NBLK);  // first sub-row of this wave's keys
  const int kbase_off = (l32 % NBLK) * PK + (wave_sub + l32 / NBLK) * ROWB + hh * 16;
  const int vbase_off = KTILE + (4 * hh + (L16 >> 2)) * PV + wave_sub * ROWB + (2 * grp1 + ((L16 & 3) >> 1)) * 16 +
                        ((L16 & 1) << 3);

  // 8-bit K/V read in place: byte offsets, inside a stage, of the lane's K operand of k-step s (key l32
  // of the wave's 32, bytes 16 s + 8 hh of its row) and of its share of the byte transpose read for
  // d block d (row = L16 >> 1 of the 8 x 16 byte matrix is key 4 hh + (row & 3) + 8 (row >> 2), as the
  // probabilities' operand layout pairs them; columns are bytes 32 d + 16 grp1 ...), with the slot
  // permutation the loads apply inside each 1 KiB piece
  int koff8[NS], voff8[ND];
  if constexpr (C::KV8_REG) {
    // piece n of the tile (keys 8 n .. 8 n + 7) was loaded by wave n / NLDK as its piece n % NLDK: its K bytes
    // sit in that wave's zone, its V bytes NLDK pieces further on
    static_assert(!C::KV8_REG || (NLDK % 2 == 0), "the slot permutation's parity bit is the piece's index in its wave's zone");
    auto piece_off = [&](int n) __attribute__((always_inline)) { return ((n / NLDK) * 2 * NLDK + n % NLDK) * 1024; };
    const int kn = wk * 4 + (l32 >> 3), kr = l32 & 7;
#pragma unroll
    for (int s2 = 0; s2 < NS; ++s2) koff8[s2] = piece_off(kn) + ((kr * 8 + (s2 ^ kr ^ (kn & 1))) << 4) + 8 * hh;
    const int row = L16 >> 1, vn = wk * 4 + (row >> 2), vr = 4 * hh + (row & 3);
#pragma unroll
    for (int d = 0; d < ND; ++d)
      voff8[d] = piece_off(vn) + NLDK * 1024 + ((vr * 8 + ((2 * (d ^ (wk * (ND / 2))) + grp1) ^ vr ^ (vn & 1))) << 4) + 8 * (L16 & 1);
  }
  constexpr int V8_SECOND = (NLDK >= 4 ? 2 : 2 * NLDK) * 1024;  // keys 16 .. 31 of the wave: two pieces further on

  auto use_reference = [&](int r) __attribute__((always_inline)) { m_use[r] = (m_run[r] == -INFINITY) ? 0.f : m_run[r]; };
  auto set_cap = [&](int r) __attribute__((always_inline)) { cap[r] = (m_run[r] == -INFINITY) ? -1.f : kLazyCap; };
  // moves row r's reference up to a block's maximum and rescales what was summed against the old one
  auto move_reference = [&](int r, float mx) __attribute__((always_inline)) {
    const float m_new = fmaxf(m_run[r], mx);
    const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2(m_run[r] - m_new);
    m_run[r] = m_new;
    l_run[r] *= alpha;
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[r][d][i] *= alpha;
  };
  // ---- one 32-key block of one tile: S^T = K Q^T, online softmax, O^T += V^T P^T ----
  auto compute_block = [&](const lds_byte *stage, auto kb_tag, int base, int limit, bool tree, auto masked_tag, auto settled_tag, auto &&refill) __attribute__((always_inline)) {
    constexpr bool AHEAD = C::AHEAD;
    constexpr bool MASKED = decltype(masked_tag)::value, SETTLED = decltype(settled_tag)::value;
    constexpr int kb = decltype(kb_tag)::value;
    constexpr int KBOFF = kb * (32 / NBLK) * ROWB;     // this 32-key block inside the wave's part of the tile
    constexpr int V8 = (NBLK == 16) ? 8 * PV : ROWB;   // V rows 8 keys further on
    const int kofs = (wk * KBW + kb) * 32;
    const lds_byte *kp = stage + kbase_off + KBOFF;
    const uint32_t va = (uint32_t)(uintptr_t)(stage + vbase_off), va_kept = va + (uint32_t)kept0 * 2u, va_other = va + (uint32_t)other0 * 2u;
    f32x16 sacc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int i = 0; i < 16; ++i) sacc[r][i] = 0.f;
    const uint32_t sb8 = (uint32_t)(uintptr_t)stage;  // (8-bit K/V read in place)
    if constexpr (C::KV8_REG) {
      static_assert(!C::KV8_REG || (NS == 8 && ND == 4 && KBW == 1), "8-bit K/V in place: D = 128, one block per wave and tile");
      u32x2 kraw[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) kraw[s] = lds_read_b64(sb8 + koff8[s]);
      lds_wait(kraw[0], kraw[1], kraw[2], kraw[3]);
      lds_wait(kraw[NS - 4], kraw[NS - 3], kraw[NS - 2], kraw[NS - 1]);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const bf16x8 ka = widen_e4m3(kraw[s]);
#pragma unroll
        for (int r = 0; r < RB; ++r)
          sacc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[r][s], sacc[r], 0, 0, 0);
      }
    } else if constexpr (!AHEAD) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bf16x8 ka = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>(kp + s * 32);
#pragma unroll
      for (int r = 0; r < RB; ++r)
        sacc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[r][s], sacc[r], 0, 0, 0);
    }
    }
    // V^T operands of the first 16 keys: in flight during the softmax arithmetic
    auto v_at = [&](int d) __attribute__((always_inline)) { return !C::PAIR ? va + d * 64 : d < ND / 2 ? va_kept + d * 64 : va_other + (d - ND / 2) * 64; };
    s16x4 vlo[2][ND], vhi[2][ND];
    u32x2 vraw[2][ND];  // (8-bit K/V read in place: one byte transpose read per operand)
    constexpr int S2OFF = (16 / NBLK) * ROWB;
    if constexpr (AHEAD) {
      // (behind the K operand waited for: those after it and as many reads of V as K operands have been used, NS - 1 in all)
      const uint32_t kp0 = (uint32_t)(uintptr_t)kp;
      bf16x8 ka[NS];
      static_for<NS>([&](auto s_tag) __attribute__((always_inline)) { lds_read_k<decltype(s_tag)::value * 32>(ka[decltype(s_tag)::value], kp0); });
      static_for<NS>([&](auto s_tag) __attribute__((always_inline)) {
        constexpr int s = decltype(s_tag)::value, d = s / 2;
        lds_wait_n<NS - 1>(ka[s]);
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qreg[0][s], s == 0 ? f32x16{} : sacc[0], 0, 0, 0);
        if constexpr (s % 2 == 0) lds_read_v<KBOFF>(vlo[0][d], v_at(d));
        else lds_read_v<KBOFF + V8>(vhi[0][d], v_at(d));
        refill(s_tag);
        __builtin_amdgcn_sched_barrier(0);
      });
      static_for<ND>([&](auto d_tag) __attribute__((always_inline)) {
        constexpr int d = decltype(d_tag)::value;
        lds_read_v<KBOFF + S2OFF>(vlo[1][d], v_at(d));
        lds_read_v<KBOFF + S2OFF + V8>(vhi[1][d], v_at(d));
      });
    }
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      if constexpr (AHEAD) {
      } else if constexpr (C::KV8_REG) {
        vraw[0][d] = lds_read_tr8(sb8 + voff8[d]);
      } else {
        vlo[0][d] = lds_read_tr<KBOFF + 0>(v_at(d));
        vhi[0][d] = lds_read_tr<KBOFF + V8>(v_at(d));
      }
    }
    // the V^T operand of the PV product over keys 16 s2 .. 16 s2 + 15, d block d
    auto v_operand = [&](int s2, int d) __attribute__((always_inline)) {
      if constexpr (C::KV8_REG) return widen_e4m3(vraw[s2][d]);
      else return __builtin_bit_cast(bf16x8, __builtin_shufflevector(vlo[s2][d], vhi[s2][d], 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // bit i of ok[r]: element i of this lane (key base+kofs+8*(i/4)+4*hh+i%4) may be attended
    unsigned ok[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      ok[r] = 0xFFFFu;
      if (MASKED) {
        ok[r] = 0;
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
          const int p0 = base + kofs + 8 * qd + 4 * hh;  // first of 4 consecutive keys
          unsigned nib;
          if (tree) {
            // bits at or above T_b can never be keys
            const int nbits = limit - (p0 & ~63);
            const uint64_t trim = nbits >= 64 ? ~0ull : nbits <= 0 ? 0ull : (1ull << nbits) - 1;
            const uint64_t mw = ((p0 < 64) ? mrow[r][0] : mrow[r][1]) & trim;
            nib = (unsigned)(mw >> (p0 & 63)) & 0xFu;
          } else {
            const int left = limit - p0;
            nib = left >= 4 ? 0xFu : (left <= 0 ? 0u : ((1u << left) - 1u));
          }
          ok[r] |= nib << (4 * qd);
        }
      }
    }
    bf16x8 pb[2][RB];
    uint64_t lo_votes = 0;
    if constexpr (!SETTLED) {
      bool need_lo = false;
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        float sv[16];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          sv[i] = sacc[r][i];
          if (MASKED) sv[i] = ((ok[r] >> i) & 1u) ? sv[i] : -INFINITY;
          mx = fmaxf(mx, sv[i]);
        }
        mx = half_max(mx) * p.scale_log2;
        // lazy reference update: only when some row's tile maximum exceeds its reference by > 2^kLazy
        if (__builtin_amdgcn_ballot_w64(mx > m_run[r] + kLazy) != 0) {
          move_reference(r, mx);
          if (C::KEEP_USE) use_reference(r);
        }
        if (!C::KEEP_USE) use_reference(r);
        float ls = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float pv = fast_exp2(fmaf(sv[i], p.scale_log2, -m_use[r]));
          ls += pv;
          pb[i / 8][r][i % 8] = (__bf16)pv;
        }
        l_run[r] += ls;
        need_lo = need_lo || (fast_exp2(mx - m_use[r]) > kLoThreshold * half_sum(l_run[r]));
      }
      lo_votes = __builtin_amdgcn_ballot_w64(need_lo);
    } else {
      // The steady part of a long split: probabilities against the reference as it stands.  What the maximum of the block
      // would be needed for -- moving the reference, the low-order pass -- is ruled out by the lane's sum of the block's 16
      // probabilities, which bounds each of them: a sum up to 2^kLazy keeps the reference, a sum up to kLoThreshold of the
      // lane's own running sum (a part of the row's) excludes a weight that large.  After the first few blocks of a split
      // that holds for every lane, and the maximum, its exchange between the lane halves and its exponential are not
      // computed at all.
      static_assert(!MASKED, "full tiles");
      float ls[RB];
      auto exponentials = [&](int r) __attribute__((always_inline)) {
        ls[r] = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float pv = fast_exp2(fmaf(sacc[r][i], p.scale_log2, -m_use[r]));
          ls[r] += pv;
          pb[i / 8][r][i % 8] = (__bf16)pv;
        }
      };
      bool look = false;
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        exponentials(r);
        look = look || !(ls[r] <= fminf(kLoThreshold * (l_run[r] + ls[r]), cap[r]));
      }
      if (__builtin_amdgcn_ballot_w64(look) != 0) {
        bool need_lo = false;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          float mx = -INFINITY;
#pragma unroll
          for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[r][i]);
          mx = half_max(mx) * p.scale_log2;
          if (__builtin_amdgcn_ballot_w64(mx > m_run[r] + kLazy) != 0) {
            move_reference(r, mx);
            use_reference(r);
            set_cap(r);
            exponentials(r);
          }
          need_lo = need_lo || (fast_exp2(mx - m_use[r]) > kLoThreshold * half_sum(l_run[r] + ls[r]));
        }
        lo_votes = __builtin_amdgcn_ballot_w64(need_lo);
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) l_run[r] += ls[r];
    }
    // O^T += V^T P^T: first 16 keys while the operands of the second 16 arrive
    static_assert(ND == 4 || ND == 2, "head dimension 128 or 64");
    if constexpr (C::KV8_REG) lds_wait(vraw[0][0], vraw[0][1], vraw[0][ND - 2], vraw[0][ND - 1]);
    else if constexpr (ND == 4) lds_wait(vlo[0][0], vlo[0][1], vlo[0][2], vlo[0][3]), lds_wait(vhi[0][0], vhi[0][1], vhi[0][2], vhi[0][3]);
    else lds_wait(vlo[0][0], vlo[0][1], vhi[0][0], vhi[0][1]);
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      if constexpr (AHEAD) {
      } else if constexpr (C::KV8_REG) {
        vraw[1][d] = lds_read_tr8(sb8 + voff8[d] + V8_SECOND);
      } else {
        vlo[1][d] = lds_read_tr<KBOFF + S2OFF>(v_at(d));
        vhi[1][d] = lds_read_tr<KBOFF + S2OFF + V8>(v_at(d));
      }
    }
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const bf16x8 vop = v_operand(0, d);
#pragma unroll
      for (int r = 0; r < RB; ++r)
        oacc[r][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop, pb[0][r], oacc[r][d], 0, 0, 0);
    }
    if constexpr (C::KV8_REG) lds_wait(vraw[1][0], vraw[1][1], vraw[1][ND - 2], vraw[1][ND - 1]);
    else if constexpr (ND == 4) lds_wait(vlo[1][0], vlo[1][1], vlo[1][2], vlo[1][3]), lds_wait(vhi[1][0], vhi[1][1], vhi[1][2], vhi[1][3]);
    else lds_wait(vlo[1][0], vlo[1][1], vhi[1][0], vhi[1][1]);
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const bf16x8 vop = v_operand(1, d);
#pragma unroll
      for (int r = 0; r < RB; ++r)
        oacc[r][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop, pb[1][r], oacc[r][d], 0, 0, 0);
    }
    // low-order pass (rare): the bf16 rounding remainder of P, recomputed from the scores
    if (lo_votes != 0) {
      bf16x8 plo[2][RB];
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          float sv = sacc[r][i];
          if (MASKED) sv = ((ok[r] >> i) & 1u) ? sv : -INFINITY;
          const float pv = fast_exp2(fmaf(sv, p.scale_log2, -m_use[r]));
          plo[i / 8][r][i % 8] = (__bf16)(pv - (float)pb[i / 8][r][i % 8]);
        }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int d = 0; d < ND; ++d) {
          const bf16x8 vop = v_operand(s2, d);
#pragma unroll
          for (int r = 0; r < RB; ++r)
            oacc[r][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop, plo[s2][r], oacc[r][d], 0, 0, 0);
        }
    }
  };

  // ---- wait until this wave's loads of tile `it` (and, paged, the table entries the tile queued
  // next needs) have landed: all but the operations queued after them are complete ----
  auto wait_tile = [&](int it) __attribute__((always_inline)) {
    constexpr int OPS = C::TILE_OPS;
    const int later = n_tiles - 1 - it;  // tiles after `it` whose loads are already queued: min(later, PD - 1)
    if constexpr (PAGED) {
      // queued after the loads of tile `it`: entries(it+LOOK), then per later tile its loads and the entries LOOK
      // tiles on.  entries(it+PD) are needed next: they came no later than the first of those.
      if (PD >= 3 && later >= 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(OPS * 2));
      else if (PD >= 2 && later >= 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(OPS));
      else if (PD == 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::NPG));
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    } else {
      if (PD >= 3 && later >= 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NLD * 2));
      else if (PD >= 2 && later >= 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NLD * 1));
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    }
  };

  // ---- 8-bit K/V widened through LDS: this wave's pieces of tile j, once landed, are widened to bf16 into
  // stage j % NSTAGE, and the landing slot they leave takes the loads of tile j + NL.  A lane widens the 16 bytes it
  // loaded itself (row row0_of(jj) + lsub, 16 head-dimension elements from 16 * lpos): 32 bytes of bf16 ----
  auto land_tile = [&](int j) __attribute__((always_inline)) {
    if constexpr (KV8 && !C::KV8_REG) {
      wait_tile(j);
      const uint32_t land = (uint32_t)(uintptr_t)(lds + C::LAND_OFF + (j % C::NL) * C::LAND_SLOT) + lane * 16;
      lds_byte *stage = lds + (j % NSTAGE) * STAGE_BYTES;
#pragma unroll
      for (int jj = 0; jj < NLDK; ++jj) {
        u32x4 kraw = lds_read_b128(land + kdst_of(jj));
        u32x4 vraw = lds_read_b128(land + vdst_of(jj));
        lds_wait(kraw, vraw);
        const int r = row0_of(jj) + lsub;
        const int at = (r / NBLK) * ROWB + lpos * 32;
        bf16x8 lo, hi;
        widen_e4m3(kraw, lo, hi);
        auto *kd = reinterpret_cast<__attribute__((address_space(3))) bf16x8 *>(stage + (r % NBLK) * PK + at);
        kd[0] = lo;
        kd[1] = hi;
        widen_e4m3(vraw, lo, hi);
        auto *vd = reinterpret_cast<__attribute__((address_space(3))) bf16x8 *>(stage + KTILE + (r % NBLK) * PV + at);
        vd[0] = lo;
        vd[1] = hi;
      }
      asm volatile("" ::: "memory");  // the slot is refilled below this line, not above
      if (j + PD < n_tiles) issue_tile(j + PD);
    }
  };

  auto no_refill = [](auto) __attribute__((always_inline)) {};
  auto compute_tile = [&](int it, bool tree, auto masked_tag, auto &&refill) __attribute__((always_inline)) {
    const int base = tree ? (it - n_ct) * TK : k0 + it * TK;
    const int limit = tree ? Tb : k1;
    const lds_byte *stage = lds + (it % NSTAGE) * STAGE_BYTES;
    static_assert(KBW <= 2, "");
    // wave-uniform: a block is skipped when none of its keys exists, and all of them by a wave
    // none of whose query rows exists (it still loads its share of every tile)
    if (!wave_has_rows) return;
    if (base + wk * KBW * 32 < limit) compute_block(stage, std::integral_constant<int, 0>{}, base, limit, tree, masked_tag, std::false_type{}, refill);
    if constexpr (KBW > 1)
      if (base + (wk * KBW + 1) * 32 < limit) compute_block(stage, std::integral_constant<int, 1>{}, base, limit, tree, masked_tag, std::false_type{}, refill);
  };

  // ---- one pipeline step: wait for tile `it`, refill the stage tile it-1 used, compute ----
  auto step = [&](int it, auto masked_tag, auto tree_tag) __attribute__((always_inline)) {
    if constexpr (KV8 && !C::KV8_REG) {
      // everyone's widened part of tile `it` is in LDS (the wait covers this wave's LDS writes);
      // everyone is done with tile it-1, whose stage tile it+1 is widened into next
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      if (it + 1 < n_tiles) land_tile(it + 1);
    } else {
    // this wave's loads of tile `it` have landed once at most the later tiles' loads are outstanding
    wait_tile(it);
    // everyone's part of tile `it` is in LDS; everyone is done with tile it-1 (no barrier where a wave
    // reads only the bytes it loaded itself)
    if (!(C::KV8_REG && WM == 1)) __builtin_amdgcn_s_barrier();
    if (it + PD < n_tiles) issue_tile(it + PD);
    }
    compute_tile(it, decltype(tree_tag)::value, masked_tag, no_refill);
  };

  // ---- the pipelined loop's loads: K and V of a tile apart ----
  constexpr int LEAD = C::LEAD, KOPS = NLDK + C::NPG;
  const bool piped = C::PIPED && n_full >= (R > BM ? C::PIPE_TILES_ROWS : C::PIPE_TILES) && (PAGED ? small_pages : tok_bytes < (1 << 26)) &&
                     (int64_t)p.Hkv * D * EB < (1 << 26);  // (a tile's rows are within 32 bits; the entry points take tokens up to 32 MiB apart)
  const bool tree_apart = p.k_tree != nullptr;
  // full cache tiles.  Dense: an address per operand, carried along from tile to tile in scalar registers, and the lane's offset
  const int64_t tile_bytes = (int64_t)TK * p.stride_tok * EB;
  const char *k_next = kc_bytes + (cache_base + (int64_t)k0 * p.stride_tok) * EB;
  const char *v_next = vc_bytes + (cache_base + (int64_t)k0 * p.stride_tok) * EB;
  // Paged: a multiply-add on the number of each row's page, for K; V of that tile, queued next, takes the same offsets.
  uint64_t row_at[NLDK];
  auto issue_full = [&](int t, auto v_tag) __attribute__((always_inline)) {
    constexpr bool V = decltype(v_tag)::value;
    lds_byte *stage = lds + (t & (NSTAGE - 1)) * STAGE_BYTES;
    const char *&next = V ? v_next : k_next;
#pragma unroll
    for (int j = 0; j < NLDK; ++j) {
      const char *src = next + lane_off[j];
      if constexpr (PAGED) {
        if constexpr (!V) row_at[j] = small_off(page_of(t, tile_row(j)), k0 + t * TK + tile_row(j), j);
        src = (V ? vc_bytes : kc_bytes) + row_at[j];
      }
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(src), stage + (V ? vdst_of(j) : kdst_of(j)), 16, 0, kLoadOnce);
    }
    if constexpr (!PAGED) next += tile_bytes;
    if constexpr (!V) request_pages(t + C::LOOK, std::integral_constant<int, 1>{});
  };
  // the partial cache tile and the tree's
  auto issue_rest = [&](int t, auto v_tag) __attribute__((always_inline)) {
    constexpr bool V = decltype(v_tag)::value;
    const bool tree = t >= n_ct, apart = tree && tree_apart;
    const int first_key = tree ? (t - n_ct) * TK : k0 + t * TK, last = (tree ? Tb : k1) - 1 - first_key;
    const int pos0 = tree ? Lb0 + first_key : first_key;
    lds_byte *stage = lds + (t & (NSTAGE - 1)) * STAGE_BYTES;
    const char *base = V ? vc_bytes : kc_bytes;
    uint32_t stride = (uint32_t)tok_bytes;
    if (apart) {
      const const_args late = late_args();
      base = reinterpret_cast<const char *>(V ? late->v_tree : late->k_tree) + ((int64_t)(t0 + first_key) * late->Hkv + kvh) * (D * EB);
      stride = (uint32_t)(late->Hkv * D * EB);
    }
    if (!PAGED && !apart) base += (cache_base + (int64_t)pos0 * p.stride_tok) * EB;
#pragma unroll
    for (int j = 0; j < NLDK; ++j) {
      if constexpr (!V || !PAGED) {
        const int row_in = row0_of(j) + lrow, row = row_in < last ? row_in : last;
        row_at[j] = (__umul24((uint32_t)row, stride >> 4) + (uint32_t)chunk_of(j)) << 4;  // (strides are multiples of 16 bytes)
        if constexpr (PAGED)
          if (!apart) row_at[j] = small_off(page_of(t, row_in), pos0 + row, j);
      }
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(base + row_at[j]), stage + (V ? vdst_of(j) : kdst_of(j)), 16, 0, kLoadOnce);
    }
    if constexpr (!V) request_pages(t + C::LOOK, std::integral_constant<int, 2>{});
  };
  auto issue_k = [&](int t) __attribute__((always_inline)) { issue_full(t, std::false_type{}); };
  auto issue_v = [&](int t) __attribute__((always_inline)) { issue_full(t, std::true_type{}); };

  // No ancestor masks passed: the tree's parent array goes to LDS (by the first two waves, with the
  // same LDS-writing loads as everything else here, so it is covered by the counted wait below).
  const bool derive_masks = has_tree && p.mask == nullptr;
  if (derive_masks && wave < 2) {
    int idx = wave * 64 + lane;
    idx = idx < Tb ? idx : Tb - 1;
    __builtin_amdgcn_global_load_lds(GLOBAL_PTR(p.parent + t0 + idx), lds + C::PARENT_OFF + wave * 256, 4, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < C::LOOK; ++t) request_pages(t, std::false_type{});
  // The first PD tiles (fewer if the chunk has fewer).  Q and the mask rows were requested before
  // them and have arrived once no more than the tiles' own operations are outstanding; that wait
  // sits in the same branch as the loads it counts, so that the number is plainly a constant.
  auto issue_first = [&](auto n_tag) __attribute__((always_inline)) {
    constexpr int n = decltype(n_tag)::value;
#pragma unroll
    for (int t = 0; t < n; ++t) {
      if constexpr (PAGED) {
        // entries(t) have landed once only what was queued after them is outstanding
        if (t == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::NPG * (C::LOOK - 1)));
        else if (t == 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::NPG * (C::LOOK - 2) + C::TILE_OPS));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::TILE_OPS * 2));
        asm volatile("" ::: "memory");  // the entries are read from LDS below this line, not above
      }
      issue_tile(t);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(vm_cap(C::LOOK * C::NPG + C::TILE_OPS * n)));
  };
  if (C::PIPED && piped) {
    // K of the first NSTAGE tiles and V of one less, in the order in which the loop queues them
    auto entries = [&](auto n_tag) __attribute__((always_inline)) {
      if constexpr (PAGED) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(decltype(n_tag)::value));
        asm volatile("" ::: "memory");  // the entries are read from LDS below this line, not above
      }
    };
    entries(std::integral_constant<int, 2 * C::NPG>{});
    issue_k(0);
    if constexpr (KBW == 2) issue_v(0);
    entries(std::integral_constant<int, C::NPG + KOPS + (KBW == 2 ? NLDK : 0)>{});
    issue_k(1);
    // Q and the mask rows are waited for here, before the rest: queueing 112 KB takes longer than they do
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(vm_cap(C::LOOK * C::NPG + 2 * KOPS + (KBW == 2 ? NLDK : 0))));
    if constexpr (KBW == 1) issue_v(0);
    else issue_v(1);
    entries(std::integral_constant<int, 2 * KOPS + (KBW == 2 ? 2 : 1) * NLDK>{});
    issue_k(2);
    if constexpr (KBW == 1) issue_v(1);
    else issue_v(2);
    entries(std::integral_constant<int, 2 * KOPS + 2 * NLDK>{});
    issue_k(3);
    if constexpr (KBW == 1) issue_v(2);
  } else if (PD >= 3 && n_tiles >= 3) issue_first(std::integral_constant<int, PD >= 3 ? 3 : 1>{});
  else if (PD >= 2 && n_tiles >= 2) issue_first(std::integral_constant<int, PD >= 2 ? 2 : 1>{});
  else issue_first(std::integral_constant<int, 1>{});
  if (derive_masks) {
    // Every wave has waited for its own loads queued before the tiles; after the barrier the parent
    // array is complete.  Each lane walks from its node to the root (paper, Tree Reranking Phase:
    // a token attends to its ancestors; and to itself), at most T_b steps whatever the array holds.
    // (A bare barrier: the fenced one would wait for the tiles in flight too.)
    __builtin_amdgcn_s_barrier();
    const auto *par = reinterpret_cast<const __attribute__((address_space(3))) int32_t *>(lds + C::PARENT_OFF);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int row = rblk * BM + (wm * RB + r) * 32 + l32;
      const int rowc = row < R ? row : R - 1;
      int node = node_off + node_of(p, rowc);
      uint64_t b0 = 0, b1 = 0;
      for (int step = 0; step < Tb && node >= 0; ++step) {
        if (node < 64) b0 |= 1ull << node;
        else b1 |= 1ull << (node - 64);
        // (read through inline assembly: an ordinary LDS load of memory an LDS-writing load filled
        // makes the compiler drain every outstanding load first, the prefetched tiles included)
        int up;
        asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(up) : "v"((uint32_t)(uintptr_t)(par + node)));
        node = up < node ? up : -1;  // a link that does not point backwards ends the walk
      }
      mrow[r][0] = b0;
      mrow[r][1] = b1;
    }
  }
  if constexpr (KV8 && !C::KV8_REG) land_tile(0);
  int it = 0;
  TL_STAMP(2);  // Q and the mask rows have arrived, the first tiles are in flight
#ifdef TVA_TIMELINE
  if (n_full > 0 && !piped) {
    step(0, std::false_type{}, std::false_type{});
    it = 1;
  }
  TL_STAMP(3);  // first full tile done (a split without one: the same moment as the stamp before; the pipelined loop stamps it anew)
#endif
  if constexpr (C::PIPED) {
    if (piped) {
      // ---- the full tiles as a software pipeline over 32-key blocks.  A step computes the scores of the next block, the
      // probabilities of this one and the output of the one before, a matrix instruction of each product and two probabilities per
      // lane at a time, with their operands read from LDS four such groups ahead: the matrix unit has work while the vector ALUs
      // exponentiate, whatever the SIMD's other wave is at.  K is fetched LEAD tiles further ahead than V, whose place it would
      // else wait for.  The partial cache tile and the tree's are queued from here as well.
      // (Per tile with 8 workgroups on the chip, without -> with: deep 64-row shape 0.97 -> 0.69 us, 128-row shape 0.95 -> 0.71,
      // 256-row shape, which had a pipeline for its middle tiles, 1.17 -> 1.16.  With 256 workgroups the chip's power bounds the two
      // large shapes: 8 sequences of 4096 keys, 64 heads, spend 17 % fewer cycles in the loop at 9 % less clock, 57.8 -> 56.4 us; 32 of
      // 2048 keys, 60 nodes, 7 % fewer, 82.4 -> 80.3.  16 of 512 .. 2048 keys, 16 nodes, deep 64-row shape: 29.8 -> 28.0.) ----
      static_assert(!C::PIPED || (RB == 1 && NS == 8 && ND == 4 && KBW <= 2), "");
      constexpr int V8 = 8 * PV, S2OFF = ROWB, BLK = KBW == 2 ? 2 * ROWB : 0;
      // In tile t: K of tile t + LEAD - 1 and V of tile t - 1 have been read everywhere, so their places take K and V of NSTAGE tiles
      // later, where those exist.  And what is read from here on has landed everywhere: with two blocks per tile K of tile t + 2 and V of
      // tile t + 1; with one K of tile t + 2 and V of tile t, whose first reads stand right behind.  So three tiles are in flight there, as
      // in the plain loop.  (One group later, behind those reads, each had to land a tile earlier: two in flight, and calls of the
      // 128-row shape bound by their reads took up to 10 % longer than in the plain loop.)
      static_assert(!C::PIPED || NSTAGE == 4, "");
      auto enter = [&](int t) __attribute__((always_inline)) {
        // (two blocks: but for the reads since those of the K and V given up)
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(KBW == 1 ? 0 : 6) : "memory");
        const int left = n_tiles - t;
        if (__builtin_expect(n_full - t > 3 + LEAD, 1)) {
          __builtin_amdgcn_s_waitcnt(vmcnt_imm((KBW == 1 ? 2 : 1) * C::TILE_OPS));
          __builtin_amdgcn_s_barrier();
          issue_v(t + 3);
          issue_k(t + 3 + LEAD);
        } else {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          if constexpr (KBW == 1) {  // queued behind them: V(t+1) K(t+3) V(t+2) K(t+4), where those exist
            if (left > 4) __builtin_amdgcn_s_waitcnt(vmcnt_imm(4 * NLDK));
            else if (left == 4) __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * NLDK));
            else if (left == 3) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * NLDK));
            else if (left == 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NLDK));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
          } else {  // V(t+2) K(t+3)
            if (left > 2 + LEAD) __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::TILE_OPS));
            else if (left > 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NLDK));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
          }
          __builtin_amdgcn_s_barrier();
          if (t + 3 < n_full) issue_v(t + 3);
          else if (left > 3) issue_rest(t + 3, std::true_type{});
          if (left > 3 + LEAD) issue_rest(t + 3 + LEAD, std::false_type{});
        }
      };
      // (two blocks) in the first tile, ahead of the first read of its V and of K of the next one
      auto first_landed = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * KOPS + 2 * NLDK));
        __builtin_amdgcn_s_barrier();
      };
      // -- arithmetic --
      bf16x8 kr[4];           // K operands: four of the next block's eight
      s16x4 vl[4], vh[4];     // V^T operands: four of the eight of the block before
      f32x16 sA, sB;          // scores of the blocks, in turn
      bf16x8 pA[2], pB[2];    // their probabilities
#pragma unroll
      for (int i = 0; i < 4; ++i) vl[i] = vh[i] = s16x4{0, 0, 0, 0};
      // Waits for all of them; what follows takes them as written here.  Until its wait the compiler takes such a register as written
      // although the value is still to come, so nothing but a straight line, the groups below and (with two blocks per tile) the barrier of a
      // tile that queues full tiles may stand between a read and its wait: every other way on starts with this one, and every loop is
      // entered and left at one place.
      // (A loop over pairs of blocks that could be left between the two had its operands in other registers on either way out: a
      // statement on one of them, and they were copied and spilled in flight.)
      auto settle_reads = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(kr[0]), "+v"(kr[1]), "+v"(kr[2]), "+v"(kr[3]), "+v"(vl[0]), "+v"(vl[1]), "+v"(vl[2]), "+v"(vl[3]), "+v"(vh[0]),
                       "+v"(vh[1]), "+v"(vh[2]), "+v"(vh[3])
                     :
                     : "memory");
      };
      const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
      auto k_at = [&](int t) __attribute__((always_inline)) { return lds0 + (uint32_t)(t & (NSTAGE - 1)) * STAGE_BYTES + kbase_off; };
      auto v_at = [&](int t) __attribute__((always_inline)) { return lds0 + (uint32_t)(t & (NSTAGE - 1)) * STAGE_BYTES + vbase_off; };
      // (two key groups: the head dimension's halves in the accumulators' order, the kept one first)
      auto v_of = [&](uint32_t va, int d) __attribute__((always_inline)) { return !C::PAIR ? va : d < ND / 2 ? va + wk * 128 : va - wk * 128; };
      const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      auto half = [&](auto &&f, auto second_tag) __attribute__((always_inline)) {
        constexpr int g0 = decltype(second_tag)::value ? 4 : 0;
        f(std::integral_constant<int, g0>{}), f(std::integral_constant<int, g0 + 1>{});
        f(std::integral_constant<int, g0 + 2>{}), f(std::integral_constant<int, g0 + 3>{});
      };
      auto pv = [&](int d, const bf16x8 &pr) __attribute__((always_inline)) {
        oacc[0][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, __builtin_shufflevector(vl[d], vh[d], 0, 1, 2, 3, 4, 5, 6, 7)), pr, oacc[0][d], 0, 0, 0);
      };
      auto pack = [&](float a, float b) __attribute__((always_inline)) {
        const bf16x2 pair = {(__bf16)a, (__bf16)b};
        return __builtin_bit_cast(uint32_t, pair);
      };
      // what two probabilities lost when they were rounded to w
      auto pack_rest = [&](float a, float b, uint32_t w) __attribute__((always_inline)) {
        return pack(a - __uint_as_float(w << 16), b - __uint_as_float(w & 0xFFFF0000u));
      };
      auto operands = [&](const uint32_t (&w)[8], bf16x8 (&out)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s) out[s] = __builtin_bit_cast(bf16x8, u32x4{w[4 * s], w[4 * s + 1], w[4 * s + 2], w[4 * s + 3]});
      };
      // a bound of a lane's largest probability of a block: of the rounded ones, which are not negative, the largest as 16-bit
      // integers, and what rounding can have taken off it
      auto largest = [&](const uint32_t (&w)[8]) __attribute__((always_inline)) {
        typedef short s16x2 __attribute__((ext_vector_type(2)));
        s16x2 top = __builtin_bit_cast(s16x2, w[0]);
#pragma unroll
        for (int i = 1; i < 8; ++i) top = __builtin_elementwise_max(top, __builtin_bit_cast(s16x2, w[i]));
        return __uint_as_float((uint32_t)(uint16_t)(top[0] > top[1] ? top[0] : top[1]) << 16) * (1.f + 1.f / 256);
      };
      auto block_max = [&](const f32x16 &sc) __attribute__((always_inline)) {
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[i]);
        return half_max(mx) * p.scale_log2;
      };
      // moves the reference if a block's maximum asks for it
      auto settle_reference = [&](float mx) __attribute__((always_inline)) {
        if (__builtin_amdgcn_ballot_w64(mx > m_run[0] + kLazy) == 0) return false;
        move_reference(0, mx);
        use_reference(0);
        set_cap(0);
        return true;
      };
      // group g of a step: K operand g of the next block, two of this block's probabilities, the read of K operands four groups on
      // (of the next block, or the first ones of the block after it)
      auto group_head = [&](auto g_tag, auto wait_tag, const f32x16 &cur, f32x16 &nxt, uint32_t ka1, uint32_t ka2, auto kb_tag, float &e0, float &e1, auto &&middle) __attribute__((always_inline)) {
        constexpr int g = decltype(g_tag)::value, d = g % 4, kb = decltype(kb_tag)::value;
        lds_wait_n<decltype(wait_tag)::value>(kr[d], vl[d], vh[d]);
        nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[d], qreg[0][g], g == 0 ? zero16 : nxt, 0, 0, 0);
        e0 = fast_exp2(fmaf(cur[2 * g], p.scale_log2, -m_use[0]));
        e1 = fast_exp2(fmaf(cur[2 * g + 1], p.scale_log2, -m_use[0]));
        if constexpr (g == 4) middle();
        if constexpr (g < 4) lds_read_k<(1 - kb) * BLK + (g + 4) * 32>(kr[d], ka1);
        else lds_read_k<kb * BLK + (g - 4) * 32>(kr[d], ka2);
        __builtin_amdgcn_sched_barrier(0);
      };
      // what a block hands to the step after it: its probabilities, rounded, and (the first blocks, whose weights are large against
      // what has been summed) what rounding took off them
      uint32_t hA[8], hB[8], rA[8], rB[8];
      bool rest = false;  // ... which is wanted
      // the step of one of the first blocks.  ka1, ka2: where K of the next block and of the one after it are, va1, va2: V of the block
      // before and of this one
      auto block_lo = [&](f32x16 &cur, f32x16 &nxt, uint32_t (&hc)[8], uint32_t (&rc)[8], uint32_t (&hp)[8], uint32_t (&rp)[8],
                          uint32_t ka1, uint32_t ka2, uint32_t va1, uint32_t va2, auto kb_tag, auto pv_tag, auto &&middle, auto &&after) __attribute__((always_inline)) {
        constexpr int kb = decltype(kb_tag)::value, HERE = kb * BLK, THERE = (1 - kb) * BLK;
        constexpr bool HASPV = decltype(pv_tag)::value;
        float ls = 0.f;
        bf16x8 pp[2], pr[2];
        if constexpr (HASPV) operands(hp, pp), operands(rp, pr);
        auto group = [&](auto g_tag) __attribute__((always_inline)) {
          constexpr int g = decltype(g_tag)::value, d = g % 4;
          float e0, e1;
          // (three reads a group; of K alone before the first)
          group_head(g_tag, std::integral_constant<int, HASPV ? 9 : g < 4 ? 3 : 3 + 2 * d>{}, cur, nxt, ka1, ka2, kb_tag, e0, e1, middle);
          if constexpr (HASPV) pv(d, pp[g / 4]);
          ls += e0;
          ls += e1;
          hc[g] = pack(e0, e1);
          rc[g] = pack_rest(e0, e1, hc[g]);
          asm volatile("" : "+v"(hc[g]), "+v"(rc[g]), "+v"(ls));  // (computed here, not where it is used)
          if constexpr (HASPV)
            if (rest) pv(d, pr[g / 4]);
          if constexpr (g >= 4) {
            lds_read_v<HERE + d * 64>(vl[d], v_of(va2, d));
            lds_read_v<HERE + V8 + d * 64>(vh[d], v_of(va2, d));
          } else if constexpr (HASPV) {
            lds_read_v<THERE + S2OFF + d * 64>(vl[d], v_of(va1, d));
            lds_read_v<THERE + S2OFF + V8 + d * 64>(vh[d], v_of(va1, d));
          }
          __builtin_amdgcn_sched_barrier(0);
          after(g_tag);
        };
        half(group, std::false_type{});
        half(group, std::true_type{});
        asm volatile("s_waitcnt lgkmcnt(9)" ::: "memory");  // (the next step's first operands)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(ls <= cap[0])) != 0, 0)) {
          settle_reads();
          if (settle_reference(block_max(cur))) {
            ls = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const float e0 = fast_exp2(fmaf(cur[2 * i], p.scale_log2, -m_use[0])), e1 = fast_exp2(fmaf(cur[2 * i + 1], p.scale_log2, -m_use[0]));
              ls += e0;
              ls += e1;
              hc[i] = pack(e0, e1);
              rc[i] = pack_rest(e0, e1, hc[i]);
            }
          }
        }
        l_run[0] += ls;
        rest = __builtin_amdgcn_ballot_w64(!(largest(hc) <= kLoThreshold * half_sum(l_run[0]))) != 0;
      };
      // any later block's step; va1, va2: where V of the block before and of this one are
      auto block = [&](f32x16 &cur, f32x16 &nxt, bf16x8 (&pc)[2], bf16x8 (&pp)[2], uint32_t ka1, uint32_t ka2, uint32_t va1, uint32_t va2,
                       auto kb_tag, auto pv_tag, auto &&middle, auto &&after) __attribute__((always_inline)) {
        constexpr int kb = decltype(kb_tag)::value, HERE = kb * BLK, THERE = (1 - kb) * BLK;
        constexpr bool HASPV = decltype(pv_tag)::value;
        float ls = 0.f;
        uint32_t pw[8];
        auto group = [&](auto g_tag) __attribute__((always_inline)) {
          constexpr int g = decltype(g_tag)::value, d = g % 4;
          float e0, e1;
          // (three reads a group; of K alone before the first)
          group_head(g_tag, std::integral_constant<int, HASPV ? 9 : g < 4 ? 3 : 3 + 2 * d>{}, cur, nxt, ka1, ka2, kb_tag, e0, e1, middle);
          if constexpr (HASPV) pv(d, pp[g / 4]);
          ls += e0;
          ls += e1;
          pw[g] = pack(e0, e1);
          asm volatile("" : "+v"(pw[g]), "+v"(ls));
          if constexpr (g >= 4) {
            lds_read_v<HERE + d * 64>(vl[d], v_of(va2, d));
            lds_read_v<HERE + V8 + d * 64>(vh[d], v_of(va2, d));
          } else if constexpr (HASPV) {
            lds_read_v<THERE + S2OFF + d * 64>(vl[d], v_of(va1, d));
            lds_read_v<THERE + S2OFF + V8 + d * 64>(vh[d], v_of(va1, d));
          }
          __builtin_amdgcn_sched_barrier(0);
          after(g_tag);
        };
        half(group, std::false_type{});
        half(group, std::true_type{});
        operands(pw, pc);
        // (the bound of compute_block's settled form)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(ls <= fminf(kLoThreshold * (l_run[0] + ls), cap[0]))) != 0, 0)) {
          settle_reads();
          // (the scores are looked at where the rounded probabilities, against the row's sum of both lane halves, leave it open)
          const bool open = __builtin_amdgcn_ballot_w64(!(ls <= cap[0]) | !(largest(pw) <= kLoThreshold * half_sum(l_run[0] + ls))) != 0;
          const float mx = open ? block_max(cur) : -INFINITY;
          if (open && settle_reference(mx)) {
            ls = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const float e = fast_exp2(fmaf(cur[i], p.scale_log2, -m_use[0]));
              ls += e;
              pc[i / 8][i % 8] = (__bf16)e;
            }
          }
          if (open && __builtin_amdgcn_ballot_w64(fast_exp2(mx - m_use[0]) > kLoThreshold * half_sum(l_run[0] + ls)) != 0) {
            // the low-order pass of this block, at once: its V^T operands are read for it alone
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
              bf16x8 plo;
#pragma unroll
              for (int i = 0; i < 8; ++i)
                plo[i] = (__bf16)(fast_exp2(fmaf(cur[8 * s2 + i], p.scale_log2, -m_use[0])) - (float)pc[s2][i]);
#pragma unroll
              for (int d = 0; d < ND; ++d) {
                s16x4 a, c;
                const uint32_t va = v_of(va2, d) + s2 * S2OFF + d * 64;
                lds_read_v<HERE>(a, va);
                lds_read_v<HERE + V8>(c, va);
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a), "+v"(c));
                oacc[0][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, c, 0, 1, 2, 3, 4, 5, 6, 7)), plo, oacc[0][d], 0, 0, 0);
              }
            }
          }
        }
        l_run[0] += ls;
      };
      // -- the loop --
      std::integral_constant<int, 0> blk0;
      std::integral_constant<int, 1> blk1;
      // K of the first tile has landed
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * KOPS + 3 * NLDK));
      __builtin_amdgcn_s_barrier();
      if (wave_has_rows) {
        const uint32_t ka = k_at(it);
        lds_read_k<0>(kr[0], ka), lds_read_k<32>(kr[1], ka), lds_read_k<64>(kr[2], ka), lds_read_k<96>(kr[3], ka);
        auto group = [&](auto g_tag) __attribute__((always_inline)) {
          constexpr int g = decltype(g_tag)::value;
          lds_wait_n<g < 5 ? 3 : 7 - g>(kr[g % 4], vl[0], vh[0]);
          sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[g % 4], qreg[0][g], g == 0 ? zero16 : sA, 0, 0, 0);
          if constexpr (g < 4) lds_read_k<(g + 4) * 32>(kr[g % 4], ka);
          __builtin_amdgcn_sched_barrier(0);
        };
        half(group, std::false_type{}), half(group, std::true_type{});
      }
      if constexpr (KBW == 1) {
        // K of the second tile has landed, that of the first has been read everywhere (each wave has waited for its reads)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * KOPS + 3 * NLDK));
        __builtin_amdgcn_s_barrier();
        issue_k(4);
      }
      if (!wave_has_rows) {
        if constexpr (KBW == 2) first_landed();
        for (; it < n_full; ++it) enter(it);
      } else {
        const uint32_t ka = k_at(KBW == 1 ? 1 : 0);  // the second block
        lds_read_k<BLK>(kr[0], ka), lds_read_k<BLK + 32>(kr[1], ka), lds_read_k<BLK + 64>(kr[2], ka), lds_read_k<BLK + 96>(kr[3], ka);
        __builtin_amdgcn_sched_barrier(0);
        m_run[0] = block_max(sA), use_reference(0), set_cap(0);
        const auto nothing = [&]() __attribute__((always_inline)) {};
        const auto none = [&](auto) __attribute__((always_inline)) {};
        // one block per tile: ahead of the first reads from the next tile of K and from this one of V; two: in the second one
        const auto enter_here = [&]() __attribute__((always_inline)) { enter(it); };
        const auto entered = [&](auto g_tag) __attribute__((always_inline)) {
          if constexpr (decltype(g_tag)::value == 1) enter(it);
        };
        auto tile_lo = [&](f32x16 &cur, f32x16 &nxt, uint32_t (&hc)[8], uint32_t (&rc)[8], uint32_t (&hp)[8], uint32_t (&rp)[8], auto first_tag) __attribute__((always_inline)) {
          constexpr bool FIRST = decltype(first_tag)::value;
          if constexpr (KBW == 2) {
            const auto started = [&](auto g_tag) __attribute__((always_inline)) {
              if constexpr (FIRST && decltype(g_tag)::value == 3) settle_reads(), first_landed();
            };
            block_lo(cur, nxt, hc, rc, hp, rp, k_at(it), k_at(it + 1), v_at(it + 3), v_at(it), blk0, std::bool_constant<!FIRST>{}, nothing, started);
            block_lo(nxt, cur, hp, rp, hc, rc, k_at(it + 1), k_at(it + 1), v_at(it), v_at(it), blk1, std::true_type{}, nothing, entered);
          } else {
            block_lo(cur, nxt, hc, rc, hp, rp, k_at(it + 1), k_at(it + 2), v_at(it + 3), v_at(it), blk0, std::bool_constant<!FIRST>{}, enter_here, none);
          }
        };
        // the output of the last block computed; va: its V, read anew (a copy of a register whose read is in flight would be made
        // ahead of any wait)
        auto drain = [&](uint32_t va, const bf16x8 (&ph)[2], const bf16x8 (&pr)[2]) __attribute__((always_inline)) {
          settle_reads();
          s16x4 a[4], c[4];
          auto read = [&](auto g_tag) __attribute__((always_inline)) {
            constexpr int g = decltype(g_tag)::value, d = g % 4;
            lds_read_v<BLK + (g / 4) * S2OFF + d * 64>(a[d], v_of(va, d));
            lds_read_v<BLK + (g / 4) * S2OFF + V8 + d * 64>(c[d], v_of(va, d));
          };
          auto product = [&](int d, const bf16x8 &x) __attribute__((always_inline)) {
            oacc[0][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, __builtin_shufflevector(a[d], c[d], 0, 1, 2, 3, 4, 5, 6, 7)), x, oacc[0][d], 0, 0, 0);
          };
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2) {
            if (s2 == 0) half(read, std::false_type{});
            else half(read, std::true_type{});
            lds_wait(a[0], a[1], a[2], a[3]), lds_wait(c[0], c[1], c[2], c[3]);
#pragma unroll
            for (int d = 0; d < ND; ++d) product(d, ph[s2]);
            if (rest)
#pragma unroll
              for (int d = 0; d < ND; ++d) product(d, pr[s2]);
          }
        };
        auto tile = [&](f32x16 &cur, f32x16 &nxt, bf16x8 (&pc)[2], bf16x8 (&pp)[2], auto pv_tag) __attribute__((always_inline)) {
          if constexpr (KBW == 2) {
            block(cur, nxt, pc, pp, k_at(it), k_at(it + 1), v_at(it + 3), v_at(it), blk0, pv_tag, nothing, none);
            block(nxt, cur, pp, pc, k_at(it + 1), k_at(it + 1), v_at(it), v_at(it), blk1, std::true_type{}, nothing, entered);
          } else {
            block(cur, nxt, pc, pp, k_at(it + 1), k_at(it + 2), v_at(it + 3), v_at(it), blk0, pv_tag, enter_here, none);
          }
        };
        bf16x8 ph[2], pr[2];
        static_assert(!C::PIPED || C::PIPE_TILES_ROWS >= C::LO_TILES + (KBW == 2 ? 2 : 3), "every loop runs");
        if constexpr (KBW == 2) {
          tile_lo(sA, sB, hA, rA, hB, rB, std::true_type{});
          for (++it; it < C::LO_TILES; ++it) tile_lo(sA, sB, hA, rA, hB, rB, std::false_type{});
          operands(hB, ph), operands(rB, pr);
          drain(v_at(it - 1), ph, pr);
          TL_STAMP(3);  // the first tiles, with the prepared low-order pass, done
          tile(sA, sB, pA, pB, std::false_type{});
          ++it;
          do {
            tile(sA, sB, pA, pB, std::true_type{});
          } while (++it < n_full);
        } else {
          // (blocks take the two sets of registers in turn: one block more or less of the first ones leaves the others an odd number)
          static_assert(KBW == 2 || (C::LO_TILES % 2 == 0 && C::LO_TILES >= 4), "");
          tile_lo(sA, sB, hA, rA, hB, rB, std::true_type{});
          do {
            ++it, tile_lo(sB, sA, hB, rB, hA, rA, std::false_type{});
            ++it, tile_lo(sA, sB, hA, rA, hB, rB, std::false_type{});
          } while (it < C::LO_TILES - 2);
          settle_reads();
          if ((n_full & 1) != 0) {
            ++it, tile_lo(sB, sA, hB, rB, hA, rA, std::false_type{});
            settle_reads();
#pragma unroll
            for (int i = 0; i < 8; ++i) hA[i] = hB[i], rA[i] = rB[i];
            sB = sA;
          }
          operands(hA, ph), operands(rA, pr);
          drain(v_at(it), ph, pr);
          TL_STAMP(3);
          ++it, tile(sB, sA, pB, pA, std::false_type{});
          do {
            ++it, tile(sA, sB, pA, pB, std::true_type{});
            ++it, tile(sB, sA, pB, pA, std::true_type{});
          } while (it + 1 < n_full);
          ++it;
        }
        rest = false;
        drain(v_at(it - 1), pB, pr);
      }
      // the partial cache tile and the tree's keys: queued long ago
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __builtin_amdgcn_s_barrier();
      for (; it < n_tiles; ++it) compute_tile(it, it >= n_ct, std::true_type{}, no_refill);
    }
  } else if constexpr (C::STEADY) {
    if (n_full >= kSteadyTiles) {
      // ---- the steady part of the loop: full cache tiles that queue full cache tiles.  One address per tile and operand, carried
      // along in scalar registers (dense), or one multiply-add per load on its page's number (paged); every wait is a constant ----
      int64_t row_off[NLDK];  // bytes from a tile's first row to the row of (load instruction j, lane 0)
#pragma unroll
      for (int j = 0; j < NLDK; ++j) row_off[j] = (int64_t)((wave * NLDK + j) * LPI) * p.stride_tok * EB;
      const char *k_next = kc_bytes + (cache_base + (int64_t)(k0 + (it + PD) * TK) * p.stride_tok) * EB;
      const char *v_next = vc_bytes + (cache_base + (int64_t)(k0 + (it + PD) * TK) * p.stride_tok) * EB;
      const int64_t tile_bytes = (int64_t)TK * p.stride_tok * EB;
      auto issue_steady = [&](int t) __attribute__((always_inline)) {
        lds_byte *stage = lds + (t % NSTAGE) * STAGE_BYTES;
        if constexpr (PAGED) {
#pragma unroll
          for (int j = 0; j < NLDK; ++j) {
            const uint64_t off = small_off(page_of(t, full_key(j)), k0 + t * TK + full_key(j), j);
            __builtin_amdgcn_global_load_lds(GLOBAL_PTR(kc_bytes + off), stage + kdst_of(j), 16, 0, kLoadOnce);
            __builtin_amdgcn_global_load_lds(GLOBAL_PTR(vc_bytes + off), stage + vdst_of(j), 16, 0, kLoadOnce);
          }
          request_pages(t + C::LOOK, std::true_type{});
        } else {
#pragma unroll
          for (int j = 0; j < NLDK; ++j) {
            __builtin_amdgcn_global_load_lds(GLOBAL_PTR(k_next + row_off[j] + lane_off2[j & 1]), stage + kdst_of(j), 16, 0, kLoadOnce);
            __builtin_amdgcn_global_load_lds(GLOBAL_PTR(v_next + row_off[j] + lane_off2[j & 1]), stage + vdst_of(j), 16, 0, kLoadOnce);
          }
          k_next += tile_bytes;
          v_next += tile_bytes;
        }
      };
      auto step_steady = [&](int t) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(PAGED && PD == 1 ? C::NPG : C::TILE_OPS * (PD - 1)));
        __builtin_amdgcn_s_barrier();
        issue_steady(t + PD);
        if (!wave_has_rows) return;
        const lds_byte *stage = lds + (t % NSTAGE) * STAGE_BYTES;
        compute_block(stage, std::integral_constant<int, 0>{}, 0, 0, false, std::false_type{}, std::true_type{}, no_refill);
        if constexpr (KBW > 1) compute_block(stage, std::integral_constant<int, 1>{}, 0, 0, false, std::false_type{}, std::true_type{}, no_refill);
      };
      static_assert(KBW <= 2, "");
#pragma unroll
      for (int r = 0; r < RB; ++r) set_cap(r);
      if (!PAGED || small_pages)
        for (; it + PD < n_full; ++it) step_steady(it);
    }
  }
  if (!C::PIPED || !piped) {
    if constexpr (C::AHEAD && !PAGED) {
      // full tiles that queue full tiles: a part of the loads behind each product of the scores
      for (; it + PD < n_full; ++it) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(NLD * (PD - 1)));
        __builtin_amdgcn_s_barrier();
        const int64_t at = (cache_base + (int64_t)(k0 + (it + PD) * TK) * p.stride_tok) * EB;
        const char *const ksrc = kc_bytes + at, *const vsrc = vc_bytes + at;
        lds_byte *const to = lds + ((it + PD) % NSTAGE) * STAGE_BYTES;
        auto load = [&](auto s_tag) __attribute__((always_inline)) {
          constexpr int s = decltype(s_tag)::value;
#pragma unroll
          for (int l = (s * NLD + NS - 1) / NS; l < ((s + 1) * NLD + NS - 1) / NS; ++l) {
            const int j = l % NLDK;
            if (l < NLDK) __builtin_amdgcn_global_load_lds(GLOBAL_PTR(ksrc + lane_off[j]), to + kdst_of(j), 16, 0, kLoadOnce);
            else __builtin_amdgcn_global_load_lds(GLOBAL_PTR(vsrc + lane_off[j]), to + vdst_of(j), 16, 0, kLoadOnce);
          }
        };
        if (wave_has_rows) compute_tile(it, false, std::false_type{}, load);
        else static_for<NS>(load);
      }
    }
    for (; it < n_full; ++it) step(it, std::false_type{}, std::false_type{});
    for (; it < n_ct; ++it) step(it, std::true_type{}, std::false_type{});   // the partial cache tile
    for (; it < n_tiles; ++it) step(it, std::true_type{}, std::true_type{});  // the tree's own keys
  }
  if constexpr (PAGED && (C::PIPED || C::SHARES)) {
    const const_args late = late_args();
    p.G = late->G, p.g_magic = late->g_magic, p.g_bits = late->g_bits, p.Hq = late->Hq, p.sum_Q = late->sum_Q, p.n_chunks = late->n_chunks;
    p.out = late->out, p.lse = late->lse, p.part_out = late->part_out, p.part_lse = late->part_lse, p.v_scale = late->v_scale;
  }
  if constexpr (PAGED) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // the last (unused) table entries have landed
  __builtin_amdgcn_s_barrier();  // all waves are done reading the ring before it is reused below
  TL_STAMP(4);  // all tiles done

  // ---- combine the two lane halves' partial sums, and the two key groups' references and sums ----
  // (factor: what a row's O is multiplied by -- to the groups' common reference, and 1 / sum)
  constexpr bool PAIR = C::PAIR;
  float l_tot[RB], factor[RB];
  float *const sm = reinterpret_cast<float *>(smem);  // [WK][WM][RB][32] references, then as many sums
  float *const sl = sm + WK * WM * RB * 32;
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    l_tot[r] = half_sum(l_run[r]);
    factor[r] = 1.f;
    if (PAIR && hh == 0) sm[((wk * WM + wm) * RB + r) * 32 + l32] = m_run[r], sl[((wk * WM + wm) * RB + r) * 32 + l32] = l_tot[r];
  }
  if constexpr (PAIR) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int other = (((1 - wk) * WM + wm) * RB + r) * 32 + l32;
      const float mo = sm[other], lo = sl[other];
      const float mf = fmaxf(m_run[r], mo), ref = (mf == -INFINITY) ? 0.f : mf;
      factor[r] = fast_exp2(m_run[r] - ref);
      l_tot[r] = l_tot[r] * factor[r] + lo * fast_exp2(mo - ref);
      m_run[r] = mf;
    }
  }
#pragma unroll
  for (int r = 0; r < RB; ++r) factor[r] *= l_tot[r] > 0.f ? p.v_scale / l_tot[r] : 0.f;

  // (A row whose sum is none -- NaN scores -- has no weight in the merge of the splits: in this launch its outputs are zeros then.)
  if (SHARED && nc > 1 && __builtin_expect(__builtin_amdgcn_ballot_w64(!(l_tot[0] > 0.f)) != 0, 0)) {
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[0][d][i] = l_tot[0] > 0.f ? oacc[0][d][i] : 0.f;
  }

  // ---- merge the WK key groups through LDS ----
  // Two key groups: each wave keeps one half of the head dimension and hands the other half to
  // its partner, so both take part in the reduction and in writing the result.
  if constexpr (PAIR) {
    constexpr int H = ND / 2;
    float *xo = sl + WK * WM * RB * 32;                      // [WM][WK][RB][H][4][64] x 16 bytes
    f32x4 *const dst = reinterpret_cast<f32x4 *>(xo) + (size_t)((wm * WK + (1 - wk)) * RB * H * 4) * 64 + lane;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int d = 0; d < H; ++d)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = oacc[r][H + d][i4 * 4 + e] * factor[r];
          dst[((r * H + d) * 4 + i4) * 64] = v;
        }
    __syncthreads();
    const f32x4 *const src = reinterpret_cast<const f32x4 *>(xo) + (size_t)((wm * WK + wk) * RB * H * 4) * 64 + lane;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
#pragma unroll
      for (int d = 0; d < H; ++d)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x4 v = src[((r * H + d) * 4 + i4) * 64];
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[r][d][i4 * 4 + e] = fmaf(oacc[r][d][i4 * 4 + e], factor[r], v[e]);
        }
    }
  }

  // ---- write (normalised) result: final when there is one split, else the partial ----
  // The accumulators hold O^T (lane = row, registers = 16 scattered d per 32-wide block); each
  // wave transposes one 32-row block at a time through its own LDS patch so that global stores
  // are whole contiguous rows (of the half of the head dimension the wave holds, when paired).
  const bool final_out = (SHARED ? nc : p.n_chunks) == 1;
  float *obase = final_out ? p.out : p.part_out + (size_t)chunk * p.sum_Q * p.Hq * D;
  float *lbase = final_out ? p.lse : p.part_lse + (size_t)chunk * p.sum_Q * p.Hq;
  constexpr int NDW = C::NDW;       // 32-wide d blocks this wave writes
  constexpr int TP = C::TP;         // patch row pitch in floats: 16 rows x 16 B apart in bank position
  constexpr int LPR = NDW * 8;      // lanes that cover one row piece with 16 bytes each
  constexpr int RPP = 64 / LPR;     // rows per wave-wide store
  float *const patches = reinterpret_cast<float *>(smem + C::PATCH_OFF);
  float *tbuf = patches + (PAIR ? wave : wm) * (32 * TP);
  const float own_lse2 = l_tot[0] > 0.f ? m_run[0] + __builtin_amdgcn_logf(l_tot[0]) : -INFINITY;
  // (lane = row, registers = 16 scattered d) -> the wave's patch
  auto to_patch = [&](int r) __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < NDW; ++d)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = PAIR ? oacc[r][d][i4 * 4 + e] : oacc[r][d][i4 * 4 + e] * factor[r];
        *reinterpret_cast<f32x4 *>(tbuf + l32 * TP + 32 * d + 8 * i4 + 4 * hh) = v;
      }
  };
  // One basic block per 32 rows: rows past the last are stored as copies of the last one (to its own address, the same values),
  // so that no store sits behind a branch of its own and the reads of all pieces are in flight together.  What remains is the
  // LDS traffic of the two exchanges.  (One sequence of 2048 keys in 7 splits, from the last tile to the last store: 1.76 us
  // with a branch, a division of the row's index and a read waited for per store, two copies of the code by key group, and
  // the sums exchanged behind the outputs; 1.30 now.  Both groups' whole rows exchanged at once instead: 1.28 there, but 0.1
  // more where two waves make a workgroup.)
  auto write_out = [&](auto once_tag) __attribute__((always_inline)) {
    // partial rows (read next by the merge kernel, then dead) are stored with the non-temporal hint; final rows,
    // which the caller's next kernel reads, are left to the caches.  Two copies of the loop: one store whose hint
    // is chosen at run time would lose it.
    constexpr bool ONCE = decltype(once_tag)::value;
    float *const first = obase + ((int64_t)tq0 * p.Hq + kvh * p.G) * D + kept0 + (lane % LPR) * 4;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      to_patch(r);
      const int row0 = rblk * BM + (wm * RB + r) * 32;
      if (row0 >= R) break;  // (wave-uniform)
      const int last = R - 1 - row0;
      f32x4 v[32 / RPP];
#pragma unroll
      for (int i = 0; i < 32 / RPP; ++i) {
        int rl = i * RPP + lane / LPR;
        rl = rl < last ? rl : last;
        v[i] = *reinterpret_cast<const f32x4 *>(tbuf + rl * TP + (lane % LPR) * 4);
      }
#pragma unroll
      for (int i = 0; i < 32 / RPP; ++i) {
        int rl = i * RPP + lane / LPR;
        rl = rl < last ? rl : last;
        const int row = row0 + rl, t = node_of(p, row);
        f32x4 *const dst = reinterpret_cast<f32x4 *>(first + (int64_t)(t * p.Hq + (row - t * p.G)) * D);
        if constexpr (ONCE) __builtin_nontemporal_store(v[i], dst);
        else *dst = v[i];
      }
      if (rvalid[r] && hh == 0 && wk == 0) lbase[orow[r]] = own_lse2 * kLn2;
    }
  };
  if (final_out) write_out(std::false_type{});
  else if constexpr (!SHARED) write_out(std::true_type{});
  if (!SHARED || final_out) {
    TL_STAMP(5);  // key groups merged, result stores issued
    TL_STORE(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), 0, 6);
    return;
  }
  if constexpr (SHARED) {
  // ---- the row block's splits merged in this launch, each workgroup a share of the rows ----
  // The nc workgroups of a (sequence, KV head, row block) take a share of its rows each.  A workgroup stores the rows of the others'
  // shares, says that it has, waits until all have, and merges its own share, which never leaves its LDS.  All that travels between
  // them is written and read at device scope (past the caches of one XCD).
  // What they say stands in the scratch memory where split 0 would keep the first row of its own share, which nobody else reads: a word
  // per split, the launch's tag and a state.  The memory may hold anything: a word of another call, or of the same launch replayed,
  // has no such tag, since tags are drawn per call and the words of a launch are cleared behind it.
  //  - ARRIVED: its rows are there for the others.
  //  - LEFT, once it has seen all arrive, or GAVE, once it has looked share_polls times: it will not look for arrivals again.  One
  //    that gives up leaves its share's rows where the results go.
  // Whoever then finds every word in one of the last two clears them; where some gave up, the one that takes the first word away does,
  // and merges their shares, with all its waves.  The last to store such a state finds them so.  So nobody relies on the others being
  // resident, and none waits longer than its looks.
  enum : uint64_t { ARRIVED = 1, LEFT = 2, GAVE = 3 };
  constexpr int LPW = D / 4, GROUPS = 64 / LPW;
  constexpr int kDevice = 16;                  // the cache policy's sc1: device scope
  constexpr uint32_t kNowhere = 0x80000000u;   // past every bound, with what may be added: neither read nor stored
  const uint64_t share_tag = late_args()->share_tag;
  const bool keeps_words = wave == C::NW - 1;  // (this wave merges no rows of its workgroup's share)
  const int Rb = R - rblk * BM < BM ? R - rblk * BM : BM;
  // (Rb / nc rounded up: whole or at least 1/32 above it, and the reciprocal is good to a few units of 2^-23)
  const int per = __builtin_amdgcn_readfirstlane((int)fmaf((float)Rb, __builtin_amdgcn_rcpf((float)nc), 0.99f));
  const int share0 = chunk * per, end = share0 + per < Rb ? share0 + per : Rb;
  const uint32_t n_rows = (uint32_t)p.sum_Q * (uint32_t)p.Hq;  // (all rows of all splits are less than 2 GiB)
  float *const own_lses = reinterpret_cast<float *>(smem + C::OWN_OFF);
  uint32_t *const rows = reinterpret_cast<uint32_t *>(own_lses + WM * 32), *const stored = rows + WM * 32 + wave * 32;
  int *const seen = reinterpret_cast<int *>(rows + WM * 32 + C::NW * 32);
  const auto parts = __builtin_amdgcn_make_buffer_rsrc(p.part_out, 0, (int)((uint32_t)p.n_chunks * n_rows * (D * 4)), 0x00020000);
  const auto part_lses = __builtin_amdgcn_make_buffer_rsrc(p.part_lse, 0, (int)((uint32_t)p.n_chunks * n_rows * 4), 0x00020000);
  const auto results = __builtin_amdgcn_make_buffer_rsrc(p.out, 0, (int)(n_rows * (D * 4)), 0x00020000);
  const auto result_lses = __builtin_amdgcn_make_buffer_rsrc(p.lse, 0, (int)(n_rows * 4), 0x00020000);
  {
    const int rl = wm * 32 + l32;
    const uint32_t at = (uint32_t)chunk * n_rows + (uint32_t)orow[0];
    if (hh == 0) stored[l32] = rl < Rb && (rl < share0 || rl >= end) ? at * (D * 4) : kNowhere;
    if (hh == 0 && wk == 0) {
      own_lses[rl] = own_lse2, rows[rl] = (uint32_t)orow[0];
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(own_lse2), part_lses, rl < Rb ? at * 4 : kNowhere, 0, kDevice);
    }
    to_patch(0);
    f32x4 v[32 / RPP];
    uint32_t to[32 / RPP];
#pragma unroll
    for (int i = 0; i < 32 / RPP; ++i) {
      to[i] = stored[i * RPP + lane / LPR];
      v[i] = *reinterpret_cast<const f32x4 *>(tbuf + (i * RPP + lane / LPR) * TP + (lane % LPR) * 4);
    }
#pragma unroll
    for (int i = 0; i < 32 / RPP; ++i)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[i]), parts, to[i] + (uint32_t)(kept0 + (lane % LPR) * 4) * 4, 0, kDevice);
  }
  TL_STAMP(5);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  uint64_t *const words = reinterpret_cast<uint64_t *>(p.part_out + (size_t)__builtin_amdgcn_readfirstlane(rows[0]) * D);
  auto look = [&]() __attribute__((always_inline)) -> uint64_t {  // a split's state, 0: none; lanes past the splits: LEFT
    if (lane >= nc) return LEFT;
    const uint64_t w = __hip_atomic_load(words + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (w & ~3ull) == share_tag ? w & 3 : 0;
  };
  auto say = [&](uint64_t state) __attribute__((always_inline)) {
    if (lane == 0) __hip_atomic_store(words + chunk, share_tag | state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  const int grp = lane / LPW, col = (lane % LPW) * 4;
  auto own_row = [&](int rl) __attribute__((always_inline)) {
    const int wave_of = (PAIR ? col / (D / 2) * WM : 0) + rl / 32;
    return *reinterpret_cast<const f32x4 *>(patches + (wave_of * 32 + rl % 32) * TP + (PAIR ? col % (D / 2) : col));
  };
  // A group of lanes takes a row, a lane 16 bytes of it: from all other splits, NI of them in flight for each of ROWS rows, and
  // without a branch between the loads and what is computed from them.  Code that runs once costs about 0.1 us for every 64 bytes of
  // it (one sequence of 2048 keys, 60 nodes: 0.9 us more with a comparison and four selections per split and row), so the
  // log-sum-exps are to the base 2 here (made natural by one multiply-add: 2.57e-7 off, root mean square, 2.73e-7 by the second
  // launch), and past the splits nothing is read (the last one again instead, for shorter addresses:
  // 2 .. 20 % of calls of 3, 4, 8 and 11 splits).
  // Merged are the rows of the workgroup's own share, by the waves that do not keep the words, or, GIVEN, those of the shares that were
  // given up, by all waves: the row block's rows one after the other, so that as many are in flight as the waves hold, whoever gave them up.
  auto merge_rows = [&](uint32_t given, auto given_tag, auto ni_tag, auto rows_tag) __attribute__((always_inline)) {
    constexpr bool GIVEN = decltype(given_tag)::value;
    constexpr int NI = decltype(ni_tag)::value, ROWS = decltype(rows_tag)::value;
    const float one_by_per = __builtin_amdgcn_rcpf((float)per);  // (GIVEN: quotients of numbers below 256, a half above whole ones)
    auto share_of = [&](int rl) __attribute__((always_inline)) { return GIVEN ? (int)(((float)rl + 0.5f) * one_by_per) : chunk; };
    const int last = GIVEN ? Rb : end;
    for (int rl0 = (GIVEN ? 0 : share0) + wave * GROUPS * ROWS; rl0 < last; rl0 += (GIVEN ? C::NW : C::NW - 1) * GROUPS * ROWS) {
      uint32_t row[ROWS];
      int share[ROWS];
      bool mine[ROWS];  // the row is one that is to be merged
      float m[ROWS], z[ROWS];
      f32x4 acc[ROWS];
#pragma unroll
      for (int j = 0; j < ROWS; ++j) {
        const int rl = rl0 + j * GROUPS + grp, rc = rl < last ? rl : last - 1;
        row[j] = rows[rc], share[j] = share_of(rc), mine[j] = rl < last && (!GIVEN || (given >> share[j] & 1));
      }
      if constexpr (GIVEN) {
        bool some = false;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) some |= mine[j];
        if (__builtin_amdgcn_ballot_w64(some) == 0) continue;
      }
      for (int k0 = 0; k0 < nc - 1; k0 += NI) {
        float l[ROWS][NI];
        f32x4 v[ROWS][NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
#pragma unroll
          for (int j = 0; j < ROWS; ++j) {
            const int k = k0 + i, s = k < share[j] ? k : k + 1;
            const uint32_t from = (uint32_t)s * n_rows, past = s < nc ? 0u : kNowhere;  // (past the splits: nothing is read)
            l[j][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(part_lses, (from + row[j]) * 4 | past, 0, kDevice));
            v[j][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(parts, ((from + row[j]) * (D * 4) + col * 4) | past, 0, kDevice));
          }
        }
        if (k0 == 0) {
          if constexpr (!GIVEN) {
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
              const int rl = rl0 + j * GROUPS + grp, rc = rl < last ? rl : last - 1;
              m[j] = own_lses[rc], acc[j] = own_row(rc);
            }
          } else {
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
              m[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(result_lses, row[j] * 4, 0, kDevice));
              acc[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(results, row[j] * (D * 4) + col * 4, 0, kDevice));
            }
          }
#pragma unroll
          for (int j = 0; j < ROWS; ++j) z[j] = m[j] > -INFINITY ? 1.f : 0.f;
        }
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
          float top = m[j];
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            if (NI > 1) l[j][i] += k0 + i < nc - 1 ? 0.f : -INFINITY;
            top = fmaxf(top, l[j][i]);
          }
          const float ref = top > -INFINITY ? top : 0.f, keep = fast_exp2(m[j] - ref);
          m[j] = top;
          z[j] *= keep;
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[j][e] *= keep;
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            const float w = fast_exp2(l[j][i] - ref);
            z[j] += w;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] = fmaf(v[j][i][e], w, acc[j][e]);
          }
        }
      }
      // A part without weight adds nothing, whatever it holds, as in merge_kernel.  Here that is told by what comes of it, 0 times
      // infinity not being a number: rows with such an element are added up again, in the same order, without those parts.
      bool lost = false;
#pragma unroll
      for (int j = 0; j < ROWS; ++j) {
        const float sum = (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
        lost |= sum != sum;
      }
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(lost) != 0, 0)) {
#pragma unroll 1
        for (int again = 0; again < ROWS; ++again) {
          const int rl = rl0 + again * GROUPS + grp, rc = rl < last ? rl : last - 1;
          const uint32_t r = rows[rc];
          const int own = share_of(rc);
          float m1 = !GIVEN ? own_lses[rc] : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(result_lses, r * 4, 0, kDevice));
          f32x4 a = !GIVEN ? own_row(rc) : __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(results, r * (D * 4) + col * 4, 0, kDevice));
#pragma unroll 1
          for (int k0 = 0; k0 < nc - 1; k0 += NI) {
            const int k1 = k0 + NI < nc - 1 ? k0 + NI : nc - 1;
            auto lse_of = [&](int k) __attribute__((always_inline)) {
              return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(part_lses, ((uint32_t)(k < own ? k : k + 1) * n_rows + r) * 4, 0, kDevice));
            };
            float top = m1;
#pragma unroll 1
            for (int k = k0; k < k1; ++k) top = fmaxf(top, lse_of(k));
            const float ref = top > -INFINITY ? top : 0.f, keep = fast_exp2(m1 - ref);
            m1 = top;
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = keep != 0.f ? a[e] * keep : 0.f;
#pragma unroll 1
            for (int k = k0; k < k1; ++k) {
              const float w = fast_exp2(lse_of(k) - ref);
              const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(parts, ((uint32_t)(k < own ? k : k + 1) * n_rows + r) * (D * 4) + col * 4, 0, kDevice));
#pragma unroll
              for (int e = 0; e < 4; ++e) a[e] = w != 0.f ? fmaf(v[e], w, a[e]) : a[e];
            }
          }
#pragma unroll
          for (int j = 0; j < ROWS; ++j) acc[j] = j == again ? a : acc[j];
        }
      }
#pragma unroll
      for (int j = 0; j < ROWS; ++j) {
        const bool any = z[j] > 0.f;
        const uint32_t past = mine[j] ? 0u : kNowhere;
        const float f0 = __builtin_amdgcn_rcpf(z[j]), f = fmaf(f0, fmaf(-z[j], f0, 1.f), f0);  // (a sum is 1 or more)
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = any ? acc[j][e] * f : 0.f;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), results, (row[j] * (D * 4) + col * 4) | past, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(any ? fmaf(m[j], kLn2, __builtin_amdgcn_logf(z[j]) * kLn2) : -INFINITY), result_lses, row[j] * 4 | (col == 0 ? past : kNowhere), 0, 0);
      }
    }
  };
  if (keeps_words) {
    say(ARRIVED);
    bool all = false;
    const int looks = late_args()->share_polls;
    for (int polls = looks >> (16 + chunk) & 1 ? 0 : looks & 0xFFFF; polls > 0; --polls) {
      all = __builtin_amdgcn_ballot_w64(look() == 0) == 0;
      if (all) break;
      __builtin_amdgcn_s_sleep(1);
    }
    if (all) say(LEFT);
    if (lane == 0) *seen = all;
  }
  __syncthreads();
  TL_STAMP(6);  // all have arrived
  // (splits x rows in flight, by what registers hold, as few past the splits as that allows.  One sequence of 256 keys a split, 12 and 60
  // nodes, three shapes: two splits by 1 x 8 rows take 0.86 .. 0.93 of 8 x 2's time and 0.92 .. 1.00 of 4 x 4's, 3 .. 5 by 4 x 4
  // 0.94 .. 1.01 of 8 x 2's, 6 .. 12 by 8 x 2 0.92 .. 0.99 of 4 x 4's.)
  auto merge = [&](uint32_t given, auto given_tag) __attribute__((always_inline)) {
    if (nc == 2) merge_rows(given, given_tag, std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
    else if (nc <= 5) merge_rows(given, given_tag, std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
    else merge_rows(given, given_tag, std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{});
  };
  if (*seen != 0) {
    if (!keeps_words) merge(0, std::false_type{});
  } else {
    for (int rl = share0 + wave * GROUPS + grp; rl < end; rl += C::NW * GROUPS) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, own_row(rl)), results, rows[rl] * (D * 4) + col * 4, 0, kDevice);
      if (col == 0) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(own_lses[rl]), result_lses, rows[rl] * 4, 0, kDevice);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (keeps_words) say(GAVE);
  }
  TL_STAMP(7);  // the share's results issued
  TL_STORE(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), 0, 8);
  if (keeps_words) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (its last word is there for the others)
    const uint64_t state = look();
    uint32_t given = 0;
    if (__builtin_amdgcn_ballot_w64(state < LEFT) == 0) {
      given = (uint32_t)__builtin_amdgcn_ballot_w64(lane < nc && state == GAVE);
      bool taken = given == 0;
      if (lane == 0 && !taken) {
        uint64_t word = share_tag | state;
        taken = __hip_atomic_compare_exchange_strong(words, &word, (uint64_t)0, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (__builtin_amdgcn_ballot_w64(taken) == 0) given = 0;
      else if (lane < nc) __hip_atomic_store(words + lane, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) seen[1] = (int)given;
  }
  __syncthreads();
  const uint32_t given = (uint32_t)__builtin_amdgcn_readfirstlane(seen[1]);
  if (__builtin_expect(given != 0, 0)) merge(given, std::true_type{});
  }
}
#undef lrow
#undef kdst_of
#undef vdst_of

// ---------------------------------------------------------------------------------------
// merge of the KV splits
// ---------------------------------------------------------------------------------------
// One wave per output row (token, head).  The lanes form GROUPS groups of D/4 lanes (16 bytes of
// the row per lane); group g takes the splits g, g + GROUPS, ...  Every load of a block of NI
// splits per group -- the partial rows and their log-sum-exps, clamped to a split that exists --
// is issued before anything is computed from them, so a row costs one memory round trip however
// many splits it has (NI is chosen on the host to cover S where it can).  The groups keep a
// running maximum each and are combined at the end.  Splits whose LSE is -inf (empty, or never
// computed because the sequence is shorter than the launch's split count) get weight zero; their
// O may be uninitialised memory and is dropped by selection, never by multiplication.
template <int D, int NI>
__global__ void __launch_bounds__(256) merge_kernel(const float *__restrict__ part_out,
                                                    const float *__restrict__ part_lse, int S, int64_t n_rows,
                                                    float *__restrict__ out, float *__restrict__ lse) {
  const int lane = threadIdx.x & 63;
  TL_DECL;
  TL_STAMP(0);
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  constexpr int LPR = D / 4;        // lanes covering one row with 16 bytes each
  constexpr int GROUPS = 64 / LPR;  // splits processed side by side in one wave
  const int grp = lane / LPR, col = (lane % LPR) * 4;
  float m = -INFINITY, z = 0.f;     // running maximum of the LSEs, sum of weights relative to it
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = grp; s0 < S; s0 += GROUPS * NI) {
    float l[NI];
    f32x4 v[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int s = s0 + i * GROUPS;
      const int sc = s < S ? s : s0;
      l[i] = part_lse[(size_t)sc * n_rows + row];
      v[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(part_out + ((size_t)sc * n_rows + row) * D + col));
      if (s >= S) l[i] = -INFINITY;
    }
    float mb = m;
#pragma unroll
    for (int i = 0; i < NI; ++i) mb = fmaxf(mb, l[i]);
    if (mb > -INFINITY) {
      const float keep = __expf(m - mb);  // 0 while nothing has been accumulated (m = -inf)
      z *= keep;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] *= keep;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const float w = __expf(l[i] - mb);
        z += w;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += (w != 0.f) ? v[i][e] * w : 0.f;
      }
      m = mb;
    }
  }
#pragma unroll
  for (int o = 32; o >= LPR; o >>= 1) {
    const float m2 = __shfl_xor(m, o), z2 = __shfl_xor(z, o);
    const float mn = fmaxf(m, m2);
    const float k1 = (m > -INFINITY) ? __expf(m - mn) : 0.f, k2 = (m2 > -INFINITY) ? __expf(m2 - mn) : 0.f;
    z = z * k1 + z2 * k2;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = acc[e] * k1 + __shfl_xor(acc[e], o) * k2;
    m = mn;
  }
  const bool any = z > 0.f;
  if (grp == 0) *reinterpret_cast<f32x4 *>(out + row * D + col) = any ? acc * (1.f / z) : f32x4{0.f, 0.f, 0.f, 0.f};
  if (lane == 0) lse[row] = any ? m + __logf(z) : -INFINITY;
  TL_STAMP(1);  // stores issued
  TL_MARK;
  TL_STORE(blockIdx.x, 6, 2);
}

// NI = splits per lane group and block: the smallest of 1, 2, 4, 8 that covers S in one block
template <int D>
void launch_merge(const float *part_out, const float *part_lse, int S, int64_t n_rows, float *out, float *lse,
                  hipStream_t st) {
  constexpr int GROUPS = 64 / (D / 4);
  const dim3 grid((unsigned)((n_rows + 3) / 4)), block(256);
  const int per_group = (S + GROUPS - 1) / GROUPS;
  if (per_group <= 1) hipLaunchKernelGGL((merge_kernel<D, 1>), grid, block, 0, st, part_out, part_lse, S, n_rows, out, lse);
  else if (per_group <= 2) hipLaunchKernelGGL((merge_kernel<D, 2>), grid, block, 0, st, part_out, part_lse, S, n_rows, out, lse);
  else if (per_group <= 4) hipLaunchKernelGGL((merge_kernel<D, 4>), grid, block, 0, st, part_out, part_lse, S, n_rows, out, lse);
  else hipLaunchKernelGGL((merge_kernel<D, 8>), grid, block, 0, st, part_out, part_lse, S, n_rows, out, lse);
}

// ---------------------------------------------------------------------------------------
// host side: validation, plan, launch
// ---------------------------------------------------------------------------------------

struct Plan {
  int variant;  // index into the kernel table
  int BM, TK;
  int n_row_blocks, n_chunks, chunk_keys;
  bool fewer;  // the splits are the fewer, longer ones that share the merge (plan_splits_of)
};

// workgroup shapes (values of tva_shape in tva.h, minus one)
enum { V_K2 = TVA_SHAPE_R32_W2 - 1, V_M2K2 = TVA_SHAPE_R64_W4 - 1, V_M2K2_3 = TVA_SHAPE_R64_W4_DEEP - 1,
       V_M4K2 = TVA_SHAPE_R128_W8 - 1, V_W8 = TVA_SHAPE_R256_W8 - 1, V_LAST = V_W8 };

// query rows of the whole batch: every tree node, or only the nodes cu_Q selects
inline int64_t query_rows(const tva_args *a) { return a->cu_Q ? a->sum_Q : a->sum_T; }

// Which sequence each workgroup slot takes, when the host knows the cache lengths (tva_args.L_host).  An unsplit
// launch of one workgroup per (sequence, KV head) with 8 KV heads and 33 .. 64 sequences, of a shape of which two
// share a CU, fits the chip at once; in dispatch order the heads go round the 8 XCDs and the sequences round an XCD's
// 32 CUs, so that slots j and j + 32 of the B share a CU for the whole launch, and a CU that got two long sequences
// ends it (measured on 64 lengths from U{512..2048}: 73.6 us as drawn, 68.0 with a long and a short one per CU,
// 60.3 with all lengths at their mean).  So: the CUs with one slot get the longest sequences, every other CU a long
// and a short one.  Where workgroups land is the dispatcher's business, not a guarantee: this is a heuristic about
// time, and slot_seq is a permutation whatever L_host holds, so no result depends on it.
void fill_slots(const tva_args *a, const Plan &pl, AttnParams *p) {
  p->pair_slots = 0;
  for (uint32_t &w : p->slot_seq) w = 0;
  p->real_splits = 0;
  const bool two_per_cu = pl.variant == V_K2 || pl.variant == V_M2K2;
  const int n = a->B;
  // A split launch of unequal sequences: a shorter one's last splits are empty.  Workgroups go to the shader engines in
  // turn whatever they do; with the empty ones among them one engine can be given more work than it has CUs while
  // another idles, and the launch then lasts two rounds (four sequences of 16384 .. 32768 keys, 31 of 40 splits filled: 176 us,
  // 146 with 25 of 32; 129 with the filled ones first).  So: the filled splits, by the lengths given, come first.  As above
  // this is a permutation whatever L_host holds.
  if (a->L_host && (pl.variant == V_W8 || pl.variant == V_M4K2) && pl.n_chunks > 1 && n > 1 && n <= 32 && (int64_t)n * pl.n_chunks <= 65535 &&
      (int64_t)n * pl.n_chunks * a->Hkv * pl.n_row_blocks > 256) {
    int filled = 0;
    for (int i = 0; i < n; ++i) {
      const int64_t L = a->L_host[i] < a->max_L ? a->L_host[i] : a->max_L;
      const int64_t nc = L > 0 ? (L + pl.chunk_keys - 1) / pl.chunk_keys : 1;
      filled += (int)nc;
      p->slot_seq[i >> 1] |= (uint32_t)filled << (16 * (i & 1));
    }
    if (filled < n * pl.n_chunks) p->real_splits = filled;
    return;
  }
  if (!a->L_host || !two_per_cu || pl.n_chunks != 1 || pl.n_row_blocks != 1 || a->Hkv != 8 || n <= 32 || n > 64) return;
  int order[64];  // sequences, longest first (equal lengths: lower index first)
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order, order + n, [&](int x, int y) { return a->L_host[x] > a->L_host[y]; });
  const int shared = n - 32;  // CUs 0 .. shared-1 of an XCD hold two slots (j and j + 32), the others one
  for (int j = 0; j < n; ++j) {
    const int rank = j >= 32 ? n - 1 - (j - 32) : j < shared ? (64 - n) + j : j - shared;
    p->slot_seq[j >> 2] |= (uint32_t)order[rank] << (8 * (j & 3));
  }
  p->pair_slots = n;
}

// The splits of one workgroup shape.  named: the shape is to be this one (else the 2 x 2 shape may take its deeper ring).
// share: fewer, longer splits that share the merge may take the place of many short ones.
void plan_splits_of(const tva_args *a, int variant, bool named, bool share, Plan *pl) {
  const int G = a->Hq / a->Hkv;
  const int rows = (a->cu_Q ? a->max_Q : a->max_T) * G;
  const int pairs = a->B * a->Hkv;
  pl->variant = variant;
  pl->BM = variant == V_W8 ? 256 : variant == V_M4K2 ? 128 : variant == V_K2 ? 32 : 64;
  pl->TK = 64;
  pl->fewer = false;
  pl->n_row_blocks = rows > 0 ? (rows + pl->BM - 1) / pl->BM : 1;
  int S = a->num_splits;
  const int max_by_len = a->max_L > 0 ? (a->max_L + pl->TK - 1) / pl->TK : 1;
  const int natural = a->B * a->Hkv * pl->n_row_blocks;
  const bool two_per_cu = variant == V_K2 || variant == V_M2K2;
  if (S == 0 && two_per_cu) {
    // The small shapes (two workgroups fit a CU): the number of splits that minimises a model of the
    // launch's duration, fitted to sweeps of the split count over B = 1 .. 8, caches of 256 .. 2048 keys and
    // trees of 1 .. 72 nodes on the benchmark head shape:
    //   (tiles of the longest split, the tree's own tiles counted with the last one) x time per tile
    //      x 1 while every workgroup has a CU to itself (256), x 1.5 while two share one (512),
    //   + with splits: a merge pass (3.0 us) and the partial rows written and read back (0.30 us per MB), as a second launch
    //     costs.  (The merge in the attention launch costs 1 us and a third less; priced so in all splits, or in short ones,
    //     the count it comes to is the slower one as often as the faster.)
    // Splits keep two tiles or more (one, in launches of at most 128 workgroups over six tiles or more) and
    // together stay within 512 workgroups.
    const int tiles = max_by_len, tree_tiles = (a->max_T + pl->TK - 1) / pl->TK;
    const double tile_us = 1.30 * a->D / 128.0;
    const double part_mb = 2.0 * query_rows(a) * a->Hq * (a->D + 1) * sizeof(float) * 1e-6;
    // Where that comes to more splits than are merged in the attention launch (merged_in_launch), and a number that is, of splits
    // of 12 tiles and more, one per CU (what the deep ring takes), promises less at what the merge costs there, that number is
    // taken, if that is what becomes of it (make_plan).  (8-bit K/V, without the deep ring, 0.88 .. 1.09 of the time; splits of fewer
    // tiles 0.89 .. 1.21.)
    double best = 0.0, shared_best = 0.0;
    int shared = 0;
    S = 1;
    for (int s = 1; s <= (tiles > 1 ? tiles : 1); ++s) {
      const int ckt = (tiles + s - 1) / s, nch = (tiles + ckt - 1) / ckt;
      if (nch != s) continue;  // the same split length as a smaller count
      const int64_t wgs = (int64_t)natural * nch;
      // splits of one tile only while half the CUs would stay empty otherwise, and not on four or five tiles
      // (measured at 256 keys: the unsplit pass is as fast as four one-tile splits and needs no merge)
      if (ckt < 2 && (wgs > 128 || tiles < 6)) break;
      // (no split once the unsplit launch already has a workgroup for every CU: measured at B = 16 and 32,
      // splitting then only adds the merge)
      if (nch > 1 && (wgs > 512 || natural >= 256)) break;
      const int last = tiles - (nch - 1) * ckt + tree_tiles;
      const int longest = nch > 1 && ckt > last ? ckt : last;
      const double share = wgs <= 256 ? 1.0 : 1.5 * (double)((wgs + 511) / 512);
      double cost = tile_us * longest * share;
      if (nch > 1 && nch <= kShareSplits && a->D == 128 && variant == V_M2K2 && !a->kv_fp8 && wgs <= 256 && ckt >= 12) {
        const double c = cost + 2.0 + 0.20 * part_mb * nch;
        if (shared == 0 || c < shared_best - 1e-9) shared_best = c, shared = nch;
      }
      if (nch > 1) cost += 3.0 + 0.30 * part_mb * nch;
      if (s == 1 || cost < best - 1e-9) best = cost, S = nch;
    }
    if (share && S > kShareSplits && shared > 0 && shared_best < best) S = shared, pl->fewer = true;
  } else if (S == 0) {
    // one workgroup per CU (256) if the batch allows, but no split shorter than two tiles:
    // every split costs a partial O of the size of the output, written and read back
    S = natural * 3 >= 512 ? 1 : (256 + natural - 1) / natural;  // two thirds of the CUs busy beats a merge pass
    if (S > 1 && natural * S > 256) --S;  // no second round for a few
    const int cap = a->max_L > 0 ? (a->max_L + 2 * pl->TK - 1) / (2 * pl->TK) : 1;
    if (S > cap) S = cap;
    if (S > max_by_len) S = max_by_len;
    // A split has to save more tile time than its merge pass costs (six tiles' worth as a second launch, with
    // the partial rows written and read back; not asked again of the merge in the attention launch): short
    // caches are split less, or not at all.
    while (S > 1 && max_by_len - (max_by_len + S - 1) / S < 6) --S;
  }
  if (S > max_by_len) S = max_by_len;
  if (S < 1) S = 1;
  int ck = a->max_L > 0 ? (a->max_L + S - 1) / S : pl->TK;
  ck = (ck + pl->TK - 1) / pl->TK * pl->TK;
  if (a->num_splits == 0 && S > 1 && a->sum_L > 0 && a->B > 1) {
    // Cache lengths known to differ (their sum is given): the plan above aims at natural * S
    // workgroups, but the splits a shorter sequence does not reach are empty.  Sequence b needs
    // ceil(L_b / c) <= L_b / c + 1 splits of c keys, so with c >= sum_L / (S * B - B) the non-empty
    // ones of the whole batch still number at most S * B per (KV head, row block): one round as
    // planned, of shorter splits.  Only where splits stay long (16 tiles), so that their length and
    // not the fixed cost per workgroup is what the time follows.
    const int64_t slots = (int64_t)S * a->B - a->B;
    int64_t c = (a->sum_L + slots - 1) / slots;
    c = (c + pl->TK - 1) / pl->TK * pl->TK;
    if (c >= 16 * pl->TK && c < ck) ck = (int)c;
  }
  if (a->num_splits == 0 && S > 1 && a->L_host && a->B > 1) {
    // The lengths themselves are known: the shortest split (whole tiles, 16 or more) with which the non-empty
    // splits of the batch still number S * B, counted instead of bounded.
    const int64_t slots = (int64_t)S * a->B;
    auto fits = [&](int c) {
      int64_t n = 0;
      for (int b = 0; b < a->B; ++b) n += a->L_host[b] > 0 ? ((int64_t)a->L_host[b] + c - 1) / c : 1;
      return n <= slots;
    };
    while (ck - pl->TK >= 16 * pl->TK && fits(ck - pl->TK)) ck -= pl->TK;
  }
  pl->chunk_keys = ck;
  pl->n_chunks = a->max_L > 0 ? (a->max_L + ck - 1) / ck : 1;
  // one 2 x 2 workgroup per CU at most and long splits: a deeper ring (two tiles in flight, with D = 128 three)
  // pays; with more workgroups the second one on the CU hides more than the deeper ring would
  if (pl->variant == V_M2K2 && !named && !a->kv_fp8 && (int64_t)pairs * pl->n_row_blocks * pl->n_chunks <= 256 && ck >= 12 * pl->TK)
    pl->variant = V_M2K2_3;
}


inline bool dense_wide(const tva_args *a) { return a->D == 128 && !a->kv_fp8 && !a->page_table; }

// A launch's duration as a model of it says, in us: fitted to 9650 timed launches (2000 calls in every shape: B = 1 .. 64,
// 64 .. 32768 keys, 4 .. 576 rows per KV head, D = 64 and 128, dense and paged, both storage types, equal and unequal lengths);
// over 4837 others its error had a standard deviation of 9 %.  The kernels have become faster since, paged ones most: 500
// calls now last 0.86 (32-row shape) .. 0.93 of what it says, paged 0.81 .. 0.92, with a standard deviation of 11 .. 16 %; what
// is compared are shapes, and the one taken is 2.6 % slower than the best in the mean (2.3 then).  A round of workgroups
// takes (tiles of the longest split) x (time per tile), more where two share a CU; workgroups beyond whole rounds take a part
// of one more, more than half of it however few they are; every round starts and drains; the launch takes no less than
// its bytes at the rate the shape streams; with splits there is a merge pass, priced as the second launch that it was in all of those.
// The dense deep 64-row shape's tile is 0.85 of that from 14 on, one begun counted, which is most of what its four-stage ring and its
// pipelined loop gained.  (The limit is the plan's own: the ring alone is worth it at 13 full tiles and a part of one, where the loop
// does not run yet.  60 calls of 833 .. 895 keys that this moves to the shape take 0.953 of their time in the others.)
// The eight-wave shapes' tiles stay as fitted: at 0.95 a few more calls moved between those two, for 0.1 % in the mean.
inline int longest_split(const tva_args *a, const Plan &pl) { return pl.n_chunks > 1 ? pl.chunk_keys / pl.TK : (a->max_L + pl.TK - 1) / pl.TK; }
inline bool deep_wide(const tva_args *a, const Plan &pl) { return pl.variant == V_M2K2_3 && dense_wide(a) && longest_split(a, pl) >= 14; }
double plan_cost(const tva_args *a, const Plan &pl) {
  struct Shape {
    double tile, fixed, round, d64, f8, paged, tb_s, tb_s8;
  };
  static const Shape shapes[V_LAST + 1] = {{1.06, 6.5, 2.0, 0.56, 0.92, 1.42, 7.1, 4.9},   // V_K2
                                           {1.13, 6.5, 3.2, 0.55, 0.94, 1.17, 7.1, 5.9},   // V_M2K2
                                           {1.03, 8.0, 4.0, 0.53, 1.00, 1.34, 7.9, 4.9},   // V_M2K2_3
                                           {1.12, 8.5, 5.5, 0.55, 0.94, 1.24, 8.5, 4.2},   // V_M4K2
                                           {1.88, 8.4, 5.8, 0.59, 0.98, 1.17, 7.0, 3.3}};  // V_W8
  const Shape &s = shapes[pl.variant];
  const int G = a->Hq / a->Hkv, rows = (a->cu_Q ? a->max_Q : a->max_T) * G;
  const int64_t keys = (int64_t)a->B * a->max_L, splits = (int64_t)a->B * pl.n_chunks;
  const double wgs = (double)splits * a->Hkv * pl.n_row_blocks;
  const bool two = pl.variant == V_K2 || pl.variant == V_M2K2;
  const double holds = two ? 512.0 : 256.0;
  double tile = pl.variant == V_W8 && rows <= 128 ? 1.18 : s.tile;  // (half of the eight waves have no rows)
  if (a->D == 64) tile *= s.d64;
  if (a->kv_fp8) tile *= s.f8;
  if (a->page_table) tile *= s.paged;
  const int longest = longest_split(a, pl), own = (a->max_T + pl.TK - 1) / pl.TK;
  if (deep_wide(a, pl)) tile *= 0.85;
  const double tiles = longest + own * (pl.n_chunks > 1 ? 0.89 : 1.0);
  double rounds = wgs > holds ? wgs / holds : 1.0;
  const double whole = std::floor(rounds), part = rounds - whole;
  if (part > 0.0) rounds = whole + std::max(part, two ? 0.57 : 0.76);
  const double compute = (tile * tiles + (rounds > 1.0 ? s.round : 0.0)) * rounds * (two && wgs > 256 ? 1.37 : 1.0);
  const double mb = ((double)(keys + a->sum_T) * a->Hkv * 2 * (a->kv_fp8 ? 1 : 2) + 6.0 * (double)query_rows(a) * a->Hq) * a->D * 1e-6;
  const double stream = mb / (a->kv_fp8 ? s.tb_s8 : s.tb_s);
  const double c2 = compute * compute, m2 = stream * stream;
  double us = s.fixed + std::sqrt(std::sqrt(c2 * c2 + m2 * m2));
  if (pl.n_chunks > 1) us += 1.6 + 0.172 * 2.0 * pl.n_chunks * (double)query_rows(a) * a->Hq * (a->D + 1) * sizeof(float) * 1e-6;
  return us;
}

// the partial rows and their LSEs
inline size_t scratch_bytes(const tva_args *a, const Plan &pl) {
  return pl.n_chunks > 1 ? (size_t)pl.n_chunks * query_rows(a) * a->Hq * (a->D + 1) * sizeof(float) : 0;
}

// The plan, and whether fewer splits that share the merge had a part in it (or in what other shapes were held against).
bool plan_of(const tva_args *a, bool share, Plan *pl, bool *fewer) {
  if (!a || a->B <= 0 || a->Hq <= 0 || a->Hkv <= 0 || a->Hq % a->Hkv) return false;
  if (a->sum_T < 0 || a->max_T < 0 || a->max_L < 0 || a->num_splits < 0) return false;
  if (a->plan_shape < TVA_SHAPE_AUTO || a->plan_shape > V_LAST + 1) return false;
  const int G = a->Hq / a->Hkv;
  const int rows = (a->cu_Q ? a->max_Q : a->max_T) * G;
  // Workgroup shape, from sweeps over the benchmark shapes and batch / length variations of them.
  // Up to 32 rows per KV head: 32-row workgroups of two waves that split the keys of 64-key tiles.
  // More rows: 64-row workgroups of 2 x 2 waves (two row groups x two key groups).  Both keep a
  // two-stage ring, small enough that two workgroups share a CU and hide each other's start-up
  // and drain.  From 128 rows on, larger workgroups that read each key fewer times take over
  // where the launch can feed them:
  //  - 128-row workgroups of 4 x 2 waves when 96 .. 256 of them exist (one per CU; with two KV
  //    splits at most, and those 16 tiles or longer);
  //  - 256-row workgroups of eight waves (32 rows each, two waves per SIMD) when there would be more
  //    than 256 of the former, or when there are fewer than 96 but the keys are many: half a million
  //    over the (sequence, KV head) pairs, or half of that with long caches, which splits then
  //    spread over the chip.
  const int pairs = a->B * a->Hkv;
  const int64_t keys = (int64_t)pairs * a->max_L;
  const int n128 = pairs * ((rows + 127) / 128);
  const int s128 = n128 * 3 >= 512 ? 1 : 256 / (n128 > 0 ? n128 : 1);
  int variant = V_M2K2;
  // (8-bit K/V from 128 K keys on, lengths known: four waves queue a tile's loads faster than two; 4 sequences of 16000
  // keys 36 -> 31.5 us; not where long and short sequences share a CU, see fill_slots: 41.4 -> 42.0)
  if (rows <= 32) variant = a->kv_fp8 && a->L_host && a->B <= 32 && keys >= (128 << 10) ? V_M2K2 : V_K2;
  // (the draft stage's attention of one or two sequences -- queries are the newest nodes, at most 48 rows per KV head: two
  // 32-row workgroups, the second three quarters empty, and a second launch for their splits against one of 64 rows that may
  // merge its own.  12 nodes, 256, 700, 1024, 2048 and 4096 keys, us: one sequence 9.2, 9.9, 10.0, 11.2, 13.6 against 9.8, 9.9,
  // 11.4, 11.9, 13.4; two 9.6, 10.6, 10.5, 13.2, 16.8 against 10.3, 10.3, 10.5, 12.8, 15.5.  From eight sequences on the 64-row
  // shape wins)
  else if (a->cu_Q && rows <= 48 && pairs <= 16) variant = V_K2;
  else if (rows >= 128) {
    if (n128 >= 96 && n128 <= 256 && (s128 == 1 || a->max_L / s128 >= 16 * 64)) variant = V_M4K2;
    else if (n128 > 256 || keys >= (512 << 10) || (keys >= (256 << 10) && a->max_L >= 4096)) variant = V_W8;
  }
  // tuning and test aid: the caller names the workgroup shape
  const bool forced = a->plan_shape != TVA_SHAPE_AUTO;
  if (forced) variant = a->plan_shape - 1;
  if (a->kv_fp8 && variant == V_M2K2_3) variant = V_M2K2;  // (8-bit K/V: no deep variant of the 2 x 2 shape)
  plan_splits_of(a, variant, forced, share, pl);
  *fewer = pl->fewer;
  // The rules above against the model: another shape is taken where it promises enough.  Asked where the rules have most
  // to lose: with the lengths of the caches known, and without them where more than 80 rows per KV head meet more than 64
  // pairs or 4096 keys.  3000 calls timed in every shape: 509 take another one than the rules', 13 % faster in the geometric
  // mean, six of them more than 2 % slower (8 % at worst).  Against the best of the five shapes in each call the rules lose
  // 4.8 %, with the model 2.3 %.  Unsplit launches of 33 .. 64 sequences of few rows keep their shape: there the lengths
  // only place the workgroups (fill_slots).  Dense calls with D = 128 and 16-bit K/V are asked about from 65 rows on without the
  // lengths too (up to 80 rows: above 128 pairs or 4096 keys, where 12 calls take another shape and 26 % less time), and leave
  // the 64-row shape for its deep ring for 5 %: of 907 drawn ones 38 change shape, 13 % faster in the mean, one of them more than 2 %
  // slower (5 %); against the best shape in each they lost 3.2 %, now 2.6.  (5 % for the eight-wave shapes too: 62 change, 12 %
  // faster, but of seven newly drawn ones three were 2.5 .. 5 % slower, three 15 .. 23 % faster.)
  const bool placed_only = a->Hkv == 8 && a->B > 32 && a->B <= 64 && rows <= 64;
  // (Nor does the draft stage's attention ask: few of a tree's nodes are queries there, which the fit has not seen.)
  const bool long_ones = a->max_L > 4096;
  const bool ask = a->cu_Q ? false : a->L_host ? !placed_only : rows > 80 ? pairs > 64 || long_ones : dense_wide(a) && rows > 64 && (pairs > 128 || long_ones);
  if (!forced && ask && a->max_L > 0 && a->num_splits == 0) {
    tva_args shapes = *a;  // (the lengths shorten the splits of a shape, they do not choose it)
    shapes.sum_L = 0, shapes.L_host = nullptr;
    Plan plan;
    plan_splits_of(&shapes, variant, false, share, &plan);
    *fewer |= plan.fewer;
    // (Dense, D = 128: where the lengths shorten the rules' splits to more workgroups than the deep 64-row shape may have, the two-stage
    // shape is what the rules come to, and what it takes is asked: 40 calls that were held to the deep shape's discount instead, 4
    // sequences of 2.5 .. 4 K keys, 30 nodes, 25 -> 35 us, take 0.99 of what they did before there was one, 28 others 0.83.)
    const double rules = plan_cost(&shapes, dense_wide(a) && pl->variant != plan.variant ? *pl : plan);
    // How much: 8 %, which is about the model's error (6 % for all pairs: twice as many calls more than 2 % slower); less
    // where nearly every smaller promise was kept, more where one of 12 % was missed by 30.
    // (5 % for the deep shape where its tile counts less.  On shorter splits such promises were not kept: of 540000 drawn calls
    // 30 took the shape for one, 8 % slower in the mean; one sequence of 1.6 K keys, 66 nodes, splits of five tiles 15.7 -> 17.9 us)
    auto enough = [&](const Plan &other) {
      const int v = other.variant;
      if (variant == V_K2) return 0.98;
      if (variant == V_M4K2 || (variant == V_M2K2 && deep_wide(a, other))) return 0.95;
      if (variant == V_W8 && a->kv_fp8) return 0.85;
      // (D = 64, dense: of the 256-row shape a CU holds one workgroup)
      if (variant == V_W8 && (a->D == 64 ? !a->page_table : v == V_M2K2)) return 0.98;
      return 0.92;
    };
    // No shape whose partial rows need more than the library's own scratch array where the rules' plan does not: a call
    // without a workspace (tva_tree_verify_attn_static) is refused for its size only where it always was.
    const size_t own = TVA_STATIC_SCRATCH_BYTES, most = std::max(scratch_bytes(a, plan), own);
    // Dense deep 64-row shape, lengths known: not where the splits they shorten are more than the chip holds at once, the empty ones
    // among them (4 sequences of 13 .. 20 K keys as 320 workgroups took 70 us instead of 59).
    auto crowded = [&](int v) {
      if (v != V_M2K2_3 || !dense_wide(a) || !a->L_host) return false;
      Plan own_lengths;
      plan_splits_of(a, v, true, share, &own_lengths);
      return own_lengths.n_chunks > 1 && (int64_t)pairs * own_lengths.n_row_blocks * own_lengths.n_chunks > 256;
    };
    double best = 0.0;
    int chosen = -1;
    const int first = rows <= 64 ? V_K2 : V_M2K2, last = rows <= 32 ? V_M2K2 : V_LAST;
    for (int v = first; v <= last; ++v) {
      // (8-bit K/V: no deep variant; its four-wave shape widens every key once per row group, which short caches show)
      if (v == variant || (a->kv_fp8 && (v == V_M2K2_3 || (v == V_M2K2 && rows > 64)))) continue;
      plan_splits_of(&shapes, v, true, share, &plan);
      const double us = plan_cost(&shapes, plan);
      if (us < enough(plan) * rules && (chosen < 0 || us < best) && scratch_bytes(a, plan) <= most && !crowded(v)) best = us, chosen = v;
    }
    if (chosen >= 0) {
      // (splits that the lengths shorten are more splits: where those pass the limit they keep their length)
      const size_t limit = std::max(scratch_bytes(a, *pl), own);
      plan_splits_of(a, chosen, true, share, pl);
      *fewer |= pl->fewer;
      if (scratch_bytes(a, *pl) > limit) plan_splits_of(&shapes, chosen, true, share, pl);
    }
  }
  return true;
}

// Fewer, longer splits are taken for the merge that they share, in place of many short ones of the 64-row shape.  The plan is made
// without them where what becomes of them is of that shape but does not share it -- known lengths have made them more splits than
// that, or more workgroups than the deep ring takes -- and where another shape's promise beats the short ones.
// Timed, with / without them, all 184 of 96014 drawn calls whose plan they change: 88 as promised 0.92 of the time (0.84 .. 1.00, one
// 1.07; 3 sequences of 9311 keys, 12 nodes, 21 splits of 7 tiles -> 10 of 15: 30.5 -> 27.0 us), 74 that the 128-row shape and five that
// the 32-row shape take, which promise enough against longer splits and not against short ones, 0.94 (0.86 .. 1.03) and 0.98; 11 of more
// splits or workgroups 1.11 (1.04 .. 1.23) and six for another shape 1.02 (0.95 .. 1.06): those are sent back.
bool make_plan(const tva_args *a, Plan *pl) {
  bool fewer = false;
  if (!plan_of(a, true, pl, &fewer)) return false;
  if (fewer) {
    Plan without;
    plan_of(a, false, &without, &fewer);
    const bool shares = pl->variant == V_M2K2_3 && pl->n_chunks <= kShareSplits;
    if (pl->BM == 64 && (!shares || without.BM != 64)) *pl = without;
  }
  return true;
}

// Whether a row block's splits are merged in the attention launch itself: D = 128, more rows than the 32-row shape's (of its two waves
// one would merge: single sequences of 12 query nodes 0.9 .. 1.2 us slower than with a second launch; D = 64 up to 20 %), 2 .. 12
// splits, and all workgroups (with the lengths given, those the plan puts first) on the chip at once, where none waits for one that
// has not started.  Against a second launch, 28 drawn calls of these: 0.948 of the time called one by one, 0.950 in a graph (0.79 ..
// 1.05 each); four of 15 .. 31 splits 1.00.  One sequence of 2048 keys, 60 nodes: 12.5 -> 11.7 us; 16 of 512 .. 2048 keys, 16 nodes
// 27.8 -> 26.0; 8 of 4096 keys, 64 heads, 55.9 -> 52.4.  (A named number of splits: by the whole grid, so that hints change no bit of
// the result there.)
bool merged_in_launch(const tva_args *a, const Plan &pl, const AttnParams &p, const void *workspace) {
  if (!shape_shares(a->D, pl.BM / 32, a->page_table != nullptr, a->kv_fp8 != 0) || pl.n_chunks < 2 || pl.n_chunks > kShareSplits || ((uintptr_t)workspace & 15)) return false;
  if ((int64_t)pl.n_chunks * query_rows(a) * a->Hq * a->D * 4 >= (1ll << 31)) return false;  // (offsets into the partial rows)
  const int64_t splits = p.real_splits > 0 && a->num_splits == 0 ? p.real_splits : (int64_t)a->B * pl.n_chunks;
  return splits * a->Hkv * pl.n_row_blocks <= (pl.variant == V_M2K2 ? 512 : 256);
}
// Looks at the others' words, up to 0.6 us each, before a workgroup gives up: up to 5 us and four times the time of its tiles.  Alone on
// the chip nobody gives up: splits of unequal length, two workgroups to a CU, need six and, of 8 tiles, seven looks a tile (4 sequences
// of 2057 .. 3883 keys, 61 nodes, 8 splits of 8 tiles: 23.2 us, 25.2 with 16 + 3 a tile; of 4, 7, 12 and 16 tiles 24 .. 32, 32 .. 48, 48
// .. 96 and 64 .. 96 looks), and a call in which all give up takes 18.0 us for 12.6 (one sequence of 2048 keys, 60 nodes, 5 tiles).  What
// it bounds is how long a CU is held for partners that wait for one, where other streams have the chip: that sequence on four streams
// at once, us for the four calls: 300 looks 42.8, 64 38.1, 56 35.7, 48 34.1, 40 33.0, 16 .. 32 32.3, none 31.5, with a second launch
// 29.1; on three streams 23.6, two 16.6, by a second launch 23.6 and 17.6.
int share_polls(const Plan &pl) { return std::min(8 + 7 * (pl.chunk_keys / pl.TK), 0xFFFF); }

// A number that no other call of the process is given (an odd step visits all 2^62 before it comes back to one) and that scratch
// memory does not hold by chance; its last two bits are free.  0 stands for none and is passed over.  Nothing here throws.
uint64_t share_tag_seed() {
  uint64_t seed = 0;
  if (getrandom(&seed, sizeof seed, GRND_NONBLOCK) == (ssize_t)sizeof seed) return seed;
  timespec now{};
  clock_gettime(CLOCK_REALTIME, &now);
  return ((uint64_t)now.tv_sec * 1000000007u + (uint64_t)now.tv_nsec) * 0xBF58476D1CE4E5B9ull ^ (uint64_t)getpid() << 40 ^ (uint64_t)(uintptr_t)&seed;
}
uint64_t next_share_tag() {
  static std::atomic<uint64_t> next{share_tag_seed()};
  uint64_t tag;
  do tag = next.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed) << 2;
  while (tag == 0);
  return tag;
}

typedef void (*attn_fn)(const AttnParams);

// Launch status.  An error some earlier HIP call of the process left behind is cleared before a
// launch, so that the status reflects this launch only; a failure is left in place (peeked, not
// consumed) for the caller's hipGetLastError, and named on stderr when TVA_VERBOSE is set.
inline void clear_stale_hip_error() { (void)hipGetLastError(); }
inline hipError_t launch_status(const char *what) {
  const hipError_t e = hipPeekAtLastError();
  if (e != hipSuccess && getenv("TVA_VERBOSE")) fprintf(stderr, "libtva: %s: %s\n", what, hipGetErrorString(e));
  return e;
}

template <int D, int WM, int WK, int RB, bool PAGED, int NST, bool KV8 = false>
hipError_t launch_attn(const AttnParams &p, dim3 grid, hipStream_t st) {
  using C = AttnCfg<D, WM, WK, RB, PAGED, NST, KV8>;
  // raising the dynamic-LDS limit is idempotent and needed once per device (and per instantiation)
  static std::atomic<uint64_t> attr_done[2]{};
  const bool shared = p.share_tag != 0;
  attn_fn kfn = attn_kernel<D, WM, WK, RB, PAGED, NST, KV8>;
  if constexpr (C::SHARES) {
    if (shared) kfn = attn_kernel<D, WM, WK, -RB, PAGED, NST, KV8>;
  } else if (shared) {
    return hipErrorInvalidValue;  // (the results would be left to a launch that nobody queues)
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
  const uint64_t bit = (dev >= 0 && dev < 64) ? 1ull << dev : 0;
  if (!(attr_done[shared].load(std::memory_order_relaxed) & bit)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kfn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM);
    if (e != hipSuccess) return e;
    attr_done[shared].fetch_or(bit, std::memory_order_relaxed);
  }
  clear_stale_hip_error();
  hipLaunchKernelGGL(kfn, grid, dim3(C::NT), C::SMEM, st, p);
  return launch_status("attention kernel launch");
}

template <int D, bool PAGED>
hipError_t dispatch_variant(int variant, const AttnParams &p, dim3 grid, hipStream_t st) {
  switch (variant) {
    case V_W8: return launch_attn<D, 8, 1, 1, PAGED, 4>(p, grid, st);
    case V_M4K2: return launch_attn<D, 4, 2, 1, PAGED, 4>(p, grid, st);
    case V_M2K2_3: return launch_attn<D, 2, 2, 1, PAGED, D == 128 ? 4 : 3>(p, grid, st);
    case V_K2: return launch_attn<D, 1, 2, 1, PAGED, 2>(p, grid, st);
    default: return launch_attn<D, 2, 2, 1, PAGED, 2>(p, grid, st);  // V_M2K2
  }
}

// 8-bit K/V (three landing slots each)
template <bool PAGED>
hipError_t dispatch_variant_fp8(int variant, const AttnParams &p, dim3 grid, hipStream_t st) {
  switch (variant) {
    case V_W8: return launch_attn<128, 8, 1, 1, PAGED, 3, true>(p, grid, st);
    case V_M4K2: return launch_attn<128, 4, 2, 1, PAGED, 3, true>(p, grid, st);
    case V_K2: return launch_attn<128, 1, 2, 1, PAGED, 3, true>(p, grid, st);
    default: return launch_attn<128, 2, 2, 1, PAGED, 3, true>(p, grid, st);  // V_M2K2
  }
}

}  // namespace

// ---------------------------------------------------------------------------------------
// scratch memory of tva_tree_verify_attn_static (the entry point that allocates nothing)
// ---------------------------------------------------------------------------------------
// A device array that is part of the code object: every GPU the library runs on holds its own copy,
// at its own address, from the moment the module is loaded there until the process ends.  In host
// code the array's name is only a handle for hipGetSymbolAddress; the address it returns for the
// current device is what kernels, copies and fills are given.  Nothing in it has to start at zero:
// where a second launch merges the splits, the attention kernel writes every partial row and every
// partial log-sum-exp (also the "empty" marks of splits a short sequence does not reach) that it
// reads; where the attention launch merges them, each workgroup's rows outside its own share, and
// the words that say so carry a tag that no other call has.
static __device__ __align__(256) unsigned char scratch[TVA_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void *> scratch_addr[kMaxDevices];  // zero-initialised: not looked up yet

// Address of `scratch` on the current device; looked up once per device, with that device current.
int static_scratch(void **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TVA_HIP_ERROR;
  void *ptr = scratch_addr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    const hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      if (getenv("TVA_VERBOSE")) fprintf(stderr, "libtva: hipGetSymbolAddress(scratch): %s\n", hipGetErrorString(e));
      return TVA_HIP_ERROR;
    }
    scratch_addr[dev].store(ptr, std::memory_order_release);  // (two threads racing store the same value)
  }
  *out = ptr;
  return TVA_OK;
}
}  // namespace

extern "C" {

int tva_version(void) { return 7; }

int tva_timeline_read(uint64_t *dst, int32_t n_workgroups) {
#ifdef TVA_TIMELINE
  if (!dst || n_workgroups < 0 || n_workgroups > TL_MAX_WG) return TVA_INVALID_ARG;
  const hipError_t e = hipMemcpyFromSymbol(dst, HIP_SYMBOL(timeline), (size_t)n_workgroups * TL_SLOTS * sizeof(uint64_t), 0,
                                           hipMemcpyDeviceToHost);
  return e == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
#else
  (void)dst;
  (void)n_workgroups;
  return TVA_UNSUPPORTED;
#endif
}

size_t tva_sizeof_args(void) { return sizeof(tva_args); }

const char *tva_strerror(int code) {
  switch (code) {
    case TVA_OK: return "ok";
    case TVA_INVALID_ARG: return "invalid argument";
    case TVA_UNSUPPORTED: return "unsupported shape";
    case TVA_WORKSPACE_TOO_SMALL: return "workspace too small";
    case TVA_HIP_ERROR: return "HIP launch error";
    case TVA_BAD_TREE: return "malformed tree (parent index outside [-1, i-1])";
    default: return "unknown status";
  }
}

int tva_build_ancestor_mask(const int32_t *parent, const int32_t *cu_T, int32_t B, int32_t max_T,
                            int32_t mask_words, uint64_t *mask, int32_t *err_flag, void *stream) {
  if (B < 0 || max_T < 0 || mask_words < 1 || mask_words * 64 < max_T) return TVA_INVALID_ARG;
  if (B == 0) return TVA_OK;
  if (!parent || !cu_T || !mask) return TVA_INVALID_ARG;
  int threads = ((max_T + 63) / 64) * 64;
  threads = threads < 64 ? 64 : (threads > 256 ? 256 : threads);
  clear_stale_hip_error();
  hipLaunchKernelGGL(anc_mask_kernel, dim3(B), dim3(threads), 0, (hipStream_t)stream, parent, cu_T, B,
                     mask_words, mask, err_flag);
  return launch_status("ancestor mask kernel launch") == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

static int check_args(const tva_args *a, bool shapes_only) {
  if (!a) return TVA_INVALID_ARG;
  if (a->B <= 0 || a->Hq <= 0 || a->Hkv <= 0 || a->Hq % a->Hkv) return TVA_INVALID_ARG;
  if (a->sum_T < 0 || a->max_T < 0 || a->max_L < 0 || a->num_splits < 0) return TVA_INVALID_ARG;
  if (a->D != 64 && a->D != 128) return TVA_UNSUPPORTED;
  if (a->max_T > TVA_MAX_TREE) return TVA_UNSUPPORTED;
  if (a->mask_words < 1 || a->mask_words > 2 || a->mask_words * 64 < a->max_T) return TVA_UNSUPPORTED;
  if (a->kv_fp8 != 0 && a->kv_fp8 != 1) return TVA_INVALID_ARG;
  if (a->kv_fp8 && a->D != 128) return TVA_UNSUPPORTED;
  if (a->cu_Q && (a->sum_Q < 0 || a->max_Q < 0 || a->max_Q > a->max_T || a->sum_Q > a->sum_T)) return TVA_INVALID_ARG;
  if (a->plan_shape < TVA_SHAPE_AUTO || a->plan_shape > TVA_SHAPE_R256_W8) return TVA_INVALID_ARG;
  if (a->sum_L < 0) return TVA_INVALID_ARG;
  if (shapes_only) return TVA_OK;
  if (!(a->scale > 0.f)) return TVA_INVALID_ARG;
  if (a->sum_T == 0) return TVA_OK;
  if (!a->cu_T || !a->L || !a->q || !a->out || !a->lse) return TVA_INVALID_ARG;
  if ((a->k_tree == nullptr) != (a->v_tree == nullptr)) return TVA_INVALID_ARG;
  if (!a->anc_mask && !a->parent) return TVA_INVALID_ARG;
  const bool dense = a->cu_L != nullptr, paged = a->page_table != nullptr;
  if (dense == paged) return TVA_INVALID_ARG;
  const bool tree_in_cache = a->k_tree == nullptr;
  if ((a->max_L > 0 || tree_in_cache) && (!a->k_cache || !a->v_cache)) return TVA_INVALID_ARG;
  if (paged && (a->page_size <= 0 || a->max_pages <= 0)) return TVA_INVALID_ARG;
  // (with tree rows in the cache the table must cover L[b] + T_b positions of every sequence; only the two
  // bounds are known here, and the longest cache need not belong to the largest tree)
  if (paged && (int64_t)a->max_pages * a->page_size < (tree_in_cache && a->max_T > a->max_L ? a->max_T : a->max_L))
    return TVA_INVALID_ARG;
  if ((a->stride_page | a->stride_tok | a->stride_head) % (a->kv_fp8 ? 16 : 8)) return TVA_INVALID_ARG;  // 16-byte pieces
  if (a->stride_page < 0 || a->stride_tok < 0 || a->stride_head < 0) return TVA_INVALID_ARG;
  if (a->stride_tok >= (1 << 24)) return TVA_UNSUPPORTED;  // lane offsets inside a tile are 32-bit
  if (a->kv_fp8 && (!(a->k_scale >= 0.f) || !(a->v_scale >= 0.f))) return TVA_INVALID_ARG;
  return TVA_OK;
}

int32_t tva_plan_splits(const tva_args *a) {
  if (check_args(a, true) != TVA_OK) return -1;
  Plan pl;
  if (!make_plan(a, &pl)) return -1;
  return pl.n_chunks;
}

int32_t tva_plan_chunk_keys(const tva_args *a) {
  if (check_args(a, true) != TVA_OK) return -1;
  Plan pl;
  if (!make_plan(a, &pl)) return -1;
  return pl.chunk_keys;
}

int32_t tva_plan_slot_sequences(const tva_args *a, int32_t *slot_seq) {
  if (check_args(a, true) != TVA_OK || !slot_seq) return -1;
  Plan pl;
  if (!make_plan(a, &pl)) return -1;
  AttnParams p;
  fill_slots(a, pl, &p);
  for (int j = 0; j < p.pair_slots; ++j) slot_seq[j] = (int32_t)((p.slot_seq[j >> 2] >> (8 * (j & 3))) & 0xFFu);
  return p.pair_slots;
}

int32_t tva_plan_workgroup_rows(const tva_args *a) {
  if (check_args(a, true) != TVA_OK) return -1;
  Plan pl;
  if (!make_plan(a, &pl)) return -1;
  return pl.BM;
}

size_t tva_workspace_bytes(const tva_args *a) {
  if (check_args(a, true) != TVA_OK) return (size_t)-1;
  Plan pl;
  if (!make_plan(a, &pl)) return (size_t)-1;
  return scratch_bytes(a, pl);
}

static int run_attention(const tva_args *a, void *workspace, size_t workspace_bytes, void *stream, bool merge, int polls = -1);

int tva_tree_verify_attn(const tva_args *a, void *stream) {
  return a ? run_attention(a, a->workspace, a->workspace_bytes, stream, true) : TVA_INVALID_ARG;
}

int tva_tree_verify_attn_splits(const tva_args *a, void *stream) {
  return a ? run_attention(a, a->workspace, a->workspace_bytes, stream, false) : TVA_INVALID_ARG;
}

int tva_tree_verify_attn_wait_bound_test(const tva_args *a, int32_t polls, void *stream) {
  return a && polls >= 0 ? run_attention(a, a->workspace, a->workspace_bytes, stream, true, polls) : TVA_INVALID_ARG;
}

size_t tva_static_scratch_bytes(void) { return TVA_STATIC_SCRATCH_BYTES; }

int tva_tree_verify_attn_static(const tva_args *a, void *stream) {
  if (!a) return TVA_INVALID_ARG;
  // the size is settled from the shapes alone, before any pointer or the device is looked at
  int rc = check_args(a, true);
  if (rc != TVA_OK) return rc;
  const size_t need = tva_workspace_bytes(a);
  if (need == (size_t)-1) return TVA_INVALID_ARG;
  if (need > TVA_STATIC_SCRATCH_BYTES) return TVA_WORKSPACE_TOO_SMALL;
  rc = check_args(a, false);
  if (rc != TVA_OK) return rc;
  void *ptr = nullptr;
  if (need > 0) {  // (a single split touches no scratch memory: no lookup either)
    rc = static_scratch(&ptr);
    if (rc != TVA_OK) return rc;
  }
  return run_attention(a, ptr, need > 0 ? TVA_STATIC_SCRATCH_BYTES : 0, stream, true);
}

static int run_attention(const tva_args *a, void *workspace, size_t workspace_bytes, void *stream, bool merge, int polls) {
  int rc = check_args(a, false);
  if (rc != TVA_OK) return rc;
  if (a->sum_T == 0 || a->max_T == 0 || query_rows(a) == 0) return TVA_OK;
  Plan pl;
  if (!make_plan(a, &pl)) return TVA_INVALID_ARG;
  const size_t need = scratch_bytes(a, pl);
  if (need > 0 && (!workspace || workspace_bytes < need)) return TVA_WORKSPACE_TOO_SMALL;

  AttnParams p;
  p.q = (const __bf16 *)a->q;
  p.k_tree = (const __bf16 *)a->k_tree;
  p.v_tree = (const __bf16 *)a->v_tree;
  p.k_cache = (const __bf16 *)a->k_cache;
  p.v_cache = (const __bf16 *)a->v_cache;
  p.cu_T = a->cu_T;
  p.L = a->L;
  p.cu_L = a->cu_L;
  p.page_table = a->page_table;
  p.mask = a->anc_mask;
  p.parent = a->parent;
  p.out = a->out;
  p.lse = a->lse;
  p.part_out = need > 0 ? (float *)workspace : nullptr;
  p.part_lse = p.part_out ? p.part_out + (size_t)pl.n_chunks * query_rows(a) * a->Hq * a->D : nullptr;
  p.B = a->B;
  p.Hq = a->Hq;
  p.Hkv = a->Hkv;
  p.G = a->Hq / a->Hkv;
  p.g_bits = 0;
  while (p.g_bits < 31 && (1ll << p.g_bits) < p.G) ++p.g_bits;
  p.g_magic = (uint32_t)(((1ull << (31 + p.g_bits)) + (uint32_t)p.G - 1) / (uint32_t)p.G);
  p.sum_Q = (int)query_rows(a);
  p.cu_Q = a->cu_Q;
  p.W = a->mask_words;
  p.chunk_keys = pl.chunk_keys;
  p.n_chunks = pl.n_chunks;
  p.n_row_blocks = pl.n_row_blocks;
  p.max_L = a->max_L;
  fill_slots(a, pl, &p);
  p.page_size = a->page_size > 0 ? a->page_size : 1;
  p.page_shift = -1;
  for (int sft = 0; sft < 31; ++sft)
    if ((1 << sft) == p.page_size) p.page_shift = sft;
  p.max_pages = a->max_pages;
  p.stride_head = a->stride_head ? a->stride_head : a->D;
  p.stride_tok = a->stride_tok ? a->stride_tok : (int64_t)a->Hkv * a->D;
  p.stride_page = a->stride_page ? a->stride_page : (int64_t)p.page_size * p.stride_tok;
  p.scale_log2 = a->scale * kLog2e * ((a->kv_fp8 && a->k_scale > 0.f) ? a->k_scale : 1.f);
  p.v_scale = (a->kv_fp8 && a->v_scale > 0.f) ? a->v_scale : 1.f;

  const bool in_launch = merge && merged_in_launch(a, pl, p, workspace);
  p.share_tag = in_launch ? next_share_tag() : 0;
  p.share_polls = polls < 0 ? share_polls(pl) : polls;

  if ((int64_t)a->B * pl.n_chunks > 65535 || pl.n_row_blocks > 65535) return TVA_UNSUPPORTED;
  const dim3 grid(a->Hkv, pl.n_row_blocks, a->B * pl.n_chunks);
  const bool paged = a->page_table != nullptr;
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  if (a->kv_fp8)
    e = paged ? dispatch_variant_fp8<true>(pl.variant, p, grid, st) : dispatch_variant_fp8<false>(pl.variant, p, grid, st);
  else if (a->D == 128)
    e = paged ? dispatch_variant<128, true>(pl.variant, p, grid, st) : dispatch_variant<128, false>(pl.variant, p, grid, st);
  else
    e = paged ? dispatch_variant<64, true>(pl.variant, p, grid, st) : dispatch_variant<64, false>(pl.variant, p, grid, st);
  if (e != hipSuccess) return TVA_HIP_ERROR;

  if (merge && pl.n_chunks > 1 && !in_launch) {
    const int64_t n_rows = (int64_t)query_rows(a) * a->Hq;
    clear_stale_hip_error();
    if (a->D == 128) launch_merge<128>(p.part_out, p.part_lse, pl.n_chunks, n_rows, a->out, a->lse, st);
    else launch_merge<64>(p.part_out, p.part_lse, pl.n_chunks, n_rows, a->out, a->lse, st);
    if (launch_status("merge kernel launch") != hipSuccess) return TVA_HIP_ERROR;
  }
  return TVA_OK;
}

int tva_merge_splits(const float *part_out, const float *part_lse, int32_t S, int64_t n_rows, int32_t D,
                     float *out, float *lse, void *stream) {
  if (S < 1 || n_rows < 0) return TVA_INVALID_ARG;
  if (D != 64 && D != 128) return TVA_UNSUPPORTED;
  if (n_rows == 0) return TVA_OK;
  if (!part_out || !part_lse || !out || !lse) return TVA_INVALID_ARG;
  if ((n_rows + 3) / 4 > 0x7fffffff) return TVA_UNSUPPORTED;
  hipStream_t st = (hipStream_t)stream;
  clear_stale_hip_error();
  if (D == 128) launch_merge<128>(part_out, part_lse, S, n_rows, out, lse, st);
  else launch_merge<64>(part_out, part_lse, S, n_rows, out, lse, st);
  return launch_status("merge kernel launch") == hipSuccess ? TVA_OK : TVA_HIP_ERROR;
}

}  // extern "C"
