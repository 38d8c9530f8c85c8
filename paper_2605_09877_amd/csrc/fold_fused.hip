// A run of folds in one launch (bf16, head_dim 128), one workgroup or several per (sequence, KV head) unit.
//
// A fold (sections "Append", "Merge" and the readout equations of the paper's Method section) is a
// chain of small dependent steps: similarity of the block to the normalised state, selection of
// the tokens to append, creation of their rows, similarity of the remaining tokens to the new
// rows, winner-take-all accumulation, readout refresh.  Units are independent of each other, and
// consecutive folds of one unit depend on each other through that unit's state alone, so the
// workgroups of a unit walk it through all of a run's folds with workgroup barriers between the steps:
// no launch boundaries inside the chain and none between its folds.  Two shapes of workgroup: 16
// waves with up to 160 KiB of LDS when the folds have the chip to themselves (a prefill whose folds
// outweigh its attention); 8 waves at 128 registers and under 96 KiB when they run beside a
// prefill's attention launches, whose workgroups leave room for exactly that on a compute unit (a
// larger workgroup would wait until a unit has drained, which a running attention launch never
// lets happen).  Per fold:
//   1. the block's memory keys k-bar = LN_s(zero_r(k)), computed by a launch of their own ahead of
//      the run (they depend on k alone, so they are not part of the chain), are read as matrix-core
//      operands by the wave that owns the 32 tokens, while the fold before merges;
//   2. D[row, token] = K-hat_tile . K-bar^T on the matrix cores, 64 state rows at a time: append
//      score s_j = max over all rows, merge target = argmax over rows >= S (a lane owns a token and
//      scans rows in ascending order: ties keep the lowest row).  The K-hat tiles stay in LDS for
//      the whole run where they fit, kept up to date by steps 3 and 5; otherwise they stream from
//      HBM / L2 through a ring of two stages;
//   3. when the budget has room for some of the block: the n_append smallest (s_j, j) are taken,
//      their rows are created, and step 2 runs again over the new rows for the tokens that were
//      not taken (a strictly larger score moves a token);
//   4. every merging token pushes itself on its target row's list in LDS (an exchange on the
//      row's head); the token that finds the list empty enters the row in the list of touched rows;
//      the tokens' memory keys and values are loaded straight into LDS, all at once;
//   5. 16 lanes per touched row (8 channels each): the sums are asked for, the row's list is
//      walked, its tokens are added in ascending position, sums and the readout row (LN_s in
//      fp64 on keys, stored radius on values) are written; rows nothing was added to are copied
//      to the new state version (prefill; with resident tiles during the next fold's exchange,
//      where nothing waits for it) or left alone (in place).
// Integer decisions rest on fp64 LN_s and fp64 key sums, as everywhere in this library.
//
// With fewer units than compute units one workgroup per unit leaves most of the chip idle, so a
// unit is given `split` workgroups (a power of two) that divide its state rows among them in
// 64-row tiles, tile t belonging to workgroup t mod split: a workgroup scores the whole block
// against its own rows, merges the tokens bound for its own rows and copies its own untouched
// rows; the normalised keys of new rows every workgroup makes for itself.  Everything a workgroup
// reads of the state it wrote itself, so the only data that crosses workgroups is each token's
// partial winner: one exchange per fold through a small table in global memory.  An entry is one
// 64-bit word (score, row, a 16-bit tag of the exchange it belongs to) written and read with relaxed
// device-scope atomics: no fences, no flags beside the data; a reader spins on the tag.
//
// Workgroups that wait for each other must all be running, and nothing promises that they are: there may be
// fewer compute units than expected, or others' work on them.  So before any of them touches the
// state they count themselves in (meet()), and when a unit's last one has not started within a time limit,
// one of those that have takes the whole unit, as with one workgroup per unit, and the others leave,
// late ones included.  Either way the fold's results are the same bits.  After that a workgroup waits for
// running ones only, whose next exchange entry depends on nothing but entries already due: every wait ends, whatever
// else the chip is doing.
//
// What bounds it: with shared rows, latency.  A fold of a 256-token block into some 300 rows (32 units x
// 8 workgroups) takes 15 us without an append and 18 us with one of a few rows, 23 us on average beside attention: scores and copies of
// the fold before 6.5, exchange 1, lists 1.5, merge 5.5 (of which a round trip to the sums 2), another 4 to select, create and
// score again.  A kernel per step took 38 us and 62 us for the same.  Prefill of 65536 tokens with a growing state
// (B 2 x H 16, 256-token blocks): 10.6 to 13.5 ms with a kernel per step (the box decides), 7.6 shared, 6.35 with one
// attention workgroup beside each of these and runs of eight folds, 5.95 with few new rows selected one by one; a
// layer's 16384 tokens with 512 rows: 3.3, 2.7 and 2.3 ms.  With one workgroup per unit (256 units and more)
// by the tiles' and rows' traffic: B 16 x H 16, 8192 tokens, 5.06 ms before, 4.61 ms
// (keys of the next run computed beside the folds, gathered tokens, no separate copy pass).
#include <cstddef>

#include <hip/hip_ext.h>

#include "kvm_device.h"
#include "kvm_internal.h"
#include "kvm_mfma.h"

namespace kvm {

namespace {

constexpr int kNoRow = 0x7fffffff;
constexpr int kTileBytes = kTileElems * 2;   // 16 KiB
constexpr int kListMax = 16;                 // tokens of a row taken from its list in one go
constexpr uint32_t kTokenBytes = 2 * kHeadDim * 2;   // memory key and value of a token
// NW waves per workgroup; a stage of the K-hat stream is NW / 4 tiles, two stages are in LDS.  A workgroup that takes
// over a unit meant for several has the LDS of its share: stages of one tile, and the scratch is those two.
__host__ __device__ constexpr int stage_tiles(int NW) { return NW / 4; }
constexpr int kStageTaken = 1, kGatherTaken = (int)(2 * kStageTaken * kTileBytes / kTokenBytes);

// LN_s parameters when the caller gave none (gamma = 1, beta = 0): read like given ones, so that
// the kernels carry no per-element branches.
__device__ const float kOnes[kHeadDim] = {
    1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1,
    1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1,
    1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1,
    1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1};
__device__ const float kZeros[kHeadDim] = {};

__device__ __forceinline__ bool beats(float sa, int ia, float sb, int ib) {
  return sa > sb || (sa == sb && ia < ib);
}

// LDS layout of one workgroup, bytes from the start of dynamic shared memory.  Everything is a fixed
// offset plus a multiple of C, so that no table of offsets has to be kept in registers.  "Local"
// rows are the rows of this workgroup's own 64-row tiles, numbered through (all rows when a unit
// has one workgroup).
//   0                   int [8] counters
//   kLdsMerge           float/int [3][NW * 32] partial winners of waves that share tokens; then the block's merge gates
//   tables(NW)          eight arrays of C words: append score s_j, winning merge score, target row, rank among
//                       the appended tokens or -1, next token on the same row's list or -1, token that creates
//                       new row number a (later: where a merging token has been gathered to), local rows
//                       that receive tokens (before that: near ties), the gathered tokens
//   then                int [local rows] last token pushed on the row's list or -1
//   then (1-KiB bound)  scratch, one use after the other: the fresh tile (K-hat of the rows this fold creates); the
//                       gathered tokens' memory keys and values
//   then                K-hat tiles: this workgroup's own for the whole run (resident); otherwise a ring of two
//                       stages, which is the scratch as well (it is idle when that is needed)
constexpr uint32_t kLdsCounters = 0, kLdsMerge = kLdsCounters + 32;
__host__ __device__ constexpr uint32_t lds_tables(int NW) { return kLdsMerge + 3u * 4u * NW * 32; }
__host__ __device__ constexpr uint32_t lds_fresh(int NW, int C, int own_tiles) {
  return (lds_tables(NW) + 32u * C + 4u * kTileKeys * own_tiles + 1023u) & ~1023u;
}
__host__ __device__ inline int own_tiles_most(int Mcap, int split) { return (Mcap / kTileKeys + split - 1) / split; }

template <int NW>
struct Ctx {
  unsigned char *smem;
  int C;                    // tokens of a block
  uint32_t fresh_at;        // LDS offset of the scratch
  int gather;               // tokens the scratch can hold (memory key and value)
  int u, tid, lane, wave;
  int part, split, shift;   // this workgroup's number among the unit's workgroups, how many they are, log2 of that
  bool resident;            // its K-hat tiles stay in LDS for the whole run
  int stage;                // otherwise: tiles per stage of the ring, a power of two
  // the workgroup that owns a state row: 64-row tiles dealt round robin
  __device__ bool owns(int row) const { return ((row >> 6) & (split - 1)) == part; }
  __device__ int local(int row) const { return ((row >> (6 + shift)) << 6) | (row & 63); }
  __device__ int global(int lr) const { return ((((lr >> 6) << shift) + part) << 6) | (lr & 63); }
  // local rows that exist when the state has m rows
  __device__ int n_local(int m) const {
    const int t = m >> 6, own = t > part ? (t - part + split - 1) >> shift : 0;   // whole tiles of this workgroup
    return 64 * own + ((m & 63) && (t & (split - 1)) == part ? (m & 63) : 0);
  }
  template <typename V>
  __device__ V *table(int k) const { return (V *)(smem + lds_tables(NW) + 4u * k * C); }
  __device__ uint16_t *s_fresh() const { return (uint16_t *)(smem + fresh_at); }
  __device__ uint16_t *s_tiles() const { return (uint16_t *)(smem + fresh_at + (resident ? (uint32_t)gather * kTokenBytes : 0u)); }
  __device__ uint16_t *s_keys(int slot) const { return (uint16_t *)(smem + fresh_at) + slot * kHeadDim; }
  __device__ uint16_t *s_vals(int slot) const { return (uint16_t *)(smem + fresh_at) + (gather + slot) * kHeadDim; }
  __device__ float *s_app() const { return table<float>(0); }
  __device__ float *s_best() const { return table<float>(1); }
  __device__ int *s_pi() const { return table<int>(2); }
  __device__ int *s_rank() const { return table<int>(3); }
  __device__ int *s_next() const { return table<int>(4); }
  __device__ int *s_creator() const { return table<int>(5); }
  __device__ int *s_rows() const { return table<int>(6); }
  __device__ int *s_slot() const { return table<int>(5); }
  __device__ int *s_own() const { return table<int>(7); }
  __device__ int *s_head() const { return table<int>(8); }
  // the block's merge gates, while its tokens merge: where the partial winners were, if they fit there
  __device__ bool gates_in_lds() const { return C <= 3 * NW * 32; }
  __device__ float *s_gate() const { return (float *)(smem + kLdsMerge); }
  __device__ int *s_cnt() const { return (int *)(smem + kLdsCounters); }
  __device__ unsigned char *s_merge() const { return smem + kLdsMerge; }
};
// counters: touched rows, near ties of the append, own merging tokens, who folds the unit, (stamps)
enum { kCntRows = 0, kCntTies = 1, kCntOwn = 2, kCntMeet = 3, kCntStamps = 4 };
enum { kShared = 0, kWhole = 1, kLeave = 2 };   // with the others; this workgroup by itself; one of the others

// Development aid (compiled in only with -DKVM_FOLD_STAMPS): the first workgroup leaves the clock
// at its phase boundaries in the `creator` scratch, which this path does not use.
#ifdef KVM_FOLD_STAMPS
#define FOLD_STAMP()                                                                        \
  do {                                                                                      \
    if (blockIdx.x == 0 && threadIdx.x == 0 && cx.s_cnt()[kCntStamps] < 240)                         \
      reinterpret_cast<long long *>(args_now().dv.creator)[cx.s_cnt()[kCntStamps]++] = (long long)wall_clock64(); \
  } while (0)
#else
#define FOLD_STAMP() \
  do {               \
  } while (0)
#endif

// ------------------------------------------------------------------------------------------------
// The exchange after the scoring pass (split > 1): every workgroup of the unit publishes its own
// winners and reads the others'; all of them end up with the same unit-wide result in LDS.
// Table, behind the arrival words: [unit][exchange parity][workgroup][2][C] 64-bit words; word 0 of a token = (merge score,
// row in 16 bits, tag), word 1 = (append score, tag), the latter only from workgroups that own sink rows (elsewhere
// every row may win, and the two scores are one).  A workgroup cannot be two exchanges ahead of
// a sibling (it needs the sibling's entries of the exchange in between), so two parities suffice.
// tag: the exchange's number, 16 bits; the host zeroes the table before numbers repeat, and 0 is never a tag.
__device__ __forceinline__ unsigned long long *exchange_table(const Dev &dv, const FoldRunArgs &run) {
  return run.xtab + (size_t)dv.U * kArrivalWords;
}
__device__ __forceinline__ unsigned long long xchg_pack(float score, uint32_t low16, uint32_t tag) {
  return ((unsigned long long)__float_as_uint(score) << 32) | ((unsigned long long)(low16 & 0xffffu) << 16) |
         (unsigned long long)(tag & 0xffffu);
}
template <int kCtrl>
__device__ __forceinline__ int dpp_int(int x) {
  return (int)__builtin_amdgcn_mov_dpp((uint32_t)x, kCtrl, 0xF, 0xF, true);
}
// whether workgroup `part` owns rows below the number of sinks (tile t belongs to workgroup t mod split)
__device__ __forceinline__ bool sink_owner(const Dev &dv, int part) { return part < (dv.S + kTileKeys - 1) / kTileKeys; }
__device__ __forceinline__ void publish_winner(unsigned long long *mine, int C, int j, float best, int best_i, float all,
                                               bool with_all, uint32_t tag) {
  __hip_atomic_store(mine + j, xchg_pack(best, best_i == kNoRow ? 0xffffu : (uint32_t)best_i, tag), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  if (with_all) __hip_atomic_store(mine + C + j, xchg_pack(all, 0, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One entry, waited for (the workgroup that owes it is running: meet()).
__device__ __forceinline__ unsigned long long xchg_wait(unsigned long long v, const unsigned long long *p, uint32_t tag) {
  while ((uint32_t)(v & 0xffffu) != tag) {
    __builtin_amdgcn_s_sleep(1);
    v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return v;
}
// Counts this workgroup in at its unit's arrival word (one thread) and says who folds the unit in this launch.  Low half of
// the word: workgroups that have arrived since the table was zeroed, `before` of them in earlier launches; high
// half: the last launch whose unit one workgroup took for itself.  The take is an exchange of the word as it was
// seen incomplete: either it succeeds, and whoever comes or looks later sees this launch's number, or another
// arrival came first.
__device__ __forceinline__ int meet(unsigned long long *word, int split, uint32_t before, uint32_t launch, uint32_t patience) {
  unsigned long long v = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((uint32_t)(v >> 32) == launch) return kLeave;
  v += 1ull;
  const unsigned long long t0 = wall_clock64();   // 100 MHz
  for (;;) {
    if ((uint32_t)(v >> 32) == launch) return kLeave;
    if ((uint32_t)v - before == (uint32_t)split) return kShared;
    if (wall_clock64() - t0 >= patience) {
      const unsigned long long taken = ((unsigned long long)launch << 32) | (uint32_t)v;
      if (__hip_atomic_compare_exchange_strong(word, &v, taken, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        return kWhole;
    } else {
      __builtin_amdgcn_s_sleep(1);
      v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}
// A pair of lanes per token: each reads half of the workgroups' entries, all of them asked for at once
// (a read goes to memory, one or two microseconds away), waits for the stragglers one by one and
// puts them together; then the two halves meet.
template <int NW, int kHalf>   // kHalf: workgroups per lane
__device__ __forceinline__ void exchange_half(const Dev &dv, const Ctx<NW> &cx, const unsigned long long *unit_tab,
                                              uint32_t tag) {
  const int C = cx.C, h = cx.tid & 1;
  const unsigned long long *theirs = unit_tab + (size_t)(h * kHalf) * 2 * C;
  const int n_sinks = (dv.S + kTileKeys - 1) / kTileKeys - h * kHalf;   // how many of this half own sink rows
#pragma unroll 1
  for (int j = cx.tid >> 1; j < C; j += 32 * NW) {
    unsigned long long w0[kHalf], w1 = 0;
#pragma unroll
    for (int o = 0; o < kHalf; ++o)
      w0[o] = __hip_atomic_load(theirs + (size_t)o * 2 * C + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n_sinks > 0) w1 = __hip_atomic_load(theirs + C + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool late = false;
#pragma unroll
    for (int o = 0; o < kHalf; ++o) late = late || (uint32_t)(w0[o] & 0xffffu) != tag;
    if (late) {
#pragma unroll
      for (int o = 0; o < kHalf; ++o) w0[o] = xchg_wait(w0[o], theirs + (size_t)o * 2 * C + j, tag);
    }
    float best = -INFINITY, all = -INFINITY;
    int best_i = kNoRow;
    auto take = [&](float ob, int oi) {
      const bool up = beats(ob, oi, best, best_i);   // (no row: score -inf and the largest number)
      best = up ? ob : best;
      best_i = up ? oi : best_i;
    };
#pragma unroll
    for (int o = 0; o < kHalf; ++o) {
      const uint32_t i16 = (uint32_t)(w0[o] >> 16) & 0xffffu;
      take(__uint_as_float((uint32_t)(w0[o] >> 32)), i16 == 0xffffu ? kNoRow : (int)i16);
    }
    take(dpp_get<0xB1>(best), dpp_int<0xB1>(best_i));   // the other lane of the pair
    // the append score counts sink rows too: their owners say what they are worth
    for (int o = 0; o < n_sinks && o < kHalf; ++o) {
      w1 = xchg_wait(o == 0 ? w1 : 0ull, theirs + ((size_t)o * 2 + 1) * C + j, tag);
      all = fmaxf(all, __uint_as_float((uint32_t)(w1 >> 32)));
    }
    all = fmaxf(fmaxf(all, dpp_get<0xB1>(all)), best);
    if (h == 0) {
      cx.s_app()[j] = all;
      cx.s_best()[j] = best;
      cx.s_pi()[j] = best_i;
      cx.s_rank()[j] = -1;
    }
  }
}
template <int NW>
__device__ __forceinline__ void exchange_winners(const Dev &dv, const Ctx<NW> &cx, const unsigned long long *unit_tab,
                                                 uint32_t tag) {
  switch (cx.split) {
    case 2: exchange_half<NW, 1>(dv, cx, unit_tab, tag); break;
    case 4: exchange_half<NW, 2>(dv, cx, unit_tab, tag); break;
    case 8: exchange_half<NW, 4>(dv, cx, unit_tab, tag); break;
    default: exchange_half<NW, 8>(dv, cx, unit_tab, tag); break;
  }
}

// ------------------------------------------------------------------------------------------------
// The memory keys of a wave's 32 tokens, as B operands of the matrix instruction: lane = 32 g + i holds
// token i, channels 16 ks + 8 g .. + 7.  Round r of a pass: token groups r * NW .. (waves share a group
// when the block has fewer groups than waves).
struct TokenGroup {
  int j;          // the lane's token
  int wpg, sub;   // waves that share the group, and which of them this is (they split the tiles)
  bool active;
};
template <int NW>
__device__ __forceinline__ TokenGroup token_group(const Ctx<NW> &cx, int C, int g0) {
  const int left = C / 32 - g0, Gp = left < NW ? left : NW;
  TokenGroup t;
  t.wpg = NW / Gp;
  const int gi = cx.wave / t.wpg;
  t.sub = cx.wave % t.wpg;
  t.active = gi < Gp;
  t.j = (g0 + (t.active ? gi : 0)) * 32 + (cx.lane & 31);
  return t;
}
__device__ __forceinline__ void fetch_keys(bf16x8 (&kreg)[8], const uint16_t *kbar_blk, int j, int lane) {
  const uint16_t *row = kbar_blk + (int64_t)j * kHeadDim + 8 * (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    Frag8 f;
    f.q = *reinterpret_cast<const uint4 *>(row + 16 * ks);
    kreg[ks] = f.v;
  }
}

// The running winner of a lane's token: a wave-uniform code (32-row block number * 16 + accumulator
// element) turned into a row at the end, so that selecting a candidate costs a scalar.
struct Winner {
  float all, best;   // best of all rows, best of those that may win
  int code;
};
// One 64-row tile (in LDS, K layout) against the wave's tokens: D[row, token] = K-hat . K-bar^T, one
// accumulation chain per 32-row block with the channels in ascending order (as score_mfma_kernel:
// both produce the same fp32 scores), rows scanned in ascending order (ties keep the lowest).
// blk0: number of the tile's first 32-row block; rows below row1 count, rows >= row_lo may win.
// fresh (the new rows of an append, all of which may win): w.all is the second best instead.
__device__ __forceinline__ void score_tile(Winner &w, const uint16_t *Kt, const uint32_t (&koff)[8],
                                           const bf16x8 (&kreg)[8], int blk0, int row1, int row_lo, int g, bool fresh) {
  f32x16 acc[2];
  {
    bf16x8 kf[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) kf[q] = ktile_frag(Kt, koff, q & 1, q >> 1);
    const f32x16 zero = {0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int rh = 0; rh < 2; ++rh) {
        const int slot2 = (2 * ks + rh) & 3;
        acc[rh] = mfma32(kf[slot2], kreg[ks], ks == 0 ? zero : acc[rh]);
        if (ks + 2 < 8) kf[slot2] = ktile_frag(Kt, koff, rh, ks + 2);
      }
    // pin that order: four LDS reads up front, then one read behind every matrix instruction, so
    // that no matrix instruction waits for the read issued just before it
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int q = 0; q < 12; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
  }
#pragma unroll
  for (int rh = 0; rh < 2; ++rh) {
    const int blk = blk0 + rh, base = 32 * blk;
    if (base < row1) {
      if (fresh) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int i2 = base + mfma_row(v, g);
          const float sc = i2 < row1 && i2 >= row_lo ? acc[rh][v] : -INFINITY;
          w.all = fmaxf(w.all, fminf(sc, w.best));
          const bool up = sc > w.best;
          w.best = up ? sc : w.best;
          w.code = up ? 16 * blk + v : w.code;
        }
      } else if (base < row_lo || base + 32 > row1) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int i2 = base + mfma_row(v, g);
          const float sc = acc[rh][v];
          if (i2 < row1) {
            w.all = fmaxf(w.all, sc);
            if (i2 >= row_lo && sc > w.best) {
              w.best = sc;
              w.code = 16 * blk + v;
            }
          }
        }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float sc = acc[rh][v];
          const bool up = sc > w.best;
          w.best = up ? sc : w.best;
          w.code = up ? 16 * blk + v : w.code;
        }
      }
    }
  }
}
// What the lanes and waves that share a token found, put together; the result is with the lanes
// g = 0 of the group's first wave.  (Every wave calls this: it holds barriers when wpg > 1.)
template <int NW>
__device__ __forceinline__ void merge_winners(const Ctx<NW> &cx, const TokenGroup &tg, Winner &w, int &best_i, bool fresh) {
  const int g = cx.lane >> 5, l32 = cx.lane & 31;
  best_i = w.code < 0 ? kNoRow : 32 * (w.code >> 4) + mfma_row(w.code & 15, g);
  if (!fresh) w.all = fmaxf(w.all, w.best);
  {
    // the other lane half holds the other rows of the same token
    const float ob = __shfl_xor(w.best, 32, kWave);
    const int oi = __shfl_xor(best_i, 32, kWave);
    float oa = __shfl_xor(w.all, 32, kWave);
    if (fresh) oa = fmaxf(oa, fminf(ob, w.best));   // second best of both halves
    if (beats(ob, oi, w.best, best_i)) {
      w.best = ob;
      best_i = oi;
    }
    w.all = fmaxf(w.all, oa);
  }
  if (tg.wpg > 1 && !fresh) {   // (the fresh tile is one wave's work)
    float *x_all = (float *)cx.s_merge(), *x_best = x_all + NW * 32;
    int *x_idx = (int *)(x_best + NW * 32);
    if (tg.active && tg.sub != 0 && g == 0) {
      const int xi = cx.wave * 32 + l32;
      x_all[xi] = w.all;
      x_best[xi] = w.best;
      x_idx[xi] = best_i;
    }
    __syncthreads();
    if (tg.active && tg.sub == 0 && g == 0) {
      for (int o = 1; o < tg.wpg; ++o) {
        const int xi = (cx.wave + o) * 32 + l32;
        w.all = fmaxf(w.all, x_all[xi]);
        if (beats(x_best[xi], x_idx[xi], w.best, best_i)) {
          w.best = x_best[xi];
          best_i = x_idx[xi];
        }
      }
    }
    __syncthreads();   // the scratch is free again
  }
}

// Where a workgroup's 64-row tile with rows from `base` on is fetched from, sixteen 1-KiB pieces of
// four rows: wave w takes pieces w, w + NW, ...  Rows at or past `valid` repeat the last one.
template <int NW>
__device__ __forceinline__ void fetch_tile(const char *khat, int base, int valid, uint32_t lds_addr, int wave,
                                           const DmaLane &dl) {
  const int wq = wave & 3;   // the chunk permutation of a piece depends on piece % 4 = wave % 4
  const uint32_t kcol = wq == 0 ? dl.kcol[0] : wq == 1 ? dl.kcol[1] : wq == 2 ? dl.kcol[2] : dl.kcol[3];
#pragma unroll
  for (int n = 0; n < 16 / NW; ++n) {
    const int piece = wave + NW * n;
    int r = 4 * piece + (int)dl.rl;
    r = r < valid ? r : valid - 1;
    dma16(khat + (uint32_t)base * (kHeadDim * 2), (uint32_t)r * (kHeadDim * 2) + kcol, lds_addr + (uint32_t)piece * 1024u);
  }
}

// Step 2, and the second pass of an append.  kreg holds the first round's memory keys on entry.
//   first: the block's tokens against this workgroup's rows of [0, m) of readout version `slot`; every
//     token's winner among these rows goes to LDS (app, best, pi) or, with more than one workgroup per
//     unit, to the exchange table.
//   otherwise: the tokens that were not taken against the n new rows from m on that are in the fresh
//     tile; a token moves to one of them when that score is strictly larger than its best.  exact:
//     small appends of short blocks, where append_kernel takes its decisions on fp32 sums in plain
//     channel order: here a token for which that order could decide otherwise than the matrix
//     cores' is only noted, and settle_ties decides it on the same sums.
template <int NW>
__device__ __forceinline__ void score_pass(const Dev &dv, const Ctx<NW> &cx, bool first, int slot, int m, int n, bool exact,
                                           const uint16_t *kbar_blk, bf16x8 (&kreg)[8], unsigned long long *mine,
                                           uint32_t tag) {
  constexpr int D = kHeadDim;
  const int ST = cx.stage;
  const int lane = cx.lane, wave = cx.wave, g = lane >> 5;
  const int C = cx.C;
  const bool ring = first && !cx.resident;
  const int n_tiles = first ? (cx.n_local(m) + kTileKeys - 1) >> 6 : 1;
  const int row1 = first ? m : n, row_lo = first ? dv.S : dv.S - m;
  uint16_t *Ks = first ? cx.s_tiles() : cx.s_fresh();
  const uint32_t ks_addr = lds_addr_of(Ks);
  const char *khat = (const char *)dv.khat + (slot * dv.slot_elems + (int64_t)cx.u * dv.Mcap * D) * 2;
  uint32_t koff[8];
  ktile_offsets(lane, koff);
  const DmaLane dl = dma_lane(lane);
  auto issue_stage = [&](int sg) {
#pragma unroll 1
    for (int i = 0; i < ST; ++i) {
      const int t = ST * sg + i;
      if (t < n_tiles) {
        const int base = cx.global(64 * t);
        fetch_tile<NW>(khat, base, m - base, ks_addr + (uint32_t)(t & (2 * ST - 1)) * kTileBytes, wave, dl);
      }
    }
  };
  for (int g0 = 0; g0 < C / 32; g0 += NW) {
    const TokenGroup tg = token_group<NW>(cx, C, g0);
    if (C / 32 > NW && (g0 > 0 || !first)) fetch_keys(kreg, kbar_blk, tg.j, lane);
    Winner w{-INFINITY, -INFINITY, -1};
    if (ring) {
      __syncthreads();   // the ring's last readers are done
      issue_stage(0);
    }
#pragma unroll 1
    for (int t = 0; t < n_tiles; ++t) {
      if (ring && (t & (ST - 1)) == 0) {   // a stage has landed for every wave, and the other one has been read
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        issue_stage((t >> __builtin_ctz(ST)) + 1);
      }
      if (tg.active && (t & (tg.wpg - 1)) == tg.sub)   // wpg is a power of two: NW and C / 32 are
        score_tile(w, Ks + (ring ? t & (2 * ST - 1) : t) * kTileElems, koff, kreg, first ? cx.global(64 * t) >> 5 : 0, row1,
                   row_lo, g, !first);
    }
    int best_i;
    merge_winners<NW>(cx, tg, w, best_i, !first);
    if (tg.active && tg.sub == 0 && g == 0) {
      if (!first) {
        const float best = cx.s_best()[tg.j];
        if (cx.s_rank()[tg.j] < 0 && best_i != kNoRow) {
          // fp32 sums of 128 exact products in two orders differ by far less than this
          const float reach = fmaxf(1e-2f, fabsf(best) * 0x1p-12f);
          if (exact && w.best > best - reach && (w.best < best + reach || w.all > w.best - reach)) {
            cx.s_rows()[atomicAdd(&cx.s_cnt()[kCntTies], 1)] = tg.j;
          } else if (w.best > best) {
            cx.s_best()[tg.j] = w.best;
            cx.s_pi()[tg.j] = m + best_i;
          }
        }
      } else if (cx.split > 1) {
        publish_winner(mine, C, tg.j, w.best, best_i, w.all, sink_owner(dv, cx.part), tag);
      } else {
        cx.s_app()[tg.j] = w.all;
        cx.s_best()[tg.j] = w.best;
        cx.s_pi()[tg.j] = best_i;
        cx.s_rank()[tg.j] = -1;
      }
    }
  }
}

// The noted tokens, a wave each: lane a sums token . new row a over the channels in ascending order.
template <int NW>
__device__ __forceinline__ void settle_ties(const Dev &dv, const Ctx<NW> &cx, int m, int n_app, const uint16_t *kbar_blk) {
  const int n = cx.s_cnt()[kCntTies], lane = cx.lane;
  const uint16_t *Kt = cx.s_fresh() + (lane & 15) * kHeadDim;   // n_app <= 16
  for (int k = cx.wave; k < n; k += NW) {
    const int j = cx.s_rows()[k];
    // the token's key, a sixteenth per lane; its pieces go round as scalars
    const uint4 piece = *reinterpret_cast<const uint4 *>(kbar_blk + (int64_t)j * kHeadDim + 8 * (lane & 15));
    float acc = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const uint4 xq = make_uint4(__builtin_amdgcn_readlane(piece.x, q), __builtin_amdgcn_readlane(piece.y, q),
                                  __builtin_amdgcn_readlane(piece.z, q), __builtin_amdgcn_readlane(piece.w, q));
      float x[8], y[8];
      unpack16<bf16_t>(xq, x);
      unpack16<bf16_t>(*reinterpret_cast<const uint4 *>(Kt + 8 * (q ^ (lane & 15))), y);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(x[e], y[e], acc);
    }
    float best = lane < n_app ? acc : -INFINITY;
    int a = lane < n_app ? lane : kNoRow;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {   // n_app <= 16
      const float ob = __shfl_xor(best, o, kWave);
      const int oa = __shfl_xor(a, o, kWave);
      if (beats(ob, oa, best, a)) {
        best = ob;
        a = oa;
      }
    }
    if (lane == 0 && m + a >= dv.S && best > cx.s_best()[j]) {
      cx.s_best()[j] = best;
      cx.s_pi()[j] = m + a;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Step 3: the n_app tokens with the smallest (s_j, position) are taken; a taken token's rank among
// the taken ones, in position order, is the new row it creates.  Every wave finds the n_app-th smallest
// score for itself, bit by bit from the top, counting with ballots over scores it holds in registers (no
// barriers, no table: comparing every token with every other one through LDS took 7 us for 256 tokens,
// this takes 1.5).  A few (a growing state appends at most folds, some four rows) are taken one by one, the smallest that is left
// each time, some 130 cycles, where the bits take 3.9 us: 65536 tokens, growing state, 32 units 6.34 -> 6.03 ms.
// (Up to 12 of 256 tokens, 32 of 512: with 32 of 256 a call of 8 x 32 heads, 16 or 32 rows a fold, was 1 % slower.)
constexpr int kMaxBlock = 1024;
constexpr int select_few(int pieces) { return pieces <= 4 ? 12 : 32; }
// Minimum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
  auto mn = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
  x = mn(x, (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true));
  x = mn(x, (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true));
  x = mn(x, (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true));
  x = mn(x, (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x140, 0xF, 0xF, true));
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = mn(r[0], r[1]);
  const auto t = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return mn(t[0], t[1]);
}
// A score's bits made monotonic as an unsigned number.
__device__ __forceinline__ uint32_t score_key(float s) {
  uint32_t f = __float_as_uint(s);
  f = f == 0x80000000u ? 0u : f;   // -0 and +0 are one score
  return (f & 0x80000000u) ? ~f : (f | 0x80000000u);
}
template <int NW, int kQ>   // kQ: 64-token pieces, at least C / 64
__device__ __forceinline__ void select_tokens(const Ctx<NW> &cx, int m, int n_app) {
  const int C = cx.C, lane = cx.lane;
  uint32_t key[kQ];   // (the largest number beyond the block)
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    key[q] = 0xffffffffu;
    if (64 * q < C) {
      key[q] = score_key(cx.s_app()[64 * q + lane]);
    }
  }
  unsigned long long taken[kQ];   // tokens taken, by piece
#pragma unroll
  for (int q = 0; q < kQ; ++q) taken[q] = 0ull;
  if (n_app <= select_few(kQ)) {
#pragma unroll 1
    for (int a = 0; a < n_app; ++a) {
      uint32_t least = key[0];
#pragma unroll
      for (int q = 1; q < kQ; ++q) least = key[q] < least ? key[q] : least;
      least = wave_min_u32(least);
      bool found = false;
#pragma unroll
      for (int q = 0; q < kQ; ++q) {   // the earliest of those with this score
        const unsigned long long eq = __builtin_amdgcn_ballot_w64(key[q] == least) & ~taken[q];
        if (!found && eq != 0 && 64 * q < C) {
          found = true;
          const unsigned long long bit = eq & (0ull - eq);
          taken[q] |= bit;
          key[q] = (bit >> lane) & 1ull ? 0xffffffffu : key[q];
        }
      }
    }
  } else {
    uint32_t T = 0;   // largest number that fewer than n_app scores lie below: the n_app-th smallest score
#pragma unroll 1
    for (int bit = 30; bit >= 0; bit -= 2) {   // two bits at a time
      const uint32_t c1 = T | (1u << bit), c2 = T | (2u << bit), c3 = T | (3u << bit);
      int n1 = 0, n2 = 0, n3 = 0;
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        n1 += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[q] < c1));
        n2 += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[q] < c2));
        n3 += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[q] < c3));
      }
      T = n3 < n_app ? c3 : n2 < n_app ? c2 : n1 < n_app ? c1 : T;
    }
    int equal = n_app;   // how many of the scores equal to it are taken: the earliest
#pragma unroll
    for (int q = 0; q < kQ; ++q) equal -= __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[q] < T));
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      unsigned long long eq = __builtin_amdgcn_ballot_w64(key[q] == T);
      while (__builtin_popcountll(eq) > equal) eq &= ~(1ull << (63 - __builtin_clzll(eq)));
      equal -= __builtin_popcountll(eq);
      taken[q] = __builtin_amdgcn_ballot_w64(key[q] < T) | eq;
    }
  }
  int base = 0;
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    if (q % NW == cx.wave) {   // a wave per 64 tokens writes what they all know
      const int j = 64 * q + lane;
      if ((taken[q] >> lane) & 1ull) {
        const int a = base + __builtin_popcountll(taken[q] & ((1ull << lane) - 1ull));
        cx.s_rank()[j] = a;
        cx.s_pi()[j] = m + a;
        cx.s_best()[j] = __uint_as_float(0x7fc00000u);
        cx.s_creator()[a] = j;
      }
    }
    base += __builtin_popcountll(taken[q]);
  }
  __syncthreads();
}

// The same for blocks of more than 512 tokens, whose scores stay in LDS: a loop instead of registers, for the rare block that is
// so long (sixteen pieces in registers made the whole kernel's code slower: 8 x 32 heads, 8192 tokens 4.51 -> 4.60 ms).
template <int NW>
__device__ __forceinline__ void select_long(const Ctx<NW> &cx, int m, int n_app) {
  const int pieces = cx.C / 64, lane = cx.lane;
  uint32_t T = 0;   // as above
#pragma unroll 1
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t c = T | (1u << bit);
    int n = 0;
#pragma unroll 1
    for (int q = 0; q < pieces; ++q) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(score_key(cx.s_app()[64 * q + lane]) < c));
    T = n < n_app ? c : T;
  }
  int equal = n_app;
#pragma unroll 1
  for (int q = 0; q < pieces; ++q) equal -= __builtin_popcountll(__builtin_amdgcn_ballot_w64(score_key(cx.s_app()[64 * q + lane]) < T));
  int base = 0;
#pragma unroll 1
  for (int q = 0; q < pieces; ++q) {
    const int j = 64 * q + lane;
    const uint32_t k = score_key(cx.s_app()[j]);
    unsigned long long eq = __builtin_amdgcn_ballot_w64(k == T);
    while (__builtin_popcountll(eq) > equal) eq &= ~(1ull << (63 - __builtin_clzll(eq)));
    equal -= __builtin_popcountll(eq);
    const unsigned long long taken = __builtin_amdgcn_ballot_w64(k < T) | eq;
    if (q % NW == cx.wave && ((taken >> lane) & 1ull)) {
      const int a = base + __builtin_popcountll(taken & ((1ull << lane) - 1ull));
      cx.s_rank()[j] = a;
      cx.s_pi()[j] = m + a;
      cx.s_best()[j] = __uint_as_float(0x7fc00000u);
      cx.s_creator()[a] = j;
    }
    base += __builtin_popcountll(taken);
  }
  __syncthreads();
}

// 1 / sqrt(x) in fp64 from the hardware estimate and two Newton steps (y <- y (1.5 - 0.5 x y^2)):
// within a few units of the last place, against some 300 instructions for the correctly rounded
// division of the correctly rounded root; the result is rounded to bf16 afterwards.
__device__ __forceinline__ double rsqrt64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  y = y * fma(-hx * y, y, 1.5);
  y = y * fma(-hx * y, y, 1.5);
  return y;
}

// A row is held by 16 lanes, 8 channels each: lane c has channels 64 q + 4 c + e, q = 0..1, e = 0..3 (element 4 q + e of
// its arrays), so that every access to a row of bf16, fp32 or fp64 is contiguous over the lanes in
// pieces of 128, 256 or 512 bytes.
__device__ __forceinline__ void load_bf16x4(const uint16_t *p, float *f) {
  const uint2 x = *reinterpret_cast<const uint2 *>(p);
  f[0] = __uint_as_float(x.x << 16);
  f[1] = __uint_as_float(x.x & 0xffff0000u);
  f[2] = __uint_as_float(x.y << 16);
  f[3] = __uint_as_float(x.y & 0xffff0000u);
}
struct Row8 {   // eight bf16 values of a lane
  uint2 q[2];
};
__device__ __forceinline__ void store_row(uint16_t *row, int c16, const Row8 &v) {
#pragma unroll
  for (int q = 0; q < 2; ++q) *reinterpret_cast<uint2 *>(row + 64 * q + 4 * c16) = v.q[q];
}
// the same into row r of tiles in the K layout (16-byte chunk k of a row sits in slot k ^ (r & 15))
__device__ __forceinline__ void store_tile_row(uint16_t *tiles, int r, int c16, const Row8 &v) {
#pragma unroll
  for (int q = 0; q < 2; ++q)
    *reinterpret_cast<uint2 *>(tiles + r * kHeadDim + 8 * ((8 * q + (c16 >> 1)) ^ (r & 15)) + 4 * (c16 & 1)) = v.q[q];
}
// Parameters of LN_s of the unit's KV head (given, or 1 and 0)
struct LnParams {
  const float *gamma, *beta;
};
__device__ __forceinline__ LnParams ln_params(const Dev &dv, int u) {
  const int h = u % dv.Hkv;
  return {dv.gamma ? dv.gamma + h * kHeadDim : kOnes, dv.beta ? dv.beta + h * kHeadDim : kZeros};
}
// LN_s of a row of key sums.
__device__ __forceinline__ Row8 normalised16(const Dev &dv, const double (&sk)[8], const LnParams &ln, int c16) {
  constexpr int D = kHeadDim;
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) s += sk[e];
  const double mean = group_sum<16>(s) * (1.0 / (double)D);   // D is a power of two: exact
  double qq = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double dl = sk[e] - mean;
    qq += dl * dl;
  }
  const double rden = rsqrt64(group_sum<16>(qq) * (1.0 / (double)D) + (double)dv.ln_eps);
  Row8 r;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float4 g4 = *reinterpret_cast<const float4 *>(ln.gamma + 64 * q + 4 * c16);
    const float4 b4 = *reinterpret_cast<const float4 *>(ln.beta + 64 * q + 4 * c16);
    const float ga[4] = {g4.x, g4.y, g4.z, g4.w}, be[4] = {b4.x, b4.y, b4.z, b4.w};
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = (float)((sk[4 * q + e] - mean) * rden * (double)ga[e] + (double)be[e]);
    r.q[q] = make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
  }
  return r;
}

// Squared norm of a row of values, added up in the order of the kernel-per-step path (write_readout, create: pairs of
// adjacent channels, then a balanced tree over the pairs): both paths have the same fp32 bits, and with them
// the same readout.
__device__ __forceinline__ float norm2_16(const float (&x)[8]) {
  float half[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float y[2][2] = {{x[4 * q], x[4 * q + 1]}, {x[4 * q + 2], x[4 * q + 3]}};
    half[q] = group_sum<16>(lane_norm2<2>(y[0]) + lane_norm2<2>(y[1]));
  }
  return half[0] + half[1];
}
// The readout row of value sums sv and radius rho whose normalised key is `khat`.  Rounding to bf16
// is the hardware's (nearest even).
__device__ __forceinline__ void store_readout16(const Dev &dv, int slot, int64_t ro, int c16, const Row8 &khat,
                                                const float (&sv)[8], float rho) {
  constexpr int D = kHeadDim;
  const float vs = rho / fmaxf(sqrtf(norm2_16(sv)), dv.norm_eps);
  Row8 v;
#pragma unroll
  for (int q = 0; q < 2; ++q)
    v.q[q] = make_uint2(pack_bf16(sv[4 * q] * vs, sv[4 * q + 1] * vs), pack_bf16(sv[4 * q + 2] * vs, sv[4 * q + 3] * vs));
  store_row((uint16_t *)dv.khat + slot * dv.slot_elems + ro * D, c16, khat);
  store_row((uint16_t *)dv.vhat + slot * dv.slot_elems + ro * D, c16, v);
}
__device__ __forceinline__ void load_sums(const Dev &dv, int64_t ro, int c16, double (&sk)[8], float (&sv)[8]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const double2 *pk = reinterpret_cast<const double2 *>(dv.sK + ro * kHeadDim + 64 * q + 4 * c16);
    const double2 a = pk[0], b = pk[1];
    const float4 v = *reinterpret_cast<const float4 *>(dv.sV + ro * kHeadDim + 64 * q + 4 * c16);
    sk[4 * q] = a.x; sk[4 * q + 1] = a.y; sk[4 * q + 2] = b.x; sk[4 * q + 3] = b.y;
    sv[4 * q] = v.x; sv[4 * q + 1] = v.y; sv[4 * q + 2] = v.z; sv[4 * q + 3] = v.w;
  }
}
__device__ __forceinline__ void store_sums(const Dev &dv, int64_t ro, int c16, const double (&sk)[8], const float (&sv)[8]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    double2 *pk = reinterpret_cast<double2 *>(dv.sK + ro * kHeadDim + 64 * q + 4 * c16);
    pk[0] = make_double2(sk[4 * q], sk[4 * q + 1]);
    pk[1] = make_double2(sk[4 * q + 2], sk[4 * q + 3]);
    *reinterpret_cast<float4 *>(dv.sV + ro * kHeadDim + 64 * q + 4 * c16) =
        make_float4(sv[4 * q], sv[4 * q + 1], sv[4 * q + 2], sv[4 * q + 3]);
  }
}

// The block a fold takes in, seen from one unit: memory keys, values, gates of its tokens.
struct Block {
  const uint16_t *vsrc, *kbar;
  const float *gsrc;
  int64_t v_t, g_t;
};
template <int NW>
__device__ __forceinline__ Block block_of(const Dev &dv, const Ctx<NW> &cx, const Src &src, int64_t tok,
                                          const uint16_t *kbar_blk) {
  Block b;
  const int bi = cx.u / dv.Hkv, h = cx.u % dv.Hkv;
  b.vsrc = (const uint16_t *)src.v + bi * src.v_b + h * src.v_h + tok * src.v_t;
  b.gsrc = src.g ? src.g + bi * src.g_b + h * src.g_h + tok * src.g_t : nullptr;
  b.kbar = kbar_blk;
  b.v_t = src.v_t;
  b.g_t = src.g_t;
  return b;
}

// New rows m + a_lo .. m + a_hi - 1 from their creator tokens: ungated copy of the memory key and the
// value, radius = the value's norm.  The row's owner writes it; with `fresh` every workgroup of the
// unit also makes the row's normalised key for itself, in the fresh tile (the same arithmetic on the
// same operands: all of them have the same bits), so that the second scoring pass needs no exchange.
template <int NW>
__device__ __forceinline__ void create_rows(const Dev &dv, const Ctx<NW> &cx, const Block &blk, int m, int a_lo, int a_hi,
                                            bool fresh, int slot_new) {
  constexpr int D = kHeadDim, NG = 4 * NW;
  const int gid = cx.tid >> 4, c16 = cx.tid & 15;
  const LnParams ln = ln_params(dv, cx.u);
  for (int a = a_lo + gid; a < a_hi; a += NG) {
    const bool own = cx.owns(m + a);
    if (!own && !fresh) continue;
    const int t = cx.s_creator()[a];
    float kf[8], vf[8] = {};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      load_bf16x4(blk.kbar + (int64_t)t * D + 64 * q + 4 * c16, kf + 4 * q);
      if (own) load_bf16x4(blk.vsrc + (int64_t)t * blk.v_t + 64 * q + 4 * c16, vf + 4 * q);
    }
    double sk[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sk[e] = (double)kf[e];
    const Row8 khat = normalised16(dv, sk, ln, c16);
    if (fresh) store_tile_row(cx.s_fresh(), a - a_lo, c16, khat);
    if (!own) continue;
    const int64_t ro = (int64_t)cx.u * dv.Mcap + m + a;
    const float rho = sqrtf(norm2_16(vf));
    store_sums(dv, ro, c16, sk, vf);
    if (c16 == 0) {
      dv.rho[ro] = rho;
      dv.w[ro] = 1.f;
      dv.n[ro] = 1;
    }
    store_readout16(dv, slot_new, ro, c16, khat, vf, rho);
    if (cx.resident) store_tile_row(cx.s_tiles(), cx.local(m + a), c16, khat);
  }
}

// Step 4: the lists.  Every token that merges pushes itself on its row's list; the one that finds
// the list empty enters the row in `rows`.  The token also gets a place in the scratch, as long as
// there are places.  (The heads and the counters were cleared earlier in the fold.)
template <int NW>
__device__ __forceinline__ void build_lists(const Dev &dv, const Ctx<NW> &cx) {
  constexpr int NT = 64 * NW;
  const int C = dv.C, tid = cx.tid, lane = cx.lane;
  int *cnt = cx.s_cnt();
  for (int j0 = 0; j0 < C; j0 += NT) {
    const int j = j0 + tid;
    bool leader = false, mine = false;
    int lr = 0;
    if (j < C && cx.s_rank()[j] < 0) {
      const int row = cx.s_pi()[j];
      if (row != kNoRow && cx.owns(row)) {   // other rows are other workgroups' work
        lr = cx.local(row);
        const int old = atomicExch(&cx.s_head()[lr], j);
        cx.s_next()[j] = old;
        leader = old < 0;
        mine = true;
      }
    }
    const unsigned long long rows = __builtin_amdgcn_ballot_w64(leader), toks = __builtin_amdgcn_ballot_w64(mine);
    const unsigned long long below = (1ull << lane) - 1ull;
    int row0 = 0, tok0 = 0;
    if (lane == 0 && toks) {
      row0 = atomicAdd(&cnt[kCntRows], __builtin_popcountll(rows));
      tok0 = atomicAdd(&cnt[kCntOwn], __builtin_popcountll(toks));
    }
    row0 = __shfl(row0, 0, kWave);
    tok0 = __shfl(tok0, 0, kWave);
    if (leader) cx.s_rows()[row0 + __builtin_popcountll(rows & below)] = lr;
    if (mine) {
      const int slot = tok0 + __builtin_popcountll(toks & below);
      cx.s_slot()[j] = slot;
      cx.s_own()[slot] = j;
    }
  }
  __syncthreads();
}

// The merging tokens' memory keys and values on their way into the scratch: all of them in flight at
// once, four tokens' rows per load instruction.  (Taken from memory where they are added, a row with
// several tokens is a chain of memory round trips.)
template <int NW>
__device__ __forceinline__ void gather_tokens(const Ctx<NW> &cx, const Block &blk) {
  if (blk.gsrc && cx.gates_in_lds()) {   // the gates of the whole block, 64 per instruction (taken where they are used, each was a round trip)
    const uint32_t gates = lds_addr_of(cx.s_gate());
    for (int j0 = 64 * cx.wave; j0 < cx.C; j0 += 64 * NW) {   // (C is a multiple of 64)
      dma4_from(blk.gsrc + (int64_t)(j0 + cx.lane) * blk.g_t, gates + 4u * (uint32_t)j0);
    }
  }
  int n = cx.s_cnt()[kCntOwn];
  n = n < cx.gather ? n : cx.gather;
  const int c16 = cx.lane & 15;
  const uint32_t keys = lds_addr_of(cx.s_keys(0)), vals = lds_addr_of(cx.s_vals(0));
#pragma unroll 1
  for (int s0 = 4 * cx.wave; s0 < n; s0 += 4 * NW) {   // (gather is a multiple of four)
    const int s = s0 + (cx.lane >> 4);
    const int64_t t = cx.s_own()[s < n ? s : n - 1];
    dma16_from(blk.kbar + t * kHeadDim + 8 * c16, keys + (uint32_t)s0 * (kHeadDim * 2));
    dma16_from(blk.vsrc + t * blk.v_t + 8 * c16, vals + (uint32_t)s0 * (kHeadDim * 2));
  }
}

// Minimum over the 16 lanes of a group, in every lane.
__device__ __forceinline__ int group_min16(int x) {
  auto mn = [](int a, int b) { return a < b ? a : b; };
  x = mn(x, (int)__builtin_amdgcn_mov_dpp((uint32_t)x, 0xB1, 0xF, 0xF, true));
  x = mn(x, (int)__builtin_amdgcn_mov_dpp((uint32_t)x, 0x4E, 0xF, 0xF, true));
  x = mn(x, (int)__builtin_amdgcn_mov_dpp((uint32_t)x, 0x141, 0xF, 0xF, true));
  x = mn(x, (int)__builtin_amdgcn_mov_dpp((uint32_t)x, 0x140, 0xF, 0xF, true));
  return x;
}

// Step 5: the touched rows, 16 lanes each.
template <int NW>
__device__ __forceinline__ void merge_rows(const Dev &dv, const Ctx<NW> &cx, const Block &blk, int slot_new) {
  constexpr int D = kHeadDim, NG = 4 * NW;
  const int C = cx.C, n_rows = cx.s_cnt()[kCntRows], c16 = cx.tid & 15;
  const int *next = cx.s_next(), *pi = cx.s_pi(), *rank = cx.s_rank();
  const LnParams ln = ln_params(dv, cx.u);
  bool landed = false;
#pragma unroll 1
  for (int ri = cx.tid >> 4; ri < n_rows || !landed; ri += NG) {
    const bool on = ri < n_rows;
    const int lr = on ? cx.s_rows()[ri] : 0, row = cx.global(lr);
    const int64_t ro = (int64_t)cx.u * dv.Mcap + row;
    // the sums are asked for first; the list is walked while they travel
    double sk[8];
    float sv[8], rho = 0.f, w = 0.f;
    int n = 0;
    if (on) {
      load_sums(dv, ro, c16, sk, sv);
      rho = dv.rho[ro];
      w = dv.w[ro];
      n = dv.n[ro];
    }
    // lane i of the group keeps the i-th token of the list (any order)
    int mine = kNoRow, len = 0;
    if (on) {
      for (int t = cx.s_head()[lr]; t >= 0 && len <= kListMax; t = next[t], ++len)
        if (len == c16) mine = t;
    }
    if (!landed) {   // the gathered tokens are there, every wave's share of them
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      landed = true;
    }
    if (!on) break;
    // The row's tokens in ascending position: from the lanes' tokens, or, when a list is longer than
    // the lanes (many tokens on one row), from the block's targets, 16 positions at a time.
    auto after = [&](int t) {
      if (len <= kListMax) return group_min16(mine > t ? mine : kNoRow);
      int found = kNoRow;
      for (int t0 = t + 1; t0 < C && found == kNoRow; t0 += 16) {
        const int x = t0 + c16;
        found = group_min16(x < C && pi[x] == row && rank[x] < 0 ? x : kNoRow);
      }
      return found;
    };
    for (int t = after(-1); t != kNoRow; t = after(t)) {
      const int slot = cx.s_slot()[t];
      float gt = 1.f, kf[8], vf[8];
      if (blk.gsrc) gt = cx.gates_in_lds() ? cx.s_gate()[t] : blk.gsrc[(int64_t)t * blk.g_t];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (slot < cx.gather) {
          load_bf16x4(cx.s_keys(slot) + 64 * q + 4 * c16, kf + 4 * q);
          load_bf16x4(cx.s_vals(slot) + 64 * q + 4 * c16, vf + 4 * q);
        } else {
          load_bf16x4(blk.kbar + (int64_t)t * D + 64 * q + 4 * c16, kf + 4 * q);
          load_bf16x4(blk.vsrc + (int64_t)t * blk.v_t + 64 * q + 4 * c16, vf + 4 * q);
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sk[e] = fma((double)gt, (double)kf[e], sk[e]);
        sv[e] = fmaf(gt, vf[e], sv[e]);
      }
      w += gt;
      n += 1;
    }
    store_sums(dv, ro, c16, sk, sv);
    if (c16 == 0) {
      dv.w[ro] = w;
      dv.n[ro] = n;
    }
    const Row8 khat = normalised16(dv, sk, ln, c16);
    store_readout16(dv, slot_new, ro, c16, khat, sv, rho);
    if (cx.resident) store_tile_row(cx.s_tiles(), lr, c16, khat);
  }
}

// Own rows of [0, m) that received no token in the fold from version slot_old to slot_new: their
// readout moves to the new version unchanged (key rows of resident tiles come from LDS).  With resident
// tiles this is done while the next fold's winners travel between the workgroups: nothing of the
// chain waits for it.  (Tiles that stream are read from the new version: then it is done before the
// next fold's scores.)  The lists' heads, which tell the rows, are cleared for the next fold on the way.
template <int NW>
__device__ __forceinline__ void copy_untouched(const Dev &dv, const Ctx<NW> &cx, int m, int m_after, int slot_old,
                                               int slot_new, int in_place) {
  constexpr int D = kHeadDim, NG = 4 * NW, kRows = 4;
  const int gid = cx.tid >> 4, c16 = cx.tid & 15, n = in_place ? 0 : cx.n_local(m), n_all = cx.n_local(m_after);
  const int64_t ubase = (int64_t)cx.u * dv.Mcap * D + 8 * c16;
  const uint16_t *ko = (const uint16_t *)dv.khat + slot_old * dv.slot_elems + ubase;
  const uint16_t *vo = (const uint16_t *)dv.vhat + slot_old * dv.slot_elems + ubase;
  uint16_t *kn = (uint16_t *)dv.khat + slot_new * dv.slot_elems + ubase;
  uint16_t *vn = (uint16_t *)dv.vhat + slot_new * dv.slot_elems + ubase;
#pragma unroll 1
  for (int lr0 = gid; lr0 < n_all; lr0 += kRows * NG) {
    uint4 kk[kRows], vv[kRows];
    bool on[kRows];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const int lr = lr0 + q * NG;
      on[q] = lr < n && cx.s_head()[lr < n ? lr : 0] < 0;
      const int64_t at = (int64_t)cx.global(on[q] ? lr : 0) * D;
      vv[q] = make_uint4(0u, 0u, 0u, 0u);
      kk[q] = make_uint4(0u, 0u, 0u, 0u);
      if (on[q]) vv[q] = *reinterpret_cast<const uint4 *>(vo + at);
      if (on[q] && !cx.resident) kk[q] = *reinterpret_cast<const uint4 *>(ko + at);
      if (on[q] && cx.resident) kk[q] = *reinterpret_cast<const uint4 *>(cx.s_tiles() + lr * D + 8 * (c16 ^ (lr & 15)));
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const int lr = lr0 + q * NG;
      const int64_t at = (int64_t)cx.global(lr) * D;
      if (on[q]) {
        *reinterpret_cast<uint4 *>(kn + at) = kk[q];
        *reinterpret_cast<uint4 *>(vn + at) = vv[q];
      }
      if (c16 == 0 && lr < n_all) cx.s_head()[lr] = -1;   // (only this group's lanes look at it before the next barrier)
    }
  }
}

// The kernel's one argument.  Steps and parameters are read from the kernel-argument segment where
// they are used: a fold is a dozen short phases, and what the compiler may keep in registers from
// one phase to the next -- pointers of arrays, addresses and lane numbers made from them, for all
// phases at once -- spilled 370 vector and 370 scalar registers.  args_now() and phase() hide where
// a value comes from, so that every phase makes its own.
struct FoldKernelArgs {
  Dev dv;
  Src src;
  FoldRunArgs run;
};
__device__ __forceinline__ const FoldKernelArgs &args_now() {
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const FoldKernelArgs *)(const __attribute__((address_space(4))) FoldKernelArgs *)p;
}
template <int NW>
__device__ __forceinline__ Ctx<NW> phase(const Ctx<NW> &cx) {
  Ctx<NW> c = cx;
  asm volatile("" : "+v"(c.tid));
  c.lane = c.tid & 63;
  asm volatile("" : "+s"(c.wave), "+s"(c.C), "+s"(c.fresh_at), "+s"(c.u), "+s"(c.gather));
  return c;
}

template <int NW>
__global__ __launch_bounds__(64 * NW, 4) void fold_fused_kernel(FoldKernelArgs) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  constexpr int D = kHeadDim, NT = 64 * NW;
  Ctx<NW> cx;
  int run_n, run_in_place;
  {
    const FoldKernelArgs &a = args_now();
    const int split = a.run.split, bid = (int)blockIdx.x;
    // Workgroup -> (unit, part).  The workgroups of a unit read the same block of tokens: where the
    // number of units allows it they get ids 8 apart, which the hardware hands to one accelerator
    // die, whose L2 then fetches the block once.
    const bool by_die = a.dv.U % 8 == 0;
    cx.smem = smem;
    cx.C = a.dv.C;
    cx.fresh_at = lds_fresh(NW, a.dv.C, own_tiles_most(a.dv.Mcap, split));
    cx.gather = a.run.gather;
    cx.u = by_die ? (bid / (8 * split)) * 8 + bid % 8 : bid / split;
    cx.part = by_die ? (bid / 8) % split : bid % split;
    cx.split = split;
    cx.shift = __builtin_ctz(split);
    cx.resident = a.run.resident > 0;
    cx.stage = stage_tiles(NW);
    cx.tid = (int)threadIdx.x;
    cx.lane = cx.tid & 63;
    cx.wave = __builtin_amdgcn_readfirstlane(cx.tid >> 6);
    run_n = a.run.n;
    run_in_place = a.run.in_place;
  }
  __builtin_amdgcn_s_setprio(3);   // ahead of an attention workgroup's waves on the same compute unit: the chain waits for this one
  const float qnan = __uint_as_float(0x7fc00000u);
#ifdef KVM_FOLD_STAMPS
  if (threadIdx.x == 0) cx.s_cnt()[kCntStamps] = 0;
#endif
  // the memory keys of a step's block: slab `kbar_block` of the scratch, this unit's C rows
  auto keys_of = [&](const FoldKernelArgs &a, int si) {
    return (const uint16_t *)a.dv.kbar + ((int64_t)a.run.s[si].kbar_block * a.dv.Ufull + cx.u) * cx.C * D;
  };
  bf16x8 kreg[8];
  auto fetch_first_keys = [&](int si) {
    const Ctx<NW> c = phase(cx);
    fetch_keys(kreg, keys_of(args_now(), si), token_group<NW>(c, c.C, 0).j, c.lane);
  };
  fetch_first_keys(0);
  if (cx.resident) {
    const FoldKernelArgs &a = args_now();
    const char *khat = (const char *)a.dv.khat + (a.run.s[0].so * a.dv.slot_elems + (int64_t)cx.u * a.dv.Mcap * D) * 2;
    const DmaLane dl = dma_lane(cx.lane);
    const uint32_t at = lds_addr_of(cx.s_tiles());
    const int m0 = a.run.s[0].m;
    for (int t = 0; 64 * t < cx.n_local(m0); ++t) {
      const int base = cx.global(64 * t);
      fetch_tile<NW>(khat, base, m0 - base, at + (uint32_t)t * kTileBytes, cx.wave, dl);
    }
  }
  if (cx.split > 1) {   // the others are waited for while the tiles travel
    if (cx.tid == 0) {
      const FoldRunArgs &run = args_now().run;
      cx.s_cnt()[kCntMeet] = meet(run.xtab + (size_t)cx.u * kArrivalWords, run.split, run.arrived, run.launch, run.patience);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int who = __builtin_amdgcn_readfirstlane(cx.s_cnt()[kCntMeet]);
    if (who == kLeave) return;
    if (who == kWhole) {
      const FoldKernelArgs &a = args_now();
      cx.split = 1;
      cx.part = cx.shift = 0;
      cx.fresh_at = lds_fresh(NW, a.dv.C, own_tiles_most(a.dv.Mcap, 1));
      cx.resident = false;
      cx.stage = kStageTaken;
      cx.gather = kGatherTaken;
    }
  }
  if (cx.resident) {   // the tiles are there, every wave's share of them
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }

  {
    const int n = own_tiles_most(args_now().dv.Mcap, cx.split) * kTileKeys;
    for (int i = cx.tid; i < n; i += NT) cx.s_head()[i] = -1;
  }

  // One pass more than there are folds: a fold's copies are made in the next one's place for them.
  int m = 0, m_after = 0, so = 0, sn = 0;   // of the fold before, until the new values are taken over
  for (int si = 0;; ++si) {
    FOLD_STAMP();
    const bool live = si < run_n;
    const int m_prev = m, m_after_prev = m_after, so_prev = so, sn_prev = sn;
    if (live) {
      const FoldStep &st = args_now().run.s[si];
      m = st.m; m_after = st.m_after; so = st.so; sn = st.sn;
    }
    const int n_app = m_after - m;
    const bool all = live && n_app == cx.C;   // room for the whole block (state creation included): no scores
    const bool exact = append_fits(cx.C, n_app);
    if (cx.tid == 0) cx.s_cnt()[kCntRows] = cx.s_cnt()[kCntTies] = cx.s_cnt()[kCntOwn] = 0;
    if (all) {
      const Ctx<NW> c = phase(cx);
      for (int j = c.tid; j < c.C; j += NT) {
        c.s_rank()[j] = j;
        c.s_pi()[j] = m + j;
        c.s_app()[j] = qnan;
        c.s_best()[j] = qnan;
        c.s_creator()[j] = j;
      }
      __syncthreads();   // create_rows reads other waves' entries
    }
    auto copy_previous = [&]() {
      copy_untouched<NW>(args_now().dv, phase(cx), m_prev, m_after_prev, so_prev, sn_prev, run_in_place);
    };
    if (!cx.resident && si > 0) {
      copy_previous();
      __syncthreads();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
    // Scoring passes: the state's rows first, then (a partial append) the rows this fold creates, 64 at a time.
    int a0 = all ? 0 : -1;   // -1: the state; otherwise the first new row of the pass
    bool begin = true;
    do {
      int a1 = 0;
      if (a0 >= 0) {
        a1 = all || n_app - a0 < kTileKeys ? n_app : a0 + kTileKeys;
        const FoldKernelArgs &a = args_now();
        const Ctx<NW> c = phase(cx);
        create_rows<NW>(a.dv, c, block_of(a.dv, c, a.src, a.run.s[si].tok, keys_of(a, si)), m, a0, a1, !all, sn);
        __syncthreads();
      }
      if (live && !all) {
        const FoldKernelArgs &a = args_now();
        const Ctx<NW> c = phase(cx);
        const uint32_t xnum = a.run.s[si].xnum;
        unsigned long long *mine = exchange_table(a.dv, a.run) + (((size_t)c.u * 2 + (xnum & 1u)) * c.split + c.part) * 2 * c.C;
        score_pass<NW>(a.dv, c, a0 < 0, so, m + (a0 < 0 ? 0 : a0), a1 - a0, exact, keys_of(a, si), kreg, mine, xnum & 0xffffu);
      }
      if (begin && cx.resident && si > 0) copy_previous();
      if (!live) return;
      // (nothing waits for a barrier between a wave's own winners and its reading of the others': each entry is waited
      // for by itself)
      const bool meet_now = a0 < 0 && cx.split > 1;
      if (!meet_now) __syncthreads();
      FOLD_STAMP();
      if (meet_now) {
        const FoldKernelArgs &a = args_now();
        const Ctx<NW> c = phase(cx);
        const uint32_t xnum = a.run.s[si].xnum;
        exchange_winners<NW>(a.dv, c, exchange_table(a.dv, a.run) + (((size_t)c.u * 2 + (xnum & 1u)) * c.split) * 2 * c.C,
                             xnum & 0xffffu);
        __syncthreads();
      }
      begin = false;
      if (a0 < 0) {
        FOLD_STAMP();
        if (n_app > 0) {
          if (cx.C <= 256)
            select_tokens<NW, 4>(phase(cx), m, n_app);
          else if (cx.C <= 512)
            select_tokens<NW, 8>(phase(cx), m, n_app);
          else
            select_long<NW>(phase(cx), m, n_app);
          FOLD_STAMP();
        }
      }
      a0 = a1;
    } while (a0 < n_app);
    if (exact && cx.s_cnt()[kCntTies] > 0) {   // rarely
      const FoldKernelArgs &a = args_now();
      settle_ties<NW>(a.dv, phase(cx), m, n_app, keys_of(a, si));
      __syncthreads();
    }
    FOLD_STAMP();
    build_lists<NW>(args_now().dv, phase(cx));
    {
      const FoldKernelArgs &a = args_now();
      const Ctx<NW> c = phase(cx);
      gather_tokens<NW>(c, block_of(a.dv, c, a.src, a.run.s[si].tok, keys_of(a, si)));
    }
    if (n_app > 0) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // merges into rows just created
    if (si + 1 < run_n) fetch_first_keys(si + 1);
    FOLD_STAMP();
    {
      const FoldKernelArgs &a = args_now();
      const Ctx<NW> c = phase(cx);
      merge_rows<NW>(a.dv, c, block_of(a.dv, c, a.src, a.run.s[si].tok, keys_of(a, si)), sn);
    }
    FOLD_STAMP();
    // what the fold decided, for the record and for the entry point's optional outputs
    if (cx.part == 0) {
      const FoldKernelArgs &a = args_now();
      const Ctx<NW> c = phase(cx);
      const int64_t base = (int64_t)c.u * c.C;
      const int trace = a.run.s[si].trace;
      for (int j = c.tid; j < c.C; j += NT) {
        const int p = c.s_pi()[j];
        const float2 sc = make_float2(c.s_app()[j], c.s_best()[j]);
        a.dv.pi[base + j] = p;
        a.dv.score[base + j] = sc;
        if (a.run.trace_assign && trace >= 0) a.run.trace_assign[trace * a.run.trace_stride + base + j] = p;
        if (a.run.trace_score && trace >= 0)
          reinterpret_cast<float2 *>(a.run.trace_score)[trace * a.run.trace_stride + base + j] = sc;
      }
    }
    // The next fold of the run reads what this one wrote, this workgroup's own stores: with resident tiles behind
    // barriers of its own that wait for them, so that this one is for LDS alone.  (With full barriers here and ahead of the
    // exchange 8192 tokens, 2 units, 128-token blocks, 600 rows 976 -> 998 us, 64 units of 64-token blocks 1947 -> 1977, 65536 tokens,
    // growing, 32 units 5.95 -> 5.99 ms; either one alone costs nothing.)
    if (cx.resident) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    } else {
      __syncthreads();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
  }
}

// The readout rows [0, m) of every unit recomputed from the stored sums (after an import), with the
// arithmetic of the folds above, so that a state that was exported and imported continues to the
// bit like one that was not.
__global__ __launch_bounds__(256) void refresh16_kernel(Dev dv, int m, int slot) {
  const int u = blockIdx.y;
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4), c16 = threadIdx.x & 15;
  if (row >= m) return;
  const int64_t ro = (int64_t)u * dv.Mcap + row;
  double sk[8];
  float sv[8];
  load_sums(dv, ro, c16, sk, sv);
  store_readout16(dv, slot, ro, c16, normalised16(dv, sk, ln_params(dv, u), c16), sv, dv.rho[ro]);
}

constexpr size_t kLdsWide = 160 * 1024, kLdsNarrow = 96 * 1024;
bool pow2(int x) { return x > 0 && (x & (x - 1)) == 0; }
constexpr int kGatherLeast = 32;   // tokens: the fresh tile's size
// K-hat tiles a workgroup keeps in LDS for a whole run, 0 when they do not fit beside the rest
int resident_tiles(const Dev &dv, int NW, int split, size_t limit) {
  const int own = own_tiles_most(dv.Mcap, split);
  const size_t rest = lds_fresh(NW, dv.C, own) + (size_t)kGatherLeast * kTokenBytes;
  return own <= 2 * stage_tiles(NW) && rest + (size_t)own * kTileBytes <= limit ? own : 0;
}
// Tokens the scratch holds: with resident tiles twice the number expected per workgroup as far as the
// limit goes; otherwise what the ring has room for.
int gather_tokens_most(const Dev &dv, int NW, int split, size_t limit) {
  const int kept = resident_tiles(dv, NW, split, limit);
  if (!kept) return 2 * stage_tiles(NW) * kTileBytes / kTokenBytes;
  const size_t rest = lds_fresh(NW, dv.C, own_tiles_most(dv.Mcap, split)) + (size_t)kept * kTileBytes;
  const int room = (int)((limit - rest) / kTokenBytes) / 4 * 4, want = 2 * dv.C / split;
  const int g = room < want ? room : want;
  return g > kGatherLeast ? g : kGatherLeast;
}
size_t lds_bytes(const Dev &dv, int NW, int split, size_t limit) {
  const size_t n = lds_fresh(NW, dv.C, own_tiles_most(dv.Mcap, split)) +
                   (size_t)resident_tiles(dv, NW, split, limit) * kTileBytes +
                   (size_t)gather_tokens_most(dv, NW, split, limit) * kTokenBytes;
  if (split == 1) return n;
  // (a workgroup that shares a unit must also be able to take over all of it)
  const size_t taken = lds_fresh(NW, dv.C, own_tiles_most(dv.Mcap, 1)) + (size_t)kGatherTaken * kTokenBytes;
  return n > taken ? n : taken;
}

}  // namespace

// The shapes this path takes: bf16, head_dim 128; blocks of 2^k * 32 tokens up to 1024 (the waves
// that share a token group split a stage's tiles by a power of two); tables that fit LDS.
bool fold_fused_fits(const Dev &dv, int split) {
  if (!(dv.io == 1 && dv.d == kHeadDim && dv.C % 64 == 0 && dv.C <= kMaxBlock && pow2(dv.C / 32))) return false;
  if (!pow2(split) || split > kFoldMaxSplit || dv.Mcap >= 0xffff) return false;   // rows travel in 16 bits
  return lds_bytes(dv, 16, split, kLdsWide) <= kLdsWide && lds_bytes(dv, 8, split, kLdsNarrow) <= kLdsNarrow;
}

bool fold_fused_resident(const Dev &dv, int split, bool narrow) {
  return fold_fused_fits(dv, split) && resident_tiles(dv, narrow ? 8 : 16, split, narrow ? kLdsNarrow : kLdsWide) > 0;
}
bool fold_fused_beside(const Dev &dv, int split) {
  return split > 1 && fold_fused_fits(dv, split) && resident_tiles(dv, 8, split, kLdsBesideAttention) > 0 &&
         lds_bytes(dv, 8, split, kLdsBesideAttention) <= kLdsBesideAttention;
}

size_t fold_exchange_bytes(int64_t units, int C, int split) {
  return split > 1 ? (size_t)units * (kArrivalWords + 2 * split * 2 * C) * sizeof(unsigned long long) : 0;
}

hipError_t launch_refresh16(const Dev &dv, int m, int slot, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(refresh16_kernel, dim3((m + 15) / 16, dv.U), dim3(256), 0, st, dv, m, slot);
  return hipGetLastError();
}

hipError_t launch_fold_fused(const Dev &dv, const Src &src, const FoldRunArgs &run_, bool narrow, hipEvent_t done,
                             hipStream_t st) {
  if (run_.n <= 0) return hipSuccess;
  FoldRunArgs run = run_;
  const int split = run.split, NW = narrow ? 8 : 16;
  if (split < 1 || (split > 1 && !run.xtab)) return hipErrorInvalidValue;
  const size_t limit = run.beside ? kLdsBesideAttention : narrow ? kLdsNarrow : kLdsWide;
  if (run.beside && (!narrow || !fold_fused_beside(dv, split))) return hipErrorInvalidValue;
  run.resident = resident_tiles(dv, NW, split, limit);
  run.gather = gather_tokens_most(dv, NW, split, limit);
  FoldKernelArgs args{dv, src, run};
  void *argv[] = {&args};
  const void *kernel = narrow ? (const void *)fold_fused_kernel<8> : (const void *)fold_fused_kernel<16>;
  static OncePerDevice<hipError_t> of_narrow, of_wide;
  if (const hipError_t e = allow_lds(narrow ? of_narrow : of_wide, kernel, narrow ? kLdsNarrow : kLdsWide); e != hipSuccess) return e;
  const dim3 grid((unsigned)(dv.U * split)), block(64 * NW);
  const size_t lds = lds_bytes(dv, NW, split, limit);
  const hipError_t e = done ? hipExtLaunchKernel(kernel, grid, block, argv, lds, st, nullptr, done, 0)
                            : hipLaunchKernel(kernel, grid, block, argv, lds, st);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace kvm
