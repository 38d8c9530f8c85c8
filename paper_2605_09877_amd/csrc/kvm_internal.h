// Internal declarations shared by the host side of the KVM library and its HIP kernels.
// Nothing here is part of the public ABI (see include/kvm.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "per_device.h"

namespace kvm {

// A kernel's launches may have `bytes` of dynamic LDS on the calling thread's device.
inline hipError_t allow_lds(OncePerDevice<hipError_t> &once, const void *kernel, size_t bytes) {
  return once([](int *dev) { return hipGetDevice(dev); },
              [&] { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes); });
}

// A strided source of per-token keys, values and merge gates for all units.
// Element strides; the head_dim axis is contiguous.  Token index 0 is `k`'s first token.
struct Src {
  const void *k, *v;
  const float *g;  // nullable: g = 1
  int64_t k_b, k_h, k_t;
  int64_t v_b, v_h, v_t;
  int64_t g_b, g_h, g_t;
};

// Device views of one bound state.  U = B * H_kv units; rows are padded to Mcap.
struct Dev {
  // state proper
  double *sK;    // [U, Mcap, d] running gated sums of memory keys (fp64: feeds the argmax)
  float *sV;     // [U, Mcap, d] running gated sums of values
  float *rho;    // [U, Mcap]    radius stored at row creation
  float *w;      // [U, Mcap]    1 + sum of merged gates (diagnostic)
  int32_t *n;    // [U, Mcap]    tokens in the row (diagnostic)
  // Normalised readout, one copy ("slot") per recent state version: version v (= number of
  // folds done) lives in slot v % NS.  A fold reads the old version and writes the new one in
  // full, so attention over earlier chunks can still be running on the old slots.
  void *khat;    // [NS, U, Mcap, d] I/O dtype: LN_s(sK)
  void *vhat;    // [NS, U, Mcap, d] I/O dtype: rho * sV / max(||sV||, eps)
  int64_t slot_elems;  // U * Mcap * d
  int32_t NS;
  // window ring: token p lives in slot p % L
  void *winK, *winV;  // [U, L, d] I/O dtype
  float *winG;        // [U, L]
  // fold scratch, per overflow token
  void *kbar;        // [U, C, d] I/O dtype memory keys (the host points this at one of the
                     //           `group` blocks that a batched memkey launch fills)
  float2 *score;     // [U, C]    x = append score s_j, y = winning merge score
  int32_t *pi;       // [U, C]    row the token goes to
  int32_t *app;      // [U, C]    rank among appended tokens, or -1
  int32_t *creator;  // [U, C]    token that creates new row number a
  // decode: the memory-key scratch, idle while a step attends, also takes the partial results of
  // workgroups that share one sequence's keys (attn_rows.hip), as many as it has room for
  int64_t kbar_bytes;
  unsigned *part_cnt;  // [kShareGroups] a counter per group of them, zero between launches
  // parameters
  const float *gamma, *beta;          // [H_kv, d] or null
  const float *tau_state, *tau_bswa;  // [H_q] or null
  int32_t B, Hq, Hkv, U, d, r, C, L, S, Mcap;
  int32_t Ufull;  // units of the whole state (a view of part of the batch keeps the state's strides)
  float ln_eps, norm_eps;
  int32_t io;  // KVM_F32 / KVM_BF16
};


// One attention launch: the queries of up to kMaxGroup consecutive chunks (prefill), or one
// query per sequence (decode).  Chunk boundaries are absolute multiples of C.
constexpr int kMaxGroup = 16;
struct AttnArgs {
  const void *q;
  void *out;
  float *lse;  // nullable
  int64_t q_b, q_t, q_h, o_b, o_t, o_h, lse_b, lse_t, lse_h;  // q/out/lse index 0 = position s
  Src in;            // keys/values of this call: token index 0 = position t0
  int64_t t0;        // positions below t0 come from the ring
  int64_t s;         // position of the first query of the launch
  int32_t n_chunks;  // chunks covered
  int32_t nq_total;  // queries covered (all chunks but the last are full)
  int32_t put_token = 0;  // decode (rows kernel): also store the token at position s into the ring
  int32_t m[kMaxGroup];     // state rows each chunk sees
  int32_t slot[kMaxGroup];  // readout slot of that state version
};

// Where the record of a fold goes (kvm_state_trace), from the first unit of the launch on; nulls: nowhere.  Written, and never
// read, by the fold's last launch: the fold works in its own scratch whatever becomes of the caller's memory.
struct Record {
  int32_t *assign = nullptr;   // [U, C]
  float *score = nullptr;      // [U, C, 2]
};

// fold.hip
hipError_t launch_memkey(const Dev &dv, const Src &src, int n_blocks, hipStream_t st);
hipError_t launch_score(const Dev &dv, int slot, int row0, int row1, bool first_pass, bool beside_attention, hipStream_t st);
hipError_t launch_select(const Dev &dv, int m, int n_app, bool take_all, hipStream_t st);
hipError_t launch_accum(const Dev &dv, const Src &src, int m_before, int m_after, int row_begin,
                        bool do_create, bool do_merge, bool do_copy, bool check_app, int slot_old,
                        int slot_new, const Record &rec, hipStream_t st);
// selection + creation + second scoring pass of a small append, one launch
constexpr int kAppendMax = 16;
__host__ __device__ inline bool append_fits(int C, int n_app) {
  return n_app > 0 && n_app <= kAppendMax && C % 2 == 0 && C <= 256;
}
hipError_t launch_append(const Dev &dv, const Src &src, int m, int n_app, int slot_new, hipStream_t st);
// the merge of a small fold in a prefill: token-centred merge into slot_new + copies of untouched rows
hipError_t launch_merge_copy(const Dev &dv, const Src &src, bool check_app, int slot_old, int slot_new,
                             int m_before, const Record &rec, hipStream_t st);
hipError_t launch_merge_inplace(const Dev &dv, const Src &src, bool check_app, int slot, const Record &rec, hipStream_t st);
hipError_t launch_refresh(const Dev &dv, int m, int slot, hipStream_t st);
hipError_t launch_ring_copy(const Dev &dv, const Src &src, int64_t src_t0, int64_t p0, int64_t p1,
                            hipStream_t st);
// fold_fused.hip (bf16, d = 128): a run of up to kFoldMaxSteps consecutive folds in one launch,
// run.split workgroups per unit.  Step i folds the block whose first token is src's token s[i].tok and
// whose memory keys are in slab s[i].kbar_block of the scratch (launch_memkey), from s[i].m to
// s[i].m_after rows, reading readout slot s[i].so and writing slot s[i].sn (the same slot when
// in_place; otherwise untouched rows are copied over).  trace >= 0: the fold's assignments and
// scores also go to trace_assign / trace_score at that fold index (trace_stride = tokens of one
// fold over all units).  narrow: the 8-wave workgroup that fits beside an attention workgroup on
// a compute unit; otherwise 16 waves and the unit to itself.
constexpr int kFoldMaxSteps = 8;   // a group's worth.  A run's border costs the chain some 15 us (launch, keys and tiles
                                   // fetched anew): 65536 tokens, growing state, 32 units: 6.85 ms in runs of 4, 6.35 in runs of 8
// LDS of a shared fold's workgroup and of an attention workgroup launched with kBesideFoldLds more: one of each fills a
// compute unit, and a second attention workgroup does not fit (attn_mfma.hip: launch_attn_mfma)
constexpr size_t kLdsBesideAttention = 78 * 1024, kBesideFoldLds = 17 * 1024;
constexpr int kFoldMaxSplit = 16;  // workgroups that may share a unit's rows
struct FoldStep {
  int32_t m, m_after, so, sn;
  int64_t tok;
  int32_t trace, kbar_block;
  uint32_t xnum, pad;   // number of the fold's exchange among the unit's workgroups (split > 1)
};
struct FoldRunArgs {
  int32_t n, in_place;
  FoldStep s[kFoldMaxSteps];
  int32_t *trace_assign;
  float *trace_score;
  int64_t trace_stride;
  int32_t split;               // workgroups per unit (a power of two); 1: none of the next four is used
  unsigned long long *xtab;    // arrival words and exchange table, fold_exchange_bytes() of zeroed device memory
  uint32_t arrived;            // workgroups per unit of the earlier launches since the table was zeroed
  uint32_t launch;             // number of this launch since then, from 1
  uint32_t patience;           // how long a workgroup waits for its unit's others to start, ticks of 10 ns
  int32_t beside;              // the launch runs beside attention: LDS of at most kLdsBesideAttention where the tiles fit that
  int32_t resident;            // (set by the launch) K-hat tiles a workgroup keeps in LDS, 0: they stream through a ring
  int32_t gather;              // (likewise) merging tokens the LDS scratch holds
};
constexpr int kArrivalWords = 8;   // an arrival word of the table to itself in 64 bytes
bool fold_fused_fits(const Dev &dv, int split = 1);
// whether each of a unit's `split` workgroups keeps its normalised keys in LDS for a whole run
bool fold_fused_resident(const Dev &dv, int split, bool narrow);
// whether they do so within kLdsBesideAttention
bool fold_fused_beside(const Dev &dv, int split);
size_t fold_exchange_bytes(int64_t units, int C, int split);
// readout rows [0, m) recomputed from the sums with the one-launch path's arithmetic
hipError_t launch_refresh16(const Dev &dv, int m, int slot, hipStream_t st);
// done: an event that stands for the end of the launch (the kernel's own completion signal: nothing more is put on the
// stream; not on a stream under capture), or null
hipError_t launch_fold_fused(const Dev &dv, const Src &src, const FoldRunArgs &run, bool narrow, hipEvent_t done,
                             hipStream_t st);
// score_mfma.hip (bf16, d = 128)
hipError_t launch_score_mfma(const Dev &dv, int slot, int row0, int row1, bool first_pass, hipStream_t st);
// attn_rows.hip
constexpr int kSplitWorkgroups = 1024;  // workgroups of a decode launch whose keys are shared
// Up to this many (sequence, head group) pairs they are.  A step alone against shared, us: 128 pairs 10.7 / 10.8 (158 rows) to
// 27.5 / 20.3 (1200 rows), 96 pairs of four heads 16.7 / 13.8 to 45.9 / 27.3; but 256 pairs 11.9 / 14.5 to 30.5 / 33.1, of
// four heads 18.0 / 26.0 to 47.0 / 47.3.
constexpr int kShareGroups = 128;
hipError_t launch_attn_rows(const Dev &dv, const AttnArgs &a, hipStream_t st);
// One decode step over sequences of several states (kvm_decode_step_multi): per sequence, where
// its arrays start (its first KV head) and where it stands.
struct SeqDesc {
  const void *khat, *vhat;  // current readout version, this sequence's first unit
  void *winK, *winV;        // window ring, this sequence's first unit
  float *winG;
  int64_t pos;              // position of the token being decoded
  int32_t m, Mcap;          // state rows now, rows per unit in the buffer
};
// The same of up to kPackStates states as a kernel argument: no table to write ahead of the launch (copied from the host it was a
// launch of its own of 4.8 us and as much of host time; 3 x 4 heads on 2, 353 rows: 12.4 us a step before,
// 10.2 now).  64 of them, 2.3 KiB, of the 4 KiB that a launch's arguments may have (16 steps, 8 heads on 2, 300 rows, table / arguments: 64 states
// 504 / 477 us; 96, 3.4 KiB: 605 / 575).
constexpr int kPackStates = 64;
struct SeqPack {
  const void *khat[kPackStates];   // current readout version, first unit; v-hat is decode_value_offset() bytes further on
  void *winK[kPackStates];         // first unit; the rings of values and gates follow, decode_ring_offset() bytes apart
  int64_t pos[kPackStates];
  int32_t m[kPackStates], Mcap[kPackStates];
  int32_t seq0[kPackStates + 1];   // first sequence of each state; [n] = one past the last
  int32_t n;
};
__host__ __device__ inline int64_t up256(int64_t x) { return (x + 255) & ~(int64_t)255; }
__host__ __device__ inline int64_t decode_value_offset(int64_t NS, int64_t U, int64_t Mcap, int64_t d, int64_t es) {
  return up256(NS * U * Mcap * d * es);
}
__host__ __device__ inline int64_t decode_ring_offset(int64_t U, int64_t L, int64_t d, int64_t es) { return up256(U * L * d * es); }
// seq: the table, or null: pack.  most_keys: the largest number of keys (state rows and window) any of the sequences attends to
hipError_t launch_decode_multi(const Dev &dv, const SeqDesc *seq, const SeqPack &pack, int n_seq, int most_keys, const void *q,
                               const void *k, const void *v, const float *gate, void *out, hipStream_t st);
// attn_mfma.hip: prompts in bf16, d = 128 or 64, blocks of a multiple of 64 tokens (tiles of 64 keys neither cross
// from the ring into the call's keys nor wrap in the ring); everything else is the row kernel's
// With d = 64 and few queries in a chunk's launch the row kernel, a workgroup per query and head, fills more of the chip.
// Attention us a launch, row kernel / tiles, by queries x heads of the chunk (64-, 256-, 512-token blocks, rows = block):
// 512: 8.8 / 10.3, 12.8 / 19.4, 20.5 / 32.0; 1024: 10.7 / 10.2, 18.0 / 19.5, 29.0 / 32.8; 2048: 15.5 / 10.2, 27.2 / 19.4,
// 46.4 / 33.0; 8192: 80.6 / 19.5 (256), 140.5 / 33.2 (512); with 1000 rows the same order at every one of them.
inline bool attention_on_mfma(const Dev &dv) {
  return dv.io == 1 && dv.C % 64 == 0 && (dv.d == 128 || (dv.d == 64 && (int64_t)dv.B * dv.Hq * dv.C > 1024));
}
// beside_folds: one workgroup per compute unit, so that those of shared folds find theirs free at any time
hipError_t launch_attn_mfma(const Dev &dv, const AttnArgs &a, bool beside_folds, hipStream_t st);

// A chunk's attention with the first scoring pass of the fold after it (rows [0, m) of readout slot `slot`, memory keys at
// dv.kbar), one launch: for states without the matrix-core folds, where its one dimension holds the workgroups (a dimension
// takes fewer than 2^32 threads; the launches apart have three) and it is the faster way.
constexpr int64_t kMostWorkgroups = (1 << 24) - 1;   // of 256 threads
bool attention_takes_scores(const Dev &dv, const AttnArgs &a, int m);
hipError_t launch_attn_score(const Dev &dv, const AttnArgs &a, int slot, int m, hipStream_t st);
bool attn_rows_take_scores(const Dev &dv, const AttnArgs &a, int m);
hipError_t launch_attn_rows_score(const Dev &dv, const AttnArgs &a, int slot, int m, hipStream_t st);

// backward.hip: the backward pass of a whole-sequence prefill that started from an empty state.
// Dense operands: q, out, dout, dq [B, T, Hq, d]; k, v, dk, dv [B, T, Hkv, d]; gate, dgate
// [B, T, Hkv]; lse [B, T, Hq]; assign [folds, U, C].  The work arrays have the state's row
// capacity (Mcap rows per unit).
struct Bwd {
  Dev dv;  // dimensions, parameters and the final sums (sK, sV, rho) of the state after the forward
  bool on_mfma;  // attention adjoints on the matrix cores (decides the workspace layout and the launches)
  int32_t launches;  // KVM_DEBUG_BACKWARD_LAUNCHES
  int64_t T;
  const void *q, *k, *v, *out, *dout;
  const float *gate, *lse;
  const int32_t *assign;
  const float *score;  // [folds, U, C, 2] the forward's record of (append score, merge score)
  void *dq, *dk, *dv_out;
  float *dgate, *dgamma, *dbeta, *dtau_state, *dtau_bswa;
  // workspace
  double *wsK;           // [U, Mcap, d] key sums of the version being visited
  float *wsV;            // [U, Mcap, d]
  float *dsK, *dsV;      // [U, Mcap, d] adjoints of the sums
  float *drho;           // [U, Mcap]
  void *khat, *vhat;     // [U, Mcap, d] I/O dtype: readout of the version being visited
  float *xhat;           // [U, Mcap, d] the key sums of that version, standardised (before gamma, beta)
  float *rden;           // [U, Mcap]    1 / sqrt(var + eps) of those rows
  float *dkhat, *dvhat;  // [U, Mcap, d] adjoint of that readout (one chunk's)
  // fp32 accumulators of dk, dv: [B, T, Hkv, d] (ring_rows = 0), or, on the matrix-core path, only
  // the share a token gets when its fold is undone, kept until the token's block is finished as
  // window keys: [U, ring_rows, d] with ring_rows = L + C, block number mod (n_bswa + 1)
  float *dk_acc, *dv_acc;
  int32_t ring_rows;
  float *delta;          // [B, T, Hq] sum over channels of dout * out
  int32_t delta_ready;   // it is there already: the dq role reads it
  float *P, *dS;         // [U, G, C, Mcap + L] probabilities and logit adjoints of one chunk
  double *par64;         // [2 * Hkv * d + 2 * Hq] fp64 accumulators of dgamma, dbeta, dtau_state, dtau_bswa
};
// one chunk of the walk: its queries, the state rows it saw, and the fold that followed it
struct BwdChunk {
  int64_t s;       // first position
  int32_t nq;      // queries
  int32_t m;       // state rows the chunk saw ( = rows before the fold that follows)
  int32_t fold;    // index of the fold that followed the chunk, or -1
  int32_t m_after; // state rows after that fold
};
// Two more streams and a few untimed events, owned by the caller, for the matrix-core path: what
// does not depend on the dq role's D, or on the state at all, runs beside the chain undo-fold ->
// dq -> dk of the state rows (see run_backward).
struct BwdStreams {
  hipStream_t side = nullptr, side2 = nullptr;  // null: everything on the one stream
  hipEvent_t fork = nullptr, dq_done = nullptr, join_state = nullptr, join_window[2] = {nullptr, nullptr};
};
hipError_t run_backward(const Bwd &a, const BwdChunk *chunks, int n_chunks, hipStream_t st, const BwdStreams &x);
// backward_mfma.hip (bf16, d = 128): one chunk's dq, dk, dv and readout adjoint on the matrix cores
bool backward_on_mfma(const Dev &dv);
// D = dout . out of `rows` queries, ahead of the walk
hipError_t launch_delta_mfma(const Bwd &a, int64_t rows, hipStream_t st);
enum { kRoleDQ = 0, kRoleKV = 1 };
enum { kSecBoth = 0, kSecWindow = 1, kSecState = 2 };
// one role of the matrix-core tile kernel over one chunk; role KV: all key workgroups, or only
// those of the chunk's own tokens (window keys), or only those of the state rows
hipError_t launch_backward_mfma(const Bwd &a, int64_t cs, int nq, int m, bool folded, int role, int section,
                                hipStream_t st);
// both roles in one launch, where a whole chunk's workgroups into m state rows are few enough; needs D.  Whole calls of training,
// launches of their own on three streams / one, us (workgroups): 224 of 32 units 1050 / 801, 8 units, growing, 8465 tokens (up to 128)
// 3990 / 2960, 12 units of 64-token chunks, 20764 tokens (120) 27300 / 17500, 512 of 96 units 2118 / 1972, 704 of 128 units 2550 / 2474,
// 768 of 128 units 3517 / 3317, 960 of 96 4514 / 4028, 1024 of 64, 1536 rows 9511 / 7917, of 64 with two heads each 2876 / 2799.  (Beyond, as far as
// measured, one launch is still ahead: 1280 of 160 units 5770 / 5416, 1536 of 128 3879 / 3660, 2048 of 256 8061 / 7728.)  But
// with four heads per KV head: 96 of 8 units 4110 / 2750, 224 of 16 1632 / 1619, but 336 of 24 1737 / 1776, 448 of 32 1910 / 2050 (their
// loops are long, and the kernel of both roles spills more in them).
constexpr unsigned kBwdOneLaunch = 1024, kBwdOneLaunchHeads = 256;   // (up to two query heads per KV head; more)
bool backward_fits_one_launch(const Dev &dv, int m);
hipError_t launch_backward_mfma_both(const Bwd &a, int64_t cs, int nq, int m, bool folded, hipStream_t st);

}  // namespace kvm
