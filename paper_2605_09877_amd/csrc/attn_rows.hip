// Row attention: one workgroup per (query, query head, sequence) runs the single softmax of the
// paper's "Readout" equations over [normalised state rows || visible window tokens], streaming
// keys and values once from HBM.  This is the decode kernel (one query per sequence, memory
// bound) and also serves fp32 prefill, where every query of a chunk gets its own workgroup.
//
// A key row of D elements is read by D/VEC adjacent lanes with one 16-byte load each, so a wave
// covers 64/(D/VEC) keys per step; each such lane group keeps its own online-softmax state
// (running max, sum, output fragment) and the groups are merged at the end.
#include "kvm_device.h"
#include "kvm_internal.h"
#include "kvm_score.h"

namespace kvm {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kMaxSplit = 64;  // shares of one sequence's keys: a lane each when they are put together

// What one workgroup needs, gathered by the kernels below: a query position of one unit and GQ
// consecutive query heads of it (GQ = 1: one head; in a decode step with grouped queries a
// workgroup takes a KV head's whole group, so that every key and value row is fetched once for
// all of its heads instead of once per head).
template <typename T>
struct RowQuery {
  const T *q, *khat, *vhat, *ring_k, *ring_v, *in_k, *in_v;  // first head's query row, this unit's arrays
  T *out;            // first head's output row
  float *lse;        // first head's slot, or null
  int64_t q_h, o_h, lse_h;  // element strides between the heads
  int64_t pos, t0;   // query position; window positions below t0 come from the ring
  int64_t in_kt, in_vt;
  int m, hq;         // state rows; first head
  // decode: the workgroup that holds a KV head's first query head also stores the new token (k,
  // v, gate at position pos, read from in_k / in_v like every key at or after t0) into its ring
  // slot; nobody reads that slot in this launch
  T *put_k, *put_v;  // ring rows of this unit, or null
  float *put_g;
  float gate;
  // keys shared among n_split workgroups (decode): this one's number, and where the group of
  // workgroups that belong to the same query heads leaves its partial results
  int split, n_split;
  float *part_acc;   // [n_split][GQ][D] unnormalised outputs
  float2 *part_ml;   // [n_split][GQ] (reference point, sum)
  unsigned *part_cnt;
};

// What crosses compute units is written and read with relaxed device-scope atomics, two floats at a
// time: such a store goes through to memory, so once the workgroup has waited for its own
// (s_waitcnt) they are there for every other one, and no cache has to be written back or dropped.
// (A release and an acquire fence around plain accesses: 24.4 instead of 12.3 us for the launch of one
// sequence, 1536 keys, 32 query heads on 8.)
__device__ __forceinline__ void put_pair(void *p, float a, float b) {
  const unsigned long long v = ((unsigned long long)__float_as_uint(b) << 32) | __float_as_uint(a);
  __hip_atomic_store((unsigned long long *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 get_pair(const void *p) {
  const unsigned long long v = __hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// The last workgroup of a group to get here puts the shares together (the counter wraps to zero by
// itself, ready for the next step).
template <typename T, int D, int GQ>
__device__ __forceinline__ void combine_shares(const RowQuery<T> &rq) {
  __shared__ int last;
  __shared__ float weight[GQ][kMaxSplit], inv_l[GQ];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) last = atomicInc(rq.part_cnt, (unsigned)rq.n_split - 1u) == (unsigned)rq.n_split - 1u;
  __syncthreads();
  if (!last) return;
  if (wave < GQ) {   // a wave per head, a lane per share
    const bool on = lane < rq.n_split;
    const float2 ml = on ? get_pair(rq.part_ml + lane * GQ + wave) : make_float2(-INFINITY, 0.f);
    const float w = exp2f(ml.x - wave_max(ml.x));
    const float l = wave_sum(ml.y * w);
    if (on) weight[wave][lane] = w;
    if (lane == 0) inv_l[wave] = 1.f / l;
  }
  __syncthreads();
  for (int e = 2 * threadIdx.x; e < GQ * D; e += 512) {   // two channels of one head
    const int hh = e / D, ch = e % D;
    float o0 = 0.f, o1 = 0.f;
#pragma unroll 8
    for (int s = 0; s < rq.n_split; ++s) {
      const float2 x = get_pair(rq.part_acc + (int64_t)(s * GQ + hh) * D + ch);
      o0 = fmaf(x.x, weight[hh][s], o0);
      o1 = fmaf(x.y, weight[hh][s], o1);
    }
    T *out = rq.out + hh * rq.o_h + ch;
    if constexpr (sizeof(T) == 4)
      *reinterpret_cast<float2 *>(out) = make_float2(o0 * inv_l[hh], o1 * inv_l[hh]);
    else
      *reinterpret_cast<uint32_t *>(out) = pack_bf16(o0 * inv_l[hh], o1 * inv_l[hh]);
  }
}

// NW: waves per workgroup.  kShared: the keys may be shared among workgroups.  A kernel of its own, because what sharing adds costs registers, in bf16
// one head at a time 82 instead of 79 and with them a wave per SIMD (five instead of six): 40 sequences of 16 heads on
// 328 rows, their fold included, 31.2 instead of 30.5 us a token, 10 of 32 heads on 16 17.0 instead of 16.7.
template <typename T, int D, int GQ, bool kShared, int NW = 4>
__device__ __forceinline__ void attn_row(const Dev &dv, const RowQuery<T> &rq) {
  static_assert(NW == 4 || !kShared, "shares are put together by four waves");
  constexpr int VEC = Vec16<T>::kN;
  constexpr int LPR = D / VEC;   // lanes per key row
  constexpr int RPW = 64 / LPR;  // key rows per wave step
  constexpr int KB = 4;          // rows in flight per lane group
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane / LPR, cl = lane % LPR;
  const int64_t pos = rq.pos;
  const int64_t cs = pos / dv.C * dv.C;                      // its chunk starts here
  const int64_t wb = cs + dv.C - dv.L > 0 ? cs + dv.C - dv.L : 0;  // first window position

  if (rq.put_k && threadIdx.x < LPR) {
    const int slot = (int)(pos % dv.L);
    float x[VEC];
    Vec16<T>::load(rq.in_k + (pos - rq.t0) * rq.in_kt + threadIdx.x * VEC, x);
    Vec16<T>::store(rq.put_k + (int64_t)slot * D + threadIdx.x * VEC, x);
    Vec16<T>::load(rq.in_v + (pos - rq.t0) * rq.in_vt + threadIdx.x * VEC, x);
    Vec16<T>::store(rq.put_v + (int64_t)slot * D + threadIdx.x * VEC, x);
    if (threadIdx.x == 0) rq.put_g[slot] = rq.gate;
  }
  const float rs = kLog2e * rsqrtf((float)D);
  float qf[GQ][VEC], c_state[GQ], c_bswa[GQ];
#pragma unroll
  for (int hh = 0; hh < GQ; ++hh) {
    Vec16<T>::load(rq.q + hh * rq.q_h + cl * VEC, qf[hh]);
    c_state[hh] = (dv.tau_state ? dv.tau_state[rq.hq + hh] : 1.f) * rs;
    c_bswa[hh] = (dv.tau_bswa ? dv.tau_bswa[rq.hq + hh] : 1.f) * rs;
  }

  const int m = rq.m;
  int total = m + (int)(pos - wb + 1);
  int n_first = 0;
  if constexpr (kShared) {
    // this workgroup's share: whole rounds of the loop below (a share can be empty)
    constexpr int kRound = 4 * RPW * KB;
    const int per = ((total + rq.n_split - 1) / rq.n_split + kRound - 1) / kRound * kRound;
    n_first = rq.split * per;
    total = total < n_first + per ? total : n_first + per;
  }
  const T *khat = rq.khat, *vhat = rq.vhat, *ring_k = rq.ring_k, *ring_v = rq.ring_v;
  const T *in_k = rq.in_k, *in_v = rq.in_v;

  float m_run[GQ], l_run[GQ], acc[GQ][VEC];
#pragma unroll
  for (int hh = 0; hh < GQ; ++hh) {
    m_run[hh] = -INFINITY;
    l_run[hh] = 0.f;
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[hh][i] = 0.f;
  }

  for (int n0 = n_first; n0 < total; n0 += NW * RPW * KB) {
    float kf[KB][VEC], vf[KB][VEC];
    bool is_state[KB], on[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int n = n0 + (kb * NW + wave) * RPW + sub;
      const int nc = n < total ? n : total - 1;
      const T *kp, *vp;
      if (nc < m) {
        kp = khat + (int64_t)nc * D;
        vp = vhat + (int64_t)nc * D;
      } else {
        const int64_t p = wb + (nc - m);
        if (p >= rq.t0) {
          kp = in_k + (p - rq.t0) * rq.in_kt;
          vp = in_v + (p - rq.t0) * rq.in_vt;
        } else {
          const int slot = (int)(p % dv.L);
          kp = ring_k + (int64_t)slot * D;
          vp = ring_v + (int64_t)slot * D;
        }
      }
      Vec16<T>::load(kp + cl * VEC, kf[kb]);
      Vec16<T>::load(vp + cl * VEC, vf[kb]);
      on[kb] = n < total;
      is_state[kb] = nc < m;
    }
#pragma unroll
    for (int hh = 0; hh < GQ; ++hh) {
      float t[KB];
      float m_new = m_run[hh];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        float dot = 0.f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) dot = fmaf(qf[hh][i], kf[kb][i], dot);
        dot = group_sum<LPR>(dot);  // over the lanes that share the key row, on the vector ALU
        t[kb] = on[kb] ? dot * (is_state[kb] ? c_state[hh] : c_bswa[hh]) : -INFINITY;
        m_new = fmaxf(m_new, t[kb]);
      }
      if (m_new != -INFINITY) {
        const float alpha = exp2f(m_run[hh] - m_new);
        l_run[hh] *= alpha;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[hh][i] *= alpha;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const float p = exp2f(t[kb] - m_new);
          l_run[hh] += p;
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[hh][i] = fmaf(p, vf[kb][i], acc[hh][i]);
        }
        m_run[hh] = m_new;
      }
    }
  }

  __shared__ float sh_m[GQ][NW], sh_l[GQ][NW], sh_acc[GQ][NW][D];
#pragma unroll
  for (int hh = 0; hh < GQ; ++hh) {
    // merge the lane groups of this wave
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
      const float m_o = __shfl_xor(m_run[hh], o, kWave);
      const float l_o = __shfl_xor(l_run[hh], o, kWave);
      const float m_n = fmaxf(m_run[hh], m_o);
      const float sa = m_n == -INFINITY ? 0.f : exp2f(m_run[hh] - m_n);
      const float sb = m_n == -INFINITY ? 0.f : exp2f(m_o - m_n);
      l_run[hh] = l_run[hh] * sa + l_o * sb;
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[hh][i] = acc[hh][i] * sa + __shfl_xor(acc[hh][i], o, kWave) * sb;
      m_run[hh] = m_n;
    }
    if (sub == 0) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) sh_acc[hh][wave][cl * VEC + i] = acc[hh][i];
      if (cl == 0) {
        sh_m[hh][wave] = m_run[hh];
        sh_l[hh][wave] = l_run[hh];
      }
    }
  }
  __syncthreads();
  // merge the waves: wave hh % 4 finishes head hh
#pragma unroll
  for (int hh = 0; hh < GQ; ++hh) {
    if (wave == (hh & 3) && sub == 0) {
      float mm = fmaxf(fmaxf(sh_m[hh][0], sh_m[hh][1]), fmaxf(sh_m[hh][2], sh_m[hh][3]));
#pragma unroll
      for (int wv = 4; wv < NW; ++wv) mm = fmaxf(mm, sh_m[hh][wv]);
      float l = 0.f, o[VEC];
#pragma unroll
      for (int i = 0; i < VEC; ++i) o[i] = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) {
        // a wave that saw no key has max -inf -> 0 (none of them did: an empty share)
        const float sc = kShared && mm == -INFINITY ? 0.f : exp2f(sh_m[hh][wv] - mm);
        l += sh_l[hh][wv] * sc;
#pragma unroll
        for (int i = 0; i < VEC; ++i) o[i] += sh_acc[hh][wv][cl * VEC + i] * sc;
      }
      if constexpr (kShared) {
        // a share's maximum is -inf when it was empty (then l and o are 0 * finite = 0)
        const int slot = rq.split * GQ + hh;
#pragma unroll
        for (int i = 0; i < VEC; i += 2) put_pair(rq.part_acc + (int64_t)slot * D + cl * VEC + i, o[i], o[i + 1]);
        if (cl == 0) put_pair(rq.part_ml + slot, mm, l);
        continue;
      }
      const float inv = 1.f / l;
#pragma unroll
      for (int i = 0; i < VEC; ++i) o[i] *= inv;
      Vec16<T>::store(rq.out + hh * rq.o_h + cl * VEC, o);
      if (rq.lse && cl == 0) rq.lse[hh * rq.lse_h] = (mm + log2f(l)) * kLn2;
    }
  }
  if constexpr (kShared) combine_shares<T, D, GQ>(rq);
}

// Where the shares of query-head group number `group` of the launch go.
template <typename T, int D, int GQ>
__device__ __forceinline__ void set_share(RowQuery<T> &rq, const Dev &dv, int group) {
  const int n_groups = (int)(gridDim.y * gridDim.z);
  rq.part_acc = (float *)dv.kbar + (int64_t)group * rq.n_split * GQ * D;
  rq.part_ml = (float2 *)((float *)dv.kbar + (int64_t)n_groups * rq.n_split * GQ * D) + group * rq.n_split * GQ;
  rq.part_cnt = dv.part_cnt + group;
}

// One workgroup per (query, group of GQ query heads, sequence) of one state; shared, a decode step's:
// several per group.
template <typename T, int D, int GQ, bool kShared, int NW = 4>
__device__ __forceinline__ void attn_rows_of(const Dev &dv, const AttnArgs &a, int x, int y, int b) {
  // a decode step has one query per sequence, and the x dimension counts the shares of its keys
  const int qi = kShared ? 0 : x, hq = y * GQ;
  const int hkv = hq / (dv.Hq / dv.Hkv);
  const int u = b * dv.Hkv + hkv;
  RowQuery<T> rq;
  rq.pos = a.s + qi;
  const int ci = (int)(rq.pos / dv.C - a.s / dv.C);  // chunk of this query within the launch
  rq.q = (const T *)a.q + b * a.q_b + (int64_t)qi * a.q_t + hq * a.q_h;
  rq.out = (T *)a.out + b * a.o_b + (int64_t)qi * a.o_t + hq * a.o_h;
  rq.lse = a.lse ? a.lse + b * a.lse_b + (int64_t)qi * a.lse_t + hq * a.lse_h : nullptr;
  rq.q_h = a.q_h;
  rq.o_h = a.o_h;
  rq.lse_h = a.lse_h;
  rq.m = a.m[ci];
  rq.hq = hq;
  rq.khat = (const T *)dv.khat + a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D;
  rq.vhat = (const T *)dv.vhat + a.slot[ci] * dv.slot_elems + (int64_t)u * dv.Mcap * D;
  rq.ring_k = (const T *)dv.winK + (int64_t)u * dv.L * D;
  rq.ring_v = (const T *)dv.winV + (int64_t)u * dv.L * D;
  rq.in_k = (const T *)a.in.k + b * a.in.k_b + hkv * a.in.k_h;
  rq.in_v = (const T *)a.in.v + b * a.in.v_b + hkv * a.in.v_h;
  rq.in_kt = a.in.k_t;
  rq.in_vt = a.in.v_t;
  rq.t0 = a.t0;
  rq.put_k = rq.put_v = nullptr;
  rq.put_g = nullptr;
  rq.gate = 1.f;
  rq.split = kShared ? x : 0;
  rq.n_split = kShared ? gridDim.x : 1;
  if constexpr (kShared) set_share<T, D, GQ>(rq, dv, b * gridDim.y + y);
  if (a.put_token && rq.split == 0 && hq == hkv * (dv.Hq / dv.Hkv)) {
    rq.put_k = (T *)dv.winK + (int64_t)u * dv.L * D;
    rq.put_v = (T *)dv.winV + (int64_t)u * dv.L * D;
    rq.put_g = dv.winG + (int64_t)u * dv.L;
    rq.gate = a.in.g ? a.in.g[b * a.in.g_b + hkv * a.in.g_h + (rq.pos - a.t0) * a.in.g_t] : 1.f;
  }
  attn_row<T, D, GQ, kShared, NW>(dv, rq);
}

template <typename T, int D, int GQ, bool kShared, int NW>
__global__ __launch_bounds__(64 * NW) void attn_rows_kernel(Dev dv, AttnArgs a) {
  attn_rows_of<T, D, GQ, kShared, NW>(dv, a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// A chunk's attention and, in further workgroups, the scores of the block that is folded after it: both read the same state
// version and neither writes what the other reads, so the chain from chunk to chunk is a launch shorter.  Us per call, apart /
// in one launch: fp32, 2 heads of 64 channels, 1024 tokens in 64-token chunks, 64 rows 305 / 211; fp32, 4 units of 128
// channels, 1500 tokens in 64-token chunks, 100 rows 655 / 523; bf16, 96-token chunks, 200 rows 437 / 355.
// The scores' workgroups come first: they are the longer ones (the last of these calls 390 us the other way round).
template <typename T, int D, bool kTwo>
__global__ __launch_bounds__(256) void attn_rows_score_kernel(Dev dv, AttnArgs a, int slot, int m) {
  const int per_unit = (dv.C + 3) / 4, n_score = per_unit * dv.U;
  int id = blockIdx.x;
  if (id < n_score) {
    score_tokens<T, D, kTwo>(dv, slot, 0, m, 1, id % per_unit, id / per_unit);
  } else {
    id -= n_score;
    attn_rows_of<T, D, 1, false>(dv, a, id % a.nq_total, id / a.nq_total % dv.Hq, id / a.nq_total / dv.Hq);
  }
}

// Decode over sequences that live in different states (each at its own position, with its own
// number of state rows): one workgroup, or several sharing the keys, per (group of GQ query heads,
// sequence); sequence s reads seq[s].  dv is the states' common configuration (heads, chunk, window, temperatures).
template <typename T, int D>
__device__ __forceinline__ SeqDesc seq_of(const Dev &dv, const SeqPack &pk, int s) {
  int i = s;
  if (pk.seq0[pk.n] != pk.n) {   // some state has several sequences
    int hi = pk.n;
    i = 0;
    while (hi - i > 1) {
      const int mid = (i + hi) / 2;
      if (pk.seq0[mid] <= s) i = mid; else hi = mid;
    }
  }
  const int64_t es = sizeof(T), U = (int64_t)(pk.seq0[i + 1] - pk.seq0[i]) * dv.Hkv, u0 = (int64_t)(s - pk.seq0[i]) * dv.Hkv;
  const int64_t ring = decode_ring_offset(U, dv.L, D, es);
  SeqDesc sd;
  sd.m = pk.m[i];
  sd.Mcap = pk.Mcap[i];
  sd.pos = pk.pos[i];
  sd.khat = (const char *)pk.khat[i] + u0 * sd.Mcap * D * es;
  sd.vhat = (const char *)sd.khat + decode_value_offset(dv.NS, U, sd.Mcap, D, es);
  sd.winK = (char *)pk.winK[i] + u0 * dv.L * D * es;
  sd.winV = (char *)sd.winK + ring;
  sd.winG = (float *)((char *)pk.winK[i] + 2 * ring) + u0 * dv.L;
  return sd;
}
template <typename T, int D, int GQ, bool kShared, int NW>
__global__ __launch_bounds__(64 * NW) void attn_rows_multi_kernel(Dev dv, const SeqDesc *seq, SeqPack pk, const void *q,
                                                              const void *k, const void *v, const float *gate,
                                                              void *out) {
  const int hq = blockIdx.y * GQ, s = blockIdx.z;
  const int hkv = hq / (dv.Hq / dv.Hkv);
  const SeqDesc sd = seq ? seq[s] : seq_of<T, D>(dv, pk, s);
  RowQuery<T> rq;
  rq.pos = sd.pos;
  rq.q = (const T *)q + ((int64_t)s * dv.Hq + hq) * D;
  rq.out = (T *)out + ((int64_t)s * dv.Hq + hq) * D;
  rq.lse = nullptr;
  rq.q_h = rq.o_h = D;
  rq.lse_h = 0;
  rq.m = sd.m;
  rq.hq = hq;
  rq.khat = (const T *)sd.khat + (int64_t)hkv * sd.Mcap * D;
  rq.vhat = (const T *)sd.vhat + (int64_t)hkv * sd.Mcap * D;
  rq.ring_k = (const T *)sd.winK + (int64_t)hkv * dv.L * D;
  rq.ring_v = (const T *)sd.winV + (int64_t)hkv * dv.L * D;
  // the new token is read from the call's k, v (position pos); everything older from the ring
  rq.in_k = (const T *)k + ((int64_t)s * dv.Hkv + hkv) * D;
  rq.in_v = (const T *)v + ((int64_t)s * dv.Hkv + hkv) * D;
  rq.in_kt = rq.in_vt = 0;
  rq.t0 = sd.pos;
  rq.put_k = rq.put_v = nullptr;
  rq.put_g = nullptr;
  rq.gate = 1.f;
  rq.split = kShared ? blockIdx.x : 0;
  rq.n_split = kShared ? gridDim.x : 1;
  if constexpr (kShared) set_share<T, D, GQ>(rq, dv, s * gridDim.y + blockIdx.y);
  if (rq.split == 0 && hq == hkv * (dv.Hq / dv.Hkv)) {
    rq.put_k = (T *)sd.winK + (int64_t)hkv * dv.L * D;
    rq.put_v = (T *)sd.winV + (int64_t)hkv * dv.L * D;
    rq.put_g = sd.winG + (int64_t)hkv * dv.L;
    rq.gate = gate ? gate[(int64_t)s * dv.Hkv + hkv] : 1.f;
  }
  attn_row<T, D, GQ, kShared, NW>(dv, rq);
}

// Query heads a decode workgroup takes together: the KV head's whole group when it has 2 or 4
// heads, four of them when it has a multiple of four (so that the group's first head, whose
// workgroup stores the token, starts a workgroup either way).
int heads_together(const Dev &dv) {
  const int G = dv.Hq / dv.Hkv;
  return G % 4 == 0 ? 4 : (G % 2 == 0 ? 2 : 1);
}

// Workgroups that share the keys of one sequence in a decode step.  n_groups workgroups, each
// walking all the keys, leave the chip idle when there are few of them, and a workgroup's walk is
// a chain of memory round trips; the shares are at least one round of the loop.  Their results must
// fit the state's scratch (gq heads' d sums and two words each).  And they are put together by one workgroup, share by share: up to
// 32 of them.  Us per 64 steps, 64 / 32 shares: fp32, 128 channels, 2048 rows, 4 x 4 heads 1314 / 889, 8 x 8 on 2 1596 / 1119; bf16, 128,
// 4000 rows, 4 x 4 1248 / 827; bf16, 64, 6000, 8 x 8 on 2 1605 / 1097; fp32, 64, 4000, 4 x 4 1339 / 932.  But fp32, 128, 4000 rows in
// one or two pairs 744 / 776.
int shares_for(const Dev &dv, int gq, int n_groups, int keys, int round) {
  if (n_groups > kShareGroups) return 1;
  const int64_t room = dv.kbar_bytes / (gq * (dv.d * 4 + 8));
  int s = (int)(room < kSplitWorkgroups ? room : kSplitWorkgroups) / n_groups;
  const int most = (keys + round - 1) / round;
  s = s < most ? s : most;
  const int at_most = n_groups <= 2 && dv.io == 0 && dv.d == 128 ? kMaxSplit : kMaxSplit / 2;
  s = s < at_most ? s : at_most;
  return s > 1 ? s : 1;
}
// Eight waves per workgroup where a decode launch, one workgroup per (sequence, head group), has no more of them than compute
// units: a workgroup walks its keys alone on its unit, and loads and sums wait for each other.  Us per step with four /
// eight waves, 2048 rows in bf16: 256 workgroups of four heads 81 / 60, of one 58 / 45, 192 of two (845 rows) 24 / 20,
// 160 of one (500) 17 / 13; but 320 of four heads (1000) 58 / 63, of two 37 / 43, of one 33 / 35, 512 of four (2048) 116 / 120.
constexpr int kWavesFew = 8, kFewGroups = 256;
bool many_waves(int n_groups) { return n_groups <= kFewGroups; }
int round_keys(const Dev &dv) { return 16 * 64 / (dv.d / (dv.io == 0 ? 4 : 8)); }

}  // namespace

#define KVM_ROWS_DISPATCH(KERNEL, GQV, SHARED, NWV, grid, ...)                                           \
  do {                                                                                              \
    if (dv.io == 0 && dv.d == 64)                                                                   \
      hipLaunchKernelGGL((KERNEL<float, 64, GQV, SHARED, NWV>), grid, dim3(64 * NWV), 0, st, __VA_ARGS__);    \
    else if (dv.io == 0 && dv.d == 128)                                                             \
      hipLaunchKernelGGL((KERNEL<float, 128, GQV, SHARED, NWV>), grid, dim3(64 * NWV), 0, st, __VA_ARGS__);   \
    else if (dv.io == 1 && dv.d == 64)                                                              \
      hipLaunchKernelGGL((KERNEL<bf16_t, 64, GQV, SHARED, NWV>), grid, dim3(64 * NWV), 0, st, __VA_ARGS__);   \
    else if (dv.io == 1 && dv.d == 128)                                                             \
      hipLaunchKernelGGL((KERNEL<bf16_t, 128, GQV, SHARED, NWV>), grid, dim3(64 * NWV), 0, st, __VA_ARGS__);  \
    else                                                                                            \
      return hipErrorInvalidValue;                                                                  \
  } while (0)
#define KVM_ROWS_LAUNCH(KERNEL, SHARED, NWV, grid, ...)             \
  do {                                                         \
    if (gq == 4)                                               \
      KVM_ROWS_DISPATCH(KERNEL, 4, SHARED, NWV, grid, __VA_ARGS__); \
    else if (gq == 2)                                          \
      KVM_ROWS_DISPATCH(KERNEL, 2, SHARED, NWV, grid, __VA_ARGS__); \
    else                                                       \
      KVM_ROWS_DISPATCH(KERNEL, 1, SHARED, NWV, grid, __VA_ARGS__); \
  } while (0)

hipError_t launch_attn_rows(const Dev &dv, const AttnArgs &a, hipStream_t st) {
  if (a.nq_total <= 0) return hipSuccess;
  // a decode step (one query per sequence) takes a KV head's query heads together; a prefill on
  // this path has queries enough to fill the GPU head by head
  const int gq = a.put_token ? heads_together(dv) : 1;
  int nx = a.nq_total;
  if (a.put_token) {
    const int64_t win = a.s % dv.C + 1 + dv.L - dv.C;   // window keys, at most
    nx = shares_for(dv, gq, dv.Hq / gq * dv.B, a.m[0] + (int)win, round_keys(dv));
  }
  dim3 grid(nx, dv.Hq / gq, dv.B);
  if (a.put_token && nx > 1)
    KVM_ROWS_LAUNCH(attn_rows_kernel, true, 4, grid, dv, a);
  else if (a.put_token && many_waves(dv.Hq / gq * dv.B))
    KVM_ROWS_LAUNCH(attn_rows_kernel, false, kWavesFew, grid, dv, a);
  else
    KVM_ROWS_LAUNCH(attn_rows_kernel, false, 4, grid, dv, a);
  return hipGetLastError();
}

static int64_t attn_rows_score_workgroups(const Dev &dv, const AttnArgs &a) {
  return (int64_t)a.nq_total * dv.Hq * dv.B + (int64_t)(dv.C + 3) / 4 * dv.U;
}
// In that launch attention has the scoring's registers, and as many of its workgroups on a compute unit as those leave: of fp32 heads of
// 64 channels five where two rows of a lane are under way, two with one (eight by itself), of 128 seven (eight); bf16, 64: three,
// two (six), 128: four, one (six).  So up to the number of workgroups that was still faster.  Us per call, apart / one launch (workgroups):
//   fp32, 64:   4 x 4 heads, 256-token blocks, 1000 rows (5120) 2791 / 2629, 2 x 8 heads on 2, 512, 1000 (8704) 2778 / 2727; but 8 x 4, 256,
//               1000 (10240) 4827 / 5040, 16 x 4, 128, 300 (10240) 2054 / 2173.  Up to 64 rows: 4 x 4, 64 (1280) 297 / 289, but 8 x 4
//               (2560) 413 / 449, 8 x 16 on 4 (8704) 744 / 1137
//   fp32, 128:  16 x 4, 512, 64 (40960) 21036 / 20793, 8 x 16 on 4, 512, 300 (69632) 30998 / 30963
//   bf16, 64:   1 x 4, 480, 900 (2400) 870 / 860, but 8 x 4, 96, 128 (3840) 404 / 438, 8 x 16 on 4, 200, 128 (27200) 2515 / 2902.  Up to 64
//               rows: 4 x 4, 48 (960) 188 / 181, but 8 x 4 (1920) 228 / 259
//   bf16, 128:  8 x 4, 480, 128 (19200) 7254 / 7080, 8 x 16 on 4, 48, 128 (6528) 662 / 660, but 8 x 16 on 4, 96, 40 (13056) 1283 / 1353.
//               Up to 64 rows: 1 x 4, 48 (240) 206 / 148, but 2 x 8 on 2 (792) 223 / 245, 8 x 16 on 4 (6528) 553 / 1138
bool attn_rows_take_scores(const Dev &dv, const AttnArgs &a, int m) {
  const bool two = m > 64;
  int64_t most = kMostWorkgroups;
  if (dv.d == 64) most = dv.io == 0 ? (two ? 9216 : 1280) : (two ? 2560 : 1024);
  else if (dv.io != 0 && !two) most = 256;
  else if (dv.io != 0 && dv.Hq > dv.Hkv) most = 6656;
  return attn_rows_score_workgroups(dv, a) <= most;
}
hipError_t launch_attn_rows_score(const Dev &dv, const AttnArgs &a, int slot, int m, hipStream_t st) {
  const dim3 grid((unsigned)attn_rows_score_workgroups(dv, a));
  // (a state of up to 64 rows has one for each lane: 223 us for the first of the calls above with a second one asked for, 211 now)
#define KVM_ROWS_SCORE(T, D)                                                                                 \
  do {                                                                                                       \
    if (m > 64)                                                                                              \
      hipLaunchKernelGGL((attn_rows_score_kernel<T, D, true>), grid, dim3(256), 0, st, dv, a, slot, m);      \
    else                                                                                                     \
      hipLaunchKernelGGL((attn_rows_score_kernel<T, D, false>), grid, dim3(256), 0, st, dv, a, slot, m);     \
  } while (0)
  if (dv.io == 0 && dv.d == 64) KVM_ROWS_SCORE(float, 64);
  else if (dv.io == 0) KVM_ROWS_SCORE(float, 128);
  else if (dv.d == 64) KVM_ROWS_SCORE(bf16_t, 64);
  else KVM_ROWS_SCORE(bf16_t, 128);
#undef KVM_ROWS_SCORE
  return hipGetLastError();
}

hipError_t launch_decode_multi(const Dev &dv, const SeqDesc *seq, const SeqPack &pack, int n_seq, int most_keys, const void *q,
                               const void *k, const void *v, const float *gate, void *out, hipStream_t st) {
  if (n_seq <= 0) return hipSuccess;
  const int gq = heads_together(dv);
  dim3 agrid(shares_for(dv, gq, dv.Hq / gq * n_seq, most_keys, round_keys(dv)), dv.Hq / gq, n_seq);
  if (agrid.x > 1)
    KVM_ROWS_LAUNCH(attn_rows_multi_kernel, true, 4, agrid, dv, seq, pack, q, k, v, gate, out);
  else if (many_waves(dv.Hq / gq * n_seq))
    KVM_ROWS_LAUNCH(attn_rows_multi_kernel, false, kWavesFew, agrid, dv, seq, pack, q, k, v, gate, out);
  else
    KVM_ROWS_LAUNCH(attn_rows_multi_kernel, false, 4, agrid, dv, seq, pack, q, k, v, gate, out);
  return hipGetLastError();
}

}  // namespace kvm
