// Attention weight preparation in front of the KVM layer (the paper's appendix "GPTAlpha-2
// Attention weight preparation"; merge gate: Method, "KVM weight preparation"), memory bound:
//   v~ <- (1 - lambda) v~ + lambda v~first          value residual
//   a  =  a~_t + alpha * (a~_{t-1} - a~_t)          token shift of q, k, v (first token unshifted)
//   q, k <- RoPE_r(LN(q)), RoPE_r(LN(k))            LayerNorm with bias per head, rotary on r channels
//   g  =  1 + ELU(x W_g)                            merge gate, one scalar per KV head
// One row (token, head) is handled by d_h / kN adjacent lanes, 16 bytes of channels each, so a
// wave takes several adjacent heads, and walks a run of consecutive tokens of them; statistics
// and the rotation partner come through lane exchanges.
// Arithmetic is fp32; the rotation angles are evaluated in fp64 once per position (a table),
// because position * frequency loses its low bits in fp32 at 32k tokens.
// The rows of q, k and v are the sections of one launch.  What that launch needs beforehand -- the
// table, and the gate's weights as two bf16 halves -- is made by one launch ahead of it; a call of
// a few tokens (generation) makes its own table in LDS, has its gate on the vector units and is a
// single launch.
#include "../../include/kvm.h"
#include "kvm_device.h"
#include "kvm_mfma.h"

namespace kvm {
namespace {

constexpr int64_t kGateFewMost = 64, kGateFewMostVector = 512, kGateShortMost = 16384;  // tokens
constexpr int kGateHeads = 32;  // matrix-core gate: heads of the operand (zero rows beyond H_kv)

// (cos, sin) of channel c < half at position pos
__device__ __forceinline__ float2 rotation(int64_t pos, int c, int half, double base) {
  const double ang = (double)pos * pow(base, -(double)c / (double)half);  // base^(-2c/r)
  return make_float2((float)cos(ang), (float)sin(ang));
}

// Ahead of the rows: workgroups [0, table_wgs) make the rotation table, the others split W_g (fp32)
// into hi = bf16(w) and lo = bf16(w - hi), transposed to [kGateHeads][d_model].
__global__ __launch_bounds__(256) void prep_setup_kernel(float2 *tab, int64_t n_pos, int64_t pos0, int half, double base,
                                                         unsigned table_wgs, const float *w, uint16_t *hi, uint16_t *lo,
                                                         int dm, int Hkv) {
  if (blockIdx.x < table_wgs) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_pos * half) tab[i] = rotation(pos0 + i / half, (int)(i % half), half, base);
    return;
  }
  const int i = (blockIdx.x - table_wgs) * 256 + threadIdx.x;  // over kGateHeads * dm
  if (i >= kGateHeads * dm) return;
  const int h = i / dm, c = i - h * dm;
  const float x = h < Hkv ? w[(int64_t)c * Hkv + h] : 0.f;
  const uint16_t a = float_to_bf16_bits(x);
  hi[i] = a;
  lo[i] = float_to_bf16_bits(x - bf16_bits_to_float(a));
}

struct RowArgs {
  const void *in;       // [B, T, H, d] simple q, k or v
  const void *first;    // [B, T, H, d] first-layer value, or null (value residual)
  const void *prev;     // [B, H, d] row of the token before this call, or null
  void *out;            // [B, T, H, d]
  const float *alpha;   // [H, d] or null
  const float *lambda;  // [H, d] or null
  const float *gamma, *beta;  // [H, d] or null
  int64_t T;
  int H, r;
  float eps;
  uint32_t n_hg, n_runs, n_waves;  // head groups, token runs, waves = batch * runs * head groups
};

// kN fp32 parameters starting at p (16-byte aligned), or the neutral value when p is null.
template <int kN>
__device__ __forceinline__ void load_params(const float *p, float neutral, float (&f)[kN]) {
  if (p) {
#pragma unroll
    for (int i = 0; i < kN; i += 4) {
      const float4 x = *reinterpret_cast<const float4 *>(p + i);
      f[i] = x.x; f[i + 1] = x.y; f[i + 2] = x.z; f[i + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kN; ++i) f[i] = neutral;
  }
}

// kNorm: LayerNorm + rotation (q, k); kResidual: value residual (v).
// A wave takes 64 / (D / kN) adjacent heads (one per lane group: together a contiguous piece of a
// token) and walks run_len consecutive tokens of them, so that the token shift's "previous token" is
// the row the lane group has just had in registers instead of a second read of it (one extra row
// per run), and the per-head parameters are fetched once per run.  Tokens go in blocks of kAhead
// whose loads are all requested before the first of them is worked on.  The run's length is 16
// where that leaves waves enough to fill the chip, and 8 or 4 in shorter calls.
// wg4: number of the workgroup within the tensor's section; tab: row 0 is the call's first token.
constexpr int kRunMost = 16, kAhead = 4;
template <typename T, int D, bool kNorm, bool kResidual>
__device__ __forceinline__ void prep_rows(const RowArgs &a, uint32_t wg4, uint32_t run_len, const float2 *tab) {
  constexpr int VEC = Vec16<T>::kN;
  constexpr int LPT = D / VEC;   // lanes per row
  constexpr int RPW = 64 / LPT;  // heads per wave
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane / LPT, cl = lane % LPT;
  const uint32_t n_hg = a.n_hg, n_runs = a.n_runs;
  const uint32_t wg = wg4 * 4u + wave;  // adjacent waves: adjacent head groups of one token run
  if (wg >= a.n_waves) return;
  const uint32_t hg = wg % n_hg, br = wg / n_hg, run = br % n_runs, b = br / n_runs;
  const uint32_t H = (uint32_t)a.H, T_ = (uint32_t)a.T;
  const uint32_t h_raw = hg * RPW + sub;
  const bool live = h_raw < H;
  const uint32_t h = live ? h_raw : H - 1;  // idle lane groups repeat the last head, store nothing
  const int c0 = cl * VEC;
  const int pc = (int)h * D + c0;  // offset into the per-head parameter arrays
  const uint32_t t_begin = run * run_len, t_end = t_begin + run_len < T_ ? t_begin + run_len : T_;
  const int64_t row_stride = (int64_t)H * D;  // elements between tokens
  const int64_t off0 = (((int64_t)b * T_ + t_begin) * H + h) * D + c0;
  const bool resid = kResidual && a.first && a.lambda;

  float al[VEC], lm[VEC], ga[VEC], be[VEC];
  load_params<VEC>(a.alpha ? a.alpha + pc : nullptr, 0.f, al);
  load_params<VEC>(resid ? a.lambda + pc : nullptr, 0.f, lm);
  if (kNorm) {
    load_params<VEC>(a.gamma ? a.gamma + pc : nullptr, 1.f, ga);
    load_params<VEC>(a.beta ? a.beta + pc : nullptr, 0.f, be);
  }
  // the row before the run (already residual-mixed when it comes from the previous call)
  float prev[VEC];
  bool have_prev = false;
  if (a.alpha) {
    if (t_begin > 0) {
      Vec16<T>::load((const T *)a.in + off0 - row_stride, prev);
      if (resid) {
        float f[VEC];
        Vec16<T>::load((const T *)a.first + off0 - row_stride, f);
#pragma unroll
        for (int i = 0; i < VEC; ++i) prev[i] = (1.f - lm[i]) * prev[i] + lm[i] * f[i];
      }
      have_prev = true;
    } else if (a.prev) {
      Vec16<T>::load((const T *)a.prev + (int64_t)(b * H + h) * D + c0, prev);
      have_prev = true;
    }
  }
  for (uint32_t t0 = t_begin; t0 < t_end; t0 += kAhead) {
    float y[kAhead][VEC], f[kAhead][VEC];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const uint32_t t = t0 + k < t_end ? t0 + k : t_end - 1;
      const int64_t off = off0 + (int64_t)(t - t_begin) * row_stride;
      Vec16<T>::load((const T *)a.in + off, y[k]);
      if (resid) Vec16<T>::load((const T *)a.first + off, f[k]);
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const uint32_t t = t0 + k;
      if (t >= t_end) break;
      if (resid) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) y[k][i] = (1.f - lm[i]) * y[k][i] + lm[i] * f[k][i];
      }
      float z[VEC];  // the row after the shift; y[k] stays the next token's "previous"
#pragma unroll
      for (int i = 0; i < VEC; ++i) z[i] = have_prev ? y[k][i] + al[i] * (prev[i] - y[k][i]) : y[k][i];
      if (a.alpha) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) prev[i] = y[k][i];
        have_prev = true;
      }
      if (kNorm) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) s += z[i];
        const float mean = group_sum<LPT>(s) * (1.f / (float)D);
        float q = 0.f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          z[i] -= mean;
          q += z[i] * z[i];
        }
        const float rstd = rsqrtf(group_sum<LPT>(q) * (1.f / (float)D) + a.eps);
#pragma unroll
        for (int i = 0; i < VEC; ++i) z[i] = z[i] * rstd * ga[i] + be[i];
        if (a.r > 0) {
          // channel c < r/2 pairs with c + r/2, which sits r/2/VEC lanes away (a power of two)
          const int half = a.r / 2, hop = half / VEC;
          float o[VEC];
#pragma unroll
          for (int i = 0; i < VEC; ++i) o[i] = __shfl_xor(z[i], hop, kWave);
          if (c0 < a.r) {
            const bool lower = c0 < half;
            float cs[2 * VEC];  // (cos, sin) of this lane's channels
            load_params<2 * VEC>((const float *)(tab + (int64_t)t * half + (lower ? c0 : c0 - half)), 0.f, cs);
#pragma unroll
            for (int i = 0; i < VEC; ++i)
              z[i] = lower ? z[i] * cs[2 * i] - o[i] * cs[2 * i + 1] : z[i] * cs[2 * i] + o[i] * cs[2 * i + 1];
          }
        }
      }
      if (live) Vec16<T>::store((T *)a.out + off0 + (int64_t)(t - t_begin) * row_stride, z);
    }
  }
}

__device__ __forceinline__ float gate_of(float z) { return 1.f + (z > 0.f ? z : expm1f(z)); }

// Merge gate: a wave takes kGateTok tokens; lanes stride over the model width, 16 bytes of x each,
// heads in blocks of eight; the per-lane partial dot products are summed across the wave at the
// end.  kFull: the number of KV heads is a multiple of 8, so a row of eight gate weights is two
// aligned 16-byte loads.
constexpr int kGateTok = 8;
template <typename T, bool kFull>
__global__ __launch_bounds__(256) void gate_kernel(const T *x, const float *w, float *gate, int64_t n_tok,
                                                   int dm, int Hkv) {
  constexpr int VEC = Vec16<T>::kN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t tok0 = ((int64_t)blockIdx.x * 4 + wave) * kGateTok;
  if (tok0 >= n_tok) return;
  const T *xr[kGateTok];
#pragma unroll
  for (int k = 0; k < kGateTok; ++k) xr[k] = x + (tok0 + k < n_tok ? tok0 + k : n_tok - 1) * dm;
  for (int h0 = 0; h0 < Hkv; h0 += 8) {
    float acc[kGateTok][8];
#pragma unroll
    for (int k = 0; k < kGateTok; ++k)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[k][j] = 0.f;
    for (int c0 = lane * VEC; c0 < dm; c0 += 64 * VEC) {
      float xv[kGateTok][VEC];
#pragma unroll
      for (int k = 0; k < kGateTok; ++k) Vec16<T>::load(xr[k] + c0, xv[k]);
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        float wv[8];
        const float *wrow = w + (int64_t)(c0 + i) * Hkv + h0;
        if (kFull) {
          load_params<8>(wrow, 0.f, wv);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) wv[j] = h0 + j < Hkv ? wrow[j] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int k = 0; k < kGateTok; ++k) acc[k][j] = fmaf(xv[k][i], wv[j], acc[k][j]);
      }
    }
#pragma unroll
    for (int k = 0; k < kGateTok; ++k)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float z = wave_sum(acc[k][j]);
        if (lane == 0 && tok0 + k < n_tok && h0 + j < Hkv)
          gate[(tok0 + k) * Hkv + h0 + j] = gate_of(z);
      }
  }
}

// The merge gate on the matrix cores (bf16 x, at most 32 KV heads, d_model a multiple of 128).
// With W_g split into two bf16 halves, x W_g = x hi + x lo with the products exact and the sums in
// fp32: the same 1e-6-relative arithmetic as the vector version.
// A workgroup takes 128 tokens, a wave 32 of them and all heads.  x comes through LDS in tiles of 128
// channels, two stages, filled by direct loads of 256-byte row pieces; W's halves go from the caches
// straight into the B operand (lane = head).  Bound by the bytes of x: read from global memory into
// the A operand directly, a load instruction touches 32 rows 32 bytes each, and 65536 tokens x 2048
// took 102 us (2.6 TB/s) with 64 or 32 tokens per wave, one step of loads ahead or none; so staged, 82 us
// (3.3 TB/s).
__global__ __launch_bounds__(256) void gate_mfma_kernel(const uint16_t *x, const uint16_t *hi, const uint16_t *lo,
                                                        float *gate, int64_t n_tok, int dm, int Hkv) {
  __shared__ __attribute__((aligned(1024))) uint16_t Xs[2][2][kTileElems];   // [stage][token half]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const int64_t wg0 = (int64_t)blockIdx.x * 128, tok0 = wg0 + 32 * wave;
  const int valid = n_tok - wg0 < 128 ? (int)(n_tok - wg0) : 128;
  const char *xb = (const char *)(x + wg0 * dm);
  const uint32_t stride = (uint32_t)dm * 2, xs_addr = lds_addr_of(&Xs[0][0][0]);
  const DmaLane dl = dma_lane(lane);
  uint32_t koff[8];
  ktile_offsets(lane, koff);
  auto issue = [&](int c0, int stage) {
    // (rows past the end repeat the last one; a second half without tokens is not loaded, nothing of it is stored)
    const uint32_t at = xs_addr + (uint32_t)stage * (2 * kTileElems * 2);
    const char *from = xb + (size_t)c0 * 2;
    tile_dma<false, 4>(from, stride, valid, at, wave, dl);
    if (valid > kTileKeys)
      tile_dma<false, 4>(from + (size_t)kTileKeys * stride, stride, valid - kTileKeys, at + kTileElems * 2, wave, dl);
  };
  const bool head_lane = l32 < ((Hkv + 7) & ~7);  // lanes of the zero rows need not load them
  const uint16_t *hr = hi + (int64_t)l32 * dm + 8 * g, *lr = lo + (int64_t)l32 * dm + 8 * g;
  f32x16 acc = {0.f};
  struct Weights {
    Frag8 h[8], l[8];
  };
  auto fetch = [&](Weights &w, int c0) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      w.h[ks].q = w.l[ks].q = make_uint4(0u, 0u, 0u, 0u);
      if (head_lane) {
        w.h[ks].q = *reinterpret_cast<const uint4 *>(hr + c0 + 16 * ks);
        w.l[ks].q = *reinterpret_cast<const uint4 *>(lr + c0 + 16 * ks);
      }
    }
  };
  // one step: everything asked for a step ago has landed; the next step's weights are asked for
  // ahead of its x (loads return in order: behind them, they would be waited for as long as x is)
  auto step = [&](int c0, int stage, const Weights &now, Weights &next) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (c0 + 128 < dm) {
      fetch(next, c0 + 128);
      issue(c0 + 128, stage ^ 1);
    }
    const uint16_t *Xt = &Xs[stage][wave >> 1][0];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const bf16x8 xf = ktile_frag(Xt, koff, wave & 1, ks);
      acc = mfma32(xf, now.h[ks].v, acc);
      acc = mfma32(xf, now.l[ks].v, acc);
    }
  };
  Weights w0, w1;
  fetch(w0, 0);
  issue(0, 0);
  for (int c0 = 0; c0 < dm; c0 += 256) {
    step(c0, 0, w0, w1);
    if (c0 + 128 < dm) step(c0 + 128, 1, w1, w0);
  }
  if (l32 < Hkv) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t t = tok0 + mfma_row(v, g);
      if (t < n_tok) gate[t * Hkv + l32] = gate_of(acc[v]);
    }
  }
}

// The gate of short calls, as a section of the rows' launch, 16 tokens per workgroup: the four waves
// take a quarter of the channels each (a wave that walks all of them is a chain of d_model / 64 memory
// round trips, and a short call has no other waves to hide it behind) and their sums meet in LDS.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
constexpr int kGateShortTok = 16;
struct GateArgs {
  const void *x;
  const float *w;
  const uint16_t *hi, *lo;
  float *gate;
  int64_t n_tok;
  int dm, Hkv;
};
__device__ __forceinline__ void gate_short(const GateArgs &a, uint32_t wg, float *sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int64_t tok0 = (int64_t)wg * kGateShortTok;
  const int64_t t_lane = tok0 + l16;
  const int c_first = wave * (a.dm / 4);
  const uint16_t *xr = (const uint16_t *)a.x + (t_lane < a.n_tok ? t_lane : a.n_tok - 1) * a.dm + c_first + 8 * g;
  const uint16_t *hr = a.hi + (int64_t)l16 * a.dm + c_first + 8 * g, *lr = a.lo + (int64_t)l16 * a.dm + c_first + 8 * g;
  const bool two = a.Hkv > 16;   // a second column tile of heads
  const int64_t tile = (int64_t)16 * a.dm;
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 8
  for (int c = 0; c < a.dm / 4; c += 32) {
    Frag8 xf, hf, lf;
    xf.q = *reinterpret_cast<const uint4 *>(xr + c);
    hf.q = *reinterpret_cast<const uint4 *>(hr + c);
    lf.q = *reinterpret_cast<const uint4 *>(lr + c);
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf.v, hf.v, acc[0], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf.v, lf.v, acc[0], 0, 0, 0);
    if (two) {
      hf.q = *reinterpret_cast<const uint4 *>(hr + tile + c);
      lf.q = *reinterpret_cast<const uint4 *>(lr + tile + c);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf.v, hf.v, acc[1], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf.v, lf.v, acc[1], 0, 0, 0);
    }
  }
  // D of the 16x16 instruction: column (head) = lane % 16, row (token) = 4 * (lane / 16) + element
#pragma unroll
  for (int ht = 0; ht < 2; ++ht)
#pragma unroll
    for (int v = 0; v < 4; ++v) sh[((wave * 2 + ht) * 16 + 4 * g + v) * 16 + l16] = acc[ht][v];
  __syncthreads();
  for (int i = threadIdx.x; i < kGateShortTok * kGateHeads; i += 256) {
    const int tok = i / kGateHeads, h = i % kGateHeads, at = ((h >> 4) * 16 + tok) * 16 + (h & 15);
    const float z = (sh[at] + sh[at + 512]) + (sh[at + 1024] + sh[at + 1536]);
    if (h < a.Hkv && tok0 + tok < a.n_tok) a.gate[(tok0 + tok) * a.Hkv + h] = gate_of(z);
  }
}

// The gate of a few tokens on the vector units, a workgroup per token: threads stride over the
// channels, eight heads at a time, fp32 weights as they are.
template <typename T>
__device__ __forceinline__ void gate_few(const GateArgs &a, uint32_t tok, float *sh) {
  constexpr int VEC = Vec16<T>::kN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const T *xr = (const T *)a.x + (int64_t)tok * a.dm;
  const bool full = a.Hkv % 8 == 0;
  for (int h0 = 0; h0 < a.Hkv; h0 += 8) {
    float acc[8] = {};
    for (int c0 = threadIdx.x * VEC; c0 < a.dm; c0 += 256 * VEC) {
      float xv[VEC], wv[VEC][8];
      Vec16<T>::load(xr + c0, xv);
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        const float *wrow = a.w + (int64_t)(c0 + i) * a.Hkv + h0;
        if (full) {
          load_params<8>(wrow, 0.f, wv[i]);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) wv[i][j] = h0 + j < a.Hkv ? wrow[j] : 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < VEC; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = fmaf(xv[i], wv[i][j], acc[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float z = wave_sum(acc[j]);
      if (lane == 0) sh[wave * 8 + j] = z;
    }
    __syncthreads();
    if (threadIdx.x < 8 && h0 + (int)threadIdx.x < a.Hkv)
      a.gate[(int64_t)tok * a.Hkv + h0 + threadIdx.x] =
          gate_of((sh[threadIdx.x] + sh[8 + threadIdx.x]) + (sh[16 + threadIdx.x] + sh[24 + threadIdx.x]));
    __syncthreads();
  }
}

// The rows of q, k and v, and with kGate the gate, as sections of one grid: the gate's workgroups
// first (the longest), then q's, k's, v's.
enum { kGateElsewhere = 0, kGateFew = 1, kGateShort = 2 };
constexpr int kTableMost = 256;   // table entries a workgroup makes for itself, one per thread
struct PrepArgs {
  RowArgs q, k, v;
  GateArgs gate;
  const float2 *tab;      // [T, r/2] (cos, sin), or null: every workgroup makes its own
  int64_t pos0;
  double base;
  uint32_t wg_gate, wg_q, wg_k;   // workgroups of the first three sections
  uint32_t run;                   // tokens a wave walks
};
template <typename T, int D, int kGate>
__global__ __launch_bounds__(256) void prep_rows_kernel(PrepArgs p) {
  __shared__ float2 own_tab[kTableMost];
  uint32_t wg = blockIdx.x;
  if constexpr (kGate != kGateElsewhere) {
    if (wg < p.wg_gate) {
      __shared__ float sh[kGate == kGateShort ? 4 * 2 * 16 * 16 : 32];
      if constexpr (kGate == kGateShort)
        gate_short(p.gate, wg, sh);
      else
        gate_few<T>(p.gate, wg, sh);
      return;
    }
    wg -= p.wg_gate;
  }
  const float2 *tab = p.tab;
  if (!tab && p.q.r > 0 && wg < p.wg_q + p.wg_k) {
    const int half = p.q.r / 2;
    if ((int64_t)threadIdx.x < p.q.T * half)
      own_tab[threadIdx.x] = rotation(p.pos0 + threadIdx.x / half, threadIdx.x % half, half, p.base);
    __syncthreads();
    tab = own_tab;
  }
  if (wg < p.wg_q)
    prep_rows<T, D, true, false>(p.q, wg, p.run, tab);
  else if (wg < p.wg_q + p.wg_k)
    prep_rows<T, D, true, false>(p.k, wg - p.wg_q, p.run, tab);
  else
    prep_rows<T, D, false, true>(p.v, wg - p.wg_q - p.wg_k, p.run, tab);
}

template <typename T, int D>
hipError_t launch_prep(const PrepArgs &p, int gate, unsigned wgs, hipStream_t st) {
  if (gate == kGateShort)
    hipLaunchKernelGGL((prep_rows_kernel<T, D, kGateShort>), dim3(wgs), dim3(256), 0, st, p);
  else if (gate == kGateFew)
    hipLaunchKernelGGL((prep_rows_kernel<T, D, kGateFew>), dim3(wgs), dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL((prep_rows_kernel<T, D, kGateElsewhere>), dim3(wgs), dim3(256), 0, st, p);
  return hipGetLastError();
}

bool al16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// Scratch layout: the rotation table, then (when the matrix-core gate applies) W_g's two bf16 halves.
bool gate_on_mfma(const kvm_prep_params *p) {
  return p->io_dtype == KVM_BF16 && p->d_model > 0 && p->d_model % 128 == 0 && p->n_kv_heads <= kGateHeads;
}
size_t rope_table_bytes(const kvm_prep_params *p, int64_t T) {
  const size_t n = (size_t)T * (size_t)(p->rope_dims / 2) * sizeof(float2);
  return ((n ? n : 16) + 255) & ~(size_t)255;
}
size_t gate_split_bytes(const kvm_prep_params *p) {
  return gate_on_mfma(p) ? 2 * (size_t)kGateHeads * (size_t)p->d_model * 2 : 0;
}

bool valid(const kvm_prep_params *p) {
  if (!p || p->batch <= 0 || p->n_q_heads <= 0 || p->n_kv_heads <= 0) return false;
  if (p->head_dim != 64 && p->head_dim != 128) return false;
  if (p->io_dtype != KVM_F32 && p->io_dtype != KVM_BF16) return false;
  const int vec = p->io_dtype == KVM_F32 ? 4 : 8;
  const int r = p->rope_dims;
  if (r < 0 || r > p->head_dim) return false;
  if (r > 0) {
    const int half = r / 2;
    if (r % 2 || half % vec) return false;
    const int hop = half / vec;
    if (hop & (hop - 1)) return false;  // the rotation partner must be a power-of-two lane hop away
  }
  if (p->d_model < 0 || p->d_model % vec) return false;
  return true;
}

}  // namespace
}  // namespace kvm

extern "C" size_t kvm_prepare_scratch_bytes(const kvm_prep_params *p, int64_t T) {
  if (!kvm::valid(p) || T <= 0) return 0;
  return kvm::rope_table_bytes(p, T) + kvm::gate_split_bytes(p);
}

extern "C" int kvm_prepare_qkv(const kvm_prep_params *p, const void *q_raw, const void *k_raw,
                               const void *v_raw, const void *v_first, const void *x, const void *prev_q,
                               const void *prev_k, const void *prev_v, void *q_out, void *k_out,
                               void *v_out, float *gate_out, void *scratch, int64_t T, int64_t pos0,
                               void *stream_) {
  using namespace kvm;
  if (!valid(p) || T <= 0 || pos0 < 0) return KVM_ERR_ARG;
  if (!q_raw || !k_raw || !v_raw || !q_out || !k_out || !v_out || !scratch) return KVM_ERR_ARG;
  if (q_raw == q_out || k_raw == k_out || v_raw == v_out) return KVM_ERR_ARG;  // the shift reads token t - 1
  const void *ptrs[] = {q_raw, k_raw, v_raw, v_first, x, prev_q, prev_k, prev_v, q_out, k_out, v_out, scratch};
  for (const void *q : ptrs)
    if (!al16(q)) return KVM_ERR_ARG;
  const void *prm[] = {p->alpha_q, p->alpha_k, p->alpha_v, p->lambda_v, p->lnq_gamma, p->lnq_beta,
                       p->lnk_gamma, p->lnk_beta, p->w_gate};
  for (const void *q : prm)
    if (!al16(q)) return KVM_ERR_ARG;
  const bool gate = x != nullptr;
  if (gate && (!p->w_gate || !gate_out || p->d_model <= 0)) return KVM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream_;
  const int d = p->head_dim, r = p->rope_dims, half = r / 2;
  const float eps = p->ln_eps > 0.f ? p->ln_eps : 1e-5f;
  float2 *tab = (float2 *)scratch;
  const double base = p->rope_base > 0.0 ? p->rope_base : 10000.0;
  const int64_t n_tok = (int64_t)p->batch * T;
  if (n_tok * p->n_q_heads >= (1ll << 31) || n_tok * p->n_kv_heads >= (1ll << 31)) return KVM_ERR_ARG;  // 32-bit row numbers
  const int dm = p->d_model, hk = p->n_kv_heads;

  // How the gate is computed: a few tokens on the vector units, up to kGateShortMost on the matrix
  // cores with the channels divided among the waves, both inside the rows' launch; beyond that by
  // a launch of its own whose waves take all channels of their tokens.
  const bool mfma = gate_on_mfma(p);
  int how = kGateElsewhere;
  if (gate && n_tok <= (mfma ? kGateFewMost : kGateFewMostVector)) how = kGateFew;
  else if (gate && mfma && n_tok < kGateShortMost) how = kGateShort;
  uint16_t *hi = (uint16_t *)((char *)scratch + rope_table_bytes(p, T)), *lo = hi + (size_t)kGateHeads * dm;
  const bool own_table = half > 0 && T * half <= kTableMost;   // every workgroup makes its own
  const unsigned table_wgs = half > 0 && !own_table ? (unsigned)((T * half + 255) / 256) : 0u;
  const unsigned split_wgs = gate && mfma && how != kGateFew ? (unsigned)((kGateHeads * dm + 255) / 256) : 0u;
  if (table_wgs + split_wgs > 0) {
    hipLaunchKernelGGL(prep_setup_kernel, dim3(table_wgs + split_wgs), dim3(256), 0, st, tab, T, pos0, half, base, table_wgs,
                       p->w_gate, hi, lo, dm, hk);
    if (hipGetLastError() != hipSuccess) return KVM_ERR_HIP;
  }

  PrepArgs a;
  const int heads_per_wave = 64 / (d * (p->io_dtype == KVM_F32 ? 4 : 2) / 16);
  // tokens per wave: long runs re-read the fewest rows for the shift, short ones make waves enough
  const int64_t waves16 = n_tok / kRunMost * ((p->n_q_heads + 2 * hk + heads_per_wave - 1) / heads_per_wave);
  a.run = waves16 >= 4096 ? kRunMost : waves16 >= 2048 ? kRunMost / 2 : kAhead;
  auto section = [&](RowArgs &r_, const void *in, const void *first, const void *prev, void *out, const float *alpha,
                     const float *lambda, const float *gamma, const float *beta, int H) -> uint32_t {
    r_.in = in; r_.first = first; r_.prev = prev; r_.out = out;
    r_.alpha = alpha; r_.lambda = lambda; r_.gamma = gamma; r_.beta = beta;
    r_.T = T; r_.H = H; r_.r = r; r_.eps = eps;
    r_.n_hg = (uint32_t)((H + heads_per_wave - 1) / heads_per_wave);
    r_.n_runs = (uint32_t)((T + a.run - 1) / a.run);
    r_.n_waves = (uint32_t)p->batch * r_.n_runs * r_.n_hg;
    return (r_.n_waves + 3) / 4;
  };
  a.wg_q = section(a.q, q_raw, nullptr, prev_q, q_out, p->alpha_q, nullptr, p->lnq_gamma, p->lnq_beta, p->n_q_heads);
  a.wg_k = section(a.k, k_raw, nullptr, prev_k, k_out, p->alpha_k, nullptr, p->lnk_gamma, p->lnk_beta, hk);
  const uint32_t wg_v = section(a.v, v_raw, v_first, prev_v, v_out, p->alpha_v, p->lambda_v, nullptr, nullptr, hk);
  a.wg_gate = how == kGateFew ? (uint32_t)n_tok
              : how == kGateShort ? (uint32_t)((n_tok + kGateShortTok - 1) / kGateShortTok) : 0u;
  a.gate = GateArgs{x, p->w_gate, hi, lo, gate_out, n_tok, dm, hk};
  a.tab = own_table ? nullptr : tab;
  a.pos0 = pos0;
  a.base = base;
  const unsigned wgs = a.wg_gate + a.wg_q + a.wg_k + wg_v;
  hipError_t e;
  if (p->io_dtype == KVM_F32)
    e = d == 64 ? launch_prep<float, 64>(a, how, wgs, st) : launch_prep<float, 128>(a, how, wgs, st);
  else
    e = d == 64 ? launch_prep<bf16_t, 64>(a, how, wgs, st) : launch_prep<bf16_t, 128>(a, how, wgs, st);
  if (e != hipSuccess) return KVM_ERR_HIP;

  if (gate && how == kGateElsewhere) {
    dim3 grid((unsigned)((n_tok + 4 * kGateTok - 1) / (4 * kGateTok)));
    const bool full = hk % 8 == 0;
    const float *wg = p->w_gate;
    if (mfma) {
      hipLaunchKernelGGL(gate_mfma_kernel, dim3((unsigned)((n_tok + 127) / 128)), dim3(256), 0, st,
                         (const uint16_t *)x, hi, lo, gate_out, n_tok, dm, hk);
    } else if (p->io_dtype == KVM_F32) {
      if (full)
        hipLaunchKernelGGL((gate_kernel<float, true>), grid, dim3(256), 0, st, (const float *)x, wg, gate_out, n_tok, dm, hk);
      else
        hipLaunchKernelGGL((gate_kernel<float, false>), grid, dim3(256), 0, st, (const float *)x, wg, gate_out, n_tok, dm, hk);
    } else {
      if (full)
        hipLaunchKernelGGL((gate_kernel<bf16_t, true>), grid, dim3(256), 0, st, (const bf16_t *)x, wg, gate_out, n_tok, dm, hk);
      else
        hipLaunchKernelGGL((gate_kernel<bf16_t, false>), grid, dim3(256), 0, st, (const bf16_t *)x, wg, gate_out, n_tok, dm, hk);
    }
    if (hipGetLastError() != hipSuccess) return KVM_ERR_HIP;
  }
  return KVM_OK;
}
