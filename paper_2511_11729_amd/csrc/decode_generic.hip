// fp32-storage decode step (Harli Sec. 2.1 decode, Sec. 4.1 index-based KV): the same steps as the bf16 path with every
// tensor -- weights, KV cache, activations -- held and computed in fp32.  This path serves small models and exact checks; it
// is written for any shape (no tile-size restrictions) with plain one-wave-per-output-row kernels and makes no use of the
// pre-shuffled weight copies.  A layer is five launches -- RMSNorm rides on the products that read it (the squares are summed
// beside them), rotation and append on q, k, v, SwiGLU on gate and up -- because at these sizes a launch is what a kernel
// costs: hidden size 256, four sequences of about 100 tokens took 106 us in fourteen launches and take 21 in five.
#include <type_traits>

#include "ctx.h"
#include "device_utils.h"

namespace harli {
namespace {

constexpr int kBT = 8;  // most batch rows a wave carries per weight row

// x[b] = emb[token[b]]
__global__ void __launch_bounds__(256) g_input(int H, const int* token_ids, const float* emb, int vocab, float* x, int* err_flag) {
  const int b = blockIdx.x;
  int t = token_ids[b];
  if (t < 0 || t >= vocab) {
    if (threadIdx.x == 0) atomicOr(err_flag, 2);
    t = 0;
  }
  const float* src = emb + (size_t)t * H;
  for (int i = threadIdx.x; i < H; i += 256) x[(size_t)b * H + i] = src[i];
}

// A product of the step: rows of the weight matrices against kBT batch rows per wave.
struct GLinear {
  const float* x;   // [B, K]
  const float* g;   // RMSNorm gain of x, or null: x enters as it is
  const float* W[3];
  const float* res; // added to y, or null
  float* y;         // [B, N]
  int B, K, N;
  float eps;
};

// What bounds these kernels is their own code: a launch finds the instruction cache cold, and the reduction of four rows written
// out as butterflies took 3 to 11 us behind 1 us of loads.  So sums are folded: a lane swap of two values and one add leaves
// either value's sum in its half of the wave, two levels four values in four rows of sixteen lanes.
__device__ __forceinline__ float g_fold32(float a, float b) {
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
__device__ __forceinline__ float g_fold16(float a, float b) {
  const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
template <int CTRL>
__device__ __forceinline__ float g_dpp(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// Sums over the wave of BT values: lane l holds that of value g_value<BT>(l, r) in out[r].
template <int BT>
constexpr int g_regs() { return BT < 4 ? 1 : BT / 4; }
template <int BT>
__device__ __forceinline__ int g_value(int lane, int r) {
  return BT == 1 ? 0 : BT == 2 ? lane >> 5 : 4 * r + ((lane >> 3) & 2) + (lane >> 5);
}
template <int BT>
__device__ __forceinline__ bool g_writes(int lane) { return lane % (BT == 1 ? 64 : BT == 2 ? 32 : 16) == 0; }
template <int BT>
__device__ __forceinline__ void g_sum(const float (&v)[BT], float (&out)[g_regs<BT>()]) {
#pragma unroll
  for (int r = 0; r < g_regs<BT>(); ++r) {
    float t;
    if constexpr (BT == 1) t = g_fold32(v[0], v[0]), t = g_fold16(t, t);
    else if constexpr (BT == 2) t = g_fold32(v[0], v[1]), t = g_fold16(t, t);
    else t = g_fold16(g_fold32(v[4 * r], v[4 * r + 1]), g_fold32(v[4 * r + 2], v[4 * r + 3]));
    t += g_dpp<0x140>(t);  // mirror of a row of sixteen
    t += g_dpp<0x141>(t);  // mirror of half a row
    t += g_dpp<0x4E>(t);   // quad permute 2 3 0 1
    t += g_dpp<0xB1>(t);   // quad permute 1 0 3 2
    out[r] = t;
  }
}

// sum_k w[k] x[b_i][k] of NW weight rows at once, with NORM of the RMSNorm of x, as g_sum leaves them.  VEC: four k per lane.
template <int BT, int NW, bool VEC, bool NORM>
__device__ __forceinline__ void g_dot(const GLinear& p, const float* const (&w)[NW], int b0, int lane, float (&out)[NW][g_regs<BT>()]) {
  constexpr int E = VEC ? 4 : 1, R = g_regs<BT>();
  float ss[BT], acc[NW][BT];
#pragma unroll
  for (int i = 0; i < BT; ++i) {
    ss[i] = 0.f;
#pragma unroll
    for (int j = 0; j < NW; ++j) acc[j][i] = 0.f;
  }
#pragma unroll 1
  for (int k = lane * E; k < p.K; k += 64 * E) {
    float wv[NW][E], gv[E], xv[BT][E];
    auto load = [&](const float* q, float (&v)[E]) {
      if constexpr (VEC) {
        const float4 t = *reinterpret_cast<const float4*>(q);
        v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
      } else {
        v[0] = *q;
      }
    };
#pragma unroll
    for (int j = 0; j < NW; ++j) load(w[j] + k, wv[j]);
#pragma unroll
    for (int i = 0; i < BT; ++i) load(p.x + (size_t)min(b0 + i, p.B - 1) * p.K + k, xv[i]);
    if (NORM) load(p.g + k, gv);
#pragma unroll
    for (int i = 0; i < BT; ++i)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        float v = xv[i][e];
        if (NORM) ss[i] += v * v, v *= gv[e];
#pragma unroll
        for (int j = 0; j < NW; ++j) acc[j][i] += wv[j][e] * v;
      }
  }
#pragma unroll
  for (int j = 0; j < NW; ++j) g_sum<BT>(acc[j], out[j]);
  if (NORM) {
    float sq[R];
    g_sum<BT>(ss, sq);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float rho = rsqrtf(sq[r] / (float)p.K + p.eps);
#pragma unroll
      for (int j = 0; j < NW; ++j) out[j][r] *= rho;
    }
  }
}

// y[b][n] = (norm(x) W^T)[b][n] (+ res[b][n]); one wave per weight row n and BT batch rows
template <int BT, bool VEC, bool NORM>
__global__ void __launch_bounds__(256) g_linear(GLinear p) {
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= p.N) return;
  const float* const w[1] = {p.W[0] + (size_t)n * p.K};
  float s[1][g_regs<BT>()];
  g_dot<BT, 1, VEC, NORM>(p, w, blockIdx.y * BT, lane, s);
#pragma unroll
  for (int r = 0; r < g_regs<BT>(); ++r) {
    const int b = blockIdx.y * BT + g_value<BT>(lane, r);
    if (g_writes<BT>(lane) && b < p.B) {
      const size_t o = (size_t)b * p.N + n;
      p.y[o] = s[0][r] + (p.res ? p.res[o] : 0.f);
    }
  }
}

// m = silu(gate) * up of one row of both matrices
template <int BT, bool VEC>
__global__ void __launch_bounds__(256) g_gate_up(GLinear p) {
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= p.N) return;
  const float* const w[2] = {p.W[0] + (size_t)n * p.K, p.W[1] + (size_t)n * p.K};
  float s[2][g_regs<BT>()];
  g_dot<BT, 2, VEC, true>(p, w, blockIdx.y * BT, lane, s);
#pragma unroll
  for (int r = 0; r < g_regs<BT>(); ++r) {
    const int b = blockIdx.y * BT + g_value<BT>(lane, r);
    if (g_writes<BT>(lane) && b < p.B) p.y[(size_t)b * p.N + n] = s[0][r] / (1.f + expf(-s[0][r])) * s[1][r];
  }
}

struct GRope {
  const float *bq, *bk, *bv;
  const int *kv_len, *page_table;
  int max_pages, layer, n_q, n_kv, d;
  const double* inv_freq;
  char* slab;
  KvGeom geom;
  int* err_flag;
};

// q, k, v: a wave computes rows i and i + d/2 of one head (a rotary pair; of v, just two rows).  q and k are rotated at position
// kv_len[b] -- angle pos * base^(-2i/d) evaluated in double -- and k and v appended to the page of that position.
template <int BT, bool VEC>
__global__ void __launch_bounds__(256) g_qkv(GLinear p, GRope r) {
  const int lane = threadIdx.x & 63, half = r.d / 2, b0 = blockIdx.y * BT;
  const int pair = blockIdx.x * 4 + (threadIdx.x >> 6);  // head by head, half a head's pairs each
  if (pair >= (r.n_q + 2 * r.n_kv) * half) return;
  int hd = pair / half;
  const int i = pair - hd * half;
  const int kind = hd < r.n_q ? 0 : hd < r.n_q + r.n_kv ? 1 : 2;
  hd -= kind == 0 ? 0 : kind == 1 ? r.n_q : r.n_q + r.n_kv;
  const float* W = p.W[kind];
  const int row = hd * r.d + i;
  const float* const w[2] = {W + (size_t)row * p.K, W + (size_t)(row + half) * p.K};
  float s[2][g_regs<BT>()];
  g_dot<BT, 2, VEC, true>(p, w, b0, lane, s);
  const float* bias = kind == 0 ? r.bq : kind == 1 ? r.bk : r.bv;
#pragma unroll 1
  for (int u = 0; u < g_regs<BT>(); ++u) {
    const int b = b0 + g_value<BT>(lane, u);
    if (!g_writes<BT>(lane) || b >= p.B) continue;
    float a = s[0][0], c = s[1][0];
    if (g_regs<BT>() > 1 && u) a = s[0][g_regs<BT>() - 1], c = s[1][g_regs<BT>() - 1];
    if (bias) a += bias[row], c += bias[row + half];  // the bias precedes the rotation
    const int pos = r.kv_len[b];
    if (kind < 2) {
      double sn, cs;
      sincos((double)pos * r.inv_freq[i], &sn, &cs);
      const float t = a;
      a = t * (float)cs - c * (float)sn;
      c = c * (float)cs + t * (float)sn;
    }
    if (kind == 0) {
      float* q = p.y + ((size_t)b * r.n_q + hd) * r.d;
      q[i] = a;
      q[i + half] = c;
      continue;
    }
    const int lp = pos / r.geom.page_tokens, slot = pos - lp * r.geom.page_tokens;
    const int page = lp < r.max_pages ? r.page_table[(size_t)b * r.max_pages + lp] : -1;
    if (page < 0 || page >= r.geom.n_pages_total) {
      if (i == 0) atomicOr(r.err_flag, 1);
      continue;
    }
    // inside a page the order is [kv head][token slot][head_dim]
    float* kp = reinterpret_cast<float*>(r.slab + kv_page_off(r.geom, page, r.layer, kind - 1)) + ((size_t)hd * r.geom.page_tokens + slot) * r.d;
    kp[i] = a;
    kp[i + half] = c;
  }
}

// attention of one (sequence, query head) over positions 0..kv_len[b], 256 tokens at a time: a thread scores one token, the
// softmax runs on across blocks of tokens (its maximum moves, the sums are rescaled), a wave adds up P.V of every fourth token
// with a lane per element.  Scores and page offsets stay in LDS; the scores of a token per wave and one thread per output
// element over all tokens took 61 us for 100 tokens, this takes 9.5.
// EL: elements per lane.  A head larger than 64 EL goes to several workgroups (blockIdx.z), which score it alike; its query is
// read from memory (EL = 16: no bound on the head size).
template <int EL>
__global__ void __launch_bounds__(256) g_attention(const float* q, const int* kv_len, const int* page_table, int max_pages,
                                                   int layer, int n_q, int n_kv, int d, const char* slab, KvGeom geom,
                                                   int max_seq_len, float* o, int* err_flag) {
  __shared__ __align__(16) float qs[EL < 16 ? 64 * EL : 4];  // the query
  __shared__ float red[4], ps[256], os[4][64 * EL];
  __shared__ long long at[256];  // element offset of a token's key from the slab's start, -1: no such page
  const int hq = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int hk = hq / (n_q / n_kv);
  const int n_tot = min(min(kv_len[b] + 1, max_seq_len), max_pages * geom.page_tokens);
  if (n_tot != kv_len[b] + 1 && threadIdx.x == 0) atomicOr(err_flag, 4);  // the sequence is longer than the step was sized for
  const float* qv = q + ((size_t)b * n_q + hq) * d;
  const int e0 = blockIdx.z * (64 * EL);
  if (EL < 16 && tid < d) qs[tid] = qv[tid];
  const float scale = rsqrtf((float)d);
  const float* base = reinterpret_cast<const float*>(slab);
  float m = -INFINITY, sum = 0.f, acc[EL];
#pragma unroll
  for (int x = 0; x < EL; ++x) acc[x] = 0.f;
  __syncthreads();
  for (int t0 = 0; t0 < n_tot; t0 += 256) {
    const int t = t0 + tid, nt = min(256, n_tot - t0);
    float s = -INFINITY;
    if (t < n_tot) {
      const int lp = t / geom.page_tokens, slot = t - lp * geom.page_tokens;
      const int page = page_table[(size_t)b * max_pages + lp];
      const size_t in_page = ((size_t)hk * geom.page_tokens + slot) * d;
      s = 0.f;
      if (page >= 0 && page < geom.n_pages_total) {
        const float* kp = base + kv_page_off(geom, page, layer, 0) / 4 + in_page;
        const float* qe = EL < 16 ? qs : qv;
        // 16 bytes a load for every head size: element by element, heads of 86 took 1414 us of a step of 256 sequences of 600
        // tokens, where this step takes 320 (the cache lines of 256 tokens do not stay in L1 for 86 visits)
        int e = 0;
#pragma unroll 4
        for (; e + 4 <= d; e += 4) {
          float kv[4];
          __builtin_memcpy(kv, kp + e, 16);
          s += qe[e] * kv[0] + qe[e + 1] * kv[1] + qe[e + 2] * kv[2] + qe[e + 3] * kv[3];
        }
        if (e < d) s += qe[e] * kp[e] + qe[e + 1] * kp[e + 1];  // (head sizes are even)
        at[tid] = (long long)(kv_page_off(geom, page, layer, 1) / 4 + in_page);
      } else {
        atomicOr(err_flag, 1);
        at[tid] = -1;
      }
      s *= scale;
    }
    float mx = s;
    mx = fmaxf(mx, g_dpp<0x140>(mx));
    mx = fmaxf(mx, g_dpp<0x141>(mx));
    mx = fmaxf(mx, g_dpp<0x4E>(mx));
    mx = fmaxf(mx, g_dpp<0xB1>(mx));
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])), m);
    const float ref = mx == -INFINITY ? 0.f : mx;  // (no score above -inf yet: the terms are zeros, not NaN)
    const float p = t < n_tot ? expf(s - ref) : 0.f, old = expf(m - ref);
    m = mx;
    ps[tid] = p;
    sum = sum * old + p;
#pragma unroll
    for (int x = 0; x < EL; ++x) acc[x] *= old;
    __syncthreads();
#pragma unroll 4
    for (int u = wave; u < nt; u += 4) {
      const long long a = at[u];
      const float pu = ps[u];
#pragma unroll
      for (int x = 0; x < EL; ++x) {
        const int e = e0 + lane + 64 * x;
        if (a >= 0 && e < d) acc[x] += pu * base[a + e];
      }
    }
    __syncthreads();  // red, ps and at are free again
  }
  const float lane_sum[1] = {sum};
  float tot[1];
  g_sum<1>(lane_sum, tot);
  if (lane == 0) red[wave] = tot[0];
#pragma unroll
  for (int x = 0; x < EL; ++x) os[wave][lane + 64 * x] = acc[x];
  __syncthreads();
  const float inv = 1.f / (red[0] + red[1] + red[2] + red[3]);
  for (int e = tid; e < min(64 * EL, d - e0); e += 256)
    o[((size_t)b * n_q + hq) * d + e0 + e] = (os[0][e] + os[1][e] + os[2][e] + os[3][e]) * inv;
}

__global__ void __launch_bounds__(256) g_argmax(const float* logits, int V, int* next) {
  __shared__ float bv[256];
  __shared__ int bi[256];
  const int b = blockIdx.x, tid = threadIdx.x;
  float best = -INFINITY;
  int idx = 0x7fffffff;
  for (int i = tid; i < V; i += 256) {
    const float v = logits[(size_t)b * V + i];
    if (v > best) best = v, idx = i;  // ascending i: the first maximum is kept
  }
  bv[tid] = best;
  bi[tid] = idx;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) {
      if (bv[tid + s] > bv[tid] || (bv[tid + s] == bv[tid] && bi[tid + s] < bi[tid])) bv[tid] = bv[tid + s], bi[tid] = bi[tid + s];
    }
    __syncthreads();
  }
  if (tid == 0) next[b] = bi[0] == 0x7fffffff ? 0 : bi[0];
}

inline bool vec4(const GLinear& p, int n_w) {
  uintptr_t bits = (uintptr_t)p.x | (uintptr_t)p.g;
  for (int j = 0; j < n_w; ++j) bits |= (uintptr_t)p.W[j];
  return p.K % 4 == 0 && bits % 16 == 0;
}

// The fewest batch rows per wave that hold the batch (up to kBT), 16-byte loads where rows and pointers allow them.
template <typename F>
void pick(const GLinear& p, int n_w, F&& go) {
  auto rows = [&](auto bt) {
    if (vec4(p, n_w)) go(bt, std::true_type{});
    else go(bt, std::false_type{});
  };
  if (p.B == 1) rows(std::integral_constant<int, 1>{});
  else if (p.B == 2) rows(std::integral_constant<int, 2>{});
  else if (p.B <= 4) rows(std::integral_constant<int, 4>{});
  else rows(std::integral_constant<int, kBT>{});
}
inline dim3 grid_of(const GLinear& p, int rows, int bt) { return dim3((rows + 3) / 4, (p.B + bt - 1) / bt); }

void linear(const float* x, const float* g, float eps, const void* W, const float* res, float* y, int B, int N, int K, hipStream_t st) {
  const GLinear p{x, g, {static_cast<const float*>(W), nullptr, nullptr}, res, y, B, K, N, eps};
  pick(p, 1, [&](auto bt, auto v4) {
    constexpr int BT = decltype(bt)::value;
    constexpr bool V = decltype(v4)::value;
    if (g) hipLaunchKernelGGL((g_linear<BT, V, true>), grid_of(p, N, BT), dim3(256), 0, st, p);
    else hipLaunchKernelGGL((g_linear<BT, V, false>), grid_of(p, N, BT), dim3(256), 0, st, p);
  });
}

}  // namespace

harli_status decode_step_f32(harli_ctx* c, const harli_decode_batch* b, hipStream_t st) {
  const harli_model_cfg& m = c->cfg;
  DecodeWs& w = c->dw;
  const int B = b->batch, H = m.hidden, d = m.head_dim, QD = m.n_q_heads * d, F = m.ffn, L = m.n_layers;
  // fp32 views of the workspace (every operand buffer is allocated at 4 bytes per element)
  float* o = static_cast<float*>(w.obuf);   // attention output
  float* mm = static_cast<float*>(w.mbuf);  // silu(gate) * up
  float* q = w.qbuf;
  const float* x = b->x_in;
  float* xn = w.xb;
  if (b->token_ids) {
    hipLaunchKernelGGL(g_input, dim3(B), dim3(256), 0, st, H, b->token_ids, static_cast<const float*>(c->emb), m.vocab, w.xa, w.err_flag);
    x = w.xa;
  }
  for (int l = 0; l < L; ++l) {
    const LayerDev& lw = c->layers[l];
    {
      const GLinear p{x, lw.g1, {static_cast<const float*>(lw.w[0]), static_cast<const float*>(lw.w[1]), static_cast<const float*>(lw.w[2])},
                      nullptr, q, B, H, QD, m.rms_eps};
      const GRope r{lw.bias[0], lw.bias[1], lw.bias[2], b->kv_len, b->page_table, b->max_pages, l, m.n_q_heads, m.n_kv_heads, d, w.inv_freq,
                    c->slab, c->geom, w.err_flag};
      pick(p, 3, [&](auto bt, auto v4) {
        constexpr int BT = decltype(bt)::value;
        hipLaunchKernelGGL((g_qkv<BT, decltype(v4)::value>), grid_of(p, (m.n_q_heads + 2 * m.n_kv_heads) * (d / 2), BT), dim3(256), 0, st, p, r);
      });
    }
#define G_ATT(EL_)                                                                                                     \
  hipLaunchKernelGGL(g_attention<EL_>, dim3(m.n_q_heads, B, (d + 64 * EL_ - 1) / (64 * EL_)), dim3(256), 0, st, q, b->kv_len, b->page_table, b->max_pages, l, \
                     m.n_q_heads, m.n_kv_heads, d, c->slab, c->geom, m.max_seq_len, o, w.err_flag)
    if (d <= 64) G_ATT(1);
    else if (d <= 128) G_ATT(2);
    else if (d <= 256) G_ATT(4);
    else G_ATT(16);
#undef G_ATT
    linear(o, nullptr, 0.f, lw.w[3], x, w.x1, B, H, QD, st);
    {
      const GLinear p{w.x1, lw.g2, {static_cast<const float*>(lw.w[4]), static_cast<const float*>(lw.w[5]), nullptr}, nullptr, mm, B, H, F,
                      m.rms_eps};
      pick(p, 2, [&](auto bt, auto v4) {
        constexpr int BT = decltype(bt)::value;
        hipLaunchKernelGGL((g_gate_up<BT, decltype(v4)::value>), grid_of(p, F, BT), dim3(256), 0, st, p);
      });
    }
    const bool last = (l == L - 1);
    float* dst = (last && b->x_out) ? b->x_out : xn;
    linear(mm, nullptr, 0.f, lw.w[6], w.x1, dst, B, H, F, st);
    x = dst;
    if (dst == xn) xn = xn == w.xb ? w.xa : w.xb;
  }
  if (b->logits) {
    linear(x, c->g_final, m.rms_eps, c->w_lm, nullptr, b->logits, B, m.vocab, H, st);
    if (b->next_token) hipLaunchKernelGGL(g_argmax, dim3(B), dim3(256), 0, st, b->logits, m.vocab, b->next_token);
  }
  HARLI_HIP(hipGetLastError());
  return HARLI_OK;
}

}  // namespace harli
