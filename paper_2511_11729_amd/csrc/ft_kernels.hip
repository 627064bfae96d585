// Element-wise, reduction and skinny kernels of the LoRA finetune unit (Harli Sec. 2.1: forward,
// backward with adapter gradients only; Sec. 6.1: one transformer layer per call).  These are
// the HBM-bound pieces between the MFMA GEMMs: every kernel reads and writes each element once
// with 8- or 16-byte accesses.
#include "ft_kernels.h"

#include <algorithm>

#include "ft_elem.h"

namespace harli {
namespace {

__device__ __forceinline__ float block_sum_256(float v, float* sh) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  const float r = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------- RMSNorm
__global__ void __launch_bounds__(256) k_rmsnorm_fwd(const float* x, const float* g, bf* h, float* rho, int H, float eps, int* flag) {
  __shared__ float sh[4];
  const int t = blockIdx.x, tid = threadIdx.x;
  const float* xr = x + (size_t)t * H;
  float s2 = 0.f;
  for (int k = tid * 4; k < H; k += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(xr + k);
    s2 += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  s2 = block_sum_256(s2, sh);
  const float r = rsqrtf(s2 / (float)H + eps);
  if (tid == 0) rho[t] = r;
  bool over = false;
  for (int k = tid * 4; k < H; k += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(xr + k);
    const float4 gg = *reinterpret_cast<const float4*>(g + k);
    *reinterpret_cast<uint2*>(h + (size_t)t * H + k) =
        make_uint2(PACK2G(v.x * r * gg.x, v.y * r * gg.y, over), PACK2G(v.z * r * gg.z, v.w * r * gg.w, over));
  }
  elem_flag(over, flag);
}

__global__ void __launch_bounds__(256) k_rmsnorm_bwd(const float* dh, const float* x, const float* rho, const float* g,
                                                     const float* dres, float* dx, bf* dx16, int H, const float* res_mul,
                                                     const float* out_mul, int* flag) {
  __shared__ float sh[4];
  const int t = blockIdx.x, tid = threadIdx.x;
  const float r = rho[t];
  const float rm = res_mul ? *res_mul : 1.f, om = out_mul ? *out_mul : 1.f;
  const float* xr = x + (size_t)t * H;
  const float* dr = dh + (size_t)t * H;
  float dot = 0.f;
  for (int k = tid * 4; k < H; k += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(xr + k);
    const float4 d = *reinterpret_cast<const float4*>(dr + k);
    const float4 gg = *reinterpret_cast<const float4*>(g + k);
    dot += d.x * gg.x * v.x + d.y * gg.y * v.y + d.z * gg.z * v.z + d.w * gg.w * v.w;
  }
  dot = block_sum_256(dot, sh);
  const float c = dot * r * r / (float)H;  // mean(dh*g*xhat) * rho, with xhat = x * rho
  bool over = false;
  for (int k = tid * 4; k < H; k += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(xr + k);
    const float4 d = *reinterpret_cast<const float4*>(dr + k);
    const float4 gg = *reinterpret_cast<const float4*>(g + k);
    const float4 rs = dres ? *reinterpret_cast<const float4*>(dres + (size_t)t * H + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 o;
    o.x = om * (rs.x * rm + r * (d.x * gg.x - v.x * c));
    o.y = om * (rs.y * rm + r * (d.y * gg.y - v.y * c));
    o.z = om * (rs.z * rm + r * (d.z * gg.z - v.z * c));
    o.w = om * (rs.w * rm + r * (d.w * gg.w - v.w * c));
    *reinterpret_cast<float4*>(dx + (size_t)t * H + k) = o;
    if (dx16) *reinterpret_cast<uint2*>(dx16 + (size_t)t * H + k) = make_uint2(PACK2G(o.x, o.y, over), PACK2G(o.z, o.w, over));
  }
  elem_flag(over, flag);
}

// ---------------------------------------------------------------- rotary embedding table
// angle reduced in double, as the oracle's positions are exact
__global__ void __launch_bounds__(256) k_rope_table(float2* out, long long n, int half, const double* inv_freq) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n) return;
  const double ang = (double)(idx / half) * inv_freq[idx % half];
  const double red = ang - 6.283185307179586476925 * rint(ang * 0.15915494309189533577);
  float sn, cs;
  sincosf((float)red, &sn, &cs);
  out[idx] = make_float2(cs, sn);
}

// ---------------------------------------------------------------- gradient scaling
// The backward pass is linear in dY, so dY is multiplied by a power of two sigma that brings its
// largest magnitude to 2^8 before it is rounded to 16 bits, and 1/sigma is applied where the
// fp32 results leave the unit (dX, dA, dB).  scale[0] = sigma, scale[1] = 1/sigma.
// Both kernels are bound by their 4 (+ 2) bytes per element.  The maxima of the workgroups go to an array that every
// workgroup of the second kernel reduces for itself: one atomic per workgroup on a single word made the first kernel
// 18 us for 33 MB, with the array it takes 8.6.
__global__ void __launch_bounds__(256) k_amax(const float* x, long long n4, float* parts) {
  // grid-stride over groups of 1024 float4, four independent 16-byte loads per thread in flight (indices past the
  // end re-read the last element)
  __shared__ float wmax[4];
  float m = 0.f;
  for (long long base = (long long)blockIdx.x * 1024 + threadIdx.x; base < n4; base += (long long)gridDim.x * 1024) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const float4*>(x)[min(base + u * 256, n4 - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      m = fmaxf(fmaxf(fmaxf(fabsf(v[u].x), fabsf(v[u].y)), fmaxf(fabsf(v[u].z), fabsf(v[u].w))), m);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) parts[blockIdx.x] = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
}
// sigma from the largest magnitude: the power of two that brings it to 2^target_log2 (1 for an all-zero or non-finite dY)
__device__ __forceinline__ float sigma_of(float a, int target_log2) {
  if (!(a > 0.f && a < INFINITY)) return 1.f;
  int e;
  frexpf(a, &e);  // a = f * 2^e, f in [0.5, 1)
  return ldexpf(1.f, min(max(target_log2 - e, -100), 100));
}
// y = 16-bit(x * sigma), 1024 groups of four elements per workgroup.  Every workgroup derives sigma from the maxima that
// k_amax left; workgroup 0 also publishes scale[0] = sigma, scale[1] = 1 / sigma for the kernels downstream.
__global__ void __launch_bounds__(256) k_f32_to_e_scaled(const float* x, bf* y, long long n4, const float* parts, int n_parts,
                                                         float* scale, int target_log2) {
  __shared__ float wmax[4];
  const long long base = (long long)blockIdx.x * 1024 + threadIdx.x;
  float4 v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const float4*>(x)[min(base + u * 256, n4 - 1)];
  float m = 0.f;
  for (int i = threadIdx.x; i < n_parts; i += 256) m = fmaxf(m, parts[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  const float sg = sigma_of(fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])), target_log2);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scale[0] = sg;
    scale[1] = 1.f / sg;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (base + u * 256 < n4)
      reinterpret_cast<uint2*>(y)[base + u * 256] = make_uint2(PACK2(v[u].x * sg, v[u].y * sg), PACK2(v[u].z * sg, v[u].w * sg));
}

// ---------------------------------------------------------------- skinny NT GEMM (LoRA down-projection x.A and dy.B^T)
// Workgroup = 16 RM rows of X, 8 waves split K, RM x NT accumulators of 16x16x32 each; one workgroup per compute unit.  What
// bounds it is what a compute unit takes in -- its rows of X and all of Bm -- and the latency of that: a wave's K steps are
// loaded U at a time, unconditionally, and where a launch has more than a round of workgroups, more rows share a read of Bm
// (ft_skinny_nt_multi).  Loading every step's registers again as soon as its products had read them was slower (4096 x 64 x
// 5120 26 -> 34 us, 2048 x 16 x 4096 10 -> 18): two neighbouring steps share the cache lines of a row.
typedef unsigned __attribute__((ext_vector_type(4))) u32x4;  // native vector: arrays of it stay in registers
__device__ __forceinline__ f32x4 mma16(const u32x4& a, const u32x4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
// K steps a wave loads together: 20 to 40 loads of 16 bytes
template <int NT, int RM>
constexpr int skinny_steps() { return NT + RM == 2 ? 16 : NT + RM <= 5 ? 8 : 4; }
template <int NT, int RM>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) k_skinny_nt(SkinnyNtJobs jobs, int M, float alpha, int* flag) {
  const SkinnyNtJob& jb = jobs.j[blockIdx.y];
  const bf* X = jb.X;
  const bf* Bm = jb.Bm;
  bf* C = jb.C;
  const long long ldx = jb.ldx, ldb = jb.ldb, ldc = jb.ldc;
  const int N = jb.N, K = jb.K;
  constexpr int NW = 8, U = skinny_steps<NT, RM>();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.x * (16 * RM);
  const bf *xr[RM], *br[NT];
#pragma unroll
  for (int q = 0; q < RM; ++q) xr[q] = X + (long long)min(m0 + q * 16 + i16, M - 1) * ldx + g * 8;
#pragma unroll
  for (int t = 0; t < NT; ++t) br[t] = Bm + (long long)min(t * 16 + i16, N - 1) * ldb + g * 8;
  f32x4 acc[RM][NT];
#pragma unroll
  for (int q = 0; q < RM; ++q)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int full = K >> 5;  // whole 32-wide steps
  const int s0 = full * wave / NW, s1 = full * (wave + 1) / NW;
  u32x4 xf[U][RM], bfr[U][NT];
  auto load = [&](int u, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < RM; ++q) xf[u][q] = *reinterpret_cast<const u32x4*>(xr[q] + (s << 5));
#pragma unroll
    for (int t = 0; t < NT; ++t) bfr[u][t] = *reinterpret_cast<const u32x4*>(br[t] + (s << 5));
  };
  auto mma = [&](int u) __attribute__((always_inline)) {  // rows of X = MFMA rows, rows of Bm = columns
#pragma unroll
    for (int q = 0; q < RM; ++q)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[q][t] = mma16(xf[u][q], bfr[u][t], acc[q][t]);
  };
  int s = s0;
  for (; s + U <= s1; s += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) load(u, s + u);
    __builtin_amdgcn_sched_barrier(0);  // every load of the group is issued before the first product waits for one
#pragma unroll
    for (int u = 0; u < U; ++u) mma(u);
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (s + u < s1) load(u, s + u);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (s + u < s1) mma(u);
  if (wave == NW - 1 && (K & 31)) {  // partial last step: lanes whose 8 k lie past K contribute zeros
    const int k = full << 5;
    const bool ok = k + g * 8 < K;
    const int kc = ok ? k : 0;
#pragma unroll
    for (int q = 0; q < RM; ++q) {
      xf[0][q] = *reinterpret_cast<const u32x4*>(xr[q] + kc);
      if (!ok) xf[0][q] = u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) bfr[0][t] = *reinterpret_cast<const u32x4*>(br[t] + kc);
    mma(0);
  }
  __shared__ float4 red[NW][NT][64];
  bool over = false;
#pragma unroll
  for (int q = 0; q < RM; ++q) {
    if (q) __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) red[wave][t][lane] = make_float4(acc[q][t][0], acc[q][t][1], acc[q][t][2], acc[q][t][3]);
    __syncthreads();
    if (wave < NT) {  // one column tile per wave
      float4 sm = red[0][wave][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const float4 o = red[w][wave][lane];
        sm.x += o.x; sm.y += o.y; sm.z += o.z; sm.w += o.w;
      }
      // lane holds D[m = 4g + e][n = i16]
      const int n = wave * 16 + i16;
      const float v[4] = {sm.x, sm.y, sm.z, sm.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + q * 16 + 4 * g + e;
        if (m < M && n < N) C[(long long)m * ldc + n] = F2EG(v[e] * alpha, over);
      }
    }
  }
  elem_flag(over, flag);
}

// ---------------------------------------------------------------- adapter gradients: G[j, r] += sum_t X[t, j] U[t, r]
// Two passes without atomics.  Pass 1: a workgroup covers 512 j x one token chunk; each thread owns two adjacent j
// and all R ranks.  The U rows are widened to fp32 in LDS 64 tokens at a time and read as wave-wide broadcasts; X is
// read as one 32-bit word per lane and token, eight tokens in flight (rows past the chunk reuse its last row against
// zero U rows).  The chunk's sums go to part[chunk][r][j].  Pass 2 adds the chunks and accumulates into G.
constexpr int kLgT = 64, kLgMaxChunks = 32;
// Half operands: two tokens per v_dot2_f32_f16 (exact products, fp32 accumulation).  U is staged in LDS as packed
// pairs (U[t][r], U[t+1][r]); the matching pairs of X are assembled from the two tokens' 32-bit words.
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
template <int R>
__global__ void __launch_bounds__(256) k_lora_grad_part(const bf* X, long long ldx, const bf* U, long long ldu, float* part,
                                                        int T, int J, int tpc) {
  __shared__ __align__(16) unsigned us2[kLgT / 2][R];
  const int tid = threadIdx.x;
  const int j0 = (blockIdx.x * 256 + tid) * 2;
  const int c0 = blockIdx.y * tpc, c1 = min(T, c0 + tpc);
  float a0[R], a1[R];
#pragma unroll
  for (int r = 0; r < R; ++r) a0[r] = a1[r] = 0.f;
  for (int t0 = c0; t0 < c1; t0 += kLgT) {
    const int nt = min(kLgT, c1 - t0);
    __syncthreads();
    for (int i = tid; i < (kLgT / 2) * R; i += 256) {
      const int tp = i / R, r = i - tp * R;
      const unsigned lo = 2 * tp < nt ? U[(long long)(t0 + 2 * tp) * ldu + r] : 0u;
      const unsigned hi = 2 * tp + 1 < nt ? U[(long long)(t0 + 2 * tp + 1) * ldu + r] : 0u;
      us2[tp][r] = lo | (hi << 16);
    }
    __syncthreads();
    const bf* xp = X + (long long)t0 * ldx + min(j0, J - 2);
    for (int tp = 0; tp < kLgT / 2; tp += 4) {
      unsigned xv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) xv[u] = *reinterpret_cast<const unsigned*>(xp + (long long)min(2 * tp + u, nt - 1) * ldx);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned w0 = xv[2 * u], w1 = xv[2 * u + 1];
        const h16x2 p0 = __builtin_bit_cast(h16x2, (w0 & 0xffffu) | (w1 << 16));        // (X[t][j0],   X[t+1][j0])
        const h16x2 p1 = __builtin_bit_cast(h16x2, (w0 >> 16) | (w1 & 0xffff0000u));   // (X[t][j0+1], X[t+1][j0+1])
#pragma unroll
        for (int r = 0; r < R; r += 4) {
          const uint4 uu = *reinterpret_cast<const uint4*>(&us2[tp + u][r]);
          const unsigned uw[4] = {uu.x, uu.y, uu.z, uu.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const h16x2 up = __builtin_bit_cast(h16x2, uw[e]);
            a0[r + e] = __builtin_amdgcn_fdot2(p0, up, a0[r + e], false);
            a1[r + e] = __builtin_amdgcn_fdot2(p1, up, a1[r + e], false);
          }
        }
      }
    }
  }
  if (j0 < J) {
    float* p = part + (long long)blockIdx.y * R * J + j0;
#pragma unroll
    for (int r = 0; r < R; ++r) *reinterpret_cast<float2*>(p + (long long)r * J) = make_float2(a0[r], a1[r]);
  }
}


// MFMA version of pass 1 for 16-byte aligned operands (J, ldx, ldu multiples of 8).  The product contracts over the
// ROW index of both operands (part[r][j] = sum_t X[t][j] U[t][r]), the layout MFMA operands do not come in: a lane must
// hold eight consecutive t of one column.  gfx950's transposing LDS read does that turn on the way out of LDS: with
// the tiles stored as they are in memory ([t][j], [t][r]) and lane q of every 16-lane group pointing at row q / 4,
// columns 4 (q % 4) .. + 3 of a 4 x 16 block, ds_read_b64_tr_b16 leaves lane i of the group with column i of the four
// rows -- two such reads give a lane its eight t of v_mfma_f32_16x16x32.  Workgroup: 256 columns j (64 per wave, four
// 16-column tiles) x all R ranks x one token chunk, 32 tokens per step through LDS.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned lg_u32x4 __attribute__((ext_vector_type(4)));  // native vector: arrays of HIP's uint4 struct were left in scratch memory
constexpr int kLmJ = 256, kLmT = 32, kLmPF = 4, kLmXS = kLmJ + 8;  // tile sizes, steps in flight; padded row of the X tile (halves)

template <int R>
__global__ void __launch_bounds__(256) k_lora_grad_mfma(LoraGradJobs jobs, float* part_all, int T) {
  const LoraGradJob& jb = jobs.j[blockIdx.z];
  if ((int)blockIdx.x >= jb.jt || (int)blockIdx.y >= jb.nch) return;  // the grid is sized for the largest job
  const bf* X = jb.X;
  const bf* U = jb.U;
  const long long ldx = jb.ldx, ldu = jb.ldu;
  const int J = jb.J, tpc = jb.tpm;
  float* part = part_all + jb.part_off;
  constexpr int RP = R < 16 ? 16 : R;  // rank padded to an MFMA tile (the padding columns of the U tile stay zero)
  constexpr int NT = RP / 16;          // 16-rank tiles
  constexpr int US = RP + 8;           // padded row of the U tile (halves)
  __shared__ __align__(16) unsigned short xs[kLmT][kLmXS];
  __shared__ __align__(16) unsigned short us[kLmT][US];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j0 = blockIdx.x * kLmJ;
  const int c0 = blockIdx.y * tpc, c1 = min(T, c0 + tpc);
  f32x4 acc[4][NT];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i = tid; i < kLmT * US; i += 256) (&us[0][0])[i] = 0;  // zero once: rows and columns never written stay zero

  // staging coordinates: X tile = 32 rows x 32 chunks of 16 bytes, four per thread; U tile = 32 rows x R / 8 chunks
  const int xc = tid & 31, xr = tid >> 5;
  const int xcol = min(j0 + xc * 8, J - 8);  // columns past J are loaded from a valid place and never stored
  constexpr int UCH = R / 8;
  const int uc = tid % UCH, ur = tid / UCH;  // threads with ur >= 32 stage nothing
  // fragment coordinates: 16-lane group g covers t = 8g .. 8g+7; lane q of it points at row q / 4, columns 4 (q % 4)
  const int g = lane >> 4, q = lane & 15;
  const int frow = 8 * g + (q >> 2), fcol = 4 * (q & 3);

  // kLmPF steps of loads are issued together (the MFMAs of a step take a fraction of a load's latency, so one step
  // of prefetch would leave every step waiting for memory)
  for (int tb = c0; tb < c1; tb += kLmT * kLmPF) {
    lg_u32x4 xv[kLmPF][4], uv[kLmPF];
#pragma unroll
    for (int p = 0; p < kLmPF; ++p) {
      const int t0 = tb + p * kLmT;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        xv[p][i] = *reinterpret_cast<const lg_u32x4*>(X + (long long)min(t0 + xr + 8 * i, T - 1) * ldx + xcol);
      // rows past the chunk are fetched from a valid row and zeroed below: they add nothing
      uv[p] = *reinterpret_cast<const lg_u32x4*>(U + (long long)min(t0 + min(ur, kLmT - 1), T - 1) * ldu + uc * 8);
    }
#pragma unroll
    for (int p = 0; p < kLmPF; ++p) {
      const int t0 = tb + p * kLmT;
      if (t0 >= c1) break;  // uniform
      __syncthreads();      // the previous step's fragments have been read
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<lg_u32x4*>(&xs[xr + 8 * i][xc * 8]) = xv[p][i];
      if (ur < kLmT) *reinterpret_cast<lg_u32x4*>(&us[ur][uc * 8]) = t0 + ur < c1 ? uv[p] : lg_u32x4{0u, 0u, 0u, 0u};
      __syncthreads();
      s16x8 bfr[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(&us[frow][nt * 16 + fcol]));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(&us[frow + 4][nt * 16 + fcol]));
        bfr[nt] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int col = wave * 64 + mt * 16 + fcol;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(&xs[frow][col]));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(&xs[frow + 4][col]));
        const s16x8 afr = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, afr), __builtin_bit_cast(f16x8, bfr[nt]), acc[mt][nt], 0, 0, 0);
        }
      }
    }
  }
  // lane holds out[j = tile + 4 (lane / 16) + v][r = tile + lane % 16], v = 0..3: four consecutive j of one rank
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    const int j = j0 + wave * 64 + mt * 16 + 4 * g;
    if (j >= J) continue;  // J % 8 == 0: the four columns are in or out together
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int r = nt * 16 + q;
      if (r < R)
        *reinterpret_cast<float4*>(part + (long long)blockIdx.y * R * J + (long long)r * J + j) =
            make_float4(acc[mt][nt][0], acc[mt][nt][1], acc[mt][nt][2], acc[mt][nt][3]);
    }
  }
}

// G[j*sj + r*sr] += out_mul * sum_c part[c][r][j]: one thread per (r, j), lanes along j (the reads of part, 2 x
// nchunk times the volume of G, are the contiguous side)
__global__ void __launch_bounds__(256) k_lora_grad_reduce(const float* part, int nchunk, float* G, long long sj, long long sr,
                                                          int J, long long RJ, const float* out_mul) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= RJ) return;
  const int r = (int)(i / J), j = (int)(i - (long long)r * J);
  float sum = 0.f;
#pragma unroll 8
  for (int c = 0; c < nchunk; ++c) sum += part[c * RJ + i];
  float* g = G + (long long)j * sj + (long long)r * sr;
  *g += sum * (out_mul ? *out_mul : 1.f);
}

// The same for several jobs.  A workgroup adds up 32 columns j x R ranks; where j is not the contiguous index of G (dA: [in, r])
// the sums turn in LDS, so that both the partial sums and G are read and written in whole rows (lanes along j at a stride of R
// floats were 64 separate accesses a wave: six sums of 64 x 5120 took 45 us).
template <int R>
__global__ void __launch_bounds__(256) k_lora_grad_reduce_multi(LoraGradJobs jobs, const float* part_all, const float* out_mul) {
  constexpr int JW = 32, RS = 256 / JW, N = R / RS;  // columns of a workgroup, ranks side by side, sums per thread
  const LoraGradJob& jb = jobs.j[blockIdx.y];
  const int J = jb.J, j0 = blockIdx.x * JW, tid = threadIdx.x;
  if (j0 >= J) return;
  const long long RJ = (long long)R * J;
  const float* part = part_all + jb.part_off;
  const float mul = out_mul ? *out_mul : 1.f;
  float sum[N];
  const int jl = tid % JW, r0 = tid / JW, j = min(j0 + jl, J - 1);
#pragma unroll
  for (int n = 0; n < N; ++n) sum[n] = 0.f;
#pragma unroll 2
  for (int c = 0; c < jb.nch; ++c)
#pragma unroll
    for (int n = 0; n < N; ++n) sum[n] += part[c * RJ + (long long)(n * RS + r0) * J + j];
  if (jb.sj == 1) {
    if (j0 + jl < J)
#pragma unroll
      for (int n = 0; n < N; ++n) {
        float* g = jb.G + (long long)(n * RS + r0) * jb.sr + j;
        *g += sum[n] * mul;
      }
    return;
  }
  __shared__ float turn[JW][R + 1];
#pragma unroll
  for (int n = 0; n < N; ++n) turn[jl][n * RS + r0] = sum[n];
  __syncthreads();
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int i = n * 256 + tid, jj = i / R, r = i % R;
    if (j0 + jj < J) {
      float* g = jb.G + (long long)(j0 + jj) * jb.sj + (long long)r * jb.sr;
      *g += turn[jj][r] * mul;
    }
  }
}

__global__ void __launch_bounds__(256) k_sum_groups(const bf* in, bf* out, long long total, int n_kv, int G, int d, int* flag) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int kvd = n_kv * d;
  const long long t = i / kvd;
  const int rem = (int)(i - t * kvd), c = rem / d, e = rem - c * d;
  float s = 0.f;
  for (int g = 0; g < G; ++g) s += E2F(in[t * (long long)kvd * G + (c * G + g) * d + e]);
  bool over = false;
  out[i] = F2EG(s, over);
  elem_flag(over, flag);
}

inline unsigned nblk(long long n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

void ft_rmsnorm_fwd(const float* x, const float* g, bf* h, float* rho, int T, int H, float eps, int* flag, hipStream_t st) {
  hipLaunchKernelGGL(k_rmsnorm_fwd, dim3(T), dim3(256), 0, st, x, g, h, rho, H, eps, flag);
}
void ft_rmsnorm_bwd(const float* dh, const float* x, const float* rho, const float* g, const float* dres, float* dx, bf* dx16,
                    int T, int H, const float* res_mul, const float* out_mul, int* flag, hipStream_t st) {
  hipLaunchKernelGGL(k_rmsnorm_bwd, dim3(T), dim3(256), 0, st, dh, x, rho, g, dres, dx, dx16, H, res_mul, out_mul, flag);
}
void ft_rope_table(float2* out, int n_pos, int d, const double* inv_freq, hipStream_t st) {
  const long long n = (long long)n_pos * (d / 2);
  hipLaunchKernelGGL(k_rope_table, dim3(nblk(n, 256)), dim3(256), 0, st, out, n, d / 2, inv_freq);
}
void ft_scale_to_e(const float* x, bf* y, long long n, float* scale, int target_log2, hipStream_t st) {
  const unsigned parts = std::min(nblk(n / 4, 1024), (unsigned)kAmaxParts);
  hipLaunchKernelGGL(k_amax, dim3(parts), dim3(256), 0, st, x, n / 4, scale + 2);
  hipLaunchKernelGGL(k_f32_to_e_scaled, dim3(nblk(n / 4, 1024)), dim3(256), 0, st, x, y, n / 4, scale + 2, (int)parts, scale, target_log2);
}
void ft_skinny_nt_multi(const SkinnyNtJobs& jobs, int M, float alpha, int* flag, hipStream_t st) {
  if (jobs.n < 1) return;
  int nmax = 0;
  for (int i = 0; i < jobs.n; ++i) nmax = std::max(nmax, jobs.j[i].N);
  const int nt = nmax <= 16 ? 1 : nmax <= 32 ? 2 : 4;  // jobs with fewer columns mask their stores
  // Rows per workgroup: the fewest bytes through the fullest compute unit, 16 (RM + NT) K 2 per workgroup of it.  Measured,
  // 4096 rows, 64 columns, us with 16 rows and as chosen: three jobs over K = 5120 74 / 43 (64 rows), two 51 / 33 (32 rows), two
  // over 13824 128 / 85 (32 rows); 2048 rows, 16 columns, three jobs over 4096 17.7 / 14.7 (32 rows).
  static const int n_cu = [] {
    int dev = 0, n = 0;
    return hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0 ? n : 256;
  }();
  int rm = 1;
  long long least = 0;
  for (int q = 1; q <= 4; q *= 2) {
    const long long wgs = (long long)((M + 16 * q - 1) / (16 * q)) * jobs.n, cost = (wgs + n_cu - 1) / n_cu * (q + nt);
    if (q == 1 || cost < least) rm = q, least = cost;
  }
  const dim3 grid((M + 16 * rm - 1) / (16 * rm), jobs.n), blk(512);
#define SKINNY(NT_)                                                                                          \
  do {                                                                                                       \
    if (rm == 1) hipLaunchKernelGGL((k_skinny_nt<NT_, 1>), grid, blk, 0, st, jobs, M, alpha, flag);          \
    else if (rm == 2) hipLaunchKernelGGL((k_skinny_nt<NT_, 2>), grid, blk, 0, st, jobs, M, alpha, flag);     \
    else hipLaunchKernelGGL((k_skinny_nt<NT_, 4>), grid, blk, 0, st, jobs, M, alpha, flag);                  \
  } while (0)
  if (nt == 1) SKINNY(1);
  else if (nt == 2) SKINNY(2);
  else SKINNY(4);
#undef SKINNY
}
// floats of partial sums one job of the MFMA path can need: nch * J with nch <= max(1, 512 / column tiles)
static size_t lora_grad_job_floats(int J, int R) { return (size_t)std::max(512 * kLmJ, (J + kLmJ - 1) / kLmJ * kLmJ) * R; }
size_t ft_lora_grad_ws_floats(int J, int R) {
  return std::max((size_t)kLgMaxChunks * J * R, (size_t)kLoraGradMaxJobs * lora_grad_job_floats(J, R));
}
template <int R>
static void lora_grad_launch(const bf* X, long long ldx, const bf* U, long long ldu, float* G, long long sj, long long sr, int T,
                             int J, const float* out_mul, float* part, hipStream_t st) {
  const int tpc = std::max(kLgT, ((T + kLgMaxChunks - 1) / kLgMaxChunks + kLgT - 1) / kLgT * kLgT);
  const int nchunk = (T + tpc - 1) / tpc;
  hipLaunchKernelGGL(k_lora_grad_part<R>, dim3((J + 511) / 512, nchunk), dim3(256), 0, st, X, ldx, U, ldu, part, T, J, tpc);
  hipLaunchKernelGGL(k_lora_grad_reduce, dim3(nblk((long long)R * J, 256)), dim3(256), 0, st, part, nchunk, G, sj, sr, J, (long long)R * J,
                     out_mul);
}
static void lora_grad_vector(const LoraGradJob& b, int T, int R, const float* out_mul, float* part, hipStream_t st) {
  if (R == 8) lora_grad_launch<8>(b.X, b.ldx, b.U, b.ldu, b.G, b.sj, b.sr, T, b.J, out_mul, part, st);
  else if (R == 16) lora_grad_launch<16>(b.X, b.ldx, b.U, b.ldu, b.G, b.sj, b.sr, T, b.J, out_mul, part, st);
  else if (R == 32) lora_grad_launch<32>(b.X, b.ldx, b.U, b.ldu, b.G, b.sj, b.sr, T, b.J, out_mul, part, st);
  else lora_grad_launch<64>(b.X, b.ldx, b.U, b.ldu, b.G, b.sj, b.sr, T, b.J, out_mul, part, st);
}
void ft_lora_grad_multi(LoraGradJobs& jobs, int T, int R, const float* out_mul, float* part, hipStream_t st) {
  if (jobs.n < 1) return;
  bool aligned = (reinterpret_cast<uintptr_t>(part) & 15) == 0;
  for (int i = 0; i < jobs.n; ++i) {
    const LoraGradJob& b = jobs.j[i];
    aligned = aligned && b.J % 8 == 0 && b.ldx % 8 == 0 && b.ldu % 8 == 0 &&
              ((reinterpret_cast<uintptr_t>(b.X) | reinterpret_cast<uintptr_t>(b.U)) & 15) == 0;
  }
  if (!aligned) {  // the vector kernels, one job after the other (each uses the whole scratch)
    for (int i = 0; i < jobs.n; ++i) lora_grad_vector(jobs.j[i], T, R, out_mul, part, st);
    return;
  }
  // About three workgroups per compute unit in all jobs together and whole groups of steps in flight: every chunk of tokens
  // costs a partial sum of R x J floats, written and read (two workgroups per compute unit for each of six jobs of 64 x 5120 x
  // 4096 wrote 126 MB beside 252 MB of operands and took 74 us, now 55).
  int max_jt = 0, max_nch = 0, max_j = 0, sum_jt = 0;
  for (int i = 0; i < jobs.n; ++i) sum_jt += (jobs.j[i].J + kLmJ - 1) / kLmJ;
  long long off = 0;
  const int unit = kLmT * kLmPF;
  for (int i = 0; i < jobs.n; ++i) {
    LoraGradJob& b = jobs.j[i];
    b.jt = (b.J + kLmJ - 1) / kLmJ;
    const int want = std::min({kLgMaxChunks, std::max(1, 512 / b.jt), std::max(1, 768 / sum_jt)});
    b.tpm = std::max(unit, ((T + want - 1) / want + unit - 1) / unit * unit);
    b.nch = (T + b.tpm - 1) / b.tpm;
    b.part_off = off;
    off += (long long)lora_grad_job_floats(b.J, R);
    max_jt = std::max(max_jt, b.jt);
    max_nch = std::max(max_nch, b.nch);
    max_j = std::max(max_j, b.J);
  }
  const dim3 grid(max_jt, max_nch, jobs.n);
  if (R == 8) hipLaunchKernelGGL(k_lora_grad_mfma<8>, grid, dim3(256), 0, st, jobs, part, T);
  else if (R == 16) hipLaunchKernelGGL(k_lora_grad_mfma<16>, grid, dim3(256), 0, st, jobs, part, T);
  else if (R == 32) hipLaunchKernelGGL(k_lora_grad_mfma<32>, grid, dim3(256), 0, st, jobs, part, T);
  else hipLaunchKernelGGL(k_lora_grad_mfma<64>, grid, dim3(256), 0, st, jobs, part, T);
  const dim3 rgrid((max_j + 31) / 32, jobs.n);
  if (R == 8) hipLaunchKernelGGL(k_lora_grad_reduce_multi<8>, rgrid, dim3(256), 0, st, jobs, part, out_mul);
  else if (R == 16) hipLaunchKernelGGL(k_lora_grad_reduce_multi<16>, rgrid, dim3(256), 0, st, jobs, part, out_mul);
  else if (R == 32) hipLaunchKernelGGL(k_lora_grad_reduce_multi<32>, rgrid, dim3(256), 0, st, jobs, part, out_mul);
  else hipLaunchKernelGGL(k_lora_grad_reduce_multi<64>, rgrid, dim3(256), 0, st, jobs, part, out_mul);
}
void ft_lora_grad(const bf* X, long long ldx, const bf* U, long long ldu, float* G, long long sj, long long sr, int T, int J,
                  int R, const float* out_mul, float* part, hipStream_t st) {
  LoraGradJobs jobs{};
  jobs.n = 1;
  jobs.j[0] = LoraGradJob{X, ldx, U, ldu, G, sj, sr, J, 0, 0, 0, 0};
  ft_lora_grad_multi(jobs, T, R, out_mul, part, st);
}
void ft_sum_groups(const bf* in, bf* out, int T, int n_kv, int G, int d, int* flag, hipStream_t st) {
  const long long total = (long long)T * n_kv * d;
  hipLaunchKernelGGL(k_sum_groups, dim3(nblk(total, 256)), dim3(256), 0, st, in, out, total, n_kv, G, d, flag);
}

}  // namespace harli
