// Fused causal attention for the finetune unit on gfx950 (the attention part of the layer forward / backward
// that the per-layer finetune unit of Harli Sec. 6.1 runs; scores never leave the chip).
//
// All three kernels use v_mfma_f32_32x32x16 with one operand held in registers for the whole kernel and the
// other streamed through LDS in blocks of 64 rows.  The accumulator layout of a 32x32 tile (lane = column,
// registers = rows 8*(v/4) + 4*(lane/32) + v%4) decides the orientation of every product:
//   * forward and dQ compute S^T = K Q^T, so that a lane owns ONE query: its running max / sum (forward) or its
//     lse / delta (backward) are per-lane scalars, and the probabilities leave the accumulator already in the
//     layout of a B operand whose contraction index is the key;
//   * dK / dV compute S = Q K^T, so that a lane owns one key and the probabilities are a B operand whose
//     contraction index is the query.
// In both cases the second product contracts over the index held in the accumulator's REGISTERS.  Register v of a
// lane half h is contraction slot v%8 of MFMA step v/8, i.e. row 16*(v/8) + 8*((v%8)/4) + 4h + v%4: the A operand
// of the second product (V^T, K^T, Q^T or dO^T) wants rows 4h..4h+3 and 8+4h..8+4h+3 of each 16-row step of the
// streamed tile, eight of them per lane for one column.  The tile lies in LDS as it lies in memory (row-major), and
// ds_read_b64_tr_b16 turns it on the way out: a 16-lane group points at a 4 x 16 block (lane q at row q/4, columns
// 4(q%4)..+3) and lane i receives column i of the four rows.  No transposed copies, in memory or in LDS.
//
// Blocks go from memory straight to LDS (buffer_load ... lds, two buffers, one barrier per block), the 16-byte chunks
// of a row permuted by swz() on the way in so that the row reads and the transposing reads are both free of bank
// conflicts.  Rows past the sequence are out of the buffer resource's range and read as zeros.
//
// In k_attn_bwd_dkv<128> the loads of the next block do not overlap the products: at two waves per SIMD its 256 registers
// are not enough, 13 are spilled (eight lane offsets of the loads, four of a key fragment), and the wait for the reloads is a
// wait for everything in flight.
//
// What bounds them at 512 to 1024 tokens is vector work per score, not MFMA: the exponent is one fma and the bare
// hardware exponential, masks are applied only to blocks that cross the diagonal, and the running output is rescaled
// only when a maximum has moved.  4 x 512 tokens, 32 heads of 128: forward 41 -> 24 us, dQ 56 -> 32, dK/dV 121 -> 55
// (before: transposed copies made by a separate kernel, 36 us; both tiles of an operand in LDS, loaded through registers).
#include "ft_attention.h"

#include "ft_elem.h"

namespace harli {
namespace {

constexpr int KB = 64;            // rows of the streamed operand per block
// native vector types: arrays of them stay in registers (arrays of the HIP uint4 struct were left in scratch)
typedef unsigned __attribute__((ext_vector_type(4))) u32x4;
typedef unsigned __attribute__((ext_vector_type(2))) u32x2;
typedef short __attribute__((ext_vector_type(4))) s16x4;
typedef short __attribute__((ext_vector_type(8))) s16x8;
typedef _Float16 __attribute__((ext_vector_type(2))) f16x2;
#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ f32x16 mma32(const u32x4& a, const u32x4& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Chunk (16 bytes) permutation of a staged row: chunk c of row r lies in slot c ^ swz(r).  Eight consecutive rows get
// eight different even values (row reads: eight lanes of a b128 read hit different slots), four consecutive rows differ
// above bit 0 (transposing reads: the two chunks a row contributes lie side by side).
template <int D>
__device__ __forceinline__ int swz(int r) {
  return D == 128 ? ((r & 7) << 1) | ((r >> 3) & 1) : ((r & 3) << 1) | ((r >> 2) & 1);
}

// Rows [64 blk, 64 blk + 64) of a [rows][D] operand (row stride ld_bytes, described by rs) to an LDS tile, by four waves.
template <int D>
__device__ __forceinline__ void stage_block(__amdgpu_buffer_rsrc_t rs, int blk, unsigned ld_bytes, char* tile, int wave, int lane) {
  constexpr int CPR = D / 8, RPI = 64 / CPR, NI = KB / RPI / 4;  // chunks per row, rows per instruction, instructions per wave
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r0 = (wave * NI + i) * RPI, r = r0 + lane / CPR;
    const unsigned off = (unsigned)(blk * KB + r) * ld_bytes + (unsigned)(((lane % CPR) ^ swz<D>(r)) * 16);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(void, tile + r0 * (D * 2)), 16, (int)off, 0, 0, 0);
  }
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const bf* base, int rows, unsigned ld_bytes, int D) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf*>(base), 0, (int)((unsigned)(rows - 1) * ld_bytes + (unsigned)D * 2u), 0x00020000);
}
// this wave's loads have landed, and every wave is past its reads of the other buffer
__device__ __forceinline__ void block_ready() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// Lane offsets into a staged tile: row reads (row lane%32, chunk 2j + lane/32) and the two transposing reads.
template <int D>
struct TileLane {
  int row, t_lo, t_hi;
  __device__ __forceinline__ explicit TileLane(int lane) {
    const int l31 = lane & 31, h = lane >> 5, q = lane & 15;
    row = l31 * (D * 2) + ((h ^ swz<D>(l31)) << 4);
    const int r_lo = 4 * h + (q >> 2), r_hi = r_lo + 8, c = ((l31 >> 4) << 1) | ((q & 3) >> 1);
    t_lo = r_lo * (D * 2) + ((c ^ swz<D>(r_lo)) << 4) + (q & 1) * 8;
    t_hi = r_hi * (D * 2) + ((c ^ swz<D>(r_hi)) << 4) + (q & 1) * 8;
  }
};
// A fragment, rows sub*32 + lane%32, k = 16j + 8h .. +7
template <int D>
__device__ __forceinline__ u32x4 frag_rows(const char* tile, const TileLane<D>& t, int sub, int j) {
  return *reinterpret_cast<const u32x4*>(tile + sub * (32 * D * 2) + (t.row ^ (j << 5)));
}
// A fragment of the transposed tile: row (= column of the tile) et*32 + lane%32, contraction slots of step (sub, jj)
template <int D>
__device__ __forceinline__ u32x4 frag_cols(char* tile, const TileLane<D>& t, int et, int sub, int jj) {
  char* p = tile + (sub * 32 + jj * 16) * (D * 2);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p + (t.t_lo ^ (et << 6))));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p + (t.t_hi ^ (et << 6))));
  return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ unsigned cvt2(float lo, float hi) { return __builtin_bit_cast(unsigned, f16x2{(_Float16)lo, (_Float16)hi}); }
__device__ __forceinline__ float clamp_h(float x) { return __builtin_amdgcn_fmed3f(x, -65504.f, 65504.f); }
// eight accumulator registers to a B fragment; CLAMP where the values may leave half's range
template <bool CLAMP>
__device__ __forceinline__ u32x4 pack8(const f32x16& a, int o) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = CLAMP ? cvt2(clamp_h(a[o + 2 * i]), clamp_h(a[o + 2 * i + 1])) : cvt2(a[o + 2 * i], a[o + 2 * i + 1]);
  return r;
}
__device__ __forceinline__ f32x16 zero16f() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
// Four head-dim rows (e*32 + 8g + 4h ..) of a gradient column and their rotation partners (d/2 further), times scale, with
// the inverse rotary embedding of the column's position applied: (lo, hi) -> (lo cos + hi sin, hi cos - lo sin).
__device__ __forceinline__ void unrotate4(const f32x16& lo, const f32x16& hi, int g, const float2* cs, float scale, float* ol, float* oh) {
  const float4 t0 = *reinterpret_cast<const float4*>(cs), t1 = *reinterpret_cast<const float4*>(cs + 2);
  const float c[4] = {t0.x, t0.z, t1.x, t1.z}, s[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = lo[4 * g + i] * scale, b = hi[4 * g + i] * scale;
    ol[i] = a * c[i] + b * s[i];
    oh[i] = b * c[i] - a * s[i];
  }
}
// maximum over the two lanes (l, l + 32) that share a column
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// -------------------------------------------------------------------------------------------- forward
// grid (Bf*n_q, ceil(S/128)): the blocks with the longest causal span of all heads start first, and (with a multiple of
// eight heads) all blocks of a head run on one XCD, whose L2 then holds the head's K and V.  A workgroup owns 128 queries
// of one head, wave w the 32 queries 32w..32w+31.
template <int D>
__global__ void __launch_bounds__(256, 2) k_attn_fwd(const bf* __restrict__ q, const bf* __restrict__ k, const bf* __restrict__ v,
                                                  bf* __restrict__ o, float* __restrict__ lse2, int S, int nq, int nkv,
                                                  float scale_log2) {
  constexpr int NJ = D / 16, NE = D / 32, TILE = KB * D * 2;
  extern __shared__ __align__(1024) char smem[];  // two buffers of (K, V)
  const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb = gridDim.y - 1 - blockIdx.y;
  const int z = blockIdx.x, b = z / nq, head = z - b * nq, hk = head / (nq / nkv);
  const int QD = nq * D;
  const unsigned kv_ld = (unsigned)(nkv * D) * 2u;
  const int q0 = qb * 128 + wave * 32, qrow = q0 + l31, qc = min(qrow, S - 1);
  const TileLane<D> tl(lane);
  const auto rsK = rows_rsrc(k + (long long)b * S * nkv * D + hk * D, S, kv_ld, D);
  const auto rsV = rows_rsrc(v + (long long)b * S * nkv * D + hk * D, S, kv_ld, D);

  const int nkb = min(qb * 128 + 127, S - 1) / KB + 1;
  stage_block<D>(rsK, 0, kv_ld, smem, wave, lane);
  stage_block<D>(rsV, 0, kv_ld, smem + TILE, wave, lane);
  u32x4 Qf[NJ];
  {
    const bf* qp = q + ((long long)b * S + qc) * QD + head * D + 8 * h;
#pragma unroll
    for (int j = 0; j < NJ; ++j) Qf[j] = *reinterpret_cast<const u32x4*>(qp + 16 * j);
  }
  f32x16 O[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) O[e] = zero16f();
  float m_run = -INFINITY, l_run = 0.f;  // maximum of the raw scores; sum over this lane half's keys

  for (int kb = 0; kb < nkb; ++kb) {
    block_ready();
    char* sK = smem + (kb & 1) * (2 * TILE);
    char* sV = sK + TILE;
    if (kb + 1 < nkb) {
      char* nx = smem + ((kb + 1) & 1) * (2 * TILE);
      stage_block<D>(rsK, kb + 1, kv_ld, nx, wave, lane);
      stage_block<D>(rsV, kb + 1, kv_ld, nx + TILE, wave, lane);
    }
    if (kb * KB > q0 + 31) continue;  // every key of the block is past this wave's queries
    f32x16 sc[2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      sc[sub] = zero16f();
#pragma unroll
      for (int j = 0; j < NJ; ++j) sc[sub] = mma32(frag_rows<D>(sK, tl, sub, j), Qf[j], sc[sub]);
    }
    if (kb * KB + KB - 1 > q0) {  // the block crosses the diagonal of this wave's queries
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int vv = 0; vv < 16; ++vv)
          if (kb * KB + sub * 32 + 8 * (vv >> 2) + 4 * h + (vv & 3) > qrow) sc[sub][vv] = -INFINITY;
    }
    float mx = m_run;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) mx = fmaxf(mx, sc[sub][vv]);
    // finite: block 0 holds key 0 <= every query, and later blocks inherit a finite running maximum
    mx = max_halves(mx);
    if (__any(mx > m_run)) {
      const float alpha = __builtin_amdgcn_exp2f((m_run - mx) * scale_log2);
      l_run *= alpha;
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) O[e][vv] *= alpha;
      m_run = mx;
    }
    const float off = -m_run * scale_log2;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sc[sub][vv], scale_log2, off));
        sc[sub][vv] = p;
        l_run += p;
      }
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const u32x4 pf = pack8<false>(sc[sub], 8 * jj);
#pragma unroll
        for (int e = 0; e < NE; ++e) O[e] = mma32(frag_cols<D>(sV, tl, e, sub, jj), pf, O[e]);
      }
  }
  const float l_all = l_run + __shfl_xor(l_run, 32, 64);
  if (qrow < S) {
    const float inv = 1.f / l_all;
    bf* op = o + ((long long)b * S + qrow) * QD + head * D;
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<u32x2*>(op + e * 32 + 8 * g + 4 * h) =
            u32x2{PACK2(O[e][4 * g] * inv, O[e][4 * g + 1] * inv), PACK2(O[e][4 * g + 2] * inv, O[e][4 * g + 3] * inv)};
    if (h == 0) lse2[(long long)z * S + qrow] = fmaf(m_run, scale_log2, log2f(l_all));
  }
}

// -------------------------------------------------------------------------------------------- backward: dQ
// Same grid and ownership as the forward kernel.  dQ^T[e][q] += K^T[e][k] dS^T[k][q].
// Also computes delta[q] = sum_e dO[q][e] O[q][e] and stores it.
template <int D>
__global__ void __launch_bounds__(256, 2) k_attn_bwd_dq(const bf* __restrict__ q, const bf* __restrict__ k, const bf* __restrict__ v,
                                                     const bf* __restrict__ dO, const bf* __restrict__ o,
                                                     const float* __restrict__ lse2, float* __restrict__ delta, bf* __restrict__ dq,
                                                     const float2* __restrict__ rope, int S, int nq, int nkv, float scale,
                                                     float scale_log2, int* flag) {
  constexpr int NJ = D / 16, NE = D / 32, TILE = KB * D * 2;
  extern __shared__ __align__(1024) char smem[];  // two buffers of (K, V)
  const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb = gridDim.y - 1 - blockIdx.y;
  const int z = blockIdx.x, b = z / nq, head = z - b * nq, hk = head / (nq / nkv);
  const int QD = nq * D;
  const unsigned kv_ld = (unsigned)(nkv * D) * 2u;
  const int q0 = qb * 128 + wave * 32, qrow = q0 + l31, qc = min(qrow, S - 1);
  const TileLane<D> tl(lane);
  const auto rsK = rows_rsrc(k + (long long)b * S * nkv * D + hk * D, S, kv_ld, D);
  const auto rsV = rows_rsrc(v + (long long)b * S * nkv * D + hk * D, S, kv_ld, D);
  const int nkb = min(qb * 128 + 127, S - 1) / KB + 1;
  stage_block<D>(rsK, 0, kv_ld, smem, wave, lane);
  stage_block<D>(rsV, 0, kv_ld, smem + TILE, wave, lane);

  u32x4 Qf[NJ], Gf[NJ];  // this lane's query row and its dO row as B operands
  float dl = 0.f;
  {
    const long long ro = ((long long)b * S + qc) * QD + head * D + 8 * h;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      Qf[j] = *reinterpret_cast<const u32x4*>(q + ro + 16 * j);
      Gf[j] = *reinterpret_cast<const u32x4*>(dO + ro + 16 * j);
    }
    // delta = rowsum(dO * O) of this lane's query: the lane holds half of the row's dO (8 of every 16 elements), its
    // partner lane the other half.  Stored for the dK / dV kernel, which runs after this one.
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const u32x4 ov = *reinterpret_cast<const u32x4*>(o + ro + 16 * j);
      float gf[8], of[8];
      UNPACK8(uint4{Gf[j].x, Gf[j].y, Gf[j].z, Gf[j].w}, gf);
      UNPACK8(uint4{ov.x, ov.y, ov.z, ov.w}, of);
#pragma unroll
      for (int e = 0; e < 8; ++e) dl += gf[e] * of[e];
    }
    dl += __shfl_xor(dl, 32, 64);
    if (h == 0 && qrow < S) delta[(long long)z * S + qrow] = dl;
  }
  const float off = -lse2[(long long)z * S + qc];
  f32x16 dQ[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) dQ[e] = zero16f();

  for (int kb = 0; kb < nkb; ++kb) {
    block_ready();
    char* sK = smem + (kb & 1) * (2 * TILE);
    char* sV = sK + TILE;
    if (kb + 1 < nkb) {
      char* nx = smem + ((kb + 1) & 1) * (2 * TILE);
      stage_block<D>(rsK, kb + 1, kv_ld, nx, wave, lane);
      stage_block<D>(rsV, kb + 1, kv_ld, nx + TILE, wave, lane);
    }
    if (kb * KB > q0 + 31) continue;
    const bool diag = kb * KB + KB - 1 > q0;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      f32x16 sc = zero16f(), dp = zero16f();
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        sc = mma32(frag_rows<D>(sK, tl, sub, j), Qf[j], sc);
        dp = mma32(frag_rows<D>(sV, tl, sub, j), Gf[j], dp);
      }
      if (diag) {
#pragma unroll
        for (int vv = 0; vv < 16; ++vv)
          if (kb * KB + sub * 32 + 8 * (vv >> 2) + 4 * h + (vv & 3) > qrow) sc[vv] = -INFINITY;
      }
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) sc[vv] = __builtin_amdgcn_exp2f(fmaf(sc[vv], scale_log2, off)) * (dp[vv] - dl);
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const u32x4 df = pack8<true>(sc, 8 * jj);
#pragma unroll
        for (int e = 0; e < NE; ++e) dQ[e] = mma32(frag_cols<D>(sK, tl, e, sub, jj), df, dQ[e]);
      }
    }
  }
  if (qrow < S) {
    bf* op = dq + ((long long)b * S + qrow) * QD + head * D;
    bool over = false;
#pragma unroll
    for (int e = 0; e < NE / 2; ++e)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int eo = e * 32 + 8 * g + 4 * h;
        float lo[4], hi[4];
        unrotate4(dQ[e], dQ[e + NE / 2], g, rope + (long long)qrow * (D / 2) + eo, scale, lo, hi);
        *reinterpret_cast<u32x2*>(op + eo) = u32x2{PACK2G(lo[0], lo[1], over), PACK2G(lo[2], lo[3], over)};
        *reinterpret_cast<u32x2*>(op + eo + D / 2) = u32x2{PACK2G(hi[0], hi[1], over), PACK2G(hi[2], hi[3], over)};
      }
    elem_flag(over, flag);
  }
}

// -------------------------------------------------------------------------------------------- backward: dK, dV
// Same grid; a workgroup owns 128 keys as seen by one QUERY head, wave w the keys 32w..32w+31, and
// streams the queries from its first key to the end of the sequence.
//   dV^T[e][k] += dO^T[e][q] P[q][k],   dK^T[e][k] += Q^T[e][q] dS[q][k]
template <int D>
__global__ void __launch_bounds__(256, 2) k_attn_bwd_dkv(const bf* __restrict__ q, const bf* __restrict__ k, const bf* __restrict__ v,
                                                      const bf* __restrict__ dO, const float* __restrict__ lse2,
                                                      const float* __restrict__ delta, bf* __restrict__ dkq,
                                                      bf* __restrict__ dvq, const float2* __restrict__ rope, int S, int nq,
                                                      int nkv, float scale, float scale_log2, int* flag) {
  constexpr int NJ = D / 16, NE = D / 32, TILE = KB * D * 2;
  constexpr int BUF = 2 * TILE + 2 * KB * 4;  // Q, dO, then lse2 and delta of the block's queries
  extern __shared__ __align__(1024) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kvb = blockIdx.y;  // block 0 has the longest span of queries
  const int z = blockIdx.x, b = z / nq, head = z - b * nq, hk = head / (nq / nkv);
  const int QD = nq * D, KVD = nkv * D;
  const unsigned q_ld = (unsigned)QD * 2u;
  const int k0 = kvb * 128 + wave * 32, krow = k0 + l31, kc_ = min(krow, S - 1);
  const TileLane<D> tl(lane);
  const auto rsQ = rows_rsrc(q + (long long)b * S * QD + head * D, S, q_ld, D);
  const auto rsG = rows_rsrc(dO + (long long)b * S * QD + head * D, S, q_ld, D);
  const auto rsL = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>((wave & 1 ? delta : lse2) + (long long)z * S), 0, S * 4, 0x00020000);
  const int qb0 = kvb * 128 / KB, nqb = (S + KB - 1) / KB;
#define KV_STAGE(qb_)                                                                                                     \
  do {                                                                                                                    \
    char* nx_ = smem + ((qb_) & 1) * BUF;                                                                                 \
    stage_block<D>(rsQ, qb_, q_ld, nx_, wave, lane);                                                                      \
    stage_block<D>(rsG, qb_, q_ld, nx_ + TILE, wave, lane);                                                               \
    if (wave < 2)                                                                                                         \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsL, LDS_PTR(void, nx_ + 2 * TILE + wave * (KB * 4)), 4, ((qb_) * KB + lane) * 4, 0, 0, 0); \
  } while (0)
  KV_STAGE(qb0);

  u32x4 Kf[NJ], Vf[NJ];  // this lane's key and value rows as B operands
  {
    const long long ro = ((long long)b * S + kc_) * KVD + hk * D + 8 * h;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      Kf[j] = *reinterpret_cast<const u32x4*>(k + ro + 16 * j);
      Vf[j] = *reinterpret_cast<const u32x4*>(v + ro + 16 * j);
    }
  }
  f32x16 dV[NE], dK[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) dV[e] = zero16f(), dK[e] = zero16f();

  for (int qb = qb0; qb < nqb; ++qb) {
    block_ready();
    char* sQ = smem + (qb & 1) * BUF;
    char* sG = sQ + TILE;
    const float* sL = reinterpret_cast<const float*>(sQ + 2 * TILE);
    if (qb + 1 < nqb) KV_STAGE(qb + 1);
    if (qb * KB + KB - 1 < k0) continue;  // every query of the block precedes this wave's keys
    const bool diag = qb * KB < k0 + 31;
#pragma unroll 1
    for (int sub = 0; sub < 2; ++sub) {
      f32x16 sc = zero16f(), dp = zero16f();
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        sc = mma32(frag_rows<D>(sQ, tl, sub, j), Kf[j], sc);
        dp = mma32(frag_rows<D>(sG, tl, sub, j), Vf[j], dp);
      }
      // rows of the accumulator are queries: their lse and delta come in runs of four.  Queries past the sequence have
      // zero rows in Q and dO (lse and delta zero as well), so whatever p is there adds nothing.
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 l4 = *reinterpret_cast<const float4*>(sL + sub * 32 + 8 * g + 4 * h);
        const float4 d4 = *reinterpret_cast<const float4*>(sL + KB + sub * 32 + 8 * g + 4 * h);
        const float ls[4] = {l4.x, l4.y, l4.z, l4.w}, ds[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int vv = 4 * g + c;
          float p = __builtin_amdgcn_exp2f(fmaf(sc[vv], scale_log2, -ls[c]));
          if (diag && qb * KB + sub * 32 + 8 * g + 4 * h + c < krow) p = 0.f;
          sc[vv] = p;
          dp[vv] = p * (dp[vv] - ds[c]);
        }
      }
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const u32x4 pf = pack8<false>(sc, 8 * jj), df = pack8<true>(dp, 8 * jj);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          dV[e] = mma32(frag_cols<D>(sG, tl, e, sub, jj), pf, dV[e]);
          dK[e] = mma32(frag_cols<D>(sQ, tl, e, sub, jj), df, dK[e]);
        }
      }
    }
  }
#undef KV_STAGE
  if (krow < S) {
    const long long ro = ((long long)b * S + krow) * QD + head * D;
    bool over = false;
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int eo = e * 32 + 8 * g + 4 * h;
        *reinterpret_cast<u32x2*>(dvq + ro + eo) =
            u32x2{PACK2G(dV[e][4 * g], dV[e][4 * g + 1], over), PACK2G(dV[e][4 * g + 2], dV[e][4 * g + 3], over)};
      }
#pragma unroll
    for (int e = 0; e < NE / 2; ++e)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int eo = e * 32 + 8 * g + 4 * h;
        float lo[4], hi[4];
        unrotate4(dK[e], dK[e + NE / 2], g, rope + (long long)krow * (D / 2) + eo, scale, lo, hi);
        *reinterpret_cast<u32x2*>(dkq + ro + eo) = u32x2{PACK2G(lo[0], lo[1], over), PACK2G(lo[2], lo[3], over)};
        *reinterpret_cast<u32x2*>(dkq + ro + eo + D / 2) = u32x2{PACK2G(hi[0], hi[1], over), PACK2G(hi[2], hi[3], over)};
      }
    elem_flag(over, flag);
  }
}

template <int D>
constexpr int fwd_lds() { return 4 * KB * D * 2; }
template <int D>
constexpr int dkv_lds() { return 2 * (2 * KB * D * 2 + 2 * KB * 4); }

template <int D>
harli_status set_attrs() {
  static bool done = false;
  if (done) return HARLI_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_fwd<D>), hipFuncAttributeMaxDynamicSharedMemorySize, fwd_lds<D>()) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_bwd_dq<D>), hipFuncAttributeMaxDynamicSharedMemorySize, fwd_lds<D>()) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_bwd_dkv<D>), hipFuncAttributeMaxDynamicSharedMemorySize, dkv_lds<D>()) != hipSuccess)
    return fail(HARLI_ERR_HIP, "attention: could not raise the dynamic LDS limit");
  done = true;
  return HARLI_OK;
}

harli_status check_shape(int Bf, int S, int nq, int nkv, int d) {
  if (!ft_attn_supported(d)) return fail(HARLI_ERR_INVALID, "attention: head_dim %d is not 64 or 128", d);
  // the kernels address a sequence's rows with 32-bit byte offsets below 2^31
  if ((long long)(S + 64) * nq * d * 2 >= (1ll << 31)) return fail(HARLI_ERR_INVALID, "attention: a sequence of %d tokens is 2 GiB or more", S);
  if (Bf < 1 || S < 8 || (S & 7) || nq < 1 || nkv < 1 || nq % nkv) return fail(HARLI_ERR_INVALID, "attention: bad shape");
  return HARLI_OK;
}

}  // namespace

harli_status ft_attn_fwd(const bf* q, const bf* k, const bf* v, bf* o, float* lse2, int Bf, int S, int n_q, int n_kv, int d,
                         hipStream_t st) {
  harli_status s = check_shape(Bf, S, n_q, n_kv, d);
  if (s != HARLI_OK) return s;
  const dim3 grid(Bf * n_q, (S + 127) / 128), blk(256);
  const float sl2 = kLog2e / sqrtf((float)d);
  if (d == 128) {
    if ((s = set_attrs<128>()) != HARLI_OK) return s;
    hipLaunchKernelGGL(k_attn_fwd<128>, grid, blk, fwd_lds<128>(), st, q, k, v, o, lse2, S, n_q, n_kv, sl2);
  } else {
    if ((s = set_attrs<64>()) != HARLI_OK) return s;
    hipLaunchKernelGGL(k_attn_fwd<64>, grid, blk, fwd_lds<64>(), st, q, k, v, o, lse2, S, n_q, n_kv, sl2);
  }
  return HARLI_OK;
}

harli_status ft_attn_bwd(const bf* q, const bf* k, const bf* v, const bf* o, const bf* dO, const float* lse2, float* delta,
                         bf* dq, bf* dkq, bf* dvq, const float2* rope, int Bf, int S, int n_q,
                         int n_kv, int d, int* flag, hipStream_t st) {
  harli_status s = check_shape(Bf, S, n_q, n_kv, d);
  if (s != HARLI_OK) return s;
  const dim3 grid(Bf * n_q, (S + 127) / 128), blk(256);
  const float sc = 1.f / sqrtf((float)d), sl2 = kLog2e * sc;
  if (d == 128) {
    if ((s = set_attrs<128>()) != HARLI_OK) return s;
    hipLaunchKernelGGL(k_attn_bwd_dq<128>, grid, blk, fwd_lds<128>(), st, q, k, v, dO, o, lse2, delta, dq, rope, S, n_q, n_kv, sc, sl2, flag);
    hipLaunchKernelGGL(k_attn_bwd_dkv<128>, grid, blk, dkv_lds<128>(), st, q, k, v, dO, lse2, delta, dkq, dvq, rope, S, n_q,
                       n_kv, sc, sl2, flag);
  } else {
    if ((s = set_attrs<64>()) != HARLI_OK) return s;
    hipLaunchKernelGGL(k_attn_bwd_dq<64>, grid, blk, fwd_lds<64>(), st, q, k, v, dO, o, lse2, delta, dq, rope, S, n_q, n_kv, sc, sl2, flag);
    hipLaunchKernelGGL(k_attn_bwd_dkv<64>, grid, blk, dkv_lds<64>(), st, q, k, v, dO, lse2, delta, dkq, dvq, rope, S, n_q,
                       n_kv, sc, sl2, flag);
  }
  return HARLI_OK;
}

}  // namespace harli
