// Weight GEMM of the finetune unit (see gemm2.h for the operand layouts).
//
// Workgroup tile (64 FM) x 256, K step 32, FOUR waves -- one per SIMD, each with the whole register file: a wave owns
// a (32 FM) x 128 block of the tile = 2 FM x 8 accumulators of v_mfma_f32_16x16x32 (256 accumulator registers at FM = 4).
// What this shape buys on gfx950, measured:
//   * operand bytes per flop through L2 and through LDS fall with the tile edge: a CU pulls no more than ~22-41 B/clk
//     from L2 and LDS serves 128 B/clk, and 64 x 64 wave tiles (two waves per SIMD) need all of the latter at the full
//     MFMA rate.  128 x 128 per wave needs half;
//   * operands go from global memory straight into LDS (buffer_load ... lds, 16 B per lane, no register staging); the
//     rows of a stage are XOR-swizzled in 16-byte chunks on the way in (each lane picks the global chunk that belongs
//     in its LDS slot), which makes the 16-row fragment reads conflict free;
//   * four LDS stages, three of them in flight: the fragments of a stage are read during the stage before, so a stage's
//     buffer is free again as soon as its products begin;
//   * one wave per SIMD has nobody to hide its waits, so reads and loads are dealt out between the products by hand;
//   * nothing but the loads' scalar offsets moves from stage to stage: every branch and mask of the cursor (end of a
//     segment, of the range, a partial K step) is behind one comparison that is false on whole stages.
// What bounds it: power.  On random operands the chip holds 1.6-1.7 GHz under this loop (2.4 on zeros, and with the loads
// bunched together the clock rises as the cycles do), so energy per product counts: v_mfma_f32_16x16x32 draws less than
// 32x32x16 and the loop takes 1105-1160 cycles a 256-row stage (1024 of them product issue; 32x32x16: 1180).  A workgroup
// spends another 3-5 us before its first product and 4 (16-bit) or 8-11 us (fp32) on its store.  Alone, 4096 x 16384 x 4096:
// 484 us with 32x32x16 products and a store through LDS, 403 now (1365 TFLOP/s; the vendor's library 368); fp32 output with
// a residual 606 -> 545; one round, 2048 x 8192 x 8192: 190 (1450 TFLOP/s; 183).
// FM = 2 (128-row tiles) doubles the tile count for outputs that would not fill the chip with 256-row tiles.
#include "gemm2.h"

#include <algorithm>
#include <type_traits>

#include "ctx.h"
#include "device_utils.h"

namespace harli {
namespace {

constexpr int BN = kG2TileN, BK = kG2StepK, NT = 256;
// LDS stages: four (128 KiB at 256-row tiles).  Six stages at 128-row tiles (144 KiB) were measured and changed nothing:
// those tiles are not short of loads in flight.
template <int FM>
constexpr int stages() { return 4; }
constexpr int BSZ = BN * BK * 2;  // 16 KiB: one stage of the weight-side tile

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define G2_WAITV(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
#define G2_SB0() __builtin_amdgcn_sched_barrier(0)

// ---- products and accumulators -----------------------------------------------------------------------------------------
// A wave owns FM x 2 by 8 accumulators of v_mfma_f32_16x16x32, in accumulator registers NAMED BY HAND: accumulator t = 8 i + j
// is a[4t .. 4t+3].  The compiler's allocator copied more than half of 64 four-register accumulators between the register
// files in every pass of the stage ring; named, none moves, and the code between two products is exactly what stands there.
// The kernel claims the whole range in its first statement and nothing else in it uses accumulator registers (the compiler
// would only to spill, and it has 256 other registers for about 150 values): tests/test_gemm2_isa.py reads that off the
// built library.  Hazards the compiler does not fill in for assembly: the products of one accumulator are 16 FM products
// apart, its first use lies a barrier behind the zeros and the reads of the epilogue behind the idle cycles of g2_drain().
// The weight fragment is the FIRST operand: a lane then holds four neighbouring columns 16 j + 4 (lane / 16) + v of row
// 16 i + lane % 16, and the epilogue stores from registers.
template <bool HALF, int T>
__device__ __forceinline__ void g2_mm(u32x4 b, u32x4 a) {
  if (HALF)
    asm volatile("v_mfma_f32_16x16x32_f16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(b), "v"(a), "n"(4 * T), "n"(4 * T + 3));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(b), "v"(a), "n"(4 * T), "n"(4 * T + 3));
}
template <int R>
__device__ __forceinline__ float g2_acc() {
  float r;
  asm volatile("v_accvgpr_read_b32 %0, a%c1" : "=v"(r) : "n"(R));
  return r;
}
template <int FM>
__device__ __forceinline__ void g2_claim() {
#define G2_R10(p) p "0", p "1", p "2", p "3", p "4", p "5", p "6", p "7", p "8", p "9"
#define G2_R128                                                                                                        \
  G2_R10("a"), G2_R10("a1"), G2_R10("a2"), G2_R10("a3"), G2_R10("a4"), G2_R10("a5"), G2_R10("a6"), G2_R10("a7"),       \
      G2_R10("a8"), G2_R10("a9"), G2_R10("a10"), G2_R10("a11"), "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127"
  if (FM == 4)
    asm volatile("" ::: G2_R128, "a128", "a129", G2_R10("a13"), G2_R10("a14"), G2_R10("a15"), G2_R10("a16"), G2_R10("a17"),
                 G2_R10("a18"), G2_R10("a19"), G2_R10("a20"), G2_R10("a21"), G2_R10("a22"), G2_R10("a23"), G2_R10("a24"), "a250",
                 "a251", "a252", "a253", "a254", "a255");
  else
    asm volatile("" ::: G2_R128);
#undef G2_R128
#undef G2_R10
}
// calls f(0), f(1), .., f(N - 1) with compile-time numbers
template <int N, int Q = 0, typename F>
__device__ __forceinline__ void g2_steps(F&& f) {
  if constexpr (Q < N) {
    f(std::integral_constant<int, Q>{});
    g2_steps<N, Q + 1>(f);
  }
}
// the last product's result may be read 18 cycles later (8 passes and the way out of the pipeline)
__device__ __forceinline__ void g2_drain() { asm volatile("s_nop 15\n\ts_nop 15"); }

// ---- epilogue: a slab of 16 rows x 128 columns, as the accumulators hold it -----------------------------------------------
// x[j] of a lane: columns 16 j + 4 (lane / 16) .. + 3 of row lane % 16.  fp32 outputs are stored like that (16 rows x 64
// bytes per instruction).  For 16-bit outputs neighbouring accumulators trade rows of 16 lanes (v_permlane16_swap), after
// which a lane holds EIGHT neighbouring columns of a pair of accumulators p -- 32 p + 16 (g & 1) + 8 (g >> 1), g = lane / 16
// -- and everything an epilogue combines (gate and up, the two halves of a rotary pair) lies in the same lane.  No LDS, no
// barrier: the store of a 256 x 256 tile takes 4.1 us with 16-bit and 8 to 11 with fp32 outputs (11 and 22 through LDS).
struct G2Pre {
  u32x4 v[8];  // what the epilogue of a slab reads: residual, or stored a and u
};

// (rows past M and columns past N read some valid element instead: loads without a condition stay in flight together)
template <int EPI>
__device__ __forceinline__ void g2_epi_load(G2Pre& e, const Gemm2Args& a, const Gemm2Out& out, int tn, int wn, int lane, int m) {
  const int mc = min(m, a.M - 1), g = lane >> 4, n0 = (tn - out.tile0) * BN + wn * 128;
  if (EPI == GEMM2_EPI_SWIGLU_BWD) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int n = n0 + p * 32 + (g & 1) * 16 + (g >> 1) * 8, nc = n < out.N ? n : 0;
      e.v[2 * p] = *reinterpret_cast<const u32x4*>(a.e0 + (long long)mc * a.lde + nc);
      e.v[2 * p + 1] = *reinterpret_cast<const u32x4*>(a.e1 + (long long)mc * a.lde + nc);
    }
  } else if (EPI == GEMM2_EPI_F32) {
    if (out.res)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int n = n0 + j * 16 + g * 4, nc = n + 3 < out.N ? n : 0;
        e.v[j] = out.N > 3 ? *reinterpret_cast<const u32x4*>(out.res + (long long)mc * out.ldcf + nc) : u32x4{0, 0, 0, 0};
      }
  }
}

template <bool HALF, int EPI>
__device__ __forceinline__ void g2_epi_store(f32x4 (&x)[8], const G2Pre& e, const Gemm2Args& a, const Gemm2Out& out, int tn, int wn,
                                             int lane, int m, bool& clamped) {
  const int g = lane >> 4;
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] *= a.alpha;
  if (EPI == GEMM2_EPI_F32) {
    const int n0 = (tn - out.tile0) * BN + wn * 128 + g * 4;
    if (m >= a.M) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int n = n0 + j * 16;
      if (n + 3 < out.N) {
        f32x4 o = x[j];
        if (out.res) o += __builtin_bit_cast(f32x4, e.v[j]);
        *reinterpret_cast<f32x4*>(out.Cf + (long long)m * out.ldcf + n) = o;
        if (out.Cb) {
          if (HALF)
#pragma unroll
            for (int v = 0; v < 4; ++v) clamped = clamped || !(fabsf(o[v]) <= 65504.f);
          *reinterpret_cast<uint2*>(out.Cb + (long long)m * out.ldcb + n) =
              HALF ? make_uint2(pack_h2(o[0], o[1]), pack_h2(o[2], o[3])) : make_uint2(pack_bf2(o[0], o[1]), pack_bf2(o[2], o[3]));
        }
      } else {  // the last columns of a matrix whose width is not a multiple of four
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (n + v < out.N) {
            float o = x[j][v];
            if (out.res) o += out.res[(long long)m * out.ldcf + n + v];
            out.Cf[(long long)m * out.ldcf + n + v] = o;
            if (out.Cb) out.Cb[(long long)m * out.ldcb + n + v] = HALF ? f2h(o) : f2bf(o);
          }
      }
    }
    return;
  }
  // 16-bit outputs: y[p][0..7] = eight columns
  float y[4][8];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[2 * p][v]), __float_as_uint(x[2 * p + 1][v]), false, false);
      y[p][v] = __uint_as_float(t[0]);
      y[p][4 + v] = __uint_as_float(t[1]);
    }
  if (m >= a.M) return;
  const int c0 = (g & 1) * 16 + (g >> 1) * 8;
  auto pack8 = [&](const float* v) {
    if (HALF) {
#pragma unroll
      for (int k = 0; k < 8; ++k) clamped = clamped || !(fabsf(v[k]) <= 65504.f);
      return make_uint4(pack_h2(v[0], v[1]), pack_h2(v[2], v[3]), pack_h2(v[4], v[5]), pack_h2(v[6], v[7]));
    }
    return make_uint4(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7]));
  };
  auto unpack = [](const uint4& wv, float* v) {
    if (HALF) unpack8h(wv, v);
    else unpack8(wv, v);
  };
  if (EPI == GEMM2_EPI_GATEUP) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // pairs 0, 2: gate; 1, 3: up of the same 32 output columns
      const int n = (tn - out.tile0) * 128 + wn * 64 + h * 32 + c0;
      if (n >= out.N) continue;
      const uint4 gp = pack8(y[2 * h]), up = pack8(y[2 * h + 1]);
      float av[8], uv[8], mv[8];
      unpack(gp, av);  // the rounded values, as the backward pass will read them
      unpack(up, uv);
#pragma unroll
      for (int k = 0; k < 8; ++k) mv[k] = av[k] / (1.f + __expf(-av[k])) * uv[k];
      *reinterpret_cast<uint4*>(out.Cb + (long long)m * out.ldcb + n) = gp;
      *reinterpret_cast<uint4*>(a.o1 + (long long)m * a.lde + n) = up;
      *reinterpret_cast<uint4*>(a.o0 + (long long)m * a.lde + n) = pack8(mv);
    }
    return;
  }
  const int n0 = (tn - out.tile0) * BN + wn * 128 + c0;
  if (EPI == GEMM2_EPI_ROPE && tn < a.rope_tiles) {
    // a wave's 128 columns hold whole heads: (lo, hi) -> (lo cos - hi sin, hi cos + lo sin), hi half a head further right
    const int half = a.rope_d >> 1;
    const float4* cs = reinterpret_cast<const float4*>(a.rope + (size_t)(m % a.rope_S) * half);
    auto rotate = [&](float* lo, float* hi, int idx) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 t = cs[(idx >> 1) + k];
        const float l0 = lo[2 * k], l1 = lo[2 * k + 1], h0 = hi[2 * k], h1 = hi[2 * k + 1];
        lo[2 * k] = l0 * t.x - h0 * t.y, hi[2 * k] = h0 * t.x + l0 * t.y;
        lo[2 * k + 1] = l1 * t.z - h1 * t.w, hi[2 * k + 1] = h1 * t.z + l1 * t.w;
      }
    };
    if (half == 64) rotate(y[0], y[2], c0), rotate(y[1], y[3], 32 + c0);
    else rotate(y[0], y[1], c0), rotate(y[2], y[3], c0);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int n = n0 + p * 32;
    if (n >= out.N) continue;
    if (EPI == GEMM2_EPI_SWIGLU_BWD) {
      float av[8], uv[8], oa[8], ou[8];
      unpack(__builtin_bit_cast(uint4, e.v[2 * p]), av);
      unpack(__builtin_bit_cast(uint4, e.v[2 * p + 1]), uv);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float sg = 1.f / (1.f + __expf(-av[k]));
        oa[k] = y[p][k] * uv[k] * sg * (1.f + av[k] * (1.f - sg));
        ou[k] = y[p][k] * av[k] * sg;
      }
      *reinterpret_cast<uint4*>(a.o0 + (long long)m * a.lde + n) = pack8(oa);
      *reinterpret_cast<uint4*>(a.o1 + (long long)m * a.lde + n) = pack8(ou);
    } else {
      *reinterpret_cast<uint4*>(out.Cb + (long long)m * out.ldcb + n) = pack8(y[p]);
    }
  }
}

// Output block of column tile tn.
__device__ __forceinline__ Gemm2Out g2_out_of(const Gemm2Args& a, int tn) {
  Gemm2Out out = a.out[0];
  if (a.nout > 1 && tn >= a.out[1].tile0) out = a.out[1];
  if (a.nout > 2 && tn >= a.out[2].tile0) out = a.out[2];
  return out;
}

// Tile t of a cut launch: bands of GM row tiles, column by column inside a band, so that consecutive tiles of an XCD's
// share form compact blocks.
__device__ __forceinline__ void g2_cut_tile(const Gemm2Cut& c, int t, int& tm, int& tn) {
  const int band = t / (c.GM * c.tiles_n), rem = t - band * (c.GM * c.tiles_n), rows = min(c.GM, c.tiles_m - band * c.GM);
  tn = rem / rows;
  tm = band * c.GM + rem - tn * rows;
}

template <int FM, bool HALF, int EPI>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_gemm2(Gemm2Args a, Gemm2Cut cut, int tiles_total, int chunk, int GM, int GN, const uint4* zero16) {
  constexpr int BM = 64 * FM, ASZ = BM * BK * 2, STG = ASZ + BSZ, NS = stages<FM>();
  constexpr int LOADS = FM + 4;  // direct-to-LDS loads a wave issues per stage
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  g2_claim<FM>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;  // 2 x 2 waves of (32 FM) x 128
  const int w = blockIdx.x;
  int tm, tn, piece = -1, split = 0;  // piece: index of this workgroup's partial tile, -1 for a whole tile
  if (cut.ks > 1) {
    // cut launch (see gemm2_cut): whole tiles first, then the remaining tiles in ranges of K, range by range; either
    // list is dealt out in eight contiguous shares, one per XCD
    int slot = (w & 7) * cut.chunk_full + (w >> 3);
    if (w < 8 * cut.chunk_full) {
      if (slot >= cut.full) return;
    } else {
      const int w2 = w - 8 * cut.chunk_full;
      piece = (w2 & 7) * cut.chunk_cut + (w2 >> 3);
      if (piece >= cut.rest * cut.ks) return;
      split = piece / cut.rest;
      slot = cut.first + piece - split * cut.rest;
    }
    g2_cut_tile(cut, slot, tm, tn);
  } else {
    // XCD-aware tile order (workgroup w runs on XCD w % 8): every XCD walks blocks of GM x GN tiles, so the workgroups
    // that share an L2 share operand panels.
    const int slot = (w & 7) * chunk + (w >> 3);
    if (slot >= tiles_total) return;
    const int nbn = (a.tiles_n + GN - 1) / GN;
    const int blk = slot / (GM * GN), within = slot - blk * (GM * GN);
    const int bm = blk / nbn, bn = blk - bm * nbn;
    tm = bm * GM + within / GN, tn = bn * GN + within % GN;
  }
  const int m0 = tm * BM;
  if (m0 >= a.M || tn >= a.tiles_n) return;

  // ---- stage bookkeeping (uniform): the segments that cover this tile, 32 k at a time -------------------------------
  int n_stage = 0;
  for (int s = 0; s < a.nseg; ++s)
    if (tn >= a.seg[s].tile0 && tn < a.seg[s].tile1) n_stage += (a.seg[s].K + BK - 1) / BK;
  int skip = 0;  // stages of this tile that belong to earlier ranges of K
  if (piece >= 0) {
    skip = n_stage * split / cut.ks;
    n_stage = n_stage * (split + 1) / cut.ks - skip;
  }

  // Loads: instruction j of a wave fills 16 rows of a stage; lane -> row lane/4, LDS slot lane%4, which receives the
  // global chunk slot ^ ((row/2)%4).  They are buffer loads (buffer_load_dwordx4 ... lds): the operand is described by
  // a resource in scalar registers, a lane contributes a 32-bit byte offset that stays the same for a whole segment,
  // and the walk along K is one scalar offset per load -- no per-lane 64-bit address arithmetic in the loop, and an
  // instruction that the wave issues faster than a global load with 64-bit addresses (measured: +8-11 % on the whole
  // kernel with nothing else changed).  What must read as zero is out of the resource's range, which the hardware
  // answers with zeros: rows past M lie behind num_records = M * lda, and lanes whose k is past the segment, stages
  // past the end and the absent half of a pair get the offset kOut (>= any num_records; the scalar offsets stay
  // below 2^31, so the sum cannot wrap back into range).
  const int drow = lane >> 2, dchunk = (lane & 3) ^ ((lane >> 3) & 3);
  constexpr unsigned kOut = 0x80000000u;
  constexpr int kRsrcFlags = 0x00020000;  // raw buffer of dwords
  const unsigned voffB = (unsigned)(drow * BK + dchunk * 8) * 2u;  // a lane's place inside a 16-row group of the weight side
  unsigned voffA[FM];                                             // and inside the activation operand: (row, chunk)
  __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(zero16), 0, 0, kRsrcFlags), rsB = rsA, rsB2 = rsA;
  unsigned soffA = 0, soffB[4] = {0u, 0u, 0u, 0u};
  bool pairseg = false;
  int seg = -1, k0 = 0, Kseg = 0, issued = 0;
  int k_last = 0;           // last k0 of this segment whose stage is a whole one of this tile
  unsigned vA[FM], vB = 0;  // the offsets the loads use: voffA, voffB or kOut

  // (macros rather than lambdas: arrays captured by reference were left in scratch memory by the compiler)
#define G2_OPEN_SEG()                                                                                                  \
  do {                                                                                                                 \
    for (++seg; seg < a.nseg; ++seg)                                                                                   \
      if (tn >= a.seg[seg].tile0 && tn < a.seg[seg].tile1 && a.seg[seg].K > 0) break;                                 \
    if (seg < a.nseg) {                                                                                                \
      const Gemm2Seg& sg = a.seg[seg];                                                                                 \
      Kseg = sg.K;                                                                                                     \
      k0 = 0;                                                                                                          \
      const unsigned ks_n = (unsigned)((sg.K + BK - 1) / BK);                                                          \
      const unsigned lda2 = (unsigned)sg.lda * 2u;                                                                     \
      rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(sg.A), 0, (int)((unsigned)a.M * lda2), kRsrcFlags); \
      soffA = 0;                                                                                                       \
      _Pragma("unroll") for (int j = 0; j < FM; ++j)                                                                   \
        voffA[j] = (unsigned)(m0 + (wave * FM + j) * 16 + drow) * lda2 + (unsigned)dchunk * 16u;                       \
      pairseg = sg.pair != 0;                                                                                          \
      const int bbytes = (int)((unsigned)((sg.rows + BN - 1) / BN) * ks_n * (unsigned)(BN * BK * 2));                  \
      rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(sg.B ? sg.B : sg.A), 0, sg.B ? bbytes : 0, kRsrcFlags);   \
      /* groups 2, 3 of a wave: the second matrix of a pair, else the same operand */                                  \
      {                                                                                                                \
        const unsigned short* b2 = pairseg ? sg.B2 : sg.B;                                                             \
        rsB2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(b2 ? b2 : sg.A), 0, b2 ? bbytes : 0, kRsrcFlags); \
      }                                                                                                                \
      _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                                  \
        const int g16 = wave * 4 + j; /* 16-row group of the tile's weight side */                                     \
        /* row of the operand this group starts at; in a pair, groups with g16 & 2 (that is, j & 2) come from B2 */    \
        const unsigned brow = pairseg ? 128u * (unsigned)(tn - sg.tile0) + 32u * (unsigned)(g16 >> 2) + 16u * (unsigned)(g16 & 1) \
                                      : 256u * (unsigned)(tn - sg.tile0) + 16u * (unsigned)g16;                        \
        soffB[j] = ((brow >> 8) * ks_n * (unsigned)BN + (brow & 255u)) * (unsigned)(BK * 2);                           \
      }                                                                                                                \
    }                                                                                                                  \
  } while (0)
  // the stage at the cursor is not simply the next 32 k of its segment: past the range, past the segment, or its tail
#define G2_TURN()                                                                                                     \
  do {                                                                                                                \
    if (issued >= n_stage) {                                                                                          \
      _Pragma("unroll") for (int j = 0; j < FM; ++j) vA[j] = kOut;                                                    \
      vB = kOut;                                                                                                      \
      soffA = soffB[0] = soffB[1] = soffB[2] = soffB[3] = 0;                                                          \
      k_last = 0x7fffffff;                                                                                            \
    } else {                                                                                                          \
      if (k0 >= Kseg) G2_OPEN_SEG();                                                                                  \
      const bool whole = Kseg - k0 >= BK;                                                                             \
      _Pragma("unroll") for (int j = 0; j < FM; ++j) vA[j] = whole || k0 + dchunk * 8 < Kseg ? voffA[j] : kOut;       \
      vB = voffB;                                                                                                     \
      k_last = whole ? min(k0 + (n_stage - issued - 1) * BK, Kseg / BK * BK - BK) : k0;                               \
    }                                                                                                                 \
  } while (0)
  // moves the cursor to the next stage; G2_TURN follows when it ends up past k_last
#define G2_NEXT()                                                                                                     \
  do {                                                                                                                \
    ++issued;                                                                                                         \
    k0 += BK;                                                                                                         \
    soffA += BK * 2;                                                                                                  \
    _Pragma("unroll") for (int j = 0; j < 4; ++j) soffB[j] += BN * BK * 2;                                            \
  } while (0)
#define G2_BL(rs, voff, soff, sp)                                                                                     \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(sp), 16, (int)(voff), (int)(soff), 0, 0)
#define G2_LDA(buf, j) G2_BL(rsA, vA[j], soffA, smem + (buf) * STG + (wave * FM + (j)) * 1024)
#define G2_LDB(buf, j) G2_BL((j) < 2 ? rsB : rsB2, vB, soffB[j], smem + (buf) * STG + ASZ + (wave * 4 + (j)) * 1024)

  // fragment reads: row lane%16, 16-byte chunk lane/16, swizzled like the loads
  const int fo = (lane & 15) * 64 + ((lane >> 4) ^ ((lane >> 1) & 3)) * 16;
  const int aoff = wm * (FM * 32) * 64 + fo, boff = ASZ + wn * 128 * 64 + fo;
  u32x4 fa[2][2 * FM], fb[2][8];
#define G2_RDA(p, buf, i) fa[p][i] = *reinterpret_cast<const u32x4*>(smem + (buf) * STG + aoff + (i) * 1024)
#define G2_RDB(p, buf, j) fb[p][j] = *reinterpret_cast<const u32x4*>(smem + (buf) * STG + boff + (j) * 1024)
  // One stage: 16 FM products from fragments p.  Behind the first kBar of them every wave has all its fragments of this
  // stage in registers and its share of the next stage has landed, so the barrier there opens the next stage's buffer for
  // reading and this one's for the stage four ahead; the fragment reads and the loads are dealt out between the other
  // products.  Rows of products alternate their direction, so that one operand stays from each product to the next.
  constexpr int kBar = 3, kRdStep = FM == 4 ? 3 : 2, kLdStep = FM == 4 ? 6 : 4, kRd0 = kBar + 1, kLd0 = kBar + 2;
  static_assert(kRd0 + (2 * FM + 8 - 1) * kRdStep < 16 * FM && kLd0 + (LOADS - 1) * kLdStep < 16 * FM, "a stage must hold its reads and loads");
#define G2_STEP(cur, p)                                                                                               \
  do {                                                                                                                \
    g2_steps<16 * FM>([&](auto q_) __attribute__((always_inline)) {                                                   \
      constexpr int q = decltype(q_)::value, i = q >> 3, j = i & 1 ? 7 - (q & 7) : q & 7;                             \
      g2_mm<HALF, i * 8 + j>(fb[p][j], fa[p][i]);                                                                     \
      if constexpr (q == kBar) {                                                                                      \
        G2_SB0();                                                                                                     \
        __builtin_amdgcn_s_waitcnt(0x0070 | ((2 * LOADS) & 15) | (((2 * LOADS) >> 4) << 14)); /* vmcnt, lgkmcnt 0 */  \
        __builtin_amdgcn_s_barrier();                                                                                 \
        G2_SB0();                                                                                                     \
      }                                                                                                               \
      if constexpr (q >= kRd0 && (q - kRd0) % kRdStep == 0 && (q - kRd0) / kRdStep < 2 * FM + 8) {                    \
        constexpr int r = (q - kRd0) / kRdStep;                                                                       \
        if constexpr (r < 8) G2_RDB((p) ^ 1, ((cur) + 1) % NS, r);                                                    \
        else G2_RDA((p) ^ 1, ((cur) + 1) % NS, r - 8);                                                                \
        G2_SB0();                                                                                                     \
      }                                                                                                               \
      if constexpr (q >= kLd0 && (q - kLd0) % kLdStep == 0 && (q - kLd0) / kLdStep < LOADS) {                         \
        constexpr int r = (q - kLd0) / kLdStep;                                                                       \
        if constexpr (r < FM) G2_LDA(cur, r);                                                                         \
        else G2_LDB(cur, r - FM);                                                                                     \
        G2_SB0();                                                                                                     \
      }                                                                                                               \
    });                                                                                                               \
    G2_NEXT();                                                                                                        \
    if (k0 > k_last) G2_TURN();                                                                                       \
    G2_SB0();                                                                                                         \
  } while (0)

  const bool probe = a.clk != nullptr && blockIdx.x == 0;
  long long c_start = 0, w_start = 0;
  if (probe) c_start = clock64(), w_start = wall_clock64();
  if (n_stage > 0) {
    G2_OPEN_SEG();
    if (skip > 0) {
      while (skip * BK >= Kseg) {
        skip -= (Kseg + BK - 1) / BK;
        G2_OPEN_SEG();
      }
      k0 = skip * BK;
      soffA += (unsigned)k0 * 2u;
#pragma unroll
      for (int j = 0; j < 4; ++j) soffB[j] += (unsigned)k0 * (BN * 2u);
    }
    G2_TURN();
#pragma unroll
    for (int b = 0; b < NS; ++b) {
#pragma unroll
      for (int j = 0; j < FM; ++j) G2_LDA(b, j);
#pragma unroll
      for (int j = 0; j < 4; ++j) G2_LDB(b, j);
      G2_NEXT();
      if (k0 > k_last) G2_TURN();
    }
    g2_steps<64 * FM>([&](auto r) __attribute__((always_inline)) { asm volatile("v_accvgpr_write_b32 a%c0, 0" ::"n"(decltype(r)::value)); });
    G2_WAITV(3 * LOADS);
    __builtin_amdgcn_s_barrier();
    G2_SB0();
#pragma unroll
    for (int j = 0; j < 8; ++j) G2_RDB(0, 0, j);
#pragma unroll
    for (int i = 0; i < 2 * FM; ++i) G2_RDA(0, 0, i);
    G2_SB0();
    for (int st = 0;; st += NS) {  // the last stages load (zeros) past the end, which nobody multiplies
      G2_STEP(0, 0);
      if (st + 1 >= n_stage) break;
      G2_STEP(1, 1);
      if (st + 2 >= n_stage) break;
      G2_STEP(2, 0);
      if (st + 3 >= n_stage) break;
      G2_STEP(3, 1);
      if (st + 4 >= n_stage) break;
    }
    G2_WAITV(0);  // no load may land after the workgroup has given its LDS back
  } else {
    g2_steps<64 * FM>([&](auto r) __attribute__((always_inline)) { asm volatile("v_accvgpr_write_b32 a%c0, 0" ::"n"(decltype(r)::value)); });
  }
  g2_drain();
  if (probe && tid == 0) a.clk[0] = clock64() - c_start, a.clk[1] = wall_clock64() - w_start;
#undef G2_OPEN_SEG
#undef G2_TURN
#undef G2_NEXT
#undef G2_BL
#undef G2_LDA
#undef G2_LDB
#undef G2_RDA
#undef G2_RDB
#undef G2_STEP

  if (piece >= 0) {
    // a range of K: the accumulators leave as they lie in the registers, 1 KiB per store instruction; k_gemm2_sum reads
    // them back in the same order
    float* p = a.part + (((size_t)piece * 4 + wave) * (FM * 4096)) + lane * 4;
    g2_steps<16 * FM>([&](auto t_) __attribute__((always_inline)) {
      constexpr int t = decltype(t_)::value;
      *reinterpret_cast<f32x4*>(p + t * 256) = f32x4{g2_acc<4 * t>(), g2_acc<4 * t + 1>(), g2_acc<4 * t + 2>(), g2_acc<4 * t + 3>()};
    });
    return;
  }

  // ---- epilogue: slab by slab, what the next two slabs read in flight --------------------------------------------------
  const Gemm2Out out = g2_out_of(a, tn);
  bool clamped = false;
  const int mrow = m0 + wm * (FM * 32) + (lane & 15);
  constexpr int SL = 2 * FM;
  G2Pre pre[3];
  g2_epi_load<EPI>(pre[0], a, out, tn, wn, lane, mrow);
  g2_epi_load<EPI>(pre[1], a, out, tn, wn, lane, mrow + 16);
  g2_steps<SL>([&](auto i_) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value;
    if constexpr (i + 2 < SL) g2_epi_load<EPI>(pre[(i + 2) % 3], a, out, tn, wn, lane, mrow + (i + 2) * 16);
    f32x4 x[8];
    g2_steps<8>([&](auto j_) __attribute__((always_inline)) {
      constexpr int t = i * 8 + decltype(j_)::value;
      x[decltype(j_)::value] = f32x4{g2_acc<4 * t>(), g2_acc<4 * t + 1>(), g2_acc<4 * t + 2>(), g2_acc<4 * t + 3>()};
    });
    g2_epi_store<HALF, EPI>(x, pre[i % 3], a, out, tn, wn, lane, mrow + i * 16, clamped);
  });
  if (clamped && a.overflow_flag) atomicOr(a.overflow_flag, 8);
}

// Sum of the K ranges of the cut tiles, in range order, and their epilogue.  A wave takes one slab of 16 rows of one wave's
// block of one tile: eight 1 KiB loads per range, up to four ranges in flight.
template <int FM, bool HALF, int EPI>
__global__ void __launch_bounds__(256) k_gemm2_sum(Gemm2Args a, Gemm2Cut cut) {
  const int lane = threadIdx.x & 63, id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = id % (2 * FM), wave = (id / (2 * FM)) & 3, r = id / (8 * FM);
  int tm, tn;
  g2_cut_tile(cut, cut.first + r, tm, tn);
  const int mrow0 = tm * (64 * FM) + (wave >> 1) * (FM * 32) + i * 16;
  if (mrow0 >= a.M) return;
  const Gemm2Out out = g2_out_of(a, tn);
  G2Pre pre;
  g2_epi_load<EPI>(pre, a, out, tn, wave & 1, lane, mrow0 + (lane & 15));
  const size_t stride = (size_t)cut.rest * (4 * FM * 4096);  // floats between two ranges of a tile
  const float* p = a.part + ((size_t)r * 4 + wave) * (FM * 4096) + i * 2048 + lane * 4;
  f32x4 x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] = *reinterpret_cast<const f32x4*>(p + j * 256);
  auto add = [&](auto n_) {
    constexpr int n = decltype(n_)::value;
    f32x4 t[n][8];
#pragma unroll
    for (int u = 0; u < n; ++u)
#pragma unroll
      for (int j = 0; j < 8; ++j) t[u][j] = *reinterpret_cast<const f32x4*>(p + (u + 1) * stride + j * 256);
#pragma unroll
    for (int u = 0; u < n; ++u)
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] += t[u][j];
    p += n * stride;
  };
  int left = cut.ks - 1;
  for (; left >= 3; left -= 3) add(std::integral_constant<int, 3>{});
  if (left == 2) add(std::integral_constant<int, 2>{});
  else if (left == 1) add(std::integral_constant<int, 1>{});
  bool clamped = false;
  g2_epi_store<HALF, EPI>(x, pre, a, out, tn, wave & 1, lane, mrow0 + (lane & 15), clamped);
  if (clamped && a.overflow_flag) atomicOr(a.overflow_flag, 8);
}

// ---- blocked copies ---------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_block_jobs(BlockJobs jobs) {
  const BlockJob jb = jobs.j[blockIdx.y];
  const long long N = jb.transpose ? jb.C : jb.R, K = jb.transpose ? jb.R : jb.C;
  const long long ks_n = (K + BK - 1) / BK;
  const long long total = (long long)(jb.plain ? (size_t)(N * K) : blocked_elems(N, K)) / 8;  // 16-byte chunks of the destination
  bool over = false;
  for (long long ci = (long long)blockIdx.x * 256 + threadIdx.x; ci < total; ci += (long long)gridDim.x * 256) {
    long long e0 = ci * 8, n, k;  // first element of the chunk
    if (jb.plain) {
      // lanes run along the contiguous side of the source
      n = jb.transpose ? ci % N : e0 / K;
      k = jb.transpose ? ci / N * 8 : e0 - n * K;
      e0 = n * K + k;
    } else {  // ((tile * ks_n + ks) * 256 + row) * 32 + kk
      const int kk = (int)(e0 & 31), row = (int)((e0 >> 5) & 255);
      const long long tk = e0 >> 13, ks = tk % ks_n, tile = tk / ks_n;
      n = tile * BN + row, k = ks * BK + kk;
    }
    unsigned short v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = 0;
      if (n < N && k + e < K) {
        const long long si = jb.transpose ? (k + e) * jb.C + n : n * jb.C + k + e;
        if (jb.src_f32 == 2) {  // already in the compute element: bits as they are
          v[e] = static_cast<const unsigned short*>(jb.src)[si];
        } else {
          const float f = jb.src_f32 ? static_cast<const float*>(jb.src)[si] : bf2f(static_cast<const unsigned short*>(jb.src)[si]);
          v[e] = jobs.half ? f2h(f) : f2bf(f);
          over = over || (jobs.half && !(fabsf(f) <= 65504.f));
        }
      }
    }
    *reinterpret_cast<uint4*>(jb.dst + e0) = make_uint4(v[0] | (unsigned)v[1] << 16, v[2] | (unsigned)v[3] << 16, v[4] | (unsigned)v[5] << 16,
                                                        v[6] | (unsigned)v[7] << 16);
  }
  if (over && jobs.flag) atomicOr(jobs.flag, 8);
}

template <int FM>
constexpr int lds_bytes() { return stages<FM>() * (64 * FM * BK * 2 + BSZ); }

int g_force_fm = 0;  // measurement hook: 2 or 4 fixes the tile height
int g_force_ks = 0;  // measurement hook: fixes the ranges of K
constexpr int kMinCutStages = 4, kMaxCut = 16;  // shortest range of K in stages (the ring holds four), most ranges of a tile
constexpr size_t kMaxPartBytes = (size_t)64 << 20;  // most partial tiles of a launch

int device_cus() {
  int dev = 0;
  hipDeviceProp_t prop;
  return hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess ? prop.multiProcessorCount : 256;
}

}  // namespace

void gemm2_force_tile_rows(int rows) { g_force_fm = rows == 256 ? 4 : rows == 128 ? 2 : 0; }

void gemm2_force_split(int ks) { g_force_ks = ks > 0 ? ks : 0; }

void gemm2_block_jobs(const BlockJobs& jobs, hipStream_t st) {
  if (jobs.n < 1) return;
  hipLaunchKernelGGL(k_block_jobs, dim3(256, jobs.n), dim3(256), 0, st, jobs);
}

// Grid of a launch whose tiles are not cut: the XCD-aware tile order of the kernel.
Gemm2Plan gemm2_plan(int M, int tiles_n, int FM, int n_cu) {
  Gemm2Plan p{};
  const int BM = 64 * FM, tiles_m = (M + BM - 1) / BM;
  // The 32 workgroups an XCD runs at a time form one GM x GN block of tiles about 1024 x 2048 outputs large, so that
  // they share GM + GN operand panels in its L2.
  p.GM = std::min(FM == 2 ? 8 : 4, tiles_m);
  p.GN = std::min(FM == 2 ? 4 : 8, tiles_n);
  p.total = ((tiles_m + p.GM - 1) / p.GM) * ((tiles_n + p.GN - 1) / p.GN) * p.GM * p.GN;  // whole blocks: slots past the matrix return at once
  p.chunk = (p.total + 7) / 8;
  p.grid = p.chunk * 8;
  p.rounds = (tiles_m * tiles_n + n_cu - 1) / n_cu;
  return p;
}

// Tile height and cut of a launch.  A launch runs in rounds of one workgroup per compute unit; the last round is partly
// idle, and outputs with fewer tiles than compute units leave the chip idle throughout (1032 x 3584: 126 tiles of 128
// rows).  So the tiles past the last full round are cut along K until the chip is full: their partial tiles go to the
// workspace and k_gemm2_sum adds them in a second launch (device-scope fences for a last-arriver sum cost more than the
// idle compute units: they write back and invalidate a whole XCD's L2).  Measured in us, uncut -> cut as chosen here:
//   M x N x K            uncut   cut
//   48 x 4096 x 4096        57    23      2048 x 3584 x 18944   319   290
//   256 x 4096 x 11008     135    43      2048 x 5120 x 13824   358   315
//   600 x 5120 x 13824     180   115      4096 x 5120 x 13824   669   563
//   1032 x 3584 x 37888    628   347      2048 x 4096 x 4096     80    80 (one full round: not cut)
// Cost in us, fitted to a sweep of ranges for these and 20 more shapes (it picks within 4 % of the best, 8 % at worst):
// a stage takes 0.68 / 0.41 us in a tile of 256 / 128 rows while few compute units run and up to 0.34 / 0.18 more when
// 256 / 140 do (clock and fabric); a round 6 beyond its stages (a fitted constant: the store of a 256-row tile alone takes
// 11 us with 16-bit and 22 with fp32 outputs, part of which the figures per stage carry); the second launch 4; partial tiles
// 0.19 per MB.  (0.15 would fit the 128-row tiles alone; among the other kernels of a unit the chip holds a lower clock and the
// 256-row tiles, which move fewer operand bytes per flop, lose less of it: 2048 x 4096 x 11008 as one round of 128-row
// tiles or as half-length ranges of 256-row ones is 194 against 192 us alone and 213 against 203 inside a unit.)
// On a stream confined to `share` of the device's compute units (Harli Sec. 6.2) the ranges of K stay the device's: they
// decide the order K is added up in, and a unit gives the same bits on every partition.  The height of the tiles does not:
// where every tile is cut or none is, it is the cheaper one on the share (2048 x 4096 x 4096, not cut: 256 tiles of 128 rows
// are one round on 256 compute units and a round and 26 stragglers on 230, where 128 tiles of 256 rows are one).  Units on
// 230 compute units: 3 x 344 tokens of hidden size 3584 2200 -> 1917 us, 4 x 512 of 4096 2767 -> 2736.
Gemm2Cut gemm2_cut(int M, int tiles_n, int stages, int n_cu, int share) {
  const double t_fixed = 6.0;
  auto step_us = [](int FM, int active) {
    const double b = std::min(1.0, active / (FM == 4 ? 256.0 : 140.0));
    return FM == 4 ? 0.68 + 0.34 * b * b : 0.41 + 0.18 * b * b;
  };
  auto sum_us = [](size_t bytes) { return bytes ? 4.0 + bytes / 1048576.0 * 0.19 : 0.0; };
  auto make = [&](int FM, int ks, int full, double cost) {
    Gemm2Cut c{};
    c.FM = FM, c.ks = ks, c.cost_us = cost, c.tiles_n = tiles_n;
    c.tiles_m = (M + 64 * FM - 1) / (64 * FM), c.GM = std::min(FM == 2 ? 8 : 4, c.tiles_m);
    const int T = c.tiles_m * tiles_n;
    c.full = c.first = ks > 1 ? full : T, c.rest = T - c.full;
    c.chunk_full = (c.full + 7) / 8, c.chunk_cut = (c.rest * ks + 7) / 8;
    return c;
  };
  Gemm2Cut best{};
  best.cost_us = -1;
  for (int FM = 4; FM >= 2; FM -= 2) {
    if ((g_force_fm && FM != g_force_fm) || (!g_force_fm && FM == 4 && M <= 128)) continue;
    const int BM = 64 * FM, tiles_m = (M + BM - 1) / BM, T = tiles_m * tiles_n;
    const int full = T / n_cu * n_cu, rest = T - full;
    const int ks_max = rest > 0 ? std::max(1, std::min(kMaxCut, stages / kMinCutStages)) : 1;
    for (int ks = 1; ks <= ks_max; ++ks) {
      const int pieces = rest * ks, r2 = (pieces + n_cu - 1) / n_cu;
      const size_t bytes = ks > 1 ? (size_t)pieces * BM * BN * 4 : 0;
      if (bytes > kMaxPartBytes) break;
      double cost = (T / n_cu) * (stages * step_us(FM, n_cu) + t_fixed);
      if (r2 > 0) cost += r2 * (((stages + ks - 1) / ks) * step_us(FM, std::min(pieces, n_cu)) + t_fixed);
      cost += sum_us(bytes);
      if (best.cost_us < 0 || (g_force_ks ? ks <= g_force_ks && (ks > best.ks || cost < best.cost_us) : cost < best.cost_us))
        best = make(FM, ks, full, cost);
    }
  }
  if (share < n_cu && !g_force_fm && M > 128 && (best.ks == 1 || best.full == 0)) {
    const int ks = best.ks, len = (stages + ks - 1) / ks;
    best.cost_us = -1;
    for (int FM = 4; FM >= 2; FM -= 2) {
      const int BM = 64 * FM, n = (M + BM - 1) / BM * tiles_n * ks, last = n % share;  // workgroups, and those of the last round
      const size_t bytes = ks > 1 ? (size_t)n * BM * BN * 4 : 0;
      if (bytes > kMaxPartBytes) continue;
      double cost = (n / share) * (len * step_us(FM, share) + t_fixed) + sum_us(bytes);
      if (last) cost += len * step_us(FM, last) + t_fixed;
      if (best.cost_us < 0 || cost < best.cost_us) best = make(FM, ks, 0, cost);
    }
  }
  return best;
}

int gemm2_pass_tiles(const Gemm2Cut& c, size_t part_bytes) {
  if (c.ks < 2) return 0;
  const size_t fit = part_bytes / ((size_t)c.ks * c.FM * (64 * BN * 4));
  if (fit >= (size_t)c.rest) return c.rest;
  if (fit < 1) return 0;
  const int passes = (c.rest + (int)fit - 1) / (int)fit;
  return (c.rest + passes - 1) / passes;
}

size_t gemm2_part_bytes(int max_M, int tiles_n, int stages) {
  const int n_cu = device_cus();
  size_t most = 0;
  for (int M = std::min(128, max_M);; M = std::min(M + 128, max_M)) {  // a plan depends on the rows through their tiles alone
    const Gemm2Cut c = gemm2_cut(M, tiles_n, stages, n_cu, n_cu);
    if (c.ks > 1) most = std::max(most, (size_t)c.rest * c.ks * c.FM * (64 * BN * 4));
    if (M == max_M) return most;
  }
}

harli_status gemm2_launch(const Gemm2Args& a, hipStream_t st) {
  if (a.M < 1 || a.nseg < 1 || a.nseg > kGemm2MaxSeg || a.nout < 1 || a.nout > kGemm2MaxOut || a.tiles_n < 1)
    return fail(HARLI_ERR_INVALID, "gemm2: bad shape M %d nseg %d nout %d tiles %d", a.M, a.nseg, a.nout, a.tiles_n);
  for (int s = 0; s < a.nseg; ++s) {
    const Gemm2Seg& g = a.seg[s];
    if (!g.A || g.K < 8 || (g.K & 7) || (g.lda & 7) || ((uintptr_t)g.A & 15) || ((uintptr_t)g.B & 15) || ((uintptr_t)g.B2 & 15) ||
        g.tile0 < 0 || g.tile1 > a.tiles_n || g.tile0 >= g.tile1 || (g.pair ? (!g.B && !g.B2) : (!g.B || g.B2)))
      return fail(HARLI_ERR_INVALID, "gemm2: segment %d needs K %% 8 == 0, 16-byte aligned operands and a tile range inside the output (K %d lda %lld tiles %d..%d)",
                  s, g.K, g.lda, g.tile0, g.tile1);
  }
  const bool f32out = a.out[0].Cf != nullptr;
  for (int s = 0; s < a.nseg; ++s) {
    // the kernel addresses row tiles of the weight operands from the tile range alone: the range must stay inside them
    const Gemm2Seg& g = a.seg[s];
    const int row_tiles = (g.rows + BN - 1) / BN, span = g.tile1 - g.tile0;
    if (g.rows < 1 || (g.pair ? (span + 1) / 2 : span) > row_tiles)
      return fail(HARLI_ERR_INVALID, "gemm2: segment %d: a weight operand of %d rows cannot cover output tiles %d..%d", s, g.rows, g.tile0, g.tile1);
    // the kernel addresses both operands with 32-bit byte offsets below 2^31
    if (((long long)a.M + 255) * g.lda * 2 >= (1ll << 31) || (long long)blocked_elems(g.rows, g.K) * 2 >= (1ll << 31))
      return fail(HARLI_ERR_INVALID, "gemm2: segment %d: an operand of 2 GiB or more (M %d, lda %lld, %d weight rows, K %d)", s, a.M, g.lda, g.rows, g.K);
  }
  for (int o = 0; o < a.nout; ++o) {
    const Gemm2Out& q = a.out[o];
    if ((q.Cf != nullptr) != f32out) return fail(HARLI_ERR_INVALID, "gemm2: the output blocks of a launch are all fp32 or all 16-bit");
    const int t_end = o + 1 < a.nout ? a.out[o + 1].tile0 : a.tiles_n;
    const int width = a.epi == GEMM2_EPI_GATEUP ? 128 : BN;  // columns of the block per tile
    if (q.tile0 < 0 || q.tile0 >= t_end || (o == 0 && q.tile0 != 0) || q.N < 1 || q.N > (t_end - q.tile0) * width)
      return fail(HARLI_ERR_INVALID, "gemm2: output block %d (tiles %d..%d) cannot hold %d columns", o, q.tile0, t_end, q.N);
    if (a.epi == GEMM2_EPI_NONE && !q.Cb && !q.Cf) return fail(HARLI_ERR_INVALID, "gemm2: output block %d has no destination", o);
    if (q.res && !q.Cf) return fail(HARLI_ERR_INVALID, "gemm2: a residual needs the fp32 output");
    if (q.Cb && !q.Cf && ((q.ldcb & 7) || (q.N & 7) || ((uintptr_t)q.Cb & 15)))
      return fail(HARLI_ERR_INVALID, "gemm2: a 16-bit output needs N and its row stride to be multiples of 8");
    if (q.Cf && ((q.ldcf & 3) || ((uintptr_t)q.Cf & 15) || ((uintptr_t)q.res & 15) || (q.Cb && ((q.ldcb & 3) || ((uintptr_t)q.Cb & 7)))))
      return fail(HARLI_ERR_INVALID, "gemm2: an fp32 output needs a row stride that is a multiple of 4 and aligned pointers");
  }
  if (a.epi == GEMM2_EPI_ROPE) {
    if (f32out || !a.rope || a.rope_S < 1 || (a.rope_d != 64 && a.rope_d != 128) || ((uintptr_t)a.rope & 15) || !a.half)
      return fail(HARLI_ERR_INVALID, "gemm2: the rotary epilogue needs 16-bit outputs, a table and a head size of 64 or 128 (got %d)", a.rope_d);
    for (int o = 0; o < a.nout; ++o)
      if (a.out[o].tile0 < a.rope_tiles && a.out[o].N % a.rope_d) return fail(HARLI_ERR_INVALID, "gemm2: output block %d holds no whole heads", o);
  } else if (a.epi != GEMM2_EPI_NONE) {
    const bool gu = a.epi == GEMM2_EPI_GATEUP;
    if ((a.epi != GEMM2_EPI_GATEUP && a.epi != GEMM2_EPI_SWIGLU_BWD) || a.nout != 1 || a.out[0].Cf || (a.out[0].N & 7) || (a.lde & 7) ||
        !a.o0 || !a.o1 || (gu ? (!a.out[0].Cb) : (!a.e0 || !a.e1 || a.out[0].Cb)) ||
        (((uintptr_t)a.e0 | (uintptr_t)a.e1 | (uintptr_t)a.o0 | (uintptr_t)a.o1) & 15))
      return fail(HARLI_ERR_INVALID, "gemm2: fused SwiGLU epilogue %d needs one block, N and lde %% 8 == 0 and its own aligned outputs", a.epi);
    for (int s = 0; s < a.nseg; ++s)
      if ((a.seg[s].pair != 0) != gu) return fail(HARLI_ERR_INVALID, "gemm2: interleaved pairs go with the gate/up epilogue and only with it");
  }
  static bool attr_set = false;
  static uint4* zero16 = nullptr;  // 256 zero bytes in device memory, kept for the life of the process
  if (!attr_set) {
    HARLI_HIP(hipMalloc(reinterpret_cast<void**>(&zero16), 256));
    HARLI_HIP(hipMemset(zero16, 0, 256));
#define G2_ATTR(F_, H_, E_) \
  HARLI_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm2<F_, H_, E_>), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes<F_>()))
#define G2_ATTR4(F_, H_) \
  G2_ATTR(F_, H_, GEMM2_EPI_NONE); G2_ATTR(F_, H_, GEMM2_EPI_F32); G2_ATTR(F_, H_, GEMM2_EPI_SWIGLU_BWD); G2_ATTR(F_, H_, GEMM2_EPI_GATEUP)
#define G2_ATTR5(F_) G2_ATTR(F_, true, GEMM2_EPI_ROPE)
    G2_ATTR5(2); G2_ATTR5(4); G2_ATTR4(2, true); G2_ATTR4(4, true); G2_ATTR4(2, false); G2_ATTR4(4, false);
#undef G2_ATTR4
#undef G2_ATTR5
#undef G2_ATTR
    attr_set = true;
  }
  const int n_cu = a.n_cu > 0 ? a.n_cu : device_cus();
  int stages = 0;  // of the longest column tile
  for (int s = 0; s < a.nseg; ++s) {
    int n = 0;
    for (int q = 0; q < a.nseg; ++q)
      if (a.seg[q].tile0 <= a.seg[s].tile0 && a.seg[q].tile1 > a.seg[s].tile0) n += (a.seg[q].K + BK - 1) / BK;
    stages = std::max(stages, n);
  }
  const int share = cu_stream_count(st);  // 0: not confined
  const Gemm2Cut plan = gemm2_cut(a.M, a.tiles_n, stages, n_cu, share > 0 ? std::min(share, n_cu) : n_cu);
  const int FM = plan.FM;
  const Gemm2Plan pl = gemm2_plan(a.M, a.tiles_n, FM, n_cu);
  const int GM = pl.GM, GN = pl.GN, total = pl.total, chunk = pl.chunk;
  const int per_pass = gemm2_pass_tiles(plan, a.part ? a.part_bytes : 0);
  if (plan.ks > 1 && per_pass < 1) return fail(HARLI_ERR_INVALID, "gemm2: no room for the partial tiles of one tile");
  // Cut launch: the whole tiles with the first pass, then pass after pass (one, unless the workspace is small).
#define G2_LAUNCH(F_, H_, E_)                                                                                                \
  do {                                                                                                                       \
    Gemm2Cut cut = plan;                                                                                                     \
    if (cut.ks < 2)                                                                                                          \
      hipLaunchKernelGGL((k_gemm2<F_, H_, E_>), dim3(pl.grid), dim3(NT), lds_bytes<F_>(), st, a, cut, total, chunk, GM, GN, zero16); \
    for (int done = 0; done < plan.rest; done += cut.rest) {                                                                 \
      cut.first = plan.first + done;                                                                                         \
      cut.rest = std::min(per_pass, plan.rest - done);                                                                       \
      cut.chunk_cut = (cut.rest * cut.ks + 7) / 8;                                                                           \
      hipLaunchKernelGGL((k_gemm2<F_, H_, E_>), dim3(8 * (cut.chunk_full + cut.chunk_cut)), dim3(NT), lds_bytes<F_>(), st, a, cut, total, \
                         chunk, GM, GN, zero16);                                                                             \
      hipLaunchKernelGGL((k_gemm2_sum<F_, H_, E_>), dim3(cut.rest * 2 * F_), dim3(256), 0, st, a, cut);                       \
      cut.full = cut.chunk_full = 0;                                                                                         \
    }                                                                                                                        \
  } while (0)
#define G2_PICK(F_)                                                                    \
  do {                                                                                 \
    if (a.epi == GEMM2_EPI_ROPE) {                                                     \
      G2_LAUNCH(F_, true, GEMM2_EPI_ROPE);                                             \
    } else if (a.half) {                                                               \
      if (a.epi == GEMM2_EPI_GATEUP) G2_LAUNCH(F_, true, GEMM2_EPI_GATEUP);            \
      else if (a.epi == GEMM2_EPI_SWIGLU_BWD) G2_LAUNCH(F_, true, GEMM2_EPI_SWIGLU_BWD); \
      else if (f32out) G2_LAUNCH(F_, true, GEMM2_EPI_F32);                             \
      else G2_LAUNCH(F_, true, GEMM2_EPI_NONE);                                        \
    } else {                                                                           \
      if (a.epi == GEMM2_EPI_GATEUP) G2_LAUNCH(F_, false, GEMM2_EPI_GATEUP);           \
      else if (a.epi == GEMM2_EPI_SWIGLU_BWD) G2_LAUNCH(F_, false, GEMM2_EPI_SWIGLU_BWD); \
      else if (f32out) G2_LAUNCH(F_, false, GEMM2_EPI_F32);                            \
      else G2_LAUNCH(F_, false, GEMM2_EPI_NONE);                                       \
    }                                                                                  \
  } while (0)
  // flops asked for: 2 M K per valid output column a segment reaches (an interleaved pair fills both halves of a tile)
  double flops = 0;
  for (int s = 0; s < a.nseg; ++s) {
    long long cols = 0;
    for (int o = 0; o < a.nout; ++o) {
      const int T0 = a.out[o].tile0, T1 = o + 1 < a.nout ? a.out[o + 1].tile0 : a.tiles_n;
      const int lo = std::max(a.seg[s].tile0, T0), hi = std::min(a.seg[s].tile1, T1);
      if (hi <= lo) continue;
      const long long width = a.epi == GEMM2_EPI_GATEUP ? 128 : BN;
      const long long c0 = (long long)(lo - T0) * width, c1 = std::min<long long>((long long)(hi - T0) * width, a.out[o].N);
      if (c1 > c0) cols += (c1 - c0) * (a.epi == GEMM2_EPI_GATEUP ? ((a.seg[s].B != nullptr) + (a.seg[s].B2 != nullptr)) : 1);
    }
    flops += 2.0 * a.M * (double)cols * a.seg[s].K;
  }
  GemmTimer timer;
  HARLI_HIP(timer.begin(flops, st));
  if (FM == 4) G2_PICK(4);
  else G2_PICK(2);
#undef G2_PICK
#undef G2_LAUNCH
  HARLI_HIP(timer.end(st));
  HARLI_HIP(hipGetLastError());
  return HARLI_OK;
}

}  // namespace harli
