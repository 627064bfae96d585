// Kernels of the finetune unit's weight GEMM (see gemm2.h for the operand layouts; gemm2.hip plans and launches,
// gemm2_rows*.hip compile one tile height each).
//
// Workgroup tile (32 RT) x 256, K step 32, FOUR waves -- one per SIMD, each with the whole register file: a wave owns
// a (16 RT) x 128 block of the tile = RT x 8 accumulators of v_mfma_f32_16x16x32 (256 accumulator registers at RT = 8).
// What this shape buys on gfx950, measured:
//   * operand bytes per flop through L2 and through LDS fall with the tile edge: a CU pulls no more than ~22-41 B/clk
//     from L2 and LDS serves 128 B/clk, and 64 x 64 wave tiles (two waves per SIMD) need all of the latter at the full
//     MFMA rate.  128 x 128 per wave needs half;
//   * operands go from global memory straight into LDS (buffer_load ... lds, 16 B per lane, no register staging); the
//     rows of a stage are XOR-swizzled in 16-byte chunks on the way in (each lane picks the global chunk that belongs
//     in its LDS slot), which makes the 16-row fragment reads conflict free;
//   * the fragments of a stage are read during the stage before, so a stage's buffer is free again as soon as its products
//     begin: of four LDS stages three are in flight;
//   * one wave per SIMD has nobody to hide its waits, so reads and loads are dealt out between the products by hand;
//   * nothing but the loads' scalar offsets moves from stage to stage: every branch and mask of the cursor (end of a
//     segment, of the range, a partial K step) is behind one comparison that is false on whole stages.
// What bounds it: power.  On random operands the chip holds 1.65-1.75 GHz under this loop (2.4 on zeros, and with the loads
// bunched together the clock rises as the cycles do), so energy per product counts: v_mfma_f32_16x16x32 draws less than
// 32x32x16.  A stage takes 1142 cycles at 256 rows (1024 of them product issue), 880 (768) at 192, 635 (512) at 128: the clock
// of workgroup 0's loop, K = 8192 less K = 4096, one round of tiles.  A workgroup spends another 3-5 us before its first
// product and 4 (16-bit) or 8-11 us (fp32) on its store.  Back to back on normal operands (harli_dbg_gemm2), 4096 x 16384 x
// 4096: 487 us with 32x32x16 products and a store through LDS, 435 now (1263 TFLOP/s; the vendor's library 382); fp32 output
// with a residual 590 -> 545; one round, 2048 x 8192 x 8192: 236 -> 208 (1320 TFLOP/s; 196); 2048 x 22016 x 4096: 339 -> 304 (410).
// RT = 4 .. 8, tiles of 128, 160, .., 256 rows: the height whose tiles fit the rows and the rounds best (gemm2_cut).
#pragma once
#include "gemm2.h"

#include <algorithm>
#include <type_traits>

#include "ctx.h"
#include "device_utils.h"

namespace harli {
namespace {

constexpr int BN = kG2TileN, BK = kG2StepK, NT = 256;
constexpr int BSZ = BN * BK * 2;  // 16 KiB: one stage of the weight-side tile
// 16-row groups of the activation side each wave loads per stage (an odd RT loads two groups too many, which lie outside
// the operand's range and cost no traffic: every wave has to count the same number of loads)
constexpr int a_groups(int RT) { return (RT + 1) / 2; }
constexpr int stage_bytes(int RT) { return a_groups(RT) * 4096 + BSZ; }
// LDS stages.  As many as fit (six at 128 rows, five at the others) are no faster: 252 units of eleven layer shapes, 8 to 4096
// tokens, take 0.7 % less time with four (the best of four runs each), a 7B unit 1865 us with four and 1864 with five, a 13B unit
// 5495 and 5479, within the runs' spread.  Four leave 64 (128 rows) to 32 KiB (256 rows) of a compute unit's LDS free.
constexpr int kStages = 4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define G2_WAITV(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
#define G2_SB0() __builtin_amdgcn_sched_barrier(0)

// ---- products and accumulators -----------------------------------------------------------------------------------------
// A wave owns RT x 8 accumulators of v_mfma_f32_16x16x32, in accumulator registers NAMED BY HAND: accumulator t = 8 i + j
// is a[4t .. 4t+3].  The compiler's allocator copied more than half of 64 four-register accumulators between the register
// files in every pass of the stage ring; named, none moves, and the code between two products is exactly what stands there.
// The kernel claims the whole range in its first statement and nothing else in it uses accumulator registers (the compiler
// would only to spill, and it has 256 other registers for about 150 values).  Hazards the compiler does not fill in for
// assembly: the products of one accumulator are 8 RT products apart, its first use lies a barrier behind the zeros and the
// reads of the epilogue behind the idle cycles of g2_drain(); a vector instruction that writes a fragment has to lie two
// slots before the product that reads it, and there is none: fragments come from LDS, whose reads the compiler waits for.  The
// build (build.py) reads the compiled kernels back and refuses any in which one of this does not hold.
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
template <int RT>
__device__ __forceinline__ void g2_claim() {
#define G2_R10(p) p "0", p "1", p "2", p "3", p "4", p "5", p "6", p "7", p "8", p "9"
#define G2_R128                                                                                                        \
  G2_R10("a"), G2_R10("a1"), G2_R10("a2"), G2_R10("a3"), G2_R10("a4"), G2_R10("a5"), G2_R10("a6"), G2_R10("a7"),       \
      G2_R10("a8"), G2_R10("a9"), G2_R10("a10"), G2_R10("a11"), "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127"
  asm volatile("" ::: G2_R128);
  if (RT > 4) asm volatile("" ::: "a128", "a129", G2_R10("a13"), G2_R10("a14"), G2_R10("a15"));
  if (RT > 5) asm volatile("" ::: G2_R10("a16"), G2_R10("a17"), G2_R10("a18"), "a190", "a191");
  if (RT > 6) asm volatile("" ::: "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", G2_R10("a20"), G2_R10("a21"), "a220", "a221", "a222", "a223");
  if (RT > 7)
    asm volatile("" ::: "a224", "a225", "a226", "a227", "a228", "a229", G2_R10("a23"), G2_R10("a24"), "a250", "a251", "a252", "a253", "a254",
                 "a255");
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

// The arguments are a kilobyte, read here and there by branches, and a cold cache line of them comes from as far away as host
// memory.  One load from each line, all at once, is one trip instead of one after the other (twelve segments looked at in turn took
// 2 us a launch).
template <int BYTES>
__device__ __forceinline__ void g2_touch_args() {
  const auto* p = (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
  int any = 0;
#pragma unroll
  for (int l = 0; l < (BYTES + 63) / 64; ++l) any |= p[l * 16];
  asm volatile("" ::"s"(any));
}
constexpr int kG2ArgBytes = sizeof(Gemm2Args) + sizeof(Gemm2Cut);

template <int RT, bool HALF, int EPI>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_gemm2(Gemm2Args a, Gemm2Cut cut, int tiles_total, int chunk, int GM, int GN) {
  constexpr int BM = 32 * RT, AG = a_groups(RT), ASZ = AG * 4096, STG = stage_bytes(RT), NS = kStages;
  constexpr int LOADS = AG + 4;  // direct-to-LDS loads a wave issues per stage
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  g2_claim<RT>();
  g2_touch_args<kG2ArgBytes>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;  // 2 x 2 waves of (16 RT) x 128
  const int w = blockIdx.x;
  int tm, tn, piece = -1, split = 0;  // piece: index of this workgroup's partial tile, -1 for a whole tile
  if (chunk == 0) {
    // banded order (see gemm2_cut): whole tiles first, then the remaining tiles in ranges of K, range by range; either
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
  unsigned voffA[AG];                                             // and inside the activation operand: (row, chunk)
  __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(a.seg[0].A), 0, 0, kRsrcFlags), rsB = rsA, rsB2 = rsA;
  unsigned soffA = 0, soffB[4] = {0u, 0u, 0u, 0u};
  bool pairseg = false;
  int seg = -1, k0 = 0, Kseg = 0, issued = 0;
  int k_last = 0;           // last k0 of this segment whose stage is a whole one of this tile
  unsigned vA[AG], vB = 0;  // the offsets the loads use: voffA, voffB or kOut

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
      _Pragma("unroll") for (int j = 0; j < AG; ++j)                                                                   \
        voffA[j] = wave * AG + j < 2 * RT ? (unsigned)(m0 + (wave * AG + j) * 16 + drow) * lda2 + (unsigned)dchunk * 16u : kOut; \
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
      _Pragma("unroll") for (int j = 0; j < AG; ++j) vA[j] = kOut;                                                    \
      vB = kOut;                                                                                                      \
      soffA = soffB[0] = soffB[1] = soffB[2] = soffB[3] = 0;                                                          \
      k_last = 0x7fffffff;                                                                                            \
    } else {                                                                                                          \
      if (k0 >= Kseg) G2_OPEN_SEG();                                                                                  \
      const bool whole = Kseg - k0 >= BK;                                                                             \
      _Pragma("unroll") for (int j = 0; j < AG; ++j) vA[j] = whole || k0 + dchunk * 8 < Kseg ? voffA[j] : kOut;       \
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
#define G2_LDA(buf, j) G2_BL(rsA, vA[j], soffA, smem + (buf) + (wave * AG + (j)) * 1024)
#define G2_LDB(buf, j) G2_BL((j) < 2 ? rsB : rsB2, vB, soffB[j], smem + (buf) + ASZ + (wave * 4 + (j)) * 1024)

  // fragment reads: row lane%16, 16-byte chunk lane/16, swizzled like the loads
  const int fo = (lane & 15) * 64 + ((lane >> 4) ^ ((lane >> 1) & 3)) * 16;
  const int aoff = wm * (RT * 16) * 64 + fo, boff = ASZ + wn * 128 * 64 + fo;
  u32x4 fa[2][RT], fb[2][8];
#define G2_RDA(p, at, i) fa[p][i] = *reinterpret_cast<const u32x4*>(smem + (at) + (i) * 1024)
#define G2_RDB(p, at, j) fb[p][j] = *reinterpret_cast<const u32x4*>(smem + (at) + (j) * 1024)
  // One stage: 8 RT products from fragments p.  Behind the first kBar of them every wave has all its fragments of this
  // stage in registers and its share of the next stage has landed, so the barrier there opens the next stage's buffer for
  // reading and this one's for the stage NS ahead; the fragment reads and the loads are dealt out between the other
  // products.  Rows of products alternate their direction, so that one operand stays from each product to the next.
  constexpr int kBar = 3, kRd0 = kBar + 1, kLd0 = kBar + 2, kRdStep = RT > 5 ? 3 : 2, kLdStep = RT > 5 ? 6 : RT == 5 ? 5 : 4;
  constexpr int kFly = (NS - 2) * LOADS;  // loads of a wave that may be in flight when the next stage has to have landed
  static_assert((NS - 1) * LOADS + LOADS < 64, "vmcnt holds six bits");
  static_assert(kRd0 + (RT + 8 - 1) * kRdStep < 8 * RT && kLd0 + (LOADS - 1) * kLdStep < 8 * RT, "a stage must hold its reads and loads");
#define G2_STEP(p)                                                                                                    \
  do {                                                                                                                \
    const int at_a = aoff + next, at_b = boff + next;                                                                 \
    g2_steps<8 * RT>([&](auto q_) __attribute__((always_inline)) {                                                   \
      constexpr int q = decltype(q_)::value, i = q >> 3, j = i & 1 ? 7 - (q & 7) : q & 7;                             \
      g2_mm<HALF, i * 8 + j>(fb[p][j], fa[p][i]);                                                                     \
      if constexpr (q == kBar) {                                                                                      \
        G2_SB0();                                                                                                     \
        __builtin_amdgcn_s_waitcnt(0x0070 | (kFly & 15) | ((kFly >> 4) << 14)); /* vmcnt, lgkmcnt 0 */                \
        __builtin_amdgcn_s_barrier();                                                                                 \
        G2_SB0();                                                                                                     \
      }                                                                                                               \
      if constexpr (q >= kRd0 && (q - kRd0) % kRdStep == 0 && (q - kRd0) / kRdStep < RT + 8) {                    \
        constexpr int r = (q - kRd0) / kRdStep;                                                                       \
        if constexpr (r < 8) G2_RDB((p) ^ 1, at_b, r);                                                                \
        else G2_RDA((p) ^ 1, at_a, r - 8);                                                                            \
        G2_SB0();                                                                                                     \
      }                                                                                                               \
      if constexpr (q >= kLd0 && (q - kLd0) % kLdStep == 0 && (q - kLd0) / kLdStep < LOADS) {                         \
        constexpr int r = (q - kLd0) / kLdStep;                                                                       \
        if constexpr (r < AG) G2_LDA(cur, r);                                                                         \
        else G2_LDB(cur, r - AG);                                                                                     \
        G2_SB0();                                                                                                     \
      }                                                                                                               \
    });                                                                                                               \
    cur = next;                                                                                                       \
    next = next == (NS - 1) * STG ? 0 : next + STG;                                                                   \
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
    for (int b = 0; b < NS * STG; b += STG) {
#pragma unroll
      for (int j = 0; j < AG; ++j) G2_LDA(b, j);
#pragma unroll
      for (int j = 0; j < 4; ++j) G2_LDB(b, j);
      G2_NEXT();
      if (k0 > k_last) G2_TURN();
    }
    g2_steps<32 * RT>([&](auto r) __attribute__((always_inline)) { asm volatile("v_accvgpr_write_b32 a%c0, 0" ::"n"(decltype(r)::value)); });
    G2_WAITV((NS - 1) * LOADS);
    __builtin_amdgcn_s_barrier();
    G2_SB0();
#pragma unroll
    for (int j = 0; j < 8; ++j) G2_RDB(0, boff, j);
#pragma unroll
    for (int i = 0; i < RT; ++i) G2_RDA(0, aoff, i);
    G2_SB0();
    int cur = 0, next = STG;  // buffers of this stage and the next
    for (int st = 0;; st += 2) {  // the last stages load (zeros) past the end, which nobody multiplies
      G2_STEP(0);
      if (st + 1 >= n_stage) break;
      G2_STEP(1);
      if (st + 2 >= n_stage) break;
    }
    G2_WAITV(0);  // no load may land after the workgroup has given its LDS back
  } else {
    g2_steps<32 * RT>([&](auto r) __attribute__((always_inline)) { asm volatile("v_accvgpr_write_b32 a%c0, 0" ::"n"(decltype(r)::value)); });
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
    float* p = a.part + (((size_t)piece * 4 + wave) * (RT * 2048)) + lane * 4;
    g2_steps<8 * RT>([&](auto t_) __attribute__((always_inline)) {
      constexpr int t = decltype(t_)::value;
      *reinterpret_cast<f32x4*>(p + t * 256) = f32x4{g2_acc<4 * t>(), g2_acc<4 * t + 1>(), g2_acc<4 * t + 2>(), g2_acc<4 * t + 3>()};
    });
    return;
  }

  // ---- epilogue: slab by slab, what the next two slabs read in flight --------------------------------------------------
  // A loop, and only the reads of the accumulators written out: every launch finds the instruction cache cold, and the whole
  // epilogue written out RT times was much of a kernel's code (with g2_touch_args 1.4 to 1.9 % of a finetune unit).
  const Gemm2Out out = g2_out_of(a, tn);
  bool clamped = false;
  const int mrow = m0 + wm * (RT * 16) + (lane & 15);
  G2Pre pre, pre1, pre2;
  g2_epi_load<EPI>(pre, a, out, tn, wn, lane, mrow);
  g2_epi_load<EPI>(pre1, a, out, tn, wn, lane, mrow + 16);
#pragma unroll 1
  for (int i = 0; i < RT; ++i) {
    g2_epi_load<EPI>(pre2, a, out, tn, wn, lane, mrow + (i + 2) * 16);  // (past the tile: a valid row, never used)
    f32x4 x[8];
    g2_steps<RT>([&](auto i_) __attribute__((always_inline)) {
      if (i == decltype(i_)::value)
        g2_steps<8>([&](auto j_) __attribute__((always_inline)) {
          constexpr int t = decltype(i_)::value * 8 + decltype(j_)::value;
          x[decltype(j_)::value] = f32x4{g2_acc<4 * t>(), g2_acc<4 * t + 1>(), g2_acc<4 * t + 2>(), g2_acc<4 * t + 3>()};
        });
    });
    g2_epi_store<HALF, EPI>(x, pre, a, out, tn, wn, lane, mrow + i * 16, clamped);
    pre = pre1;
    pre1 = pre2;
  }
  if (clamped && a.overflow_flag) atomicOr(a.overflow_flag, 8);
}

// Sum of the K ranges of the cut tiles, in range order, and their epilogue.  A wave takes one slab of 16 rows of one wave's
// block of one tile: eight 1 KiB loads per range, up to four ranges in flight.
template <int RT, bool HALF, int EPI>
__global__ void __launch_bounds__(256) k_gemm2_sum(Gemm2Args a, Gemm2Cut cut) {
  g2_touch_args<kG2ArgBytes>();
  const int lane = threadIdx.x & 63, id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = id % RT, wave = (id / RT) & 3, r = id / (4 * RT);
  int tm, tn;
  g2_cut_tile(cut, cut.first + r, tm, tn);
  const int mrow0 = tm * (32 * RT) + (wave >> 1) * (RT * 16) + i * 16;
  if (mrow0 >= a.M) return;
  const Gemm2Out out = g2_out_of(a, tn);
  G2Pre pre;
  g2_epi_load<EPI>(pre, a, out, tn, wave & 1, lane, mrow0 + (lane & 15));
  const size_t stride = (size_t)cut.rest * (RT * 8192);  // floats between two ranges of a tile
  const float* p = a.part + ((size_t)r * 4 + wave) * (RT * 2048) + i * 2048 + lane * 4;
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

template <int RT>
constexpr int lds_bytes() { return kStages * stage_bytes(RT); }

}  // namespace

// The kernels need more dynamic LDS than the default limit.
template <int RT>
harli_status gemm2_init() {
  auto set = [](auto kernel) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes<RT>());
  };
  for (auto kernel : {&k_gemm2<RT, true, GEMM2_EPI_NONE>, &k_gemm2<RT, true, GEMM2_EPI_F32>, &k_gemm2<RT, true, GEMM2_EPI_SWIGLU_BWD>,
                      &k_gemm2<RT, true, GEMM2_EPI_GATEUP>, &k_gemm2<RT, true, GEMM2_EPI_ROPE>})
    HARLI_HIP(set(kernel));
  if constexpr (RT == 4 || RT == 8)
    for (auto kernel : {&k_gemm2<RT, false, GEMM2_EPI_NONE>, &k_gemm2<RT, false, GEMM2_EPI_F32>, &k_gemm2<RT, false, GEMM2_EPI_SWIGLU_BWD>,
                        &k_gemm2<RT, false, GEMM2_EPI_GATEUP>})
      HARLI_HIP(set(kernel));
  return HARLI_OK;
}

// A launch of one tile height: the whole tiles with the first pass, then pass after pass (one, unless the workspace is small).
template <int RT>
harli_status gemm2_run(const Gemm2Args& a, const Gemm2Cut& plan, const Gemm2Plan& pl, bool banded, int per_pass, hipStream_t st) {
  const bool f32out = a.out[0].Cf != nullptr;
  auto launch = [&](auto kernel, auto sum) -> harli_status {
    Gemm2Cut cut = plan;
    const int chunk = banded ? 0 : pl.chunk;
    if (cut.ks < 2)
      hipLaunchKernelGGL(kernel, dim3(banded ? 8 * cut.chunk_full : pl.grid), dim3(NT), lds_bytes<RT>(), st, a, cut, pl.total, chunk, pl.GM, pl.GN);
    for (int done = 0; done < plan.rest; done += cut.rest) {
      cut.first = plan.first + done;
      cut.rest = std::min(per_pass, plan.rest - done);
      cut.chunk_cut = (cut.rest * cut.ks + 7) / 8;
      hipLaunchKernelGGL(kernel, dim3(8 * (cut.chunk_full + cut.chunk_cut)), dim3(NT), lds_bytes<RT>(), st, a, cut, pl.total, chunk, pl.GM, pl.GN);
      hipLaunchKernelGGL(sum, dim3(cut.rest * RT), dim3(256), 0, st, a, cut);
      cut.full = cut.chunk_full = 0;
    }
    return HARLI_OK;
  };
  auto pick = [&](auto half) -> harli_status {
    constexpr bool H = decltype(half)::value;
    switch (a.epi) {
      case GEMM2_EPI_GATEUP: return launch(&k_gemm2<RT, H, GEMM2_EPI_GATEUP>, &k_gemm2_sum<RT, H, GEMM2_EPI_GATEUP>);
      case GEMM2_EPI_SWIGLU_BWD: return launch(&k_gemm2<RT, H, GEMM2_EPI_SWIGLU_BWD>, &k_gemm2_sum<RT, H, GEMM2_EPI_SWIGLU_BWD>);
      default:
        return f32out ? launch(&k_gemm2<RT, H, GEMM2_EPI_F32>, &k_gemm2_sum<RT, H, GEMM2_EPI_F32>)
                      : launch(&k_gemm2<RT, H, GEMM2_EPI_NONE>, &k_gemm2_sum<RT, H, GEMM2_EPI_NONE>);
    }
  };
  if (a.epi == GEMM2_EPI_ROPE) return launch(&k_gemm2<RT, true, GEMM2_EPI_ROPE>, &k_gemm2_sum<RT, true, GEMM2_EPI_ROPE>);
  if (a.half) return pick(std::true_type{});
  if constexpr (RT == 4 || RT == 8) return pick(std::false_type{});
  return fail(HARLI_ERR_INVALID, "gemm2: bfloat16 operands have tiles of 128 or 256 rows");
}

}  // namespace harli
