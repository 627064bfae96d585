// Weight GEMM of the finetune unit: tile height and cut of a launch, blocked copies (kernels: gemm2_kernel.h).
#include "gemm2.h"

#include <algorithm>
#include <mutex>

#include "ctx.h"
#include "device_utils.h"

namespace harli {
namespace {

constexpr int BN = kG2TileN, BK = kG2StepK;

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

int g_force_rt = 0;  // measurement hook: 4 .. 8 fixes the tile height
int g_force_ks = 0;  // measurement hook: fixes the ranges of K
constexpr int kMinCutStages = 4, kMaxCut = 16;  // shortest range of K in stages (the ring holds four), most ranges of a tile
constexpr size_t kMaxPartBytes = (size_t)64 << 20;  // most partial tiles of a launch

// row tiles of the block of 32 tiles an XCD works on at a time: about 1024 x 2048 outputs
int band_rows(int RT) { return RT < 6 ? 8 : 4; }

int device_cus() {
  int dev = 0;
  hipDeviceProp_t prop;
  return hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess ? prop.multiProcessorCount : 256;
}

}  // namespace

void gemm2_force_tile_rows(int rows) { g_force_rt = rows >= 128 && rows <= 256 && rows % 32 == 0 ? rows / 32 : 0; }

void gemm2_force_split(int ks) { g_force_ks = ks > 0 ? ks : 0; }

void gemm2_block_jobs(const BlockJobs& jobs, hipStream_t st) {
  if (jobs.n < 1) return;
  hipLaunchKernelGGL(k_block_jobs, dim3(256, jobs.n), dim3(256), 0, st, jobs);
}

// Uncut outputs that whole blocks of tiles cover go out block by block.  Any other would pad the blocks, and the XCDs whose
// shares hold the fewest empty slots would run a round more than the rest (12 x 20 tiles of 3000 x 5120 x 13824 took 550 us
// in blocks, 347 in bands): bands have no empty slots.
bool gemm2_banded(const Gemm2Cut& c, const Gemm2Plan& p) { return c.ks > 1 || p.total != c.tiles_m * c.tiles_n; }

// Grid of a launch in blocks of tiles: the XCD-aware tile order of the kernel.
Gemm2Plan gemm2_plan(int M, int tiles_n, int RT, int n_cu) {
  Gemm2Plan p{};
  const int BM = 32 * RT, tiles_m = (M + BM - 1) / BM;
  // The 32 workgroups an XCD runs at a time form one GM x GN block of tiles about 1024 x 2048 outputs large, so that
  // they share GM + GN operand panels in its L2.
  p.GM = std::min(band_rows(RT), tiles_m);
  p.GN = std::min(32 / band_rows(RT), tiles_n);
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
// idle compute units: they write back and invalidate a whole XCD's L2).  And rows that no whole number of tiles fits are
// multiplied as zeros: of the five heights the one that wastes least over rows and rounds is taken (1032 rows are five
// tiles of 256 with a fifth of them idle, or five of 224).  Measured, us,
// with operands that come from HBM as a unit's weights do (fp32 outputs with a residual):
//   M x N x K                  256 rows, uncut   best of 128 and 256 rows   as chosen
//   600 x 5120 x 13824  fp32       266               101 (256 rows / 4)        98 (224 / 4)
//   1032 x 4608 x 3584              78                54 (128, uncut)          47 (160 / 2)
//   1032 x 37888 x 3584            282               282 (256, uncut)         274 (224, uncut)
//   1032 x 3584 x 37888 fp32       673               282 (128 / 2)            264 (192 / 3)
//   2048 x 4096 x 11008 fp32       262               171 (256 / 2)            171 (256 / 2)
//   2048 x 22016 x 4096            309               309                      309 (256, uncut)
//   4096 x 5120 x 13824 fp32       653               477 (256 / 4)            477 (256 / 4)
// Cost in us, fitted to a sweep of heights and ranges for 43 shapes (48 to 4096 rows; its choices take 0.8 % longer than the
// best ones on average, 14 % at worst): a stage takes 0.21 + 0.047 RT while few compute units run and up to 0.026 RT - 0.018
// more when all do (the clock falls); a round 9 beyond its stages, 14 more where it reads a residual and stores fp32; the
// second launch 1.0 and 0.29 per MB of partials.  With operands from the memory-side cache small tiles would look better than
// they are in a unit (2048 x 4096 x 11008 as 128 rows uncut: 147 against 192 us): their stages are too short to cover the
// way to HBM.
// On a stream confined to `share` of the device's compute units (Harli Sec. 6.2) the ranges of K stay the device's: they
// decide the order K is added up in, and a unit gives the same bits on every partition.  The height of the tiles does not:
// where every tile is cut or none is, it is the cheapest there of the device's choice, 128 and 256 rows (2048 x 4096 x 4096,
// not cut: 256 tiles of 128 rows are one round on 256 compute units and a round and 26 stragglers on 230, where 128 tiles of
// 256 rows are one).
Gemm2Cut gemm2_cut(int M, int tiles_n, int stages, int n_cu, int share, bool half, bool f32out) {
  const double t_fixed = 9.0, t_store = f32out ? 14.0 : 0.0;
  auto step_us = [](int RT, int active) {
    const double b = std::min(1.0, active / 256.0);
    return 0.21 + 0.047 * RT + (0.026 * RT - 0.018) * b * b;
  };
  auto sum_us = [](size_t bytes) { return bytes ? 1.0 + bytes / 1048576.0 * 0.29 : 0.0; };
  auto make = [&](int RT, int ks, int full, double cost) {
    Gemm2Cut c{};
    c.RT = RT, c.ks = ks, c.cost_us = cost, c.tiles_n = tiles_n;
    c.tiles_m = (M + 32 * RT - 1) / (32 * RT), c.GM = std::min(band_rows(RT), c.tiles_m);
    const int T = c.tiles_m * tiles_n;
    c.full = c.first = ks > 1 ? full : T, c.rest = T - c.full;
    c.chunk_full = (c.full + 7) / 8, c.chunk_cut = (c.rest * ks + 7) / 8;
    return c;
  };
  auto allowed = [&](int RT) {  // a taller tile than the rows need only multiplies zeros
    return g_force_rt ? RT == g_force_rt : (half || RT == 4 || RT == 8) && (RT == 4 || M > 32 * (RT - 1));
  };
  Gemm2Cut best{};
  best.cost_us = -1;
  for (int RT = 8; RT >= 4; --RT) {
    if (!allowed(RT)) continue;
    const int BM = 32 * RT, tiles_m = (M + BM - 1) / BM, T = tiles_m * tiles_n;
    const int full = T / n_cu * n_cu, rest = T - full;
    const int ks_max = rest > 0 ? std::max(1, std::min(kMaxCut, stages / kMinCutStages)) : 1;
    for (int ks = 1; ks <= ks_max; ++ks) {
      const int pieces = rest * ks, r2 = (pieces + n_cu - 1) / n_cu;
      const size_t bytes = ks > 1 ? (size_t)pieces * BM * BN * 4 : 0;
      if (bytes > kMaxPartBytes) break;
      double cost = (T / n_cu) * (stages * step_us(RT, n_cu) + t_fixed + t_store);
      if (r2 > 0) cost += r2 * (((stages + ks - 1) / ks) * step_us(RT, std::min(pieces, n_cu)) + t_fixed + (ks == 1 ? t_store : 0.0));
      cost += sum_us(bytes);
      if (best.cost_us < 0 || (g_force_ks ? ks <= g_force_ks && (ks > best.ks || cost < best.cost_us) : cost < best.cost_us))
        best = make(RT, ks, full, cost);
    }
  }
  if (share < n_cu && !g_force_rt && M > 128 && (best.ks == 1 || best.full == 0)) {
    const int ks = best.ks, own = best.RT, len = (stages + ks - 1) / ks;
    best.cost_us = -1;
    for (int RT = 8; RT >= 4; --RT) {
      if (!allowed(RT) || (RT != 4 && RT != 8 && RT != own)) continue;
      const int BM = 32 * RT, n = (M + BM - 1) / BM * tiles_n * ks, last = n % share;  // workgroups, and those of the last round
      const size_t bytes = ks > 1 ? (size_t)n * BM * BN * 4 : 0;
      if (bytes > kMaxPartBytes) continue;
      const double fixed = t_fixed + (ks == 1 ? t_store : 0.0);
      double cost = (n / share) * (len * step_us(RT, share) + fixed) + sum_us(bytes);
      if (last) cost += len * step_us(RT, last) + fixed;
      if (best.cost_us < 0 || cost < best.cost_us) best = make(RT, ks, 0, cost);
    }
  }
  return best;
}

int gemm2_pass_tiles(const Gemm2Cut& c, size_t part_bytes) {
  if (c.ks < 2) return 0;
  const size_t fit = part_bytes / ((size_t)c.ks * c.RT * (32 * BN * 4));
  if (fit >= (size_t)c.rest) return c.rest;
  if (fit < 1) return 0;
  const int passes = (c.rest + (int)fit - 1) / (int)fit;
  return (c.rest + passes - 1) / passes;
}

size_t gemm2_part_bytes(int max_M, int tiles_n, int stages) {
  const int n_cu = device_cus();
  size_t most = 0;
  for (int M = std::min(128, max_M);; M = std::min(M + 32, max_M)) {  // a plan depends on the rows through their tiles alone
    for (bool f32out : {false, true}) {
      const Gemm2Cut c = gemm2_cut(M, tiles_n, stages, n_cu, n_cu, true, f32out);
      if (c.ks > 1) most = std::max(most, (size_t)c.rest * c.ks * c.RT * (32 * BN * 4));
    }
    if (M == max_M) return most;
  }
}

// Once per process, whichever thread comes first; a failure is not kept, the next caller tries again.
harli_status gemm2_prepare() {
  static std::mutex mu;
  static bool ready = false;
  std::lock_guard<std::mutex> lk(mu);
  if (ready) return HARLI_OK;
  for (harli_status (*init)() : {&gemm2_init<4>, &gemm2_init<5>, &gemm2_init<6>, &gemm2_init<7>, &gemm2_init<8>}) {
    const harli_status rc = init();
    if (rc != HARLI_OK) return rc;
  }
  ready = true;
  return HARLI_OK;
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
  {
    const harli_status rc = gemm2_prepare();
    if (rc != HARLI_OK) return rc;
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
  const Gemm2Cut plan = gemm2_cut(a.M, a.tiles_n, stages, n_cu, share > 0 ? std::min(share, n_cu) : n_cu, a.half != 0, f32out);
  const Gemm2Plan pl = gemm2_plan(a.M, a.tiles_n, plan.RT, n_cu);
  const bool banded = gemm2_banded(plan, pl);
  const int per_pass = gemm2_pass_tiles(plan, a.part ? a.part_bytes : 0);
  if (plan.ks > 1 && per_pass < 1) return fail(HARLI_ERR_INVALID, "gemm2: no room for the partial tiles of one tile");
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
  harli_status rc = HARLI_OK;
  switch (plan.RT) {
    case 4: rc = gemm2_run<4>(a, plan, pl, banded, per_pass, st); break;
    case 5: rc = gemm2_run<5>(a, plan, pl, banded, per_pass, st); break;
    case 6: rc = gemm2_run<6>(a, plan, pl, banded, per_pass, st); break;
    case 7: rc = gemm2_run<7>(a, plan, pl, banded, per_pass, st); break;
    case 8: rc = gemm2_run<8>(a, plan, pl, banded, per_pass, st); break;
  }
  if (rc != HARLI_OK) return rc;
  HARLI_HIP(timer.end(st));
  HARLI_HIP(hipGetLastError());
  return HARLI_OK;
}

}  // namespace harli
