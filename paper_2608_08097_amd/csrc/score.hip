// Block importance from the lookahead queries (paper §4.2.1): Quest upper bound
// of every candidate block for every draft row, maximum over the G x D rows of
// a KV head.
//
// The bound is a dense [rows x 256] x [256 x 16] product per tile of 16 blocks
// (score_core.h: [q+ | q-] . [kmax ; kmin], exact bf16 operands, fp32
// accumulation on v_mfma_f32_16x16x32_bf16) for the 5 to 64 rows of a KV head
// (fewer go to the vector-ALU scorer of score_valu.hip), and the row maximum is
// taken in the epilogue with two cross-lane exchanges.
//
// Memory: every summary byte is read once. A wave owns TPW consecutive tiles
// of 16 blocks; for a tile, lane (g, n) loads 16 bytes of block n at byte
// offset 64*step + 16*g of its kmax row and of its kmin row, so four lanes
// read 64 contiguous bytes and the wave covers the tile's 2 x 4 KiB in 8
// load instructions. All loads of a wave are issued before its first MFMA.
//
// The operands of the rows go to LDS once per workgroup and each wave holds
// one row tile's operands at a time (4 summary tiles per wave with one row
// tile, 2 with more). Measured on MI355X against keeping all operands in
// every wave's registers: 64 rows (16 requests x 65,536 tokens, B = 32,
// 134 MB) 30.1 us against 38.5 us (4 waves per SIMD instead of 2); 16 rows
// (8 x 131,072 tokens, 268 MB) 48.6 us against 49.9 us (fewer query reads;
// 3, 5, 6 and 8 summary tiles per wave: 48.6, 50.8, 51.7 and 56.6 us).
// Summary addresses are a wave-uniform base and a 32-bit lane offset
// (score_tiles_load): per-lane 64-bit addresses and zero-filled lanes past the
// candidates took registers that cost a wave per SIMD. Scores and selection
// before and after: the 64-row case 35.0 -> 32.1 us, the 16-row case 56.7 ->
// 55.6, 32 requests of 16K-32K tokens (16 rows, 204 MB) 49.7 -> 46.1 us.
#include "oasis_internal.h"
#include "score_core.h"

namespace oasis {

namespace {

// The [q+ | q-] operands of the KV head's rows are built once per workgroup in
// LDS, laid out per lane so that each MFMA operand is one conflict-free
// 16-byte LDS read, and a wave walks the row tiles in its outer loop. Only one
// row tile's operands are then live in registers, which leaves room for more
// summary tiles in flight per CU, and the queries are read once per workgroup
// rather than once per wave.
template <int NRT, int TPW>
__global__ __launch_bounds__(256) void score_kernel(ScoreArgs a) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4;
  const int n = lane & 15;
  const int rh = blockIdx.y;
  const int r = rh / a.Hkv;
  const int h = rh - r * a.Hkv;
  const Ctx c = ctx_blocks(a.ctx_len[r], a.B, a.NBmax);
  const int ntiles = (a.NBmax + 15) >> 4;
  // Workgroups are dealt to the 8 XCDs round-robin by linear id, so with a
  // grid 8 (or a multiple of 8) tile groups wide one XCD would always get the
  // same tile group of every row, and the tail groups of short rows (no live
  // blocks) would leave their XCDs idle; rotating the group by the row spreads
  // every group over all XCDs (ragged 16K-32K-token rows: 48.0 -> 47.0 us).
  const int group = (int)((blockIdx.x + blockIdx.y) % gridDim.x);
  float* srow = a.scores + (long long)rh * a.NBmax;
  const int tile0 = (group * 4 + wave) * TPW;
  __shared__ ScoreQOperands<NRT> s_q;

  // A workgroup past the candidates only writes padding: tables are sized for the
  // longest context, so with short contexts in long tables most workgroups end
  // here. Measured on MI355X, scores and selection, without and with this exit
  // (8 KV heads): 16 requests of 4K-8K tokens in 8,000-block tables, 16 rows 32.2
  // and 21.7 us, 64 rows 43.1 and 22.6; 64 requests of 1.5K-2.5K in 2,032-block
  // tables, 32 rows 37.9 and 24.3.
  auto padding = [&]() __attribute__((always_inline)) {
    const int blk0 = group * 4 * TPW * 16;
    if (blk0 < c.n_cand) return false;
    const int end = min(blk0 + 4 * TPW * 16, a.NBmax);
    for (int b = blk0 + threadIdx.x; b < end; b += 256) srow[b] = -INFINITY;
    return true;
  };
  // One row tile loads its queries before it waits for the context length (full
  // rows of 8 x 131,072 tokens 56.9 -> 56.0 us); with more there is no difference
  // in full rows, and the workgroups that end need not read them (64 rows, 16
  // requests as above: 29.9 -> 22.6).
  if constexpr (NRT > 1) {
    if (padding()) return;
  }

  // queries first (cache-resident, needed first), then the summaries of all TPW tiles
  u32x4 qraw[NRT];
#pragma unroll
  for (int j = 0; j < NRT; ++j) qraw[j] = score_q_raw(a, r, h, threadIdx.x + j * 256);
  if constexpr (NRT == 1) {
    asm volatile("" ::: "memory");  // the loads stay before the exit
    if (padding()) return;
  }
  const long long sum_base = (long long)rh * a.NBmax * kHeadDim;
  const uint16_t* kmx = a.kmax + sum_base;
  const uint16_t* kmn = a.kmin + sum_base;
  u32x4 vmax[TPW][4], vmin[TPW][4];
  // a wave past the candidates, in a workgroup with some, reads one row instead
  const bool alive = tile0 * 16 < c.n_cand;
  score_tiles_load<TPW>(kmx, kmn, alive ? tile0 : 0, alive ? c.n_cand : 1, g, n, vmax, vmin);
#pragma unroll
  for (int j = 0; j < NRT; ++j) score_q_store<NRT>(s_q, threadIdx.x + j * 256, qraw[j]);
  __syncthreads();  // every wave reaches it: waves past the last tile return only below
  if (tile0 >= ntiles) return;

  float best[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) best[t] = -INFINITY;
  if (alive) {
#pragma unroll
    for (int v = 0; v < NRT; ++v) {
      bf16x8 ap[4], an[4];
      score_q_tile<NRT>(s_q, v, lane, ap, an);
#pragma unroll
      for (int t = 0; t < TPW; ++t) best[t] = score_tile_fold(ap, an, vmax[t], vmin[t], best[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int tile = tile0 + t;
    if (tile >= ntiles) break;
    const float b = score_lane_reduce(best[t]);
    const int blk = tile * 16 + n;
    if (g == 0 && blk < a.NBmax) srow[blk] = blk < c.n_cand ? b : -INFINITY;
  }
}

template <int NRT, int TPW>
hipError_t launch_t(const ScoreArgs& a, hipStream_t s, const LaunchTiming& t) {
  const int ntiles = (a.NBmax + 15) / 16;
  const dim3 grid((unsigned)((ntiles + 4 * TPW - 1) / (4 * TPW)), (unsigned)(a.R * a.Hkv));
  launch_kernel(score_kernel<NRT, TPW>, grid, dim3(256), s, t, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score(const ScoreArgs& a, hipStream_t s, const LaunchTiming& t) {
  const int rows = a.num_draft * a.G;
  // a quarter of a 16-row tile or less: no MFMA
  if (rows <= kScoreValuMaxRows) return launch_score_valu(a, s, t);
  switch ((rows + 15) / 16) {
    case 1: return launch_t<1, 4>(a, s, t);
    case 2: return launch_t<2, 2>(a, s, t);
    case 3: return launch_t<3, 2>(a, s, t);
    case 4: return launch_t<4, 2>(a, s, t);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace oasis
