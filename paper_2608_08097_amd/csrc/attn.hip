// Block-sparse GQA decode attention over the HBM working set (paper §4.2.1:
// the normal and draft queries are stacked and attend one resident KV set in
// one call; §5.2: the K selected blocks plus the active local block).
//
// Work decomposition. The rows of one KV head are its G query heads times the
// T stacked query tokens (20 at G = 4, T = 5). The attended tokens of a
// (request, KV head) are cut into units of 32 tokens (two slots at B = 16,
// one at B = 32); a workgroup of 4 waves handles a contiguous range of units
// (a split) and every wave a strided subset of them, with its own online
// softmax. The waves are merged through LDS; with one split the workgroup
// writes the bf16 outputs and the log-sum-exp itself, otherwise each split
// writes one partial (unnormalised output, running max, running sum) per row
// and a second kernel merges the splits. (A merge by the last-arriving
// workgroup of a head inside the same kernel needs an agent-scope release
// per workgroup, which on MI355X writes back the XCD's L2; measured on a
// 256-workgroup stand-in, that cost 14.8 us per call against 2.6 us for the
// second launch.)
//
// One 32-token unit for one 16-row tile:
//   S^T (tokens x rows) = K (tokens x d) . Q^T (d x rows): 2 token tiles x
//       4 k-steps of v_mfma_f32_16x16x32_bf16. Token tile tau assigns MFMA row
//       i to unit token 8*(i/4) + 4*tau + i%4, so after both tiles lane (g, n)
//       holds query row n against unit tokens 8g .. 8g+7.
//   P (bf16) is then directly the B operand of
//   O^T (d x rows) += V^T (d x tokens) . P^T (tokens x rows): 8 d-tiles, one
//       MFMA each; lane (g, i) of the A operand needs V[8g .. 8g+7][d = i],
//       which is one 16-byte load because the pool keeps V transposed per
//       slot and head (d x B).
// So K and V go straight from HBM into MFMA registers with 16-byte loads and
// no LDS round trip; every lane owns one query row, so the running max and sum
// need only two cross-lane exchanges per unit.
//
// With more than two row tiles (G * T > 32 rows) the registers of one wave no
// longer hold every tile's accumulators next to two units of K and V; there a
// workgroup has two waves per row tile and the unit's K and V cross HBM once,
// into LDS, for all of them (attn_split_rows_kernel).
#include <mutex>

#include "oasis_internal.h"

namespace oasis {
namespace {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// XCD-aware placement of the `parts` items of each (request, KV head) pair:
// workgroup ids are dealt round-robin over the 8 XCDs, so id i works on item
// (i % 8) * ceil(items / 8) + i / 8 and every XCD takes one contiguous run of
// the items in pair order. The parts of a pair share query rows and partials
// in one L2, the heads of a request, whose slots are adjacent in the pools,
// share its XCD, and any number of pairs spreads over all XCDs. (Pairs dealt
// modulo 8, as before: 90 requests x 8 KV heads, 761 MB, 143 against 124 us a
// call, 116 with V past the caches; 64 x 8, 544 MB, 103 and 94.) With fewer than 8 pairs each takes an
// XCD of its own, so that its merge reads the partials from the L2 that holds
// them (1 pair: 9.3 us, spread over the XCDs 10.2). Returns -1 past the last item.
__device__ __forceinline__ int xcd_item(int wg, int pairs, int parts) {
  const int items = pairs * parts;
  const int per = pairs < 8 ? parts : (items + 7) >> 3;
  const int item = (wg & 7) * per + (wg >> 3);
  return item < items ? item : -1;
}
inline unsigned xcd_grid(long long pairs, long long parts) {
  return (unsigned)(pairs < 8 ? parts * 8 : (pairs * parts + 7) / 8 * 8);
}

// K and V registers of one 32-token unit (the operands of its MFMAs).
struct UnitRegs {
  u32x4 k[2][4];
  u32x4 v[8];
};

// Byte offsets of a lane's operands inside a unit, from the unit's first slot:
// with every unit address a wave-uniform base plus a 32-bit lane offset and a
// constant, a load costs no 64-bit vector arithmetic. The second slot of a
// B = 16 unit sits slot_bytes further (k1, v1); offsets k0, v0 stay in the first.
struct UnitOffsets {
  uint32_t k0, v0, k1, v1;
};
template <int BS>
__device__ __forceinline__ UnitOffsets unit_offsets(long long slot_elems, int g, int i) {
  UnitOffsets o;
  // K: lane (g, i), token tile tau -> unit token 8*(i/4) + 4*tau + i%4 (the tile is in the constant part)
  const uint32_t tok = 8 * (i >> 2) + (i & 3);
  o.k0 = ((BS == 16 ? tok & 15 : tok) * kHeadDim + g * 8) * 2;
  // V^T: lane (g, i), d-tile dt -> V[tokens 8g .. 8g+7][d = dt*16 + i]
  o.v0 = (i * BS + (BS == 16 ? g & 1 : g) * 8) * 2;
  const uint32_t slot_bytes = BS == 16 ? (uint32_t)slot_elems * 2 : 0;
  o.k1 = o.k0 + (i >= 8 ? slot_bytes : 0);
  o.v1 = o.v0 + (g >= 2 ? slot_bytes : 0);
  return o;
}

// Unit u (wave-uniform) covers slots s0 = 2u, s1 = 2u + 1 at B = 16 or slot u
// at B = 32. Every load is unconditional: a second slot past the pool is
// replaced by the first (always inside the pool) and only the token counts
// n0 / n1 decide which tokens count. Free slots may hold anything, even NaN;
// their K only yields masked scores and their V is cleared below.
//
// u < 0 is a placeholder unit: the loads are issued anyway (every lane on the
// first bytes of the local slot, one cache line) and count nothing. Issuing the
// same number of loads on every path keeps the compiler's wait counts exact,
// so waiting for the current unit never drains the prefetched one. With STREAM
// (kStreamBytes) V is read past the caches; K is not, since two of its loads
// share each line (22 requests x 8 heads, 187 MB: plain 36.9 us, V 32.2, K 37.7,
// both 37.5).
template <int BS, bool STREAM>
__device__ __forceinline__ void load_unit(UnitRegs& ur, int u, int ks, const uint16_t* pk, const uint16_t* pv,
                                          long long slot_elems, const UnitOffsets& o) {
  const bool real = u >= 0;
  const int s0 = real ? (BS == 16 ? 2 * u : u) : ks;
  const bool two = BS == 16 && s0 < ks;
  const uint32_t ok = real ? (two ? o.k1 : o.k0) : 0u;
  const uint32_t ov = real ? (two ? o.v1 : o.v0) : 0u;
  const char* kb = reinterpret_cast<const char*>(pk + (long long)s0 * slot_elems);
  const char* vb = reinterpret_cast<const char*>(pv + (long long)s0 * slot_elems);
#pragma unroll
  for (int tau = 0; tau < 2; ++tau)
#pragma unroll
    for (int st = 0; st < 4; ++st) ur.k[tau][st] = ldg16(kb + ok + (tau * 4 * kHeadDim + st * 32) * 2);
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) ur.v[dt] = ldg16_once<STREAM>(vb + ov + dt * 16 * BS * 2);
}

// Attended tokens of the two slots of unit u (u < 0: none): a slot below k_slots
// counts B tokens when bit `bit` (first slot) / `bit + 1` (second slot, B = 16)
// of the validity mask is set; slot k_slots is the local block.
template <int BS>
__device__ __forceinline__ void unit_counts(int u, int ks, int local_len, uint64_t vmask, int bit, int& n0,
                                            int& n1) {
  const int s0 = BS == 16 ? 2 * u : u;
  const int s1 = s0 + 1;
  n0 = u < 0 ? 0 : (s0 < ks ? (((vmask >> bit) & 1) ? BS : 0) : (s0 == ks ? local_len : 0));
  n1 = (BS == 16 && u >= 0) ? (s1 < ks ? (((vmask >> (bit + 1)) & 1) ? BS : 0) : (s1 == ks ? local_len : 0)) : 0;
}

// Tokens of the unit that lane (g, i) scores: 8g .. 8g+7 of the unit (slot 0 holds
// unit tokens 0 .. B-1). The first `keep` of them are attended (0 .. 8).
template <int BS>
__device__ __forceinline__ int lane_keep(int n0, int n1, int g) {
  const int cnt = BS == 16 ? (g < 2 ? n0 : n1) : n0;
  const int k = cnt - (BS == 16 ? (g & 1) * 8 : 8 * g);
  return k < 0 ? 0 : (k > 8 ? 8 : k);
}

// Zero the V values of tokens that are not attended (their probability is 0,
// but 0 * NaN would poison the accumulator). Lane (g, i) holds V^T of the same
// 8 tokens it scores; only lanes with keep < 8 change anything.
__device__ __forceinline__ void mask_unit_v(UnitRegs& ur, int keep) {
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t lo = (2 * w) < keep ? 0x0000FFFFu : 0u;
      const uint32_t hi = (2 * w + 1) < keep ? 0xFFFF0000u : 0u;
      ur.v[dt][w] &= (lo | hi);
    }
}

// Online-softmax update of one wave with one 32-token unit (all row tiles).
//
// Lazy rescaling: every row keeps a reference maximum m_ref (the same in the
// four lanes of the row) and each lane a partial sum over its own tokens.
// Probabilities are exp2(x - m_ref); only when some score of the wave exceeds
// its row reference by more than kLazyTh (a wave-uniform branch, rare once the
// first unit has been seen) are the row maxima exchanged across lanes and the
// accumulators rescaled. Probabilities stay below 2^kLazyTh, far inside the
// fp32 range, and the result is the same softmax.
//
// `partial` (wave-uniform) is set when some lane has keep < 8: only then are
// unattended scores set to -inf; a fully attended unit skips that work.
constexpr float kLazyTh = 8.f;

template <int NT, int BS>
__device__ __forceinline__ void process_unit(const UnitRegs& cur, int keep, bool partial, const bf16x8 (&qb)[NT][4],
                                             float (&m_ref)[NT], float (&l_part)[NT], f32x4 (&acc)[NT][8],
                                             float scale_log2) {
#pragma unroll
  for (int v = 0; v < NT; ++v) {
    f32x4 sc[2];
#pragma unroll
    for (int tau = 0; tau < 2; ++tau) {
      f32x4 s4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < 4; ++st)
        s4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(cur.k[tau][st]), qb[v][st], s4, 0, 0, 0);
      sc[tau] = s4;
    }
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = sc[e >> 2][e & 3] * scale_log2;
    if (partial) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = e < keep ? x[e] : -INFINITY;
    }
    const float lmax = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    if (__builtin_amdgcn_ballot_w64(lmax > m_ref[v] + kLazyTh)) {
      float rmax = fmaxf(lmax, __shfl_xor(lmax, 16));
      rmax = fmaxf(rmax, __shfl_xor(rmax, 32));
      const float m_new = fmaxf(m_ref[v], rmax);
      const float alpha = m_new == -INFINITY ? 1.f : fast_exp2(m_ref[v] - m_new);
      l_part[v] *= alpha;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) acc[v][dt] *= alpha;
      m_ref[v] = m_new;
    }
    const float m_use = m_ref[v] == -INFINITY ? 0.f : m_ref[v];
    bf16x8 pb;
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float pe = fast_exp2(x[e] - m_use);
      psum += pe;
      pb[e] = (__bf16)pe;
    }
    l_part[v] += psum;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      acc[v][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(cur.v[dt]), pb, acc[v][dt], 0, 0, 0);
  }
}

// Normalised bf16 output of 4 dimensions of one row, and its log-sum-exp.
__device__ __forceinline__ void write_output(const AttnArgs& a, int r, int h, int row, int c4, f32x4 o, float M,
                                             float L) {
  const int t = row / a.G;
  const int qh = h * a.G + (row - t * a.G);
  const long long orow = ((long long)r * a.T + t) * a.Hq + qh;
  const float inv = L > 0.f ? 1.f / L : 0.f;
  const uint32_t w0 = f32_to_bf16_bits(o[0] * inv) | (f32_to_bf16_bits(o[1] * inv) << 16);
  const uint32_t w1 = f32_to_bf16_bits(o[2] * inv) | (f32_to_bf16_bits(o[3] * inv) << 16);
  *reinterpret_cast<uint2*>(a.out + orow * kHeadDim + c4 * 4) = make_uint2(w0, w1);
  if (c4 == 0 && a.lse) a.lse[orow] = L > 0.f ? (M + __log2f(L)) * 0.69314718055994531f : -INFINITY;
}

// Slot-map validity of the wave's units t0 .. t0 + kChunk - 1 (unit t of the wave is
// u_first + t * kW): lane l reads the map entry of slot l % 2 of unit t0 + l / 2
// (B = 16) or of unit t0 + l (B = 32); ballot(slot < k_slots && entry >= 0) is then
// the mask unit_counts reads (bit 2j + e or j), so the unit loop loads no slot map.
// The load is split from the test: it is issued unconditionally (index clamped
// into the map; with k_slots = 0, where the map may be NULL, from `fallback`,
// any valid int, whose value the slot test then ignores), so that nothing waits
// for it until the mask is needed.
template <int BS>
__device__ __forceinline__ int unit_slot(int u_first, int t0, int lane) {
  const int j = BS == 16 ? lane >> 1 : lane;
  return BS == 16 ? 2 * (u_first + (t0 + j) * kW) + (lane & 1) : u_first + (t0 + j) * kW;
}
__device__ __forceinline__ const int32_t* map_addr(const int32_t* smap, int ks, int slot, const int32_t* fallback) {
  return ks > 0 ? smap + (slot < ks ? slot : ks - 1) : fallback;
}
__device__ __forceinline__ int map_load(const int32_t* smap, int ks, int slot, const int32_t* fallback) {
  return *map_addr(smap, ks, slot, fallback);
}
__device__ __forceinline__ uint64_t map_mask(int ks, int slot, int entry) {
  return __builtin_amdgcn_ballot_w64(slot < ks && entry >= 0);
}

// Split kernel for one or two row tiles (up to 32 rows): K and V straight
// into registers, every wave a strided subset of the part's units.
//
// Units whose slots are all free are not read: the first two units of a wave
// are loaded before the slot map has arrived, every later one is the next unit
// with an attended slot. At 64 requests x 8 KV heads with contexts of 200 to
// 3,000 tokens in 128-slot pools (383 of 541 MB attended) a call takes 75.7 us
// (71.4 with V past the caches), against 104 when every slot is read. Every unit's addresses are a
// wave-uniform base and a 32-bit lane offset (UnitOffsets); 64-bit vector
// addresses took 17.9 against 16.9 us at 8 x 131,072 tokens (68 MB).
template <int NT, int BS, bool STREAM>
__global__ __launch_bounds__(kW * 64) void attn_split_kernel(AttnArgs a) {
  static_assert(NT <= 2, "three or more row tiles take attn_split_rows_kernel");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4;
  const int i = lane & 15;
  const int item = xcd_item(blockIdx.x, a.R * a.Hkv, a.nsplit);
  if (item < 0) return;
  const int ks = a.k_slots;
  const long long slot_elems = (long long)a.Hkv * BS * kHeadDim;
  const int rh = item / a.nsplit;
  const int split = item - rh * a.nsplit;
  const int r = rh / a.Hkv;
  const int h = rh - r * a.Hkv;
  const long long pool_off = (long long)r * (ks + 1) * slot_elems + (long long)h * BS * kHeadDim;
  const uint16_t* pk = a.pool_k + pool_off;
  const uint16_t* pv = a.pool_v + pool_off;
  const int32_t* smap = a.slot_map + (long long)rh * ks;
  const UnitOffsets uo = unit_offsets<BS>(slot_elems, g, i);
  const int u_begin = split * a.units_per_split;
  const int u_end = min(a.n_units, u_begin + a.units_per_split);
  // unit t of this wave is u_first + t * kW, t < nt
  const int u_first = u_begin + wave;
  const int nt = u_first < u_end ? (u_end - u_first + kW - 1) / kW : 0;
  auto unit = [&](int t) { return t < nt ? u_first + t * kW : -1; };
  constexpr int kChunk = BS == 16 ? 32 : 64;  // units per validity mask

  // The first unit's loads go out before anything else, so that no wave starts
  // by waiting for a scalar or query load; the queries, the slot map and the
  // context length follow.
  UnitRegs ua, ub;
  load_unit<BS, STREAM>(ua, unit(0), ks, pk, pv, slot_elems, uo);

  // Q^T operand: lane (g, i) holds row v*16 + i of tile v, dims st*32 + 8g .. +8.
  bf16x8 qb[NT][4];
#pragma unroll
  for (int v = 0; v < NT; ++v) {
    const int row = v * 16 + i;
    if (row < a.rows) {
      const int tq = row / a.G;
      const int qh = h * a.G + (row - tq * a.G);
      const uint16_t* qrow = a.q + (((long long)r * a.T + tq) * a.Hq + qh) * kHeadDim;
#pragma unroll
      for (int st = 0; st < 4; ++st) qb[v][st] = as_bf16x8(ldg16(qrow + st * 32 + g * 8));
    } else {
#pragma unroll
      for (int st = 0; st < 4; ++st) qb[v][st] = as_bf16x8(u32x4{0, 0, 0, 0});
    }
  }
  int map_entry = map_load(smap, ks, unit_slot<BS>(u_first, 0, lane), a.ctx_len + r);
  // a vector load (relaxed atomic) whose value is pinned to a VGPR until the
  // next unit's loads are out, so that the wait for it comes after them
  int ctx_raw = __hip_atomic_load(a.ctx_len + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __builtin_amdgcn_sched_barrier(0);
  load_unit<BS, STREAM>(ub, unit(1), ks, pk, pv, slot_elems, uo);
  __builtin_amdgcn_sched_barrier(0);  // both units' loads are issued before the first wait

  float m_run[NT], l_run[NT];  // row reference maximum (log2 units) and this lane's partial sum
  f32x4 acc[NT][8];
#pragma unroll
  for (int v = 0; v < NT; ++v) {
    m_run[v] = -INFINITY;
    l_run[v] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[v][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // the map entries and the context length are in
  asm volatile("" : "+v"(map_entry), "+v"(ctx_raw));
  const int local_len = ctx_blocks(__builtin_amdgcn_readfirstlane(ctx_raw), BS, a.NBmax).local_len;
  int chunk = 0;
  uint64_t vmask = map_mask(ks, unit_slot<BS>(u_first, 0, lane), map_entry);
  // Units of the current chunk with an attended slot, one bit each at the
  // position of their first slot in vmask; the unit of the local block counts.
  auto live_units = [&]() {
    uint64_t m = BS == 16 ? (vmask | (vmask >> 1)) & 0x5555555555555555ull : vmask;
    const int tl = a.n_units - 1 - u_first;  // t of the local unit, times kW
    if (tl >= 0 && tl % kW == 0) {
      const int t = tl / kW - chunk * kChunk;
      if (t >= 0 && t < kChunk) m |= 1ull << (BS == 16 ? 2 * t : t);
    }
    return m;
  };
  uint64_t live = live_units();
  // The next unit of this wave after t to attend (nt: none): the next one of its
  // chunk with an attended slot, or the chunk's last one (which then counts no
  // token); a new chunk's map is read when its first unit is reached.
  auto next_unit = [&](int t) __attribute__((always_inline)) {
    ++t;
    if ((t & (kChunk - 1)) == 0 && t < nt) {
      chunk = t / kChunk;
      const int slot = unit_slot<BS>(u_first, t, lane);
      vmask = map_mask(ks, slot, map_load(smap, ks, slot, a.ctx_len + r));
      live = live_units();
    }
    const int p = t & (kChunk - 1);
    const uint64_t rest = live >> (BS == 16 ? 2 * p : p) | 1ull << (BS == 16 ? 2 * (kChunk - 1 - p) : kChunk - 1 - p);
    return min(nt, t + (BS == 16 ? __builtin_ctzll(rest) / 2 : __builtin_ctzll(rest)));
  };
  // attended tokens of the slots of unit t, from the current chunk's mask
  auto counts = [&](int t, int& n0, int& n1) __attribute__((always_inline)) {
    unit_counts<BS>(unit(t), ks, local_len, vmask, BS == 16 ? 2 * (t & (kChunk - 1)) : (t & (kChunk - 1)), n0, n1);
  };
  // One unit: V of unattended tokens cleared, then the online softmax.
  auto run = [&](UnitRegs& cur, int n0, int n1) __attribute__((always_inline)) {
    const int keep = lane_keep<BS>(n0, n1, g);
    const bool partial = __builtin_amdgcn_ballot_w64(keep < 8) != 0;
    if (partial) mask_unit_v(cur, keep);
    process_unit<NT, BS>(cur, keep, partial, qb, m_run, l_run, acc, a.scale_log2);
  };

  // The next unit's K/V loads are issued before the current unit is computed
  // (one exposed memory latency per wave, not per unit). Loads past the wave's
  // last unit are placeholders on the local slot (cache-resident), so the
  // compiler's wait counts stay exact.
  int ta = 0, tb = 1, na0, na1, nb0, nb1;
  counts(0, na0, na1);
  counts(1, nb0, nb1);
  if (nt > 0) for (;;) {
    run(ua, na0, na1);
    if (tb >= nt) break;
    ta = next_unit(tb);
    load_unit<BS, STREAM>(ua, unit(ta), ks, pk, pv, slot_elems, uo);
    counts(ta, na0, na1);
    run(ub, nb0, nb1);
    tb = next_unit(ta);
    load_unit<BS, STREAM>(ub, unit(tb), ks, pk, pv, slot_elems, uo);
    counts(tb, nb0, nb1);
    if (ta >= nt) break;
  }
  // row sums: add the partial sums of the four lanes of every row
#pragma unroll
  for (int v = 0; v < NT; ++v) {
    l_run[v] += __shfl_xor(l_run[v], 16);
    l_run[v] += __shfl_xor(l_run[v], 32);
  }

  // ---- merge the waves of this workgroup through LDS -----------------------
  // Each wave publishes its row maxima and sums; every lane then reads those of
  // all waves for its rows (all reads issued before any is used, no branch on
  // them), rescales its accumulators to the merged maximum and writes them to
  // its slice; finally every thread sums the slices of a few (row, 4-dimension)
  // positions, all their reads again issued at once.
  constexpr int kRows = NT * 16;
  constexpr int kPad = kHeadDim + 4;
  __shared__ float s_m[kW][kRows], s_l[kW][kRows], s_ml[2][kRows];
  __shared__ __align__(16) float s_o[kW][kRows][kPad];
  if (g == 0) {
#pragma unroll
    for (int v = 0; v < NT; ++v) {
      s_m[wave][v * 16 + i] = m_run[v];
      s_l[wave][v * 16 + i] = l_run[v];
    }
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NT; ++v) {
    const int row = v * 16 + i;
    float mw[kW], lw[kW];
#pragma unroll
    for (int w = 0; w < kW; ++w) {
      mw[w] = s_m[w][row];
      lw[w] = s_l[w][row];
    }
    float M = mw[0];
#pragma unroll
    for (int w = 1; w < kW; ++w) M = fmaxf(M, mw[w]);
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < kW; ++w) L += mw[w] == -INFINITY ? 0.f : lw[w] * fast_exp2(mw[w] - M);
    const float f = m_run[v] == -INFINITY ? 0.f : fast_exp2(m_run[v] - M);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[v][dt] *= f;
    if (wave == 0 && g == 0) {
      s_ml[0][row] = M;
      s_ml[1][row] = L;
    }
  }
#pragma unroll
  for (int v = 0; v < NT; ++v)
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      *reinterpret_cast<f32x4*>(&s_o[wave][v * 16 + i][dt * 16 + 4 * g]) = acc[v][dt];
  __syncthreads();

  const int nsplit = a.nsplit;
  const long long pbase = ((long long)rh * nsplit + split) * a.rows;
  constexpr int kPer = (kRows * (kHeadDim / 4) + kW * 64 - 1) / (kW * 64);  // positions per thread
  const int npos = a.rows * (kHeadDim / 4);
  f32x4 o[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int pos = threadIdx.x + j * kW * 64;
    const int row = (pos < npos ? pos : 0) >> 5;
    const int c4 = pos & 31;
    o[j] = *reinterpret_cast<const f32x4*>(&s_o[0][row][c4 * 4]);
#pragma unroll
    for (int sl = 1; sl < kW; ++sl) o[j] += *reinterpret_cast<const f32x4*>(&s_o[sl][row][c4 * 4]);
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int pos = threadIdx.x + j * kW * 64;
    if (pos >= npos) break;
    const int row = pos >> 5;
    const int c4 = pos & 31;
    const float M = s_ml[0][row], L = s_ml[1][row];
    if (nsplit == 1) {  // the only split: finish here
      write_output(a, r, h, row, c4, o[j], M, L);
    } else {
      *reinterpret_cast<f32x4*>(a.part_o + (pbase + row) * kHeadDim + c4 * 4) = o[j];
      if (c4 == 0) {
        a.part_ml[(pbase + row) * 2 + 0] = M;
        a.part_ml[(pbase + row) * 2 + 1] = L;
      }
    }
  }
}

// Split kernel for many row tiles (NT >= 3: G * T > 32 rows). Each unit's K and
// V cross HBM once: its 16 chunks (8 of K, 8 of V, 16 bytes a lane, in the MFMA
// operand layout of load_unit) are loaded straight into LDS, and one wave per
// row tile reads all 16 back as conflict-free 16-byte LDS reads. A workgroup
// has two such teams of waves, on alternate units (kTeams = 1: launch_t): with one (3 to 5 waves)
// a unit's chain of LDS reads, score products, softmax and PV products paces
// the loads, since a SIMD then has one wave, or none, to issue from. A step
// holds one unit per team; a ring of kRowsStages steps keeps kRowsStages - 1 in
// flight; one barrier per step publishes it to every wave and frees the stage
// of the one before. The teams' softmax states are merged through LDS at the
// end, so that the workgroup still leaves one partial per row.
//
// Measured on MI355X, per call: 22 requests x 8 KV heads at 20,000 tokens, 72
// rows (B = 16, 2,048-token budget, 189 MB) 68 us with one team, 45 us with two;
// 25 requests at B = 32 and budget 4,096 (429 MB) 109 and 83 us; 16 x 65,536
// tokens (B = 32, 72 rows, 274 MB; two splits per head and a merge) 63 and
// 61 us (with plain loads, as the figures below; 53.3 past the caches). Three or four teams (two stages fit) 62.9 us at the last, four stages
// 62.0, two 63.7. Each team's operands of a unit are read together and then
// used: reading a K chunk, waiting and reading the next took 47 us at the first.
// Short splits pay for the second team's part of the merge: 16 pairs in 15
// splits of 9 units 17.4 us, one team 16.3.
constexpr int kRowsStages = 3;
// 16 bytes a lane from global memory (base + offset, base wave-uniform) straight
// into LDS (global_load_lds_dwordx4): lane L's bytes land at lds_row + 16 L,
// lds_row being the same in every lane.
// Written as inline assembly because the compiler, which cannot tell the ring's
// stages apart once they are reused, would otherwise wait for every earlier
// such load before each one (a full drain per unit); the waits are the
// explicit vmcnt counts of the kernel instead. The "memory" clobber keeps LDS
// reads and writes in program order around it, and M0 (the LDS base operand
// of the load) is restored after it.
template <bool STREAM = false>
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t offset, void* lds_row) {
  const uint32_t lds =
      __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_row);
  uint32_t saved;
  if constexpr (STREAM)
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %3\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2 nt\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(offset), "s"(base), "s"(lds)
        : "memory");
  else
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %3\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(offset), "s"(base), "s"(lds)
        : "memory");
}

// 4 bytes a lane, as lds_dma16 (lane L's bytes land at lds_row + 4 L).
__device__ __forceinline__ void lds_dma4(const void* gsrc, void* lds_row) {
  const uint32_t lds =
      __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_row);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %1, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(gsrc), "s"(lds)
      : "memory");
}

// s_waitcnt vmcnt(N) alone (expcnt and lgkmcnt left at their maxima)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// Online softmax and PV products of one 32-token unit of one row tile, as in
// process_unit; the V operands are read by `load_v` once the scores are known.
template <typename LoadV>
__device__ __forceinline__ void unit_softmax_pv(const f32x4 (&sc)[2], int keep, bool partial, float& m_ref,
                                                float& l_part, f32x4 (&acc)[8], float scale_log2, LoadV&& load_v) {
  u32x4 v[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) v[dt] = load_v(dt);
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = sc[e >> 2][e & 3] * scale_log2;
  if (partial) {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = e < keep ? x[e] : -INFINITY;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t lo = (2 * w) < keep ? 0x0000FFFFu : 0u;
        const uint32_t hi = (2 * w + 1) < keep ? 0xFFFF0000u : 0u;
        v[dt][w] &= (lo | hi);
      }
  }
  const float lmax = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
  if (__builtin_amdgcn_ballot_w64(lmax > m_ref + kLazyTh)) {
    float rmax = fmaxf(lmax, __shfl_xor(lmax, 16));
    rmax = fmaxf(rmax, __shfl_xor(rmax, 32));
    const float m_new = fmaxf(m_ref, rmax);
    const float alpha = m_new == -INFINITY ? 1.f : fast_exp2(m_ref - m_new);
    l_part *= alpha;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[dt] *= alpha;
    m_ref = m_new;
  }
  const float m_use = m_ref == -INFINITY ? 0.f : m_ref;
  bf16x8 pb;
  float psum = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float pe = fast_exp2(x[e] - m_use);
    psum += pe;
    pb[e] = (__bf16)pe;
  }
  l_part += psum;
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
    acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(v[dt]), pb, acc[dt], 0, 0, 0);
}

template <int NT, int kTeams, int BS, bool STREAM>
__global__ __launch_bounds__(NT * kTeams * 64) void attn_split_rows_kernel(AttnArgs a) {
  constexpr int kWaves = NT * kTeams;
  constexpr int kPer = (16 + NT - 1) / NT;  // chunk loads per wave and step
  constexpr int kLook = kRowsStages - 1;    // steps in flight
  // ring of kRowsStages steps: [team][chunk][lane]; the surplus loads of every step share one row
  __shared__ __align__(16) u32x4 s_ring[kRowsStages][kTeams][16][64];
  __shared__ __align__(16) u32x4 s_junk[64];
  __shared__ __align__(16) u32x4 s_q[NT][4][64];  // the row tiles' query operands (4 k-steps)
  __shared__ int s_misc[kWaves][3][64];           // each wave's context length and two map chunks
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int team = wave / NT;       // takes every kTeams-th unit
  const int v = wave - team * NT;   // this wave's row tile
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4;
  const int i = lane & 15;
  const int item = xcd_item(blockIdx.x, a.R * a.Hkv, a.nsplit);
  if (item < 0) return;
  const int rh = item / a.nsplit;
  const int split = item - rh * a.nsplit;
  const int r = rh / a.Hkv;
  const int h = rh - r * a.Hkv;
  const int ks = a.k_slots;
  const long long slot_elems = (long long)a.Hkv * BS * kHeadDim;
  const long long pool_off = (long long)r * (ks + 1) * slot_elems + (long long)h * BS * kHeadDim;
  const uint16_t* pk = a.pool_k + pool_off;
  const uint16_t* pv = a.pool_v + pool_off;
  const int32_t* smap = a.slot_map + (long long)rh * ks;
  const UnitOffsets uo = unit_offsets<BS>(slot_elems, g, i);
  const int u_begin = split * a.units_per_split;
  const int u_end = min(a.n_units, u_begin + a.units_per_split);

  // This wave's chunk loads of its team's unit u into ring stage st (u < 0, past
  // the last unit: every lane on the first bytes of the local slot, one cache
  // line). Chunk j < 8 is K token tile j / 4 at k-step j % 4, j >= 8 V d-tile
  // j - 8, in the MFMA operand layout of load_unit.
  auto issue = [&](int u, int st) __attribute__((always_inline)) {
    const bool real = u >= 0;
    const int s0 = real ? (BS == 16 ? 2 * u : u) : ks;
    const bool two = BS == 16 && s0 < ks;
    const long long slot = (long long)s0 * slot_elems;
#pragma unroll
    for (int c = 0; c < kPer; ++c) {
      const int j = v + c * NT;
      const bool is_k = j < 8;
      const uint32_t off = is_k ? (two ? uo.k1 : uo.k0) : (two ? uo.v1 : uo.v0);
      const uint16_t* base = (is_k ? pk : pv) + slot +
                             (is_k ? (j >> 2) * 4 * kHeadDim + (j & 3) * 32 : j < 16 ? (j - 8) * 16 * BS : 0);
      lds_dma16<STREAM>(base, real && j < 16 ? off : 0u, j < 16 ? &s_ring[st][team][j][0] : &s_junk[0]);
    }
  };
  // validity mask chunks: units ch * kChunk .. of the split (lane l: map entry of
  // slot l % 2 of unit l / 2 at B = 16, of unit l at B = 32)
  constexpr int kChunk = BS == 16 ? 32 : 64;
  auto mask_slot = [&](int ch) __attribute__((always_inline)) {
    const int u = u_begin + ch * kChunk;
    return BS == 16 ? 2 * u + lane : u + lane;
  };
  // Everything else the unit loop reads (the context length, the slot-map
  // entries of the first two mask chunks, the query operands) takes the same
  // LDS-DMA path, ahead of the ring's first steps: the compiler cannot count
  // the DMA loads, so its wait for any load it issues after them would drain
  // the ring. Rows past the end load row 0's queries and are zeroed.
  const int row = v * 16 + i;
  lds_dma4(a.ctx_len + r, &s_misc[wave][0][0]);
  lds_dma4(map_addr(smap, ks, mask_slot(0), a.ctx_len + r), &s_misc[wave][1][0]);
  lds_dma4(map_addr(smap, ks, mask_slot(1), a.ctx_len + r), &s_misc[wave][2][0]);
  {
    const int qr = row < a.rows ? row : 0;
    const int tq = qr / a.G;
    const int qh = h * a.G + (qr - tq * a.G);
    const uint32_t qoff = (uint32_t)(((tq * a.Hq + qh) * kHeadDim + g * 8) * 2);
    const uint16_t* qbase = a.q + (long long)r * a.T * a.Hq * kHeadDim;
    // a tile's 4 k-steps are loaded by its wave of the first team
    if (team == 0) {
#pragma unroll
      for (int st = 0; st < 4; ++st) lds_dma16(qbase + st * 32, qoff, &s_q[v][st][0]);
    }
  }
  // units of the first kLook steps go out before the slot map is known
  auto unit = [&](int t) __attribute__((always_inline)) { return u_begin + t < u_end ? u_begin + t : -1; };
#pragma unroll
  for (int st = 0; st < kLook; ++st) issue(unit(st * kTeams + team), st);
  wait_vmcnt<kPer * kLook>();  // all but the ring's steps are in
  __syncthreads();             // the other team's queries too

  // Q^T operand of row tile v
  bf16x8 qb[4];
#pragma unroll
  for (int st = 0; st < 4; ++st) qb[st] = as_bf16x8(row < a.rows ? s_q[v][st][lane] : u32x4{0, 0, 0, 0});
  const Ctx c = ctx_blocks(__builtin_amdgcn_readfirstlane(s_misc[wave][0][lane]), BS, a.NBmax);
  const int local_len = c.local_len;
  int chunk = 0;
  uint64_t vmask = map_mask(ks, mask_slot(0), s_misc[wave][1][lane]);
  // attended tokens of the slots of the split's unit t (in the current mask chunk), n0 | n1 << 8
  auto counts = [&](int t) __attribute__((always_inline)) {
    int n0, n1;
    unit_counts<BS>(unit(t), ks, local_len, vmask, BS == 16 ? 2 * (t & (kChunk - 1)) : (t & (kChunk - 1)), n0, n1);
    return n0 | n1 << 8;
  };

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 acc[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nt = u_end > u_begin ? u_end - u_begin : 0;
  const int nsteps = (nt + kTeams - 1) / kTeams;
  int cnt[kLook];
#pragma unroll
  for (int st = 0; st < kLook; ++st) cnt[st] = counts(st * kTeams + team);
  int stage = 0;
  for (int s = 0; s < nsteps; ++s) {
    // this wave's loads of step s are done (those of the later step may still fly); the
    // barrier publishes every wave's loads of step s and tells that the stage of step
    // s - 1 is no longer read
    wait_vmcnt<kPer * (kLook - 1)>();
    __syncthreads();
    const int tn = (s + kLook) * kTeams + team;
    const int ch = tn / kChunk;
    if (ch != chunk) {
      // the map entries of chunk ch came in while the chunk before was attended; the next ones go out now
      chunk = ch;
      vmask = map_mask(ks, mask_slot(ch), s_misc[wave][1 + (ch & 1)][lane]);
      lds_dma4(map_addr(smap, ks, mask_slot(ch + 1), a.ctx_len + r), &s_misc[wave][1 + ((ch + 1) & 1)][0]);
    }
    const int nstage = stage == 0 ? kRowsStages - 1 : stage - 1;  // (s + kLook) % kRowsStages
    issue(unit(tn), nstage);
    const u32x4(&buf)[16][64] = s_ring[stage][team];
    f32x4 sc[2];
    // all of the unit's operands are read at once (left alone, the compiler reads
    // a K chunk, waits for it, and reads the next); the two token tiles' chains alternate
    u32x4 kr[8], vr[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) kr[j] = buf[j][lane];
    __builtin_amdgcn_sched_barrier(0);
    sc[0] = sc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int tau = 0; tau < 2; ++tau)
        sc[tau] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kr[tau * 4 + st]), qb[st], sc[tau], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 8; ++j) vr[j] = buf[8 + j][lane];
    __builtin_amdgcn_sched_barrier(0);
    const int keep = lane_keep<BS>(cnt[0] & 0xFF, cnt[0] >> 8, g);
    const bool partial = __builtin_amdgcn_ballot_w64(keep < 8) != 0;
    unit_softmax_pv(sc, keep, partial, m_run, l_run, acc, a.scale_log2, [&](int dt) { return vr[dt]; });
#pragma unroll
    for (int st = 0; st + 1 < kLook; ++st) cnt[st] = cnt[st + 1];
    cnt[kLook - 1] = counts(tn);
    stage = stage == kRowsStages - 1 ? 0 : stage + 1;
  }
  wait_vmcnt<0>();  // the placeholder loads past the last unit land before the ring is reused

  float L = l_run + __shfl_xor(l_run, 16);
  L += __shfl_xor(L, 32);
  float M = m_run;
  static_assert(kTeams == 1 || kTeams == 2, "the merge below");
  if constexpr (kTeams == 1) {
    if (row >= a.rows) return;
    if (a.nsplit == 1) {
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) write_output(a, r, h, row, dt * 4 + g, acc[dt], M, L);
      return;
    }
    const long long pr = ((long long)rh * a.nsplit + split) * a.rows + row;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      *reinterpret_cast<f32x4*>(a.part_o + pr * kHeadDim + dt * 16 + 4 * g) = acc[dt];
    if (g == 0) *reinterpret_cast<float2*>(a.part_ml + pr * 2) = make_float2(M, L);
  } else {
    // ---- merge the two teams: each takes one half of the dimensions of the row
    // tiles, d-tiles 4 * team .. +4, and gets the other team's part of them through LDS
    constexpr int kHalf = kHeadDim / 2 + 4;
    float(*s_o)[16][kHalf] = reinterpret_cast<float(*)[16][kHalf]>(&s_ring[0][0][0][0]);  // [wave]
    float(*s_ml)[2][16] = reinterpret_cast<float(*)[2][16]>(&s_q[0][0][0]);               // [wave]
    static_assert(sizeof(float) * 32 * kWaves <= sizeof(s_q), "maxima and sums fit the query area");
    static_assert(sizeof(float) * 16 * kHalf * kWaves <= sizeof(s_ring), "the states fit the ring");
    __syncthreads();  // the ring and the queries are no longer read
    f32x4 mine[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      mine[dt] = team == 0 ? acc[dt] : acc[dt + 4];
      *reinterpret_cast<f32x4*>(&s_o[wave][i][dt * 16 + 4 * g]) = team == 0 ? acc[dt + 4] : acc[dt];
    }
    if (g == 0) {
      s_ml[wave][0][i] = M;
      s_ml[wave][1][i] = L;
    }
    __syncthreads();
    if (row >= a.rows) return;
    const int other = wave < NT ? wave + NT : wave - NT;
    const float mo = s_ml[other][0][i], lo = s_ml[other][1][i];
    const float mm = fmaxf(M, mo);
    const float f = M == -INFINITY ? 0.f : fast_exp2(M - mm);
    const float fo = mo == -INFINITY ? 0.f : fast_exp2(mo - mm);
    L = L * f + lo * fo;
    M = mm;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      mine[dt] = mine[dt] * f + *reinterpret_cast<const f32x4*>(&s_o[other][i][dt * 16 + 4 * g]) * fo;
    if (a.nsplit == 1) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) write_output(a, r, h, row, (team * 4 + dt) * 4 + g, mine[dt], M, L);
      return;
    }
    const long long pr = ((long long)rh * a.nsplit + split) * a.rows + row;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      *reinterpret_cast<f32x4*>(a.part_o + pr * kHeadDim + (team * 4 + dt) * 16 + 4 * g) = mine[dt];
    if (team == 0 && g == 0) *reinterpret_cast<float2*>(a.part_ml + pr * 2) = make_float2(M, L);
  }
}

// Merge of the NS splits: a workgroup takes kMergeRows rows of one (request,
// KV head), 32 threads a row, each thread 4 dimensions; every thread issues its
// NS partial loads (16 bytes each) and the row's NS (max, sum) pairs at once.
// The items are dealt over the XCDs as the splits are (xcd_item, pairs in
// order), so most partials are read from the L2 that holds them.
constexpr int kMergeRows = 8;

template <int NS>
__global__ __launch_bounds__(kMergeRows * 32) void attn_merge_kernel(AttnArgs a) {
  const int groups = (a.rows + kMergeRows - 1) / kMergeRows;
  const int item = xcd_item(blockIdx.x, a.R * a.Hkv, groups);
  const int rh = item / groups;
  const int row = (item - rh * groups) * kMergeRows + (threadIdx.x >> 5);
  if (item < 0 || row >= a.rows) return;
  const int c4 = threadIdx.x & 31;
  const int r = rh / a.Hkv;
  const int h = rh - r * a.Hkv;
  const long long base = (long long)rh * NS * a.rows + row;
  float2 ml[NS];
  f32x4 os[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const long long idx = base + (long long)s * a.rows;
    ml[s] = *reinterpret_cast<const float2*>(a.part_ml + idx * 2);
    os[s] = *reinterpret_cast<const f32x4*>(a.part_o + idx * kHeadDim + c4 * 4);
  }
  float M = ml[0].x;
#pragma unroll
  for (int s = 1; s < NS; ++s) M = fmaxf(M, ml[s].x);
  // a split with no attended token (max -inf) weighs 0; with none at all, L = 0
  float L = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const float f = ml[s].x == -INFINITY ? 0.f : fast_exp2(ml[s].x - M);
    L += ml[s].y * f;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] += os[s][e] * f;
  }
  float res[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) res[e] = L > 0.f ? o[e] / L : 0.f;
  const int t = row / a.G;
  const int qh = h * a.G + (row - t * a.G);
  const long long orow = ((long long)r * a.T + t) * a.Hq + qh;
  const uint32_t w0 = f32_to_bf16_bits(res[0]) | (f32_to_bf16_bits(res[1]) << 16);
  const uint32_t w1 = f32_to_bf16_bits(res[2]) | (f32_to_bf16_bits(res[3]) << 16);
  *reinterpret_cast<uint2*>(a.out + orow * kHeadDim + c4 * 4) = make_uint2(w0, w1);
  if (c4 == 0 && a.lse) a.lse[orow] = L > 0.f ? (M + __log2f(L)) * 0.69314718055994531f : -INFINITY;
}

template <int NS>
void launch_merge_ns(const AttnArgs& a, hipStream_t s, const LaunchTiming& t) {
  const long long groups = (a.rows + kMergeRows - 1) / kMergeRows;
  launch_kernel(attn_merge_kernel<NS>, dim3(xcd_grid(a.R * a.Hkv, groups)), dim3(kMergeRows * 32), s, t, a);
}

void launch_merge(const AttnArgs& a, hipStream_t s, const LaunchTiming& t) {
  switch (a.nsplit) {
    case 2: return launch_merge_ns<2>(a, s, t);
    case 3: return launch_merge_ns<3>(a, s, t);
    case 4: return launch_merge_ns<4>(a, s, t);
    case 5: return launch_merge_ns<5>(a, s, t);
    case 6: return launch_merge_ns<6>(a, s, t);
    case 7: return launch_merge_ns<7>(a, s, t);
    case 8: return launch_merge_ns<8>(a, s, t);
    case 9: return launch_merge_ns<9>(a, s, t);
    case 10: return launch_merge_ns<10>(a, s, t);
    case 11: return launch_merge_ns<11>(a, s, t);
    case 12: return launch_merge_ns<12>(a, s, t);
    case 13: return launch_merge_ns<13>(a, s, t);
    case 14: return launch_merge_ns<14>(a, s, t);
    case 15: return launch_merge_ns<15>(a, s, t);
    default: return launch_merge_ns<kMaxSplits>(a, s, t);
  }
}

template <int NT, int BS>
hipError_t launch_t(const AttnArgs& a, hipStream_t s, const LaunchTiming& t) {
  const long long nrh = (long long)a.R * a.Hkv;
  const bool merge = a.nsplit > 1;
  // timed as one span: from the split kernel's start to the merge kernel's end
  const LaunchTiming ts{t.start, merge ? nullptr : t.stop};
  // Bytes at most: no context has more than NBmax blocks. (Counting every slot at
  // contexts a quarter of the pool took 21.9 -> 23.1 us.)
  const long long blocks = a.k_slots + 1ll < a.NBmax ? a.k_slots + 1ll : a.NBmax;
  const bool stream = nrh * blocks * BS * (2 * kHeadDim * 2) >= kStreamBytes;
  if constexpr (NT >= 3) {
    // With more pairs than CUs there are no splits, and at most two pairs per CU
    // fit it together with one team each (two teams' ring fills the LDS), instead
    // of in two rounds. Measured with two teams against one (8 KV heads, 40 rows,
    // budget 1,024): 33 requests 46.3 and 37.3 us, 60 requests 52.9 and 49.2; past
    // two pairs per CU level (70 requests 72.9 and 71.4). Five row tiles' single
    // teams hold a CU less well together: 33 requests 52.3 and 66.5 us.
    constexpr bool kShare = NT <= 4;
    // Reading past the caches (kStreamBytes) pays here at B = 32 where the CUs are
    // full, so that bandwidth bounds the call: 128 pairs in two splits (72 rows, 274
    // MB) 61.7 -> 54.1 us, 256 pairs 106 -> 94.5; at 176 of 256 workgroups 74.6 and
    // 79.8 us, and at B = 16, where half a wave reads each slot, 44.4 and 47.7.
    const bool fill = BS == 32 && stream && 8 * nrh * a.nsplit >= 7 * kTargetWorkgroups;
    const dim3 grid(xcd_grid(nrh, a.nsplit));
    if (kShare && nrh > kTargetWorkgroups && nrh <= 2 * kTargetWorkgroups)
      launch_kernel(attn_split_rows_kernel<NT, kShare ? 1 : 2, BS, false>, grid, dim3(NT * (kShare ? 1 : 2) * 64), s, ts,
                    a);
    else
      launch_kernel(fill ? attn_split_rows_kernel<NT, 2, BS, BS == 32> : attn_split_rows_kernel<NT, 2, BS, false>, grid,
                    dim3(NT * 2 * 64), s, ts, a);
  } else {
    launch_kernel(stream ? attn_split_kernel<NT, BS, true> : attn_split_kernel<NT, BS, false>,
                  dim3(xcd_grid(nrh, a.nsplit)), dim3(kW * 64), s, ts, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !merge) return e;
  launch_merge(a, s, LaunchTiming{nullptr, t.stop});
  return hipGetLastError();
}

template <int BS>
hipError_t launch_bs(const AttnArgs& a, hipStream_t s, const LaunchTiming& t) {
  switch ((a.rows + 15) / 16) {
    case 1: return launch_t<1, BS>(a, s, t);
    case 2: return launch_t<2, BS>(a, s, t);
    case 3: return launch_t<3, BS>(a, s, t);
    case 4: return launch_t<4, BS>(a, s, t);
    case 5: return launch_t<5, BS>(a, s, t);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_attn(const AttnArgs& a, hipStream_t s, const LaunchTiming& t) {
  return a.B == 16 ? launch_bs<16>(a, s, t) : launch_bs<32>(a, s, t);
}

// Scratch of the allocation-free attention entry point: the split partials, in
// a file-scope device array that every GPU the library runs on holds from
// module load until the process ends (kNoAllocScratchBytes each). Host code
// never passes the array's name to a kernel: that is a host-side stand-in, not
// a device address. Its address on each device comes from hipGetSymbolAddress,
// taken once per device with that device current, and only that address is
// handed to the kernels.
namespace {
__device__ __align__(256) float scratch[kNoAllocScratchBytes / sizeof(float)];
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;
}  // namespace

hipError_t noalloc_scratch(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace oasis
