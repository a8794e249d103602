// Exact top-K of one (request, KV head) score row by a workgroup (paper
// §4.2.1-§4.2.2: top-K prediction per KV head; ties go to the lowest block id).
//
// Scores are mapped to order-preserving uint32 keys (-0 folded into +0); thread
// t holds ids t, t + NTHR, ... (KPT keys in registers, or re-read with KPT ==
// 0), so that every read of the row is coalesced and nothing is staged. A radix
// select over an LDS histogram finds the exact key tau of the k-th largest
// score and how many keys equal to tau are needed. It runs on the offsets of
// the keys from the row's smallest key, 8 bits per pass from the highest bit of
// the row's key range down: scores of one row share their sign and most
// exponent bits, which would put nearly every key in one bin of a first pass
// over the raw top byte (LDS atomics on one address), and a narrow range needs
// fewer passes. As soon as the wanted bin holds at most kSelectCand keys (after
// the first pass for a row of 8,191 scores with a few strong blocks), they are
// gathered in LDS and one wave ranks them against each other, in place of the
// remaining passes.
//
// Ids ascend over (j, wave, lane) for id j * NTHR + 64 * wave + lane: each wave
// counts its keys above tau and equal to tau for each j by ballots, one wave
// scans the counts, and a selected block's output position is the number of
// greater keys before it plus that of taken ties before it (lowest ids win), so
// the selection is written in ascending id order without a sort.
//
// The kernel is a chain of barriers and LDS round trips, not bandwidth (4 bytes
// per candidate): 64 rows of 8,191 scores 9.3 us on MI355X, against 10.6 us with
// the keys staged in LDS, contiguous ids per thread and every pass made.
#pragma once

#include "oasis_internal.h"

namespace oasis {

__device__ __forceinline__ uint32_t select_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;  // -0.0 == +0.0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Wave-wide minimum and maximum of uint32 values, returned to every lane (the
// same DPP steps; lanes without a source keep the identity).
__device__ __forceinline__ void wave_min_max(uint32_t& mn, uint32_t& mx) {
  int a = (int)mn, b = (int)mx;
#define OASIS_DPP_MINMAX(CTRL, ROWS)                                                              \
  a = (int)min((uint32_t)a, (uint32_t)__builtin_amdgcn_update_dpp((int)0xFFFFFFFF, a, CTRL, ROWS, 0xF, false)); \
  b = (int)max((uint32_t)b, (uint32_t)__builtin_amdgcn_update_dpp(0, b, CTRL, ROWS, 0xF, false));
  OASIS_DPP_MINMAX(0x111, 0xF)
  OASIS_DPP_MINMAX(0x112, 0xF)
  OASIS_DPP_MINMAX(0x114, 0xF)
  OASIS_DPP_MINMAX(0x118, 0xF)
  OASIS_DPP_MINMAX(0x142, 0xA)
  OASIS_DPP_MINMAX(0x143, 0xC)
#undef OASIS_DPP_MINMAX
  mn = (uint32_t)__builtin_amdgcn_readlane(a, 63);
  mx = (uint32_t)__builtin_amdgcn_readlane(b, 63);
}

// Lanes below this one whose bit is set in `mask`.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

constexpr int kSelectCand = 64;   // candidates ranked directly: one per lane
constexpr int kSelectChunk = 32;  // with KPT == 0: keys per thread counted and written at a time

template <int NTHR, int KPT>
struct SelectShared {
  static constexpr int kWaves = NTHR / 64;
  static constexpr int kPer = KPT > 0 ? KPT : kSelectChunk;
  uint32_t hist[2][256];  // one per pass, alternately: the next is cleared while the current fills
  int digit, rem, eq_total, ncand;
  uint32_t tau;
  uint32_t cand[kSelectCand];
  uint32_t wmin[kWaves], wmax[kWaves];
  // per (j, wave): keys above tau | keys equal to tau << 16, then their exclusive prefix sums
  uint32_t cnt[kPer * kWaves];
  uint32_t total;
};

// Select the top k of the n keys key_of(0) .. key_of(n - 1) into out[0..k)
// (ascending ids, -1 padded when n < k) and set *count; every thread of the
// workgroup calls it. key_of may read memory (it is called once per id with
// KPT > 0, with ids clamped into the row). With lout (LDS, k entries) the
// selection is also left there for the workgroup.
template <int NTHR, int KPT, typename Key>
__device__ void select_row(Key&& key_of, int n, int k, int32_t* out, int32_t* count, SelectShared<NTHR, KPT>& sh,
                           int* lout = nullptr) {
  constexpr int kWaves = NTHR / 64;
  const int tid = threadIdx.x;
  if (n <= k) {  // every candidate fits the budget
    for (int i = tid; i < k; i += NTHR) {
      out[i] = i < n ? i : -1;
      if (lout) lout[i] = i < n ? i : -1;
    }
    if (tid == 0) *count = n;
    return;
  }
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int jn = (n + NTHR - 1) / NTHR;  // keys per thread
  constexpr int kRegs = KPT > 0 ? KPT : 1;
  uint32_t keys[kRegs];
  if constexpr (KPT > 0) {
#pragma unroll
    for (int j = 0; j < kRegs; ++j) keys[j] = key_of(min(tid + j * NTHR, n - 1));
  }
  auto key_at = [&](int j) __attribute__((always_inline)) -> uint32_t {
    if constexpr (KPT > 0) return keys[j];
    else return key_of(tid + j * NTHR);
  };
  // f(j) for each of this thread's keys j = 0 .. cnt - 1 (cnt is uniform)
  auto each = [&](int cnt, auto&& f) __attribute__((always_inline)) {
    if constexpr (KPT > 0) {
#pragma unroll
      for (int j = 0; j < kRegs; ++j)
        if (j < cnt) f(j);
    } else {
      for (int j = 0; j < cnt; ++j) f(j);
    }
  };

  // range of the row's keys: wave minima / maxima, then over the waves
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  each(jn, [&](int j) {
    if (tid + j * NTHR >= n) return;
    const uint32_t key = key_at(j);
    kmin = min(kmin, key);
    kmax = max(kmax, key);
  });
  wave_min_max(kmin, kmax);
  if (lane == 0) {
    sh.wmin[wave] = kmin;
    sh.wmax[wave] = kmax;
  }
  if (tid == 0) sh.ncand = 0;
  if (tid < 256) sh.hist[0][tid] = 0u;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    kmin = min(kmin, sh.wmin[w]);
    kmax = max(kmax, sh.wmax[w]);
  }
  const uint32_t range = kmax - kmin;
  // offsets from kmin have `top` significant bits; passes resolve them 8 at a time
  int top = range ? 32 - __clz((int)range) : 0;
  uint32_t prefix = 0u;  // resolved high bits of the wanted offset (bits >= top)
  int rem = k;           // rank (from the top) of the wanted key among keys matching the prefix
  int eq_total = n;      // keys matching the prefix
  // Two barriers per pass: after the histogram is filled, and after the
  // digit is found (the next pass fills the other histogram, cleared here).
  for (int pass = 0; top > 0; ++pass) {
    if (pass > 0 && eq_total <= kSelectCand) break;
    const int shift = top > 8 ? top - 8 : 0;
    const uint32_t dmask = (1u << (top - shift)) - 1u;  // this pass resolves bits [shift, top)
    uint32_t* hist = sh.hist[pass & 1];
    if (tid < 256) sh.hist[(pass & 1) ^ 1][tid] = 0u;
    uint32_t cur = 0xFFFFFFFFu;
    uint32_t run = 0u;
    each(jn, [&](int j) {
      if (tid + j * NTHR >= n) return;
      const uint32_t off = key_at(j) - kmin;
      if (top < 32 && (off >> top) != prefix) return;
      const uint32_t dg = (off >> shift) & dmask;
      if (dg == cur) {
        ++run;
      } else {
        if (run) atomicAdd(&hist[cur], run);
        cur = dg;
        run = 1u;
      }
    });
    if (run) atomicAdd(&hist[cur], run);
    __syncthreads();
    if (tid < 64) {
      // lane L looks at bins 255-4L .. 252-4L (descending)
      uint32_t hb[4];
      int local = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        hb[j] = hist[255 - 4 * tid - j];
        local += (int)hb[j];
      }
      const int incl = wave_incl_sum(local);
      const int excl = incl - local;
      if (excl < rem && rem <= incl) {
        int acc = excl;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (acc + (int)hb[j] >= rem) {
            sh.digit = 255 - 4 * tid - j;
            sh.rem = rem - acc;
            sh.eq_total = (int)hb[j];
            break;
          }
          acc += (int)hb[j];
        }
      }
    }
    __syncthreads();
    prefix = (prefix << (top - shift)) | (uint32_t)sh.digit;
    rem = sh.rem;
    eq_total = sh.eq_total;
    top = shift;
  }
  uint32_t tau = kmin + prefix;
  if (top > 0) {
    // at most kSelectCand keys match the prefix: gather them, and rank them in every wave
    each(jn, [&](int j) {
      if (tid + j * NTHR >= n) return;
      const uint32_t key = key_at(j);
      if (((key - kmin) >> top) == prefix) sh.cand[atomicAdd(&sh.ncand, 1)] = key;
    });
    __syncthreads();
    if (wave == 0) {  // one wave: the others' issue slots would be its own
      const uint32_t mine = lane < eq_total ? sh.cand[lane] : 0u;
      int above = 0, same = 0;  // candidates greater than / equal to this lane's
      for (int t = 0; t < eq_total; ++t) {
        const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, t);
        above += other > mine;
        same += other == mine;
      }
      // the wanted key is the one with above < rem <= above + same (equal lanes write equal values)
      if (lane < eq_total && above < rem && rem <= above + same) {
        sh.tau = mine;
        sh.rem = rem - above;
      }
    }
    __syncthreads();
    tau = sh.tau;
    rem = sh.rem;
  }
  const int need_eq = rem;  // how many tau-valued keys are taken, lowest ids first

  int gt_base = 0, eq_base = 0;  // keys before the current chunk
  constexpr int kPer = SelectShared<NTHR, KPT>::kPer;
  for (int j0 = 0; j0 < jn; j0 += kPer) {
    const int jc = min(kPer, jn - j0);
    // The ballots are taken again when the positions are known (they are cheap,
    // and holding them would take two registers per key).
    auto masks = [&](int j, uint64_t& gt, uint64_t& eq) __attribute__((always_inline)) {
      const bool in = tid + (j0 + j) * NTHR < n;
      uint32_t key = 0u;
      if constexpr (KPT > 0) key = keys[j];
      else if (in) key = key_of(tid + (j0 + j) * NTHR);
      gt = __ballot(in && key > tau);
      eq = __ballot(in && key == tau);
    };
    each(jc, [&](int j) {
      uint64_t gt, eq;
      masks(j, gt, eq);
      if (lane == 0) sh.cnt[j * kWaves + wave] = (uint32_t)__popcll(gt) | (uint32_t)__popcll(eq) << 16;
    });
    __syncthreads();
    if (wave == 0) {  // a lane takes consecutive entries, the wave scans the lanes' sums
      const int ne = jc * kWaves;
      constexpr int kEach = (kPer * kWaves + 63) / 64;
      uint32_t e[kEach], sum = 0u;
#pragma unroll
      for (int u = 0; u < kEach; ++u) {
        const int at = lane * kEach + u;
        e[u] = at < ne ? sh.cnt[at] : 0u;
        sum += e[u];
      }
      const uint32_t incl = (uint32_t)wave_incl_sum((int)sum);
      uint32_t excl = incl - sum;
#pragma unroll
      for (int u = 0; u < kEach; ++u) {
        const int at = lane * kEach + u;
        if (at < ne) sh.cnt[at] = excl;
        excl += e[u];
      }
      if (lane == 63) sh.total = incl;
    }
    __syncthreads();
    each(jc, [&](int j) {
      uint64_t gt, eq;
      masks(j, gt, eq);
      if ((gt | eq) == 0) return;  // wave-uniform
      const uint32_t pre = sh.cnt[j * kWaves + wave];
      const int gt_before = gt_base + (int)(pre & 0xFFFFu) + lanes_below(gt);
      const int eq_before = eq_base + (int)(pre >> 16) + lanes_below(eq);
      const bool is_eq = (eq >> lane) & 1;
      if (((gt >> lane) & 1) || (is_eq && eq_before < need_eq)) {
        const int pos = gt_before + min(eq_before, need_eq);
        const int id = tid + (j0 + j) * NTHR;
        out[pos] = id;
        if (lout) lout[pos] = id;
      }
    });
    if (KPT == 0) {
      gt_base += (int)(sh.total & 0xFFFFu);
      eq_base += (int)(sh.total >> 16);
      __syncthreads();  // the counts are rewritten by the next chunk
    }
  }
  if (tid == 0) *count = k;
}

}  // namespace oasis
