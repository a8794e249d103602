// How an attention call is cut into workgroups: host code, no HIP.
//
// The units of a (request, KV head) pair (32 tokens: two slots at B = 16, one at
// B = 32; the local block is the last slot) are dealt to nsplit workgroups in
// runs of units_per_split. With several splits each leaves a partial per row in
// the workspace and the merge kernel combines them.
#pragma once

#include <cstddef>

namespace oasis {

constexpr int kHeadDim = 128;
constexpr int kW = 4;  // waves per workgroup of the kernel for up to two row tiles
constexpr int kTargetWorkgroups = 256;  // one per CU
constexpr int kMaxSplits = 16;
constexpr int kRegisterRows = 32;  // rows up to which K and V go straight into registers (attn_split_kernel)

struct AttnPlan {
  int rows, n_units, nsplit, units_per_split;
  std::size_t part_o_floats, bytes;  // bytes: what oasis_attn_workspace_bytes returns
};

// `busy`: CUs that other kernels hold while the call runs (the staging
// workgroups of a pipelined step), to the exclusion of a many-row workgroup.
inline AttnPlan attn_plan(int R, int Hq, int Hkv, int T, int B, int k_slots, int busy = 0) {
  AttnPlan p{};
  const int G = Hq / Hkv;
  p.rows = G * T;
  p.n_units = B == 16 ? (k_slots + 2) / 2 : k_slots + 1;
  const long long nrh = (long long)R * Hkv;
  // `want` splits of at least `least` units each, at most kMaxSplits
  auto split = [&](long long want, int least) {
    const long long most = (p.n_units + least - 1) / least;
    want = want < most ? want : most;
    want = want < kMaxSplits ? want : kMaxSplits;
    want = want > 1 ? want : 1;
    p.units_per_split = (int)((p.n_units + want - 1) / want);
    p.nsplit = (p.n_units + p.units_per_split - 1) / p.units_per_split;
  };
  // The workspace holds the partials of the smallest split that gives every CU
  // a workgroup and every wave a unit, the finest split that can pay.
  long long want = (kTargetWorkgroups + nrh - 1) / (nrh > 0 ? nrh : 1);
  split(want, kW);
  p.bytes = p.nsplit > 1 ? (std::size_t)nrh * p.nsplit * p.rows * (kHeadDim + 2) * sizeof(float) : 0;
  // The split launched is the largest with at most one workgroup per CU. Of two
  // row tiles a CU holds one (264 to 268 registers, one wave per SIMD), so a few
  // workgroups more take a round of their own. Measured on MI355X (8 KV heads, 20
  // rows, budget 2,048), smallest split that fills against this one: 3 requests
  // 17.3 against 12.8 us, 5 requests 18.1 and 13.0, 17 requests 43.0 and 33.6, 22
  // requests (two splits against one, no merge) 46.3 and 35.5. Of one row tile a
  // CU holds two (204 to 208 registers), so both splits fit one round, but the
  // merge and the shorter chains cost more than the second workgroup hides: 8
  // rows, 17 requests 37.5 and 30.2 us, 22 requests 38.4 and 31.7; 16 rows 38.5
  // and 30.9, 40.1 and 32.6.
  if (p.nsplit > 1 && nrh * p.nsplit > kTargetWorkgroups) want = kTargetWorkgroups / nrh;
  const int least = p.rows <= kRegisterRows ? kW : 6;
  split(want, least);
  // Fewer splits where no wave's chain gets longer: 65 units in 13 splits of 5
  // leave one wave of four with two units, and so do 9 splits of 8 (1 request x 8
  // KV heads, 20 rows, per call: 10.8 and 10.5 us; 2 requests 12.1 and 11.4 us).
  // One row tile has little to merge (8.3 against 8.5 us), and the many-row
  // kernel's two teams take at least three units each (72 rows: 14.1 -> 13.6 us).
  if (p.rows > 16 && p.rows <= kRegisterRows && p.nsplit > 1) {
    const int depth = (p.units_per_split + kW - 1) / kW;
    split((p.n_units + depth * kW - 1) / (depth * kW), kW);
  }
  // A many-row workgroup of two teams (116 to 127 KB of LDS) and a staging one
  // (77 KB and more) do not fit one CU's 160 KB, and a pipelined step's staging
  // workgroups hold their CUs from before its attention until its transfer ends.
  // There the split is the one with the fewest units in sequence, rounds of
  // workgroups over the CUs left times units per split (ties: more splits).
  // Measured on MI355X, pipelined steps planned for 256 CUs and for the ones left
  // (us a layer): 24 pairs of 35 rows, B = 32, 51.9 and 47.3; 64 pairs of 36 rows,
  // B = 16, 62.0 and 57.8; 128 pairs of 72 rows, B = 32, budget 4,096, 167 and 153.
  // (One team a workgroup, which fits beside staging, takes 46.7 and 59.3 in the
  // first two, but 90.3 against 81.4 at 96 pairs of 36 rows.)
  if (p.rows > kRegisterRows && p.nsplit > 1 && busy > 0) {
    const long long left = busy < kTargetWorkgroups ? kTargetWorkgroups - busy : 1;
    int best = p.nsplit;
    long long least_chain = 0;
    for (int n = p.nsplit; n >= 1; --n) {
      split(n, least);
      const long long chain = (nrh * p.nsplit + left - 1) / left * p.units_per_split;
      if (n == best || chain < least_chain) {
        least_chain = chain;
        best = n;
      }
    }
    split(best, least);
  }
  // partials exist only with several splits (one split writes the outputs itself)
  p.part_o_floats = p.nsplit > 1 ? (std::size_t)nrh * p.nsplit * p.rows * kHeadDim : 0;
  return p;
}

}  // namespace oasis
