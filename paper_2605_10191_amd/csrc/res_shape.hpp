// Shapes and workspaces of the resident recurrence (resident.hip): how the
// columns of a batch go to teams, and where a call's small arrays lie.  Plain
// C++, read by the launches and by everything that sizes a buffer for them, so
// that the two cannot differ.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace polfed {

// The K steps of a column or a pair of columns in one launch, by a team of
// workgroups on one XCD.
constexpr int kResThreads = 512;  // up to 256 VGPRs a lane for the rows' state
constexpr int kResWaves = kResThreads / 64;
constexpr int kResMaxL = 20;
constexpr int kResMaxPairRows = 3;  // rows a thread of a pair of columns
constexpr int kResMaxRows = 6;      // rows a thread of a single column
constexpr int kResMaxSlabs = 32;
constexpr int kResTeamsPerXcd = 16;
struct ResTeam {
  int joined, n, group[2];
  int pad0[12];
  int flag[kResMaxSlabs];  // barriers each member has reached
};
struct ResState {
  int slots[16 * 16];  // workgroups that joined, per XCD, a cache line apart
  int queue, err;
  int home;  // 1 + the XCD of a launch for one column group, see team_join
  int pad[13];
  ResTeam teams[16 * kResTeamsPerXcd];
};

// Whether word i of a ResState is cleared before a launch: all of them before a
// call's first one, and before the launches that go on with its recurrence all
// but err, which says that a barrier gave up in one of those before.
constexpr bool res_clears(size_t i, bool first) {
  return first || i != offsetof(ResState, err) / sizeof(int);
}
// How long a barrier waits, in ticks of the 100 MHz clock.  Every member runs,
// so it ends by itself; the bound only keeps a broken device from hanging.
constexpr long long kResTicksPerSecond = 100000000, kResWait = 30 * kResTicksPerSecond;

// Slabs of a column (a power of two), pairs of columns sharing a team, rows a
// thread.
struct ResShape {
  int nslab = 0, pairs = 0, ngrp = 0, teams = 0, R = 0;
  double us = 1e30;  // of a step, by the model below
};

inline int res_rows(int64_t D, int nslab) { return (int)((D + nslab - 1) / nslab); }
inline int res_r(int64_t D, int nslab) {
  return (res_rows(D, nslab) + kResThreads - 1) / kResThreads;
}

// Measured on an MI355X (FP64, us a step): one workgroup with one row a thread
// 0.68, with two 0.97 (two slabs of one row 1.15), pairs of columns with two
// rows 2.2; 8, 16, 32 slabs with one row 1.4, 1.6, 2.0, where another row a
// thread adds 0.75 and one of a pair of columns is 1.2.  The model below follows
// these within 15% and picks the cheapest shape: one workgroup up to 1,024
// rows, one row a thread as long as 32 slabs allow it, pairs once there are
// more columns than teams.  (nslab 0: none.)
inline ResShape res_shape_at(int64_t D, int nb, int nslab) {
  ResShape best;
  const int R = res_r(D, nslab);
  if (R > kResMaxRows || (nslab == 1 && R > 2)) return best;
  const int teams = nslab == 1 ? 256 : 8 * std::min(kResMaxSlabs / nslab, kResTeamsPerXcd);
  const bool alone = nslab == 1;  // no barriers between workgroups
  const double base = alone ? 0.39 : 0.5 + 0.0235 * nslab;
  const double row = alone ? 0.29 : 0.75, pair_row = alone ? 0.9 : 1.2;
  for (int pair = 0; pair < 2; ++pair) {
    ResShape x;
    x.nslab = nslab;
    x.teams = teams;
    x.R = R;
    if (pair && R > kResMaxPairRows) continue;
    const int per = pair ? 2 : 1;
    const int rounds = (nb + per * teams - 1) / (per * teams);
    if (pair) {
      // as many single columns as the rounds have room for
      x.pairs = std::max(0, nb - rounds * teams);
      if (x.pairs == 0) continue;
    }
    x.ngrp = nb - x.pairs;
    x.us = rounds * (base + (pair ? pair_row : row) * R);
    if (x.us < best.us) best = x;
  }
  return best;
}
inline ResShape res_shape(int64_t D, int nb) {
  ResShape best;
  for (int nslab = 1; nslab <= kResMaxSlabs; nslab *= 2) {
    const ResShape x = res_shape_at(D, nb, nslab);
    if (x.us < best.us) best = x;
  }
  return best;
}

// Workgroups of a launch on one XCD that stay for all of its steps.
inline int res_per_xcd(const ResShape& x) {
  return x.nslab <= 1 ? (std::min(x.ngrp, 256) + 7) / 8
                      : std::min(x.teams / 8, (x.ngrp + 7) / 8) * x.nslab;
}
// Where several streams share the device (the server with more than one group
// of solves), a resident launch leaves half of the compute units of every XCD
// to the others.  One that fills an XCD keeps every other launch waiting for
// the workgroups of its own that were dealt to that XCD, until it ends: 48
// requests at once (L = 14, 16, 18, 50 pairs) went at 2.7 a second, at 4.3 with
// launches where this says no; at 1.17 a second the median of L = 14 was 1.5 s
// and is 0.09, of all 2.4 s and 1.1.
constexpr int kResSharedPerXcd = 16;
inline bool res_shares(const ResShape& x) { return res_per_xcd(x) <= kResSharedPerXcd; }

inline size_t res_align(size_t n) { return (n + 255) / 256 * 256; }

// Steps from which a filter goes this way: the resident launch itself
// (joining, tables, two small kernels) takes about 20 us.
constexpr int kResMinSteps = 16;
constexpr int kResChunk = 8192;  // steps of one launch

// What a single column's filter keeps behind the D elements of its first
// recurrence buffer, as byte offsets from the next multiple of 256: the team
// state, the scale (two elements) and a chunk's coefficients.
struct ResTail {
  static constexpr size_t st = 0, sc = (sizeof(ResState) + 255) / 256 * 256, A = sc + 256,
                          end = A + (size_t)(kResChunk + 1) * sizeof(double);
  // bytes to allocate behind an element that may lie anywhere
  static constexpr size_t bytes = 255 + end;
};

// Steps of the moments form in one launch: their partial products are summed
// before the next one, so that they take no more room with more moments.
constexpr int kResMomentSteps = 256;

// M steps of the Chebyshev vectors of nb columns out of groups of width
// columns (kpm.hip): the byte offsets of the scales, the sums and the partial
// products behind the team state (the sums have one element more), and the bytes in all.  Every group takes the
// slabs of a full one, so that a shorter last group needs no more room and
// reads the same tables (its own best shape can have more slabs than there are
// columns fewer: D = 5,005 4 slabs for 64 columns, 16 for 32).
struct ResMomentsPlan {
  ResShape shape;
  int64_t count = 0;  // products: M x nb
  size_t sc = 0, sums = 0, part = 0, bytes = 0;
};
inline ResMomentsPlan res_moments_plan(int64_t D, int M, int width, int nb) {
  ResMomentsPlan p;
  const int nslab = res_shape(D, width).nslab;
  if (nslab == 0 || nb > width) return p;
  p.shape = res_shape_at(D, nb, nslab);
  p.count = (int64_t)M * nb;
  p.sc = res_align(sizeof(ResState));
  p.sums = res_align(p.sc + (size_t)2 * nb * sizeof(double));
  p.part = p.sums + (size_t)(p.count + 1) * sizeof(double);
  p.bytes = p.part + (size_t)std::min(M, kResMomentSteps) * nb * nslab * kResWaves * sizeof(double);
  return p;
}

}  // namespace polfed
