// Host-side rules: the launches of a run of n steps, the form of an
// initialisation.  Plain C++ without HIP and without allocation: they run inside
// entry points that must not throw.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace lbmh {

constexpr int PLAN_MAX_STEPS = 10;  // most steps of a launch
constexpr int PLAN_DIVIDED = 4;     // launches of T steps that may be divided anew

// `head` launches of T steps, then those of `tail`.
struct LaunchPlan {
  int64_t head;
  int T;
  int ntail;
  int tail[PLAN_DIVIDED + PLAN_MAX_STEPS - 1];
  int64_t launches() const { return head + ntail; }
  int steps(int64_t l) const { return l < head ? T : tail[l - head]; }
};

// Plan of a run of n steps with a variant of T <= PLAN_MAX_STEPS steps.
// ms[t], 1 <= t <= maxt <= PLAN_MAX_STEPS: time of a launch of t steps, as far
// as known (else <= 0); one_launch: the n mod T steps left take one launch
// (else one each).  Where every time needed is known, the last up to four
// launches of T steps and the steps left are divided into the launches, no
// more than these, whose times add up to least, if that saves more than the 1%
// by which such times scatter: a launch of one or two steps costs as much as
// three or four more steps in a longer one (1000 x 777, periodic: 7 steps
// 31 us, a single step 18.6; initialisation, 50 steps and moments 262 us as
// 7 x 7 + 1, 251 as 6 x 7 + 8).
// More launches of fewer steps can look cheaper than they are, since the
// autotuner's launches all read one buffer, which a cache may hold (900 x
// 1500, 33 steps: 425 to 436 us with eight shorter launches allowed, 418 as
// 5 x 6 + 3).
inline LaunchPlan plan_launches(int64_t n, int T, bool one_launch, const double* ms, int maxt) {
  LaunchPlan p{n / T, T, 0, {}};
  const int r = (int)(n % T);
  if (r == 0) return p;
  p.ntail = one_launch ? 1 : r;
  for (int l = 0; l < p.ntail; ++l) p.tail[l] = one_launch ? r : 1;
  const double rest = one_launch ? ms[r] : r * ms[1];
  if (ms[T] <= 0.0 || rest <= 0.0) return p;
  constexpr int MOST_L = PLAN_DIVIDED + PLAN_MAX_STEPS - 1;
  constexpr int MOST_K = (PLAN_DIVIDED + 1) * PLAN_MAX_STEPS - 1;
  const int q = (int)(p.head < PLAN_DIVIDED ? p.head : PLAN_DIVIDED), K = q * T + r;
  const int most = q + p.ntail;
  // cost[l][k]: k steps in l launches, last[..]: the last one's steps
  double cost[MOST_L + 1][MOST_K + 1];
  int last[MOST_L + 1][MOST_K + 1] = {};
  for (int l = 0; l <= most; ++l)
    for (int k = 0; k <= K; ++k) cost[l][k] = 1e300;
  cost[0][0] = 0.0;
  int best = 0;
  for (int l = 1; l <= most; ++l) {
    for (int k = 1; k <= K; ++k)
      for (int t = 1; t <= maxt && t <= k; ++t)
        if (ms[t] > 0.0 && cost[l - 1][k - t] + ms[t] < cost[l][k]) {
          cost[l][k] = cost[l - 1][k - t] + ms[t];
          last[l][k] = t;
        }
    if (cost[l][K] < cost[best][K]) best = l;
  }
  if (cost[best][K] >= 0.99 * (q * ms[T] + rest)) return p;
  p.head -= q;
  p.ntail = 0;
  for (int l = best, k = K; l > 0; --l) {
    p.tail[p.ntail++] = last[l][k];
    k -= last[l][k];
  }
  return p;
}

// Time of a plan's launches, ms[t] for one of t steps; of an unknown one (<= 0)
// that of t single steps.
inline double plan_ms(const LaunchPlan& p, const double* ms) {
  auto launch = [&](int t) { return ms[t] > 0.0 ? ms[t] : t * ms[1]; };
  double sum = p.head ? (double)p.head * launch(p.T) : 0.0;
  for (int l = 0; l < p.ntail; ++l) sum += launch(p.tail[l]);
  return sum;
}

// A cached graph of a run.  The buffer that holds the state after it follows
// from the launches it was built with: a plan made later can divide the same
// run into another number (launch times measured since, or a stream now being
// captured).
template <class Exec>
struct RunGraph {
  Exec exec;
  int64_t launches;
  int buffer_after(int cur) const { return cur ^ (int)(launches & 1); }
};

// Form of an initialisation pass: tiles of 64 x 4 nodes with nontemporal or plain
// stores, or consecutive nodes with plain stores.
enum InitForm { INIT_NT, INIT_PLAIN, INIT_FLAT };

// Nontemporal stores are for states whose two buffers the last-level cache
// cannot hold: they keep smaller ones out of it, also for the launches after the
// first (initialisation, 45 steps in 9 launches and moments of 1794 x 559, three
// lattices in turn: 550 us with nontemporal stores, 54 a launch, 470 with plain
// ones; 900 x 1500, 33 steps 440 and 427; 2048 x 1024, 336 MB, 20 steps 389 and
// 402).
constexpr size_t INIT_NT_BYTES = (size_t)128 << 20;  // half of the cache
// They also need rows that fill cache lines, of 32 values: part of a line goes
// to memory as a read and a write.  And such rows leave more than half of a
// tile's lanes without a node.
constexpr int INIT_FULL_ROW = 32;

inline InitForm init_form(int nx, size_t state_bytes) {
  if (nx < INIT_FULL_ROW) return INIT_FLAT;
  return state_bytes > INIT_NT_BYTES ? INIT_NT : INIT_PLAIN;
}

// Whether a batch's initialisation stores nontemporally: as init_form for the
// pool, if most of it (full_row_bytes) belongs to instances whose rows fill
// cache lines (1024 instances of 8 x 128, a pool of 671 MB: 110 us with
// nontemporal stores, 38 with plain ones; 512 of 48 x 128: 57 and 134).
inline bool batch_init_nt(size_t pool_bytes, size_t full_row_bytes) {
  return pool_bytes > INIT_NT_BYTES && 2 * full_row_bytes > pool_bytes;
}

}  // namespace lbmh
