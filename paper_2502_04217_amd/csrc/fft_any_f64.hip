// FP64 passes of the lengths without instantiated kernels (fft_any.h), and
// the radix plan of both precisions.
#include "fft_any.h"

namespace csipm {
namespace fftk {

namespace {

// the radices of the in-place stages (with_radix), largest first
constexpr int kRadices[] = {10, 9, 8, 7, 6, 5, 4, 3, 2};

// Fewest stages, then the smallest sum of radices (balanced stages: about as
// many butterflies in each as the pencil has threads), radices not increasing.
bool search(int L, int top, int depth, int* cur, int sum, int* best, int& nbest, int& sbest) {
  if (L == 1) {
    if (depth == 0) return false;
    if (nbest == 0 || depth < nbest || (depth == nbest && sum < sbest)) {
      nbest = depth;
      sbest = sum;
      std::copy(cur, cur + depth, best);
    }
    return true;
  }
  if (depth == kAnyMaxStages || (nbest && depth >= nbest)) return false;
  bool ok = false;
  for (int r : kRadices)
    if (r <= top && L % r == 0) {
      cur[depth] = r;
      ok = search(L / r, r, depth + 1, cur, sum + r, best, nbest, sbest) || ok;
    }
  return ok;
}

// butterflies of a pencil in the stage of the largest radix
int butterflies(const AnyPlan& pl) {
  const int top = *std::max_element(pl.r, pl.r + pl.nst);
  return (pl.L + top - 1) / top;
}
// threads per pencil: as many, within kMaxThreads, in whole waves
void set_threads(AnyPlan& pl) {
  const int tm = 1 << pl.tmlog, unit = 64 / tm;
  pl.nt = std::min((butterflies(pl) + unit - 1) / unit * unit, any::kMaxThreads / tm);
}

unsigned magic(int d) { return (unsigned)((0x100000000ull + d - 1) / d); }

}  // namespace

bool any_plan(int L, int w, AnyPlan& pl) {
  if (L < 1 || L > kAnyMaxLen) return false;
  int rest = L;
  for (int f : {2, 3, 5, 7})
    while (rest % f == 0) rest /= f;
  if (rest != 1) return false;
  pl = AnyPlan{};
  pl.L = L;
  int cur[kAnyMaxStages], n = 0, sum = 0;
  if (L == 1 || !search(L, 10, 0, cur, 0, pl.r, n, sum)) {
    if (L != 1) return false;
    pl.r[0] = 1;
    n = 1;
  }
  if (n == 1) {   // (the passes want a first and a last stage)
    pl.r[1] = pl.r[0];
    pl.r[0] = 1;
    n = 2;
  }
  pl.nst = n;
  int B = L;
  for (int s = 0; s < n; ++s) {
    pl.step[s] = L / B;
    pl.ms[s] = B / pl.r[s];
    pl.mm[s] = pl.ms[s] > 1 ? magic(pl.ms[s]) : 0u;
    pl.rm[s] = pl.r[s] > 1 ? magic(pl.r[s]) : 0u;
    B /= pl.r[s];
  }
  pl.hm = L / 2 + 1 > 1 ? magic(L / 2 + 1) : 0u;
  pl.lm = L > 1 ? magic(L) : 0u;
  // pencils per workgroup: a run of one 128-byte line; more (at most 64) while
  // the pencils are too short for a whole wave.
  pl.tmlog = w == 8 ? 4 : 3;
  while ((1 << pl.tmlog) * butterflies(pl) < 64 && pl.tmlog < 6) ++pl.tmlog;
  set_threads(pl);
  return true;
}

// A pass over few long pencils has few workgroups of 16 (FP32) or 8 (FP64), and
// its time is that of one: narrower ones spread it, though a run of 4 pencils is
// a part of a line, which such an array's size makes cheap.  Tiles of one line
// against this, in us, FP32: apply_K at 1000 x 16 x 16 81, 48, at 875 x 16 x 16
// 68, 42, at 600 x 16 x 16 54, 38; apply_A at 16 x 16 x 875 38.5, 19.4, at
// 1 x 1024 x 875 50.7, 30.0; apply_At at 1 x 1 x 945 27, 16.  From kFewGroups
// workgroups on one more compute unit at work is worth less than whole lines.
void any_few(AnyPlan& pl, long long pencils, int lowest) {
  const int least = butterflies(pl);
  while (pl.tmlog > lowest && (pencils + (1 << pl.tmlog) - 1) >> pl.tmlog < kFewGroups && (1 << pl.tmlog) / 2 * least >= 64)
    --pl.tmlog;
  set_threads(pl);
}

int any_tm(int w, int L, int pencils) {
  AnyPlan pl;
  if (!any_plan(L, w, pl)) return 1;
  any_few(pl, pencils, kStridedLowest);
  return 1 << pl.tmlog;
}

CSIPM_ANY(double)
CSIPM_ANY12(double, 1, -1, EpiR)
CSIPM_ANY12(double, 1, -1, EpiRX)

}  // namespace fftk
}  // namespace csipm
