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
  // the pencils are too short for a whole wave.  Threads per pencil: as many
  // as the stage with the largest radix has butterflies, within kMaxThreads.
  const int top = *std::max_element(pl.r, pl.r + n);
  const int least = (L + top - 1) / top;
  pl.tmlog = w == 8 ? 4 : 3;
  while ((1 << pl.tmlog) * least < 64 && pl.tmlog < 6) ++pl.tmlog;
  const int tm = 1 << pl.tmlog, unit = 64 / tm;
  pl.nt = std::min((least + unit - 1) / unit * unit, any::kMaxThreads / tm);
  return true;
}

int any_tm(int w, int L) {
  AnyPlan pl;
  return any_plan(L, w, pl) ? 1 << pl.tmlog : 1;
}

CSIPM_ANY(double)
CSIPM_ANY12(double, 1, -1, EpiR)
CSIPM_ANY12(double, 1, -1, EpiRX)

}  // namespace fftk
}  // namespace csipm
