// Batches of small problems solved in one launch: one workgroup runs the
// whole interior-point solve of one problem (paper: sec. "Primal-dual
// interior-point method", equations "kkt", "kktmu" and "condensedkkt"; the
// Newton systems by PCG with the paper's preconditioner, equation
// "invprecond1"), with every scalar decision taken on the device, so a
// batch needs no host round trip until it is done.
//
// The steps are those of the library's standard form in FP64 (the readings
// of the barrier strategy, right-hand side and stopping rules); H beta is
// recomputed by a full H-apply at every iterate.
//
// An H-apply works on the half spectrum W[k1][k2][m], m <= N3 / 2, in LDS
// (row stride MS, odd: consecutive rows start on different banks).  All
// stages of all axes run in place over the whole tile, a butterfly per
// thread and round: decimation in frequency on the way to real space, which
// leaves each axis in digit-reversed slots, and decimation in time, which
// starts from them, on the way back, so nothing is ever reordered (fft_any.h
// states the two).  Two rows g and g + HR share one complex transform along
// axis 3: Z_e = A_e + i B_e takes A's slot e and Z_{N3-e} = conj A_e +
// i conj B_e B's slot e, so packing and unpacking are in place too.  Radices
// up to 8; a prime factor above 8 is one stage of direct sums.
// A grid whose tile exceeds kResident keeps W in the workspace, takes it
// through LDS in tiles of axis-1 columns and of (k2, m) planes, and is solved by
// a team of workgroups (below), which share the tiles and the vectors.
//
// What bounds it: for a resident grid the chain of stages (12 at 16^3, a
// barrier each, 2-3 thousand cycles) and the passes over the vectors at the 28
// bytes per cycle that one compute unit reaches; for a team that rate times its
// workgroups, and its four barriers per Krylov step (7 us each with 32 teams on
// the chip, 1.5 us for one alone).  Against complex transforms of the whole
// spectrum, a pencil per thread in registers (2 to 32 points) or direct DFTs in
// the workspace, one workgroup per problem, a batch takes, in ms: 64 of 16^3
// 2.6 -> 2.0; 32 of 48 x 40 x 36 397 -> 8.8; 64 of 32^3 29.6 -> 8.7; 16 of 64^3
// 2810 -> 16; 50 of 24^3 38 -> 4.8.  For the larger of these grids
// csipm_solve_batch was the better route before: on 8 host threads it took 35 ms
// for 32 problems of 48 x 40 x 36 that take 9.6 here, 57 for 64 of 32^3 (10.3),
// 28 for 16 of 64^3 (20.5).
// Sixteen waves of 128 registers instead of eight of 170 spill and lose a
// quarter.  A problem's result does not depend on the others in the batch: a
// batch of one gives the same bits.
#include "small.h"

#include "fft_any.h"

#include "../../include/csipm.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>
#include <vector>

namespace csipm {

namespace {

using fftk::any::dft_r;

constexpr int kMaxThreads = 512;
constexpr int kMaxWaves = kMaxThreads / 64;
// complex values of LDS tile at most (150 KB)
constexpr int kTile = 9600;
// largest tile that a grid is solved in by one workgroup
constexpr int kResident = 4800;
// outputs per thread and round in a stage of direct sums
constexpr int kDirect = 4;
// Fixed parts of every tile loop and sum over a grid that is not in LDS
// (Plan::parts, at most kParts), and so the most workgroups of a team: 8, and
// 16 from kLarge points.  With 16 everywhere the sums' barriers and the smaller
// tiles cost a team of 8 more than a tenth (32 problems of 48 x 40 x 36: 10.3
// against 9.2 ms); with 8 everywhere 16 problems of 64^3 leave half of the
// compute units idle (22.7 against 16.2 ms).
constexpr int kParts = 16, kLarge = 131072;

// n / d by multiplication, n d < 2^32
struct Div {
  int d;
  unsigned m;
  __device__ __forceinline__ int operator()(int n) const { return d == 1 ? n : (int)__umulhi((unsigned)n, m); }
};
Div make_div(int d) { return Div{d, d > 1 ? (unsigned)((0x100000000ull + d - 1) / d) : 0u}; }

constexpr int kStages = 6;
struct Axis {
  int L, nst;
  int r[kStages], step[kStages];
  Div ms[kStages];   // stride of a butterfly's values, B_s / R_s
};
struct Plan {
  Axis ax[3];
  int n1, n2, n3, M, MS, n;
  int resident;      // the whole half spectrum in one LDS tile
  int cols, planes;  // else: axis-1 columns and planes per tile
  int tile;          // LDS tile (complex values)
  int threads, parts;
  Div dM, dMS, dn2, dn3, dcols;
  Div dH[2], dplane[2];   // row pairs and (plane, m) pencils of a tile: all but the last, the last
  Div dcw;                // threads side by side on a tile's columns
  int cgroups;            // groups of them
};

// The plan, read where it is used: behind this the compiler cannot hoist the
// scalar loads of its fields (nor the array bases) to the top of the solver,
// where the 104 scalar registers would spill three times over and every use
// would read a vector lane.
__device__ __forceinline__ const Plan& fresh(uint64_t kernarg) {
  asm volatile("" : "+s"(kernarg));
  return *(const Plan*)(const __attribute__((address_space(4))) Plan*)kernarg;
}

// ------------------------------------------------------- block reductions --
// Sums, maxima and minima over the workgroup (every thread calls this and
// gets the result; red holds NQ kMaxWaves doubles): within the waves, then
// over the waves' values by the same exchange.
// op 0: sum, 1: max, 2: min
__device__ __forceinline__ double combine(int op, double a, double b) {
  return op == 0 ? a + b : op == 1 ? fmax(a, b) : fmin(a, b);
}
template <int NQ>
__device__ __forceinline__ void block_reduce(double* v, const int* op, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = combine(op[q], v[q], __shfl_xor(v[q], o, 64));
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < NQ; ++q) red[q * kMaxWaves + wv] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) v[q] = red[q * kMaxWaves + (lane & (nw - 1))];   // (nw is a power of two)
  for (int o = nw >> 1; o > 0; o >>= 1)
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = combine(op[q], v[q], __shfl_xor(v[q], o, 64));
}

// ------------------------------------------------------------------ teams --
// The G workgroups of a problem (one for a resident grid).  All of them take
// every decision from the same values: a sum is made of Plan::parts parts,
// part p by workgroup p mod G, combined in order by each, so the bits do not
// depend on G.  The launch makes sure that all workgroups are resident together,
// and a barrier gives up after kTeamWait all the same (work of other streams may
// hold a compute unit for long): the team then leaves kAbort in its count and
// ends, and a second launch of one workgroup per problem, which returns at once
// where the count is clean, solves those problems again.
constexpr unsigned kAbort = 0x40000000u;
struct Team {
  int G, rank;
  unsigned target;   // arrivals the next barrier waits for
  unsigned* count;   // arrivals so far (device memory, 0 at launch)
  double* parts;     // [2][kParts][5] partial sums, used in turn
  int turn;
  int* bad;          // LDS: the barrier gave up
  long long wait;    // ticks of the 100 MHz clock after which it does
};
__device__ __forceinline__ void team_sync(Team& t) {
  // Every wave waits for its own stores before the workgroup's barrier, which
  // does not: the release of thread 0 waits for those of its own wave alone.
  // (The same fence by all eight waves, each writing back the L2: 32 problems
  // of 48 x 40 x 36 23.0 ms, this 9.7.)
  if (t.G > 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (t.G == 1) return;
  t.target += t.G;
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(t.count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const long long t0 = wall_clock64();
    unsigned n;
    while ((n = __hip_atomic_load(t.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < t.target) {
      __builtin_amdgcn_s_sleep(1);
      if (wall_clock64() - t0 > t.wait) {
        __hip_atomic_fetch_or(t.count, kAbort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        n = kAbort;
        break;
      }
    }
    if (n >= kAbort) *t.bad = 1;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

// ----------------------------------------------------------------- stages --
// Calls f(std::integral_constant<int, R>) for the runtime radix r <= 8 (with 9
// and 10 as well every batch takes longer: 64 of 16^3 1.88 -> 1.94 ms, 32 of
// 48 x 40 x 36 9.65 -> 9.75, 64 of 32^3 10.3 -> 10.45).
constexpr int kMaxRadix = 8;
template <class F>
__device__ __forceinline__ void with_radix(int r, F f) {
  switch (r) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}

// Pencils of a tile: pencil b is (b / inner, b % inner), element e of it at
// (b / inner) outer + b % inner + e es.
struct Lin {
  Div inner;
  int outer, es;
  __device__ __forceinline__ int base(int b) const {
    const int q = inner(b);
    return q * outer + (b - q * inner.d);
  }
  __device__ __forceinline__ int first(int base, int e) const { return base + e * es; }
  __device__ __forceinline__ int next(int at, int, int, int q, int ms) const { return at + q * ms * es; }
  __device__ __forceinline__ int at(int base, int e) const { return base + e * es; }
};
// The row pairs of the axis-3 transform: element e < M in row g, else in row
// g + H at N3 - e.
struct Rows {
  int MS, M, L, H;
  __device__ __forceinline__ int base(int b) const { return b * MS; }
  __device__ __forceinline__ int first(int base, int e) const { return at(base, e); }
  __device__ __forceinline__ int next(int, int base, int e, int q, int ms) const { return at(base, e + q * ms); }
  __device__ __forceinline__ int at(int base, int e) const { return e < M ? base + e : base + H * MS + (L - e); }
};

__device__ __forceinline__ cx<double> tw_of(const cx<double>* tw, int i, int sgn) {
  cx<double> w = tw[i];
  if (sgn > 0) w.im = -w.im;
  return w;
}

// Stage s of np pencils in place (TIME: decimation in time).
template <int SGN, bool TIME, class Addr>
__device__ __forceinline__ void stage(cx<double>* w, const Addr& ad, uint64_t kp, int x, int s, Div np,
                                      const cx<double>* tw) {
  const Axis& ax = fresh(kp).ax[x];
  const int L = ax.L, R0 = ax.r[s], step = ax.step[s];
  const Div ms = ax.ms[s];
  __syncthreads();
  if (R0 <= kMaxRadix) {
    with_radix(R0, [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      const int total = np.d * (L / R);
#pragma unroll 1
      for (int b = threadIdx.x; b < total; b += blockDim.x) {
        const int bf = np(b), base = ad.base(b - bf * np.d);
        const int blk = ms(bf), j = bf - blk * ms.d, e0 = blk * ms.d * R + j, a0 = ad.first(base, e0);
        cx<double> v[R];
#pragma unroll
        for (int q = 0; q < R; ++q) v[q] = w[ad.next(a0, base, e0, q, ms.d)];
        const int js = j * step;
        if (TIME && ms.d > 1) {
#pragma unroll
          for (int q = 1; q < R; ++q) v[q] = cmul(v[q], tw_of(tw, q * js, SGN));
        }
        dft_r<R, SGN, double>(v);
        if (!TIME && ms.d > 1) {
#pragma unroll
          for (int q = 1; q < R; ++q) v[q] = cmul(v[q], tw_of(tw, q * js, SGN));
        }
#pragma unroll
        for (int q = 0; q < R; ++q) w[ad.next(a0, base, e0, q, ms.d)] = v[q];
      }
    });
  } else {
    // direct sums, output p of a butterfly by its own thread: a group of
    // pencils at a time, all its outputs in registers before any is written
    const int group = max(1, kDirect * (int)blockDim.x / L), unit = L / R0;
#pragma unroll 1
    for (int g0 = 0; g0 < np.d; g0 += group) {
      const int ng = min(group, np.d - g0);
      cx<double> o[kDirect];
      int dst[kDirect];
#pragma unroll
      for (int k = 0; k < kDirect; ++k) {
        const int b = threadIdx.x + k * blockDim.x;
        dst[k] = -1;
        if (b < ng * L) {
          const int e = b / ng, base = ad.base(g0 + b - e * ng);
          const int B = ms.d * R0, blk = e / B, rem = e - blk * B, p = ms(rem), j = rem - p * ms.d;
          const int inc = TIME ? (p * unit + j * step) % L : p * unit;
          double re = 0.0, im = 0.0;
          int idx = 0;
#pragma unroll 1
          for (int q = 0; q < R0; ++q) {
            const cx<double> x = w[ad.at(base, blk * B + j + q * ms.d)], t = tw_of(tw, idx, SGN);
            re += x.re * t.re - x.im * t.im;
            im += x.re * t.im + x.im * t.re;
            idx += inc;
            if (idx >= L) idx -= L;
          }
          o[k] = {re, im};
          if (!TIME) o[k] = cmul(o[k], tw_of(tw, j * p * step, SGN));
          dst[k] = ad.at(base, e);
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kDirect; ++k)
        if (dst[k] >= 0) w[dst[k]] = o[k];
      __syncthreads();
    }
  }
}

template <int SGN, bool TIME, class Addr>
__device__ __forceinline__ void axis_stages(cx<double>* w, const Addr& ad, uint64_t kp, int x, int lo, int hi, Div np,
                                            const cx<double>* tw) {
#pragma unroll 1
  for (int i = lo; i < hi; ++i) stage<SGN, TIME>(w, ad, kp, x, TIME ? hi - 1 - (i - lo) : i, np, tw);
}

// ------------------------------------------------------------- one problem --
// the per-problem arrays, each of n doubles, in the problem's workspace
// (p_beta twice: the H-apply of the new direction reads the old one at k and
// -k while it writes the new one)
enum SmallVec {
  SV_XI, SV_B, SV_Z, SV_N1, SV_N2, SV_HB, SV_S1, SV_S2, SV_XB, SV_XZ, SV_RB, SV_RZ, SV_PB, SV_PB2, SV_PZ, SV_QB,
  SV_QZ, SV_COUNT
};

// what the spectrum is formed from and what becomes of it
enum Mode {
  M_XI,      // xi = A^T b
  M_RESID,   // H beta and the residual parts of the iterate
  M_K,       // q = K p, p.q
  M_KP       // the same after p <- z + bt p
};

struct Ctx {
  uint64_t kp;                // the kernel's arguments: the plan
  int n;
  cx<double>* w;              // LDS tile
  cx<double>* wg;             // the spectrum in the workspace (not resident)
  const cx<double>* tw;       // LDS: the twiddle tables of axes 1, 2, 3
  const uint8_t* nat;         // LDS: natural index of a slot, kSmallMaxExtent per axis
  const uint8_t* obs;
  const double* sig;
  double* red;
  double *v;                  // the arrays
  double *pb, *pb_old;
  double lam, bt;
  __device__ __forceinline__ double* a(int k) const {
    uint64_t b = (uint64_t)v;   // (as fresh)
    asm volatile("" : "+s"(b));
    return (double*)(__attribute__((address_space(1))) double*)b + (long long)k * n;
  }
};

// element i of a vector, by a 32-bit offset from its (uniform) base
__device__ __forceinline__ double& el(double* p, int i) {
  return *reinterpret_cast<double*>(reinterpret_cast<char*>(p) + ((uint32_t)i << 3));
}
__device__ __forceinline__ double el(const double* p, int i) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(p) + ((uint32_t)i << 3));
}

// Loops over a tile's or a vector's values take kBatch of them per thread and
// round: the loads of all go out before the first is used (one load's
// latency per round is what such a loop costs on one compute unit).
constexpr int kBatch = 4;

// A thread's column (k2, m) of the beta side and the external indices of its
// frequencies k and -k: k1 enters as f0 + k1 s and g0 - k1 s (g0 at k1 = 0 less
// n1 s), so a loop over k1 costs no division.
struct Col {
  int k2, m, f0, g0, s;
  bool plane;   // m = 0 or N3 / 2: k and -k are two values of the spectrum
  __device__ __forceinline__ int f(int k1) const { return f0 + k1 * s; }
  __device__ __forceinline__ int g(int k1, int n1) const { return g0 + (k1 ? n1 - k1 : 0) * s; }
};
__device__ __forceinline__ Col column(const Plan& pl, int q) {
  Col c;
  c.k2 = pl.dMS(q);
  c.m = q - c.k2 * pl.MS;
  c.s = pl.n2 * pl.n3;
  c.f0 = c.k2 * pl.n3 + c.m;
  c.g0 = (c.k2 ? pl.n2 - c.k2 : 0) * pl.n3 + (c.m ? pl.n3 - c.m : 0);
  c.plane = c.m == 0 || 2 * c.m == pl.n3;
  return c;
}

// kBatch spectrum values k1 = k, k + dk, .. of a column of the input vector
// (derivation "map") into LDS (at + k1 as), the direction updated on the way
// for M_KP.
__device__ __forceinline__ void map_in(const Ctx& c, const Plan& pl, int mode, const Col& col, int k, int dk, int at,
                                       int as) {
  const double rs2 = 0.70710678118654752440;
  double b[kBatch], bm[kBatch], z[kBatch], zm[kBatch];
  const double* const x = mode == M_RESID ? c.a(SV_B) : (mode == M_K ? c.pb : c.pb_old);
#pragma unroll
  for (int u = 0; u < kBatch; ++u) {
    const int k1 = min(k + u * dk, pl.n1 - 1);
    b[u] = el(x, col.f(k1));
    bm[u] = el(x, col.g(k1, pl.n1));
  }
  if (mode == M_KP) {
    const double* const y = c.a(SV_QB);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int k1 = min(k + u * dk, pl.n1 - 1);
      z[u] = el(y, col.f(k1));
      zm[u] = el(y, col.g(k1, pl.n1));
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      b[u] = z[u] + c.bt * b[u];
      bm[u] = zm[u] + c.bt * bm[u];
    }
  }
#pragma unroll
  for (int u = 0; u < kBatch; ++u) {
    const int k1 = k + u * dk;
    if (k1 >= pl.n1) break;
    if (mode == M_KP) {
      el(c.pb, col.f(k1)) = b[u];
      if (!col.plane) el(c.pb, col.g(k1, pl.n1)) = bm[u];
    }
    const int cl = col.plane ? cls3(k1, col.k2, col.m, pl.n1, pl.n2, pl.n3) : 1;
    c.w[at + k1 * as] = cl == 0 ? cx<double>{b[u], 0.0}
                                : (cl == 1 ? cx<double>{rs2 * b[u], rs2 * bm[u]} : cx<double>{rs2 * bm[u], -rs2 * b[u]});
  }
}

// The output y = H (input) (or xi) at the coordinates of NU values; acc:
// three maxima, two sums.
template <int NU>
__device__ __forceinline__ void out_values(const Ctx& c, int mode, const int* f, const double* h, double* acc) {
  if (mode == M_XI) {
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (f[u] >= 0) {
        el(c.a(SV_XI), f[u]) = h[u];
        acc[0] = fmax(acc[0], fabs(h[u]));
      }
    return;
  }
  double x[5][NU];
  const double* const p0 = mode == M_RESID ? c.a(SV_B) : c.a(SV_S1);
  const double* const p1 = mode == M_RESID ? c.a(SV_Z) : c.a(SV_S2);
  const double* const p2 = mode == M_RESID ? c.a(SV_N1) : c.pb;
  const double* const p3 = mode == M_RESID ? c.a(SV_N2) : c.a(SV_PZ);
  const double* const p4 = mode == M_RESID ? c.a(SV_XI) : c.a(SV_QZ);
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int i = max(f[u], 0);
    x[0][u] = el(p0, i);
    x[1][u] = el(p1, i);
    x[2][u] = el(p2, i);
    x[3][u] = el(p3, i);
    x[4][u] = mode == M_K ? 0.0 : el(p4, i);
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    if (f[u] < 0) continue;
    if (mode == M_RESID) {
      const double b = x[0][u], z = x[1][u], a1 = x[2][u], a2 = x[3][u];
      const double fb = h[u] - x[4][u] - a1 + a2, fz = c.lam - a1 - a2;
      const double c1 = (z + b) * a1, c2 = (z - b) * a2;
      el(c.a(SV_HB), f[u]) = h[u];
      acc[0] = fmax(acc[0], fabs(fb));
      acc[1] = fmax(acc[1], fabs(fz));
      acc[2] = fmax(acc[2], fmax(c1, c2));
      acc[3] += c1 + c2;
      if (!isfinite(fb) || !isfinite(c1) || !isfinite(c2)) acc[4] += 1.0;
    } else {
      const double g1 = x[0][u], g2 = x[1][u], pb = x[2][u];
      double pz = x[3][u];
      if (mode == M_KP) {
        pz = x[4][u] + c.bt * pz;
        el(c.a(SV_PZ), f[u]) = pz;
      }
      const double L1 = g1 + g2, L2 = g1 - g2;
      const double qb = h[u] + L1 * pb + L2 * pz, qz = L2 * pb + L1 * pz;
      el(c.a(SV_QB), f[u]) = qb;
      el(c.a(SV_QZ), f[u]) = qz;
      acc[3] += pb * qb + pz * qz;
    }
  }
}
// Two spectrum values k1 = k, k + dk of a column: up to four coordinates.
__device__ __forceinline__ void map_out(const Ctx& c, const Plan& pl, int mode, const Col& col, int k, int dk, int at,
                                        int as, double* acc) {
  const double sq2 = 1.41421356237309504880;
  int f[4];
  double h[4];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int k1 = k + u * dk, kk = min(k1, pl.n1 - 1);
    const bool on = k1 < pl.n1;
    const cx<double> x = c.w[at + kk * as];
    const int cl = col.plane ? cls3(kk, col.k2, col.m, pl.n1, pl.n2, pl.n3) : 1;
    f[2 * u] = on ? col.f(kk) : -1;
    f[2 * u + 1] = on && !col.plane ? col.g(kk, pl.n1) : -1;
    h[2 * u] = cl == 0 ? x.re : (cl == 1 ? sq2 * x.re : -sq2 * x.im);
    h[2 * u + 1] = sq2 * x.im;
  }
  out_values<4>(c, mode, f, h, acc);
}

// v: this workgroup's parts (acc of part p passed to put as they are done)
// combined over the team.
__device__ __forceinline__ void put_part(const Team& t, int part, const double* acc, int nq) {
  if (threadIdx.x == 0)
    for (int q = 0; q < nq; ++q) t.parts[(t.turn * kParts + part) * 5 + q] = acc[q];
}
template <int NQ>
__device__ __forceinline__ void take_parts(Team& t, int parts, double* v, const int* op) {
  team_sync(t);
  const double* const p = t.parts + t.turn * kParts * 5;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double a = p[q];
    for (int k = 1; k < parts; ++k) a = combine(op[q], a, p[k * 5 + q]);
    v[q] = a;
  }
  t.turn ^= 1;
}

// The whole apply, in one pass over the resident tile, or in three over
// tiles of axis-1 columns, planes and columns again; v: the maxima and sums
// of the output.  (Every kind of stage has one call here, and the solver one
// call of this: the butterflies of each would be compiled in again.)
__device__ __forceinline__ void apply(const Ctx& c, Team& team, int mode, double* v) {
  constexpr int NQ = 5;
  constexpr int op[NQ] = {1, 1, 1, 0, 0};
  cx<double>* const w = c.w;
  const Plan& pl0 = fresh(c.kp);
  const bool res = pl0.resident, xi = mode == M_XI;
  for (int ph = xi && !res ? 1 : 0; ph < (res ? 1 : 3); ++ph) {
    const Plan& plp = fresh(c.kp);
    const bool cols = !res && ph != 1;             // tiles of axis-1 columns
    const bool inv1 = !xi && ph == 0, mid = res || ph == 1, out = res || ph == 2;
    const int nt = res ? 1 : (cols ? (plp.n2 * plp.MS + plp.cols - 1) / plp.cols : (plp.n1 + plp.planes - 1) / plp.planes);
    const int parts = plp.parts;
#pragma unroll 1
    for (int part = res ? 0 : team.rank; part < parts; part += team.G) {
      double acc[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
#pragma unroll 1
      for (int t = part; t < nt; t += parts) {
        const Plan& pl = fresh(c.kp);
        const int C = pl.n2 * pl.MS, T = pl.cols, n3 = pl.n3, last = pl.ax[2].nst - 1;
        const bool prime = pl.ax[2].r[last] > kMaxRadix;
        const int q0 = t * T, nc = min(T, C - q0);               // columns
        const int s0 = res ? 0 : t * pl.planes, np1 = res ? pl.n1 : min(pl.planes, pl.n1 - s0);   // planes
        const int lt = t == nt - 1 ? 1 : 0, NR = np1 * pl.n2;
        const Div dH = pl.dH[lt], d2 = pl.dplane[lt];
        const int H = dH.d;
        const Rows ad3{pl.MS, pl.M, n3, H};
        // the thread's columns of the tile on the beta side: column cq + i cw,
        // k1 = ck, ck + cg, ..
        const int cw = pl.dcw.d, cg = pl.cgroups, ck = pl.dcw(threadIdx.x), cq = threadIdx.x - ck * cw;
        // row of the tile and natural index along axis 3 -> sample
        auto sample = [&](int row, int e) {
          const int q = pl.dn2(row);
          return (c.nat[s0 + q] * pl.n2 + c.nat[kSmallMaxExtent + row - q * pl.n2]) * n3 + e;
        };
        __syncthreads();
        if (inv1) {
#pragma unroll 1
          for (int q = cq; q < nc; q += cw) {
            const Col col = column(pl, q0 + q);
            if (ck >= cg) break;
            if (col.m < pl.M) {
#pragma unroll 1
              for (int k = ck; k < pl.n1; k += kBatch * cg) map_in(c, pl, mode, col, k, cg, q, T);
            } else {
#pragma unroll 1
              for (int k = ck; k < pl.n1; k += cg) w[k * T + q] = {0.0, 0.0};
            }
          }
        } else if (cols) {
#pragma unroll 1
          for (int i = threadIdx.x; i < pl.n1 * T; i += blockDim.x) {
            const int s = pl.dcols(i), q = i - s * T;
            w[i] = q < nc ? c.wg[s * C + q0 + q] : cx<double>{0.0, 0.0};
          }
        } else if (!xi) {
#pragma unroll 1
          for (int i = threadIdx.x; i < np1 * C; i += blockDim.x) w[i] = c.wg[s0 * C + i];
        }
        // axes 1 and 2 to real space
#pragma unroll 1
        for (int x = 0; x < 2; ++x)
          if (!xi && (x == 0 ? inv1 : mid) && pl.ax[x].L > 1)
            axis_stages<+1, false>(w, x == 0 ? Lin{pl.dcols, 0, T} : Lin{pl.dMS, C, pl.MS}, c.kp, x, 0, pl.ax[x].nst,
                                   x == 0 ? pl.dcols : d2, c.tw + (x == 0 ? 0 : pl.n1));
        if (mid) {
          const cx<double>* const tw3 = c.tw + pl.n1 + pl.n2;
          __syncthreads();
          if (xi) {
#pragma unroll 1
            for (int i = threadIdx.x; i < H * n3; i += blockDim.x) {
              const int g = pl.dn3(i), s = i - g * n3, e = c.nat[2 * kSmallMaxExtent + s];
              const int fa = sample(g, e), fb = g + H < NR ? sample(g + H, e) : -1;
              w[ad3.at(ad3.base(g), s)] = {c.obs[fa] ? c.sig[fa] : 0.0, fb >= 0 && c.obs[fb] ? c.sig[fb] : 0.0};
            }
          } else {
#pragma unroll 1
            for (int i = threadIdx.x; i < H * pl.M; i += blockDim.x) {
              const int g = pl.dM(i), e = i - g * pl.M;
              const cx<double> x = w[g * pl.MS + e];
              const cx<double> y = g + H < NR ? w[(g + H) * pl.MS + e] : cx<double>{0.0, 0.0};
              if (e == 0 || 2 * e == n3) {   // (real values)
                w[g * pl.MS + e] = {x.re, y.re};
              } else {
                w[g * pl.MS + e] = {x.re - y.im, x.im + y.re};
                w[(g + H) * pl.MS + e] = {x.re + y.im, y.re - x.im};
              }
            }
            axis_stages<+1, false>(w, ad3, c.kp, 2, 0, prime ? last + 1 : last, dH, tw3);
            __syncthreads();
            if (prime) {
#pragma unroll 1
              for (int i = threadIdx.x; i < H * n3; i += blockDim.x) {
                const int s = dH(i), g = i - s * H, e = c.nat[2 * kSmallMaxExtent + s];
                cx<double>& x = w[ad3.at(ad3.base(g), s)];
                if (!c.obs[sample(g, e)]) x.re = 0.0;
                if (g + H >= NR || !c.obs[sample(g + H, e)]) x.im = 0.0;
              }
            } else {
              // the last inverse stage, the mask and the first forward stage
              // on the same values
              with_radix(pl.ax[2].r[last], [&](auto rc) {
                constexpr int R = decltype(rc)::value;
                const int total = H * (n3 / R);
#pragma unroll 1
                for (int b = threadIdx.x; b < total; b += blockDim.x) {
                  const int bf = dH(b), g = b - bf * H, base = ad3.base(g);
                  cx<double> u[R];
#pragma unroll
                  for (int q = 0; q < R; ++q) u[q] = w[ad3.at(base, bf * R + q)];
                  dft_r<R, +1, double>(u);
                  // (a row without a partner: the imaginary part is dropped when unpacked)
                  const int ra = sample(g, 0), rb = sample(min(g + H, NR - 1), 0);
#pragma unroll
                  for (int q = 0; q < R; ++q) {
                    const int e = c.nat[2 * kSmallMaxExtent + bf * R + q];
                    const int oa = c.obs[ra + e], ob = c.obs[rb + e];
                    u[q].re = oa ? u[q].re : 0.0;
                    u[q].im = ob ? u[q].im : 0.0;
                  }
                  dft_r<R, -1, double>(u);
#pragma unroll
                  for (int q = 0; q < R; ++q) w[ad3.at(base, bf * R + q)] = u[q];
                }
              });
            }
          }
          axis_stages<-1, true>(w, ad3, c.kp, 2, 0, xi || prime ? last + 1 : last, dH, tw3);
          __syncthreads();
          const double sc = xi ? 0.5 / sqrt((double)pl.n) : 0.5 / (double)pl.n;
#pragma unroll 1
          for (int i = threadIdx.x; i < H * pl.M; i += blockDim.x) {
            const int g = pl.dM(i), e = i - g * pl.M;
            const cx<double> y = w[g * pl.MS + e];
            cx<double> x0, x1;
            if (e == 0 || 2 * e == n3) {
              x0 = {2.0 * sc * y.re, 0.0};
              x1 = {2.0 * sc * y.im, 0.0};
            } else {
              const cx<double> z = w[(g + H) * pl.MS + e];
              x0 = cscale(cx<double>{y.re + z.re, y.im - z.im}, sc);
              x1 = cscale(cx<double>{y.im + z.im, z.re - y.re}, sc);
            }
            w[g * pl.MS + e] = x0;
            if (g + H < NR) w[(g + H) * pl.MS + e] = x1;
          }
        }
        // axes 2 and 1 back
#pragma unroll 1
        for (int x = 1; x >= 0; --x)
          if ((x == 0 ? out : mid) && pl.ax[x].L > 1)
            axis_stages<-1, true>(w, x == 0 ? Lin{pl.dcols, 0, T} : Lin{pl.dMS, C, pl.MS}, c.kp, x, 0, pl.ax[x].nst,
                                  x == 0 ? pl.dcols : d2, c.tw + (x == 0 ? 0 : pl.n1));
        __syncthreads();
        if (out) {
#pragma unroll 1
          for (int q = cq; q < nc; q += cw) {
            const Col col = column(pl, q0 + q);
            if (ck >= cg || col.m >= pl.M) continue;
#pragma unroll 1
            for (int k = ck; k < pl.n1; k += 2 * cg) map_out(c, pl, mode, col, k, cg, q, T, acc);
          }
        } else if (cols) {
#pragma unroll 1
          for (int i = threadIdx.x; i < pl.n1 * T; i += blockDim.x) {
            const int s = pl.dcols(i), q = i - s * T;
            if (q < nc) c.wg[s * C + q0 + q] = w[i];
          }
        } else {
#pragma unroll 1
          for (int i = threadIdx.x; i < np1 * C; i += blockDim.x) c.wg[s0 * C + i] = w[i];
        }
      }
      if (out) {
        if (mode == M_RESID) block_reduce<NQ>(acc, op, c.red);
        else if (xi) block_reduce<1>(acc, op, c.red);
        else block_reduce<1>(acc + 3, op + 3, c.red);
        if (res) {
#pragma unroll
          for (int q = 0; q < NQ; ++q) v[q] = acc[q];
        } else {
          put_part(team, part, acc, NQ);
        }
      }
    }
    if (!res) {
      if (out) take_parts<NQ>(team, plp.parts, v, op);
      else team_sync(team);
    }
  }
}

// P^{-1} of one 2x2 block (equation "invprecond1", C = I)
__device__ __forceinline__ void pinv1(double rb, double rz, double s1, double s2, double& zb, double& zz) {
  const double L1 = s1 + s2, L2 = s1 - s2;
  const double D = L1 + 4.0 * s1 * s2;
  zb = (L1 * rb - L2 * rz) / D;
  zz = (-L2 * rb + (1.0 + L1) * rz) / D;
}

// largest a with v + a dv >= 0 over this thread's share (inf if none)
__device__ __forceinline__ double ratio(double v, double dv) { return dv < 0.0 ? -v / dv : INFINITY; }

__global__ void __launch_bounds__(kMaxThreads)
k_small_solve(Plan pl, const double* __restrict__ signals, const uint8_t* __restrict__ observed,
              const double* __restrict__ lambdas, double lambda_frac, double* __restrict__ beta_out,
              double* __restrict__ info, char* __restrict__ ws, long long ws_stride, const cx<double>* __restrict__ tw,
              unsigned* __restrict__ counters, int count, int G, SmallOpts o, long long wait, int again) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[5 * kMaxWaves];
  __shared__ uint8_t nat[3 * kSmallMaxExtent];
  __shared__ int bad;
  // workgroups go to the 8 XCDs in turn: a team stays on one (its vectors and
  // spectrum in that L2)
  const int n = pl.n, prob = G == 1 ? (int)blockIdx.x : (int)blockIdx.x / (8 * G) * 8 + (int)blockIdx.x % 8;
  if (prob >= count) return;
  if (again && counters[16 * prob] < kAbort) return;   // (solved by its team)
  if (threadIdx.x == 0) bad = 0;
  double* const v = reinterpret_cast<double*>(ws + (long long)prob * ws_stride);
  cx<double>* const twl = reinterpret_cast<cx<double>*>(smem);
#pragma unroll 1
  for (int i = threadIdx.x; i < pl.n1 + pl.n2 + pl.n3; i += blockDim.x) twl[i] = tw[i];
  // slot -> natural index of each axis
#pragma unroll 1
  for (int x = 0; x < 3; ++x)
#pragma unroll 1
    for (int k = threadIdx.x; k < pl.ax[x].L; k += blockDim.x) {
      int slot = 0, r = k;
      for (int s = 0; s < pl.ax[x].nst; ++s) {
        slot = slot * pl.ax[x].r[s] + r % pl.ax[x].r[s];
        r /= pl.ax[x].r[s];
      }
      nat[x * kSmallMaxExtent + slot] = (uint8_t)k;
    }
  __syncthreads();
  Ctx c;
  c.kp = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();   // (the plan is the first argument)
  c.n = n;
  c.w = twl + (pl.n1 + pl.n2 + pl.n3);
  c.wg = reinterpret_cast<cx<double>*>(v + ((long long)SV_COUNT * n + 1) / 2 * 2);
  c.tw = twl;
  c.nat = nat;
  c.obs = observed + (long long)prob * n;
  c.sig = signals + (long long)prob * n;
  c.red = red;
  c.v = v;
  c.pb = c.a(SV_PB);
  c.pb_old = c.a(SV_PB2);
  const int parts = pl.parts;
  Team team{G, G == 1 ? 0 : (int)blockIdx.x / 8 % G, 0u, counters + 16 * (G == 1 ? 0 : prob),
            reinterpret_cast<double*>(c.wg + (pl.resident ? 0 : pl.n1 * pl.n2 * pl.MS)), 0, &bad, wait};
  // sum (or minimum) over the coordinates, in fixed parts: f(load(i)) with the
  // loads of two coordinates ahead of the first use
  auto over = [&](int op, auto load, auto f) {
    double tot = 0.0;
#pragma unroll 1
    for (int part = team.rank; part < parts; part += team.G) {
      const int lo = (int)((long long)n * part / parts), hi = (int)((long long)n * (part + 1) / parts);
      double a = op == 2 ? INFINITY : 0.0;
#pragma unroll 1
      for (int i = lo + (int)threadIdx.x; i < hi; i += 2 * blockDim.x) {
        const int j = i + blockDim.x;
        const auto x = load(i), y = load(min(j, n - 1));
        a = combine(op, a, f(i, x));
        if (j < hi) a = combine(op, a, f(j, y));
      }
      block_reduce<1>(&a, &op, red);
      tot = a;
      if (parts > 1) put_part(team, part, &a, 1);
    }
    if (parts > 1) take_parts<1>(team, parts, &tot, &op);
    return tot;
  };

  // One apply after another; what follows each decides on the next:
  //   xi = A^T b_hat: lambda, the starting point beta = 0, z = |xi|_inf (1 if
  //     0), nu = lambda / 2 (reading "barrier strategy"), then the residual;
  //   H beta: the KKT residual, then the Newton system and its first q = K p;
  //   q = K p: a PCG step, then the next direction's, or the step of the
  //     iterate and the next residual.
  int it = 0, cg = 0, cg_total = 0, status = 1;   // 1: not converged (iteration limit)
  double rel = INFINITY, mu = 0.0, xinf = 0.0, smu = 0.0, rho = 0.0, tol = 0.0;
  c.lam = 0.0;
  c.bt = 0.0;
  for (int mode = M_XI;;) {
    double q[5];
    apply(c, team, mode, q);
    if (bad) break;   // (written before a barrier that all have passed)
    if (mode == M_XI) {
      xinf = q[0];
      c.lam = lambdas ? lambdas[prob] : lambda_frac * xinf;
      const double z0 = xinf > 0.0 ? xinf : 1.0;
      double *const be = c.a(SV_B), *const zv = c.a(SV_Z), *const nu1 = c.a(SV_N1), *const nu2 = c.a(SV_N2);
      for (int f = team.rank * blockDim.x + threadIdx.x; f < n; f += team.G * blockDim.x) {
        el(be, f) = 0.0;
        el(zv, f) = z0;
        el(nu1, f) = 0.5 * c.lam;
        el(nu2, f) = 0.5 * c.lam;
      }
      team_sync(team);
      mode = M_RESID;
      continue;
    }
    if (mode == M_RESID) {
      // the iterate's relative residual (equation "kkt")
      mu = q[3] / (2.0 * (double)n);
      rel = fmax(fmax(q[0], q[1]), q[2]) / (1.0 + xinf);
      if (q[4] > 0.0) {
        status = -2;   // non-finite iterate
        break;
      }
      if (rel <= o.tol) {
        status = 0;
        break;
      }
      if (it >= o.max_iter) break;
      // Newton system (equation "condensedkkt"): Sigma_j = nu_j / s_j and the
      // right-hand side from equation "kktmu" (reading "Newton RHS"), in r;
      // PCG from x = 0 on K with the paper's P
      smu = o.sigma * mu;
      const double eta = fmin(o.cg_rtol, 0.1 * rel), lam = c.lam;
      const double *const be = c.a(SV_B), *const zv = c.a(SV_Z), *const nu1 = c.a(SV_N1), *const nu2 = c.a(SV_N2),
                   *const hb = c.a(SV_HB), *const xi = c.a(SV_XI);
      double *const g1 = c.a(SV_S1), *const g2 = c.a(SV_S2), *const rb = c.a(SV_RB), *const rz = c.a(SV_RZ),
             *const pz = c.a(SV_PZ);
      struct State { double b, z, a1, a2, h, x; };
      rho = over(0, [&](int f) { return State{el(be, f), el(zv, f), el(nu1, f), el(nu2, f), el(hb, f), el(xi, f)}; }, [&](int f, State s) {
        const double s1 = s.z + s.b, s2 = s.z - s.b;
        const double i1 = 1.0 / s1, i2 = 1.0 / s2;
        const double a1 = s.a1 * i1, a2 = s.a2 * i2;
        el(g1, f) = a1;
        el(g2, f) = a2;
        const double r1 = -(s.h - s.x) + smu * (i1 - i2);
        const double r2 = -lam + smu * (i1 + i2);
        el(rb, f) = r1;
        el(rz, f) = r2;
        double w1v, w2v;
        pinv1(r1, r2, a1, a2, w1v, w2v);
        el(c.pb, f) = w1v;
        el(pz, f) = w2v;
        return r1 * w1v + r2 * w2v;
      });
      tol = fmax(o.cg_atol, eta * sqrt(fmax(rho, 0.0)));
      cg = 0;
    } else {
      const double alpha = rho / q[3];
      const bool first = cg == 0;
      const double *const pz = c.a(SV_PZ), *const g1 = c.a(SV_S1), *const g2 = c.a(SV_S2);
      double *const xb = c.a(SV_XB), *const xz = c.a(SV_XZ), *const rb = c.a(SV_RB), *const rz = c.a(SV_RZ),
             *const qb = c.a(SV_QB), *const qz = c.a(SV_QZ);
      struct Krylov { double pb, pz, xb, xz, rb, rz, qb, qz, g1, g2; };
      auto load = [&](int f) {
        return Krylov{el(c.pb, f), el(pz, f), first ? 0.0 : el(xb, f), first ? 0.0 : el(xz, f), el(rb, f), el(rz, f), el(qb, f), el(qz, f), el(g1, f),
                      el(g2, f)};
      };
      const double rn = over(0, load, [&](int f, Krylov k) {
        el(xb, f) = k.xb + alpha * k.pb;
        el(xz, f) = k.xz + alpha * k.pz;
        const double r1 = k.rb - alpha * k.qb, r2 = k.rz - alpha * k.qz;
        el(rb, f) = r1;
        el(rz, f) = r2;
        double w1v, w2v;
        pinv1(r1, r2, k.g1, k.g2, w1v, w2v);
        el(qb, f) = w1v;   // z = P^{-1} r, kept in q until the direction update
        el(qz, f) = w2v;
        return r1 * w1v + r2 * w2v;
      });
      c.bt = rn / rho;
      rho = rn;
      ++cg;
    }
    if (sqrt(fmax(rho, 0.0)) > tol && cg < o.cg_max) {
      mode = cg == 0 ? M_K : M_KP;
      if (cg > 0) {
        double* const t = c.pb;
        c.pb = c.pb_old;
        c.pb_old = t;
      }
      continue;
    }
    cg_total += cg;
    // multiplier direction, step to the boundary and update
    const bool none = cg == 0;
    double *const be = c.a(SV_B), *const zv = c.a(SV_Z), *const nu1 = c.a(SV_N1), *const nu2 = c.a(SV_N2),
           *const xb = c.a(SV_XB), *const xz = c.a(SV_XZ), *const rb = c.a(SV_RB), *const rz = c.a(SV_RZ);
    const double *const g1 = c.a(SV_S1), *const g2 = c.a(SV_S2);
    struct Dir { double b, z, a1, a2, d1, d2, g1, g2; };
    auto load = [&](int f) {
      return Dir{el(be, f), el(zv, f), el(nu1, f), el(nu2, f), none ? 0.0 : el(xb, f), none ? 0.0 : el(xz, f), el(g1, f), el(g2, f)};
    };
    const double amax = over(2, load, [&](int f, Dir d) {
      if (none) {
        el(xb, f) = 0.0;
        el(xz, f) = 0.0;
      }
      const double s1 = d.z + d.b, s2 = d.z - d.b;
      const double ds1 = d.d1 + d.d2, ds2 = d.d2 - d.d1;
      const double dn1 = smu / s1 - d.a1 - d.g1 * ds1;
      const double dn2 = smu / s2 - d.a2 - d.g2 * ds2;
      el(rb, f) = dn1;
      el(rz, f) = dn2;
      return fmin(fmin(ratio(s1, ds1), ratio(s2, ds2)), fmin(ratio(d.a1, dn1), ratio(d.a2, dn2)));
    });
    const double step = fmin(1.0, o.tau * amax);
#pragma unroll 1
    for (int part = team.rank; part < parts; part += team.G) {
      const int lo = (int)((long long)n * part / parts), hi = (int)((long long)n * (part + 1) / parts);
#pragma unroll 1
      for (int i = lo + (int)threadIdx.x; i < hi; i += 2 * blockDim.x) {
        struct Step { double b, z, a1, a2, xb, xz, r1, r2; };
        auto get = [&](int f) { return Step{el(be, f), el(zv, f), el(nu1, f), el(nu2, f), el(xb, f), el(xz, f), el(rb, f), el(rz, f)}; };
        auto put = [&](int f, const Step& d) {
          el(be, f) = d.b + step * d.xb;
          el(zv, f) = d.z + step * d.xz;
          el(nu1, f) = d.a1 + step * d.r1;
          el(nu2, f) = d.a2 + step * d.r2;
        };
        const int j = i + blockDim.x;
        const Step x = get(i), y = get(min(j, n - 1));
        put(i, x);
        if (j < hi) put(j, y);
      }
    }
    team_sync(team);
    mode = M_RESID;
    ++it;
  }
  __syncthreads();
  for (int f = team.rank * blockDim.x + threadIdx.x; f < n; f += team.G * blockDim.x)
    beta_out[(long long)prob * n + f] = el(c.a(SV_B), f);
  if (threadIdx.x == 0 && team.rank == 0) {
    double* out = info + (long long)prob * CSIPM_SMALL_INFO;
    out[0] = (double)status;
    out[1] = (double)it;
    out[2] = (double)cg_total;
    out[3] = rel;
    out[4] = mu;
    out[5] = c.lam;
  }
}

// Radices of an axis: primes above 8 first, then the fewest of 2 .. 8 (the
// smallest sum among those, largest first).
void search(int L, int top, int depth, int* cur, int sum, int* best, int& nbest, int& sbest) {
  if (L == 1) {
    if (nbest == 0 || depth < nbest || (depth == nbest && sum < sbest)) {
      nbest = depth;
      sbest = sum;
      std::copy(cur, cur + depth, best);
    }
    return;
  }
  if (depth == kStages || (nbest && depth >= nbest)) return;
  for (int r = std::min(top, kMaxRadix); r >= 2; --r)
    if (L % r == 0) {
      cur[depth] = r;
      search(L / r, r, depth + 1, cur, sum + r, best, nbest, sbest);
    }
}

Axis make_axis(int L) {
  Axis ax{};
  ax.L = L;
  int rest = L, n = 0;
  for (int p = 11; p <= L; ++p)
    while (rest % p == 0 && [&] { for (int d = 2; d * d <= p; ++d) if (p % d == 0) return false; return true; }()) {
      ax.r[n++] = p;
      rest /= p;
    }
  if (rest > 1) {
    int cur[kStages], best[kStages], nb = 0, sb = 0;
    search(rest, kMaxRadix, 0, cur, 0, best, nb, sb);
    for (int i = 0; i < nb; ++i) ax.r[n++] = best[i];
  }
  if (n == 0) ax.r[n++] = 1;
  ax.nst = n;
  int B = L;
  for (int s = 0; s < n; ++s) {
    ax.step[s] = L / B;
    ax.ms[s] = make_div(B / ax.r[s]);
    B /= ax.r[s];
  }
  return ax;
}

Plan make_plan(int n1, int n2, int n3) {
  Plan pl{};
  pl.n1 = n1;
  pl.n2 = n2;
  pl.n3 = n3;
  pl.n = n1 * n2 * n3;
  pl.M = n3 / 2 + 1;
  pl.MS = pl.M | 1;
  const int L[3] = {n1, n2, n3};
#pragma unroll 1
  for (int x = 0; x < 3; ++x) pl.ax[x] = make_axis(L[x]);
  const int C = n2 * pl.MS, rows = (n1 * n2 + 1) / 2 * 2;
  pl.resident = rows * pl.MS <= kResident;
  if (pl.resident) {
    pl.tile = rows * pl.MS;
    pl.cols = C;
    pl.parts = 1;
  } else {
    // about as many tiles of columns and of planes as parts
    auto up8 = [](int x) { return (x + 7) / 8 * 8; };
    pl.parts = pl.n < kLarge ? kParts / 2 : kParts;
    pl.cols = std::min({up8((C + pl.parts - 1) / pl.parts), kMaxThreads, kTile / n1 / 8 * 8});
    pl.planes = std::min((n1 + pl.parts - 1) / pl.parts, std::max(1, kTile / ((n2 + 1) / 2 * 2 * pl.MS)));
    pl.tile = std::max(pl.cols * n1, ((pl.planes * n2 + 1) / 2 * 2) * pl.MS);
  }
  pl.threads = kMaxThreads;
  pl.dM = make_div(pl.M);
  pl.dMS = make_div(pl.MS);
  pl.dn2 = make_div(n2);
  pl.dn3 = make_div(n3);
  pl.dcols = make_div(pl.cols);
  const int full = pl.resident ? n1 : pl.planes, rest = n1 % full ? n1 % full : full;
  for (int k = 0; k < 2; ++k) {
    const int np = k ? rest : full;
    pl.dH[k] = make_div((np * n2 + 1) / 2);
    pl.dplane[k] = make_div(np * pl.MS);
  }
  pl.dcw = make_div(std::min(pl.cols, pl.threads));
  pl.cgroups = std::max(1, pl.threads / pl.cols);
  return pl;
}

}  // namespace

bool small_supported(int n1, int n2, int n3) {
  return n1 >= 1 && n2 >= 1 && n3 >= 1 && n1 <= kSmallMaxExtent && n2 <= kSmallMaxExtent &&
         n3 <= kSmallMaxExtent;
}

size_t small_front_bytes(int n1, int n2, int n3) {
  const size_t b = sizeof(cx<double>) * (size_t)(n1 + n2 + n3) + 64 * (size_t)kSmallTeams;
  return (b + 255) & ~(size_t)255;
}

size_t small_problem_bytes(int n1, int n2, int n3) {
  if (tiny_grid(n1, n2, n3)) return tiny_problem_bytes(n1, n2, n3);
  const Plan pl = make_plan(n1, n2, n3);
  // SV_COUNT real arrays, and, when the spectrum does not sit in LDS, it and
  // the parts of the sums
  size_t b = sizeof(double) * (((size_t)pl.n * (size_t)SV_COUNT + 1) / 2 * 2) +
             (pl.resident ? 0 : (size_t)n1 * n2 * pl.MS * sizeof(cx<double>) + 2 * kParts * 5 * sizeof(double));
  return (b + 255) & ~(size_t)255;
}

hipError_t small_launch(int n1, int n2, int n3, int count, const double* signals, const uint8_t* observed,
                        const double* lambdas, double lambda_frac, double* beta_out, double* info, char* ws,
                        const cx<double>* tw, unsigned* counters, const SmallOpts& o, long long wait, hipStream_t s) {
  if (tiny_grid(n1, n2, n3))
    return tiny_launch(n1, n2, n3, count, signals, observed, lambdas, lambda_frac, beta_out, info, ws, tw, o, s);
  const Plan pl = make_plan(n1, n2, n3);
  const size_t shm = (size_t)(pl.tile + n1 + n2 + n3) * sizeof(cx<double>);
  if (shm > 65536) {
    const hipError_t e =
        hipFuncSetAttribute((const void*)k_small_solve, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
  }
  long long stride = (long long)small_problem_bytes(n1, n2, n3);
  int G = 1, again = 0;
  if (!pl.resident && count <= kSmallTeams) {
    // teams of as many workgroups as are resident together, launched
    // cooperatively (which guarantees it, whatever else the device runs)
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, (const void*)k_small_solve, pl.threads, shm) == hipSuccess) {
      const int slots = (count + 7) / 8 * 8;
      while (2 * G <= pl.parts && 2 * G * slots <= cus * per) G *= 2;
    }
    if (G > 1) {
      Plan plan = pl;
      SmallOpts opts = o;
      void* args[] = {&plan, &signals, &observed, &lambdas, &lambda_frac, &beta_out, &info, &ws, &stride, &tw,
                      &counters, &count, &G, &opts, &wait, &again};
      const hipError_t e = hipLaunchCooperativeKernel((const void*)k_small_solve, dim3((count + 7) / 8 * 8 * G),
                                                      dim3(pl.threads), args, (unsigned)shm, s);
      if (e == hipSuccess) again = 1;
      else (void)hipGetLastError();   // (refused: one workgroup per problem)
    }
  }
  hipLaunchKernelGGL(k_small_solve, dim3(count), dim3(pl.threads), shm, s, pl, signals, observed, lambdas, lambda_frac,
                     beta_out, info, ws, stride, tw, counters, count, 1, o, wait, again);
  return hipGetLastError();
}

}  // namespace csipm

using csipm::cx;

extern "C" size_t csipm_small_workspace_bytes(int n1, int n2, int n3, int count) {
  if (!csipm::small_supported(n1, n2, n3) || count < 1) return 0;
  return csipm::small_front_bytes(n1, n2, n3) + (size_t)count * csipm::small_problem_bytes(n1, n2, n3);
}

extern "C" csipm_status csipm_solve_small_batch(int n1, int n2, int n3, int count, const double* d_signals,
                                                const uint8_t* d_observed, const double* d_lambdas,
                                                double lambda_frac, const csipm_options* opts, double* d_beta_out,
                                                double* d_info, void* d_workspace, size_t workspace_bytes,
                                                void* hip_stream) {
  return csipm_solve_small_batch_wait(n1, n2, n3, count, d_signals, d_observed, d_lambdas, lambda_frac, opts,
                                      d_beta_out, d_info, d_workspace, workspace_bytes, hip_stream,
                                      csipm::kTeamWait);
}

extern "C" csipm_status csipm_solve_small_batch_wait(int n1, int n2, int n3, int count, const double* d_signals,
                                                     const uint8_t* d_observed, const double* d_lambdas,
                                                     double lambda_frac, const csipm_options* opts,
                                                     double* d_beta_out, double* d_info, void* d_workspace,
                                                     size_t workspace_bytes, void* hip_stream, long long wait) {
  if (count < 1 || !d_signals || !d_observed || !opts || !d_beta_out || !d_info || !d_workspace ||
      (!d_lambdas && !(lambda_frac > 0.0 && std::isfinite(lambda_frac)))) {
    csipm::noctx_set_error("solve_small_batch: bad argument");
    return CSIPM_EINVAL;
  }
  if ((reinterpret_cast<uintptr_t>(d_workspace) & 255) != 0) {
    csipm::noctx_set_error("solve_small_batch: workspace not 256-byte aligned");
    return CSIPM_EINVAL;
  }
  if (!csipm::small_supported(n1, n2, n3)) {
    csipm::noctx_set_error("solve_small_batch: extents must lie in [1, 64]");
    return CSIPM_EUNSUPPORTED;
  }
  if (!(opts->tol > 0.0) || opts->max_iter < 0 || opts->cg_max < 0 || !(opts->tau > 0.0 && opts->tau < 1.0) ||
      !(opts->sigma > 0.0 && opts->sigma <= 1.0) || !(opts->cg_rtol >= 0.0) || !(opts->cg_atol >= 0.0)) {
    csipm::noctx_set_error("solve_small_batch: options out of range");
    return CSIPM_EINVAL;
  }
  const size_t need = csipm_small_workspace_bytes(n1, n2, n3, count);
  if (workspace_bytes < need) {
    csipm::noctx_set_error("solve_small_batch: workspace smaller than csipm_small_workspace_bytes");
    return CSIPM_ENOMEM;
  }
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  // twiddle tables exp(-2 pi i q / L) for L = n1, n2, n3, from long double
  // rounded once, at the front of the workspace
  std::vector<cx<double>> h;
  for (int L : {n1, n2, n3})
    for (int q = 0; q < L; ++q) {
      const long double a = -2.0L * 3.141592653589793238462643383279502884L * (long double)q / (long double)L;
      h.push_back({(double)cosl(a), (double)sinl(a)});
    }
  // and, behind them, the team counters, 0 (64 bytes each)
  const size_t ntw = h.size();
  h.resize(ntw + 4 * (size_t)csipm::kSmallTeams, cx<double>{0.0, 0.0});
  char* ws = reinterpret_cast<char*>(d_workspace);
  hipError_t e = hipMemcpyAsync(ws, h.data(), h.size() * sizeof(cx<double>), hipMemcpyHostToDevice, s);
  // (the host vector must outlive the copy)
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  const csipm::SmallOpts o{opts->tol, opts->max_iter, opts->cg_max, opts->cg_rtol, opts->cg_atol, opts->sigma,
                           opts->tau};
  if (e == hipSuccess)
    e = csipm::small_launch(n1, n2, n3, count, d_signals, d_observed, d_lambdas, lambda_frac, d_beta_out, d_info,
                            ws + csipm::small_front_bytes(n1, n2, n3), reinterpret_cast<const cx<double>*>(ws),
                            reinterpret_cast<unsigned*>(ws + ntw * sizeof(cx<double>)), o, wait, s);
  if (e != hipSuccess) {
    csipm::noctx_set_error(std::string("solve_small_batch: ") + hipGetErrorString(e));
    return CSIPM_EHIP;
  }
  return CSIPM_OK;
}
