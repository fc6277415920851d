// The operator applies of a small grid as one launch: the whole half spectrum in the
// LDS of one workgroup, through every stage of every axis in place (fft_any.h
// states the stages, fft_kernels.h the m = 0 plane and the epilogues).
//
// Grids of a few thousand points are bound by their launches: an apply_K of
// 16^3 in FP64 took five dependent passes of about 4 us each, most of it the
// way into and out of a kernel; here it is one chain of some twelve stages with
// a barrier each, bound by one compute unit's FP64 rate and LDS from 16^3 on.
// Operator applies one after the other, five passes and this, in us: K in FP64
// 8^3 21.8, 11.5; 12^3 26.2, 16.1; 16^3 22.8, 19.9; 20 x 14 x 18 36.8, 23.6;
// in FP32 at 16^3 K 22.9, 16.5, H 22.0, 14.4, A 14.7, 11.0, A^T 15.2, 10.2.
// Queued back to back on the GPU alone, K in FP64 takes 14.6, 9.8 at 8^3; 17.8,
// 17.4 at 16^3; 21.5, 21.3 at 24 x 16 x 16 (kCubeMax); 18.6, 27.3 at 32 x 16 x
// 16.  (The solves keep the five passes: they replay them from graphs.)
#include "fft_any.h"

#include <cmath>

namespace csipm {
namespace fftk {

namespace cube {

using any::div_m;
using any::slot_of;
using any::with_radix;

constexpr int kMaxThreads = 1024;

// pencils of an axis: pencil b starts at (b / d) S + b % d, elements es apart
struct Axis {
  AnyPlan pl;
  int np, d, S, es;
  unsigned npm, dm;
};
struct Plan {
  Axis ax[3];
  int n1, n2, M, MS, total;   // total = n1 n2 M; MS: row stride in LDS
  unsigned qm, mm, n2m, hm;   // ceil(2^32 / (n2 M)), / M, / n2, / (M / 2 + 1)
};
__device__ __forceinline__ int div_1(int n, int d, unsigned m) { return d == 1 ? n : div_m(n, m); }

// All stages lo .. hi - 1 of an axis (TIME: in time, from hi - 1 down).
template <typename T, int SGN, bool TIME>
__device__ __forceinline__ void stages(cx<T>* w, const Axis& ax, int lo, int hi, const cx<T>* twl) {
#pragma unroll 1
  for (int i = lo; i < hi; ++i) {
    const int s = TIME ? hi - 1 - (i - lo) : i, r = ax.pl.r[s];
    if (r == 1) continue;
    const int ms = ax.pl.ms[s], step = ax.pl.step[s], np = ax.np, es = ax.es;
    const unsigned mm = ax.pl.mm[s];
    __syncthreads();
    with_radix(r, [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      const int total = np * (ax.pl.L / R);
#pragma unroll 1
      for (int k = threadIdx.x; k < total; k += blockDim.x) {
        const int b = div_1(k, np, ax.npm), pen = k - b * np, q0 = div_1(pen, ax.d, ax.dm);
        const int blk = s == 0 ? 0 : (ms == 1 ? b : div_m(b, mm));
        const int j = b - blk * ms;
        cx<T>* const x = w + q0 * ax.S + (pen - q0 * ax.d) + (blk * ms * R + j) * es;
        cx<T> v[R];
#pragma unroll
        for (int q = 0; q < R; ++q) v[q] = x[q * ms * es];
        if (TIME && ms > 1) any::twiddle_powers<R, SGN, T>(v, twl, j * step);
        any::dft_r<R, SGN, T>(v);
        if (!TIME && ms > 1) any::twiddle_powers<R, SGN, T>(v, twl, j * step);
#pragma unroll
        for (int q = 0; q < R; ++q) x[q * ms * es] = v[q];
      }
    });
  }
}

// Real samples instead of a vector of the beta side (src, the input of A^T, and
// dst, the output of A).
struct Real {
  static constexpr int NRED = 0;
};

template <typename T, class In, class Out>
__global__ void __launch_bounds__(kMaxThreads)
k_cube(const cx<T>* src, cx<T>* dst, const uint32_t* __restrict__ mask, const cx<T>* __restrict__ tw1,
       const cx<T>* __restrict__ tw2, const cx<T>* __restrict__ twm, const cx<T>* __restrict__ tw3, T sc_c2r, T sc_dc,
       T sc_ac, In in, Out out, Plan pl) {
  constexpr bool INV = !std::is_same<In, Real>::value, FWD = !std::is_same<Out, Real>::value;
  const int n1 = pl.n1, n2 = pl.n2, M = pl.M, MS = pl.MS, NR = n1 * n2, H = M / 2 + 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* const w = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* const t1 = w + NR * MS;
  cx<T>* const t2 = t1 + n1;
  cx<T>* const t3 = t2 + n2;
  uint16_t* const nat1 = reinterpret_cast<uint16_t*>(t3 + M);   // natural index of a slot
  uint16_t* const nat2 = nat1 + n1;
  const StridedGeom<T> geo{n2 * M, 0, (long long)n2 * M, n2 * M};
  for (int i = threadIdx.x; i < n1; i += blockDim.x) {
    t1[i] = tw1[i];
    nat1[slot_of(i, pl.ax[0].pl)] = (uint16_t)i;
  }
  for (int i = threadIdx.x; i < n2; i += blockDim.x) {
    t2[i] = tw2[i];
    nat2[slot_of(i, pl.ax[1].pl)] = (uint16_t)i;
  }
  for (int i = threadIdx.x; i < M; i += blockDim.x) t3[i] = twm[i];
  // element k1 of pencil q = k2 M + m of the beta side
  auto lane = [&](int i, int& e) {
    e = div_1(i, n2 * M, pl.qm);
    const int q = i - e * (n2 * M);
    Lane12 ln;
    ln.base = q;
    ln.k2 = div_1(q, M, pl.mm);
    ln.active = true;
    ln.m0 = q == ln.k2 * M;
    ln.canon = true;
    ln.ded = false;
    return ln;
  };
  auto slot = [&](const Lane12& ln, int e) { return (e * n2 + ln.k2) * MS + ((int)ln.base - ln.k2 * M); };
  const int last = pl.ax[2].pl.nst - 1;
  if constexpr (INV) {
#pragma unroll 4
    for (int i = threadIdx.x; i < pl.total; i += blockDim.x) {
      int e;
      const Lane12 ln = lane(i, e);
      cx<T> x = read_input<T, +1>(src, e, n1, geo, ln, xlane<IO_EXT>(ln, M, n2), n2, false, T(0), in, false);
      if (ln.m0) {
        const cx<T> y = partner_value<T, +1>(src, ln.k2 ? n2 - ln.k2 : 0, e ? n1 - e : 0, geo, M, n2, in, false, T(0));
        x = plane0_mix<T, +1>(x, y, e, ln, n1, n2);
      }
      w[slot(ln, e)] = x;
    }
#pragma unroll 1
    for (int a = 0; a < 2; ++a) stages<T, +1, false>(w, pl.ax[a], 0, pl.ax[a].pl.nst, a ? t2 : t1);
    __syncthreads();
    for (int i = threadIdx.x; i < NR * H; i += blockDim.x) {
      const int row = div_1(i, H, pl.hm), e = i - row * H;
      cx<T>* const x = w + row * MS;
      if (e == 0) {
        x[0] = c2r_dc(x[0]);
      } else {
        const cx<T> a = x[e], b = cconj(x[M - e]), sm = cadd(a, b);
        const cx<T> it = cmul_i<1>(cmul(cconj(tw3[e]), csub(a, b)));
        x[e] = cadd(sm, it);
        x[M - e] = cconj(csub(sm, it));
      }
    }
    stages<T, +1, false>(w, pl.ax[2], 0, FWD ? last : last + 1, t3);
    __syncthreads();
    if constexpr (FWD) {
      // the last inverse stage, the mask and the first forward stage
      with_radix(pl.ax[2].pl.r[last], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        const int nbf = M / R;
#pragma unroll 1
        for (int i = threadIdx.x; i < NR * nbf; i += blockDim.x) {
          const int b = div_1(i, NR, pl.ax[2].npm), row = i - b * NR, s1 = div_1(row, n2, pl.n2m);
          cx<T>* const x = w + row * MS + b * R;
          cx<T> v[R];
#pragma unroll
          for (int q = 0; q < R; ++q) v[q] = x[q];
          any::dft_r<R, +1, T>(v);
          const int bit0 = (nat1[s1] * n2 + nat2[row - s1 * n2]) * (2 * M) + 2 * any::block_freq(b, pl.ax[2].pl);
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int bit = bit0 + 2 * q * nbf;
            v[q] = mask_pair(v[q], mask[bit >> 5], bit & 31);
          }
          any::dft_r<R, -1, T>(v);
#pragma unroll
          for (int q = 0; q < R; ++q) x[q] = v[q];
        }
      });
    } else {
      for (int i = threadIdx.x; i < pl.total; i += blockDim.x) {
        const int row = div_1(i, M, pl.mm), j1 = div_1(row, n2, pl.n2m);
        const int r = slot_of(j1, pl.ax[0].pl) * n2 + slot_of(row - j1 * n2, pl.ax[1].pl);
        dst[i] = cscale(w[r * MS + slot_of(i - row * M, pl.ax[2].pl)], sc_c2r);
      }
      return;
    }
  } else {
    for (int i = threadIdx.x; i < pl.total; i += blockDim.x) {
      const int row = div_1(i, M, pl.mm), j1 = div_1(row, n2, pl.n2m);
      const int r = slot_of(j1, pl.ax[0].pl) * n2 + slot_of(row - j1 * n2, pl.ax[1].pl);
      w[r * MS + slot_of(i - row * M, pl.ax[2].pl)] = src[i];
    }
  }
  if constexpr (FWD) {
    stages<T, -1, true>(w, pl.ax[2], 0, INV ? last : last + 1, t3);
    __syncthreads();
    for (int i = threadIdx.x; i < NR * H; i += blockDim.x) {
      const int row = div_1(i, H, pl.hm), e = i - row * H;
      cx<T>* const x = w + row * MS;
      if (e == 0) {
        x[0] = r2c_dc(x[0], sc_dc);
      } else {
        const cx<T> a = x[e], b = cconj(x[M - e]), sm = cadd(a, b);
        const cx<T> it = cmul_i<-1>(cmul(tw3[e], csub(a, b)));
        x[e] = cscale(cadd(sm, it), sc_ac);
        x[M - e] = cscale(cconj(csub(sm, it)), sc_ac);   // (the same value when 2 e = M)
      }
    }
#pragma unroll 1
    for (int a = 1; a >= 0; --a) stages<T, -1, true>(w, pl.ax[a], 0, pl.ax[a].pl.nst, a ? t2 : t1);
    __syncthreads();
    constexpr int NQ = Out::NRED > 0 ? Out::NRED : 1;
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    const T rs2 = T(0.70710678118654752440);
#pragma unroll 2
    for (int i = threadIdx.x; i < pl.total; i += blockDim.x) {
      int e;
      const Lane12 ln = lane(i, e);
      cx<T> h = w[slot(ln, e)];
      if (ln.m0) {   // the unmixed pair (k1, k2), (-k1, -k2)
        const cx<T> y = w[((e ? n1 - e : 0) * n2 + (ln.k2 ? n2 - ln.k2 : 0)) * MS];
        const int c = cls2(e, ln.k2, n1, n2);
        h = c == 0 ? h : (c == 1 ? cscale(cadd(h, y), rs2) : cscale(cmul_i<1>(csub(h, y)), rs2));
      }
      write_output<T, 1, -1>(dst, e, h, n1, geo, ln, xlane<IO_EXT>(ln, M, n2), n2, out, acc);
    }
    if constexpr (Out::NRED > 0)
      any::block_sums_rt<Out::NRED, Out::NMAX>(acc, out.partial, out.pstride, reinterpret_cast<double*>(smem_raw));
  }
}

unsigned magic(int d) { return d > 1 ? (unsigned)((0x100000000ull + d - 1) / d) : 0u; }

bool plan(int n1, int n2, int M, int w, Plan& pl) {
  const int n[3] = {n1, n2, M};
  for (int a = 0; a < 3; ++a)
    if (!any_plan(n[a], w, pl.ax[a].pl)) return false;
  pl.n1 = n1;
  pl.n2 = n2;
  pl.M = M;
  pl.MS = M | 1;
  pl.total = n1 * n2 * M;
  pl.qm = magic(n2 * M);
  pl.mm = magic(M);
  pl.n2m = magic(n2);
  pl.hm = magic(M / 2 + 1);
  auto set = [&](int a, int np, int d, int S, int es) {
    pl.ax[a].np = np;
    pl.ax[a].d = d;
    pl.ax[a].S = S;
    pl.ax[a].es = es;
    pl.ax[a].npm = magic(np);
    pl.ax[a].dm = magic(d);
  };
  set(0, n2 * M, M, pl.MS, n2 * pl.MS);
  set(1, n1 * M, M, n2 * pl.MS, pl.MS);
  set(2, n1 * n2, 1, pl.MS, 1);
  return true;
}
size_t lds_bytes(const Plan& pl, int w) {
  return (size_t)(pl.n1 * pl.n2 * pl.MS + pl.n1 + pl.n2 + pl.M) * w + 2 * (size_t)(pl.n1 + pl.n2);
}

template <typename T, class In, class Out>
void launch(const Grid& g, const T* src, T* dst, const uint32_t* mask, const Twiddles<T>& tw, T sc_c2r, T sc_dc,
            T sc_ac, In in, Out out, hipStream_t s) {
  Plan pl;
  if (!plan(g.n1, g.n2, g.m, (int)sizeof(cx<T>), pl)) return;   // (cube_pass has checked)
  const size_t shm = std::max(lds_bytes(pl, (int)sizeof(cx<T>)), (size_t)(2 * kMaxThreads / 64) * sizeof(double));
  auto kern = k_cube<T, In, Out>;
  if (shm > 65536)
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  // (few values: fewer waves at the barriers; apply_K of 8^3 9.8 us with 512 threads, 10.6 with 1024)
  hipLaunchKernelGGL(kern, dim3(1), dim3(pl.total <= 512 ? kMaxThreads / 2 : kMaxThreads), shm, s, reinterpret_cast<const cx<T>*>(src),
                     reinterpret_cast<cx<T>*>(dst), mask, tw.t1, tw.t2, tw.tm, tw.t3, sc_c2r, sc_dc, sc_ac, in, out,
                     pl);
}

}  // namespace cube
}  // namespace fftk

bool cube_pass(const Grid& g) {
  if (g.odd3() || g.n > kCubeMax) return false;
  fftk::cube::Plan pl;
  return fftk::cube::plan(g.n1, g.n2, g.m, 16, pl) && fftk::cube::lds_bytes(pl, 16) <= 163840;
}

template <typename T>
void launch_cube(const Grid& g, CubeOp op, const T* in, T* out, const uint32_t* mask, const Twiddles<T>& tw,
                 const EpiArgs<T>* ea, hipStream_t s) {
  using namespace fftk;
  using cube::Real;
  // (the scales of launch_axis3)
  const double rn = 1.0 / std::sqrt((double)g.n), r2 = std::sqrt(2.0);
  const T c2r = (T)(rn / r2), dc = (T)(op == CUBE_AT ? rn : rn * rn / r2),
          ac = (T)(op == CUBE_AT ? rn / r2 : rn * rn / 2.0);
  auto run = [&](auto i, auto o) { cube::launch<T>(g, in, out, mask, tw, c2r, dc, ac, i, o, s); };
  const EpiIn<T, IO_EXT> xin{in, nullptr, nullptr, nullptr};
  const EpiOut<T, IO_EXT> xout{out, -1};
  if (op == CUBE_A) run(xin, Real{});
  else if (op == CUBE_AT) run(Real{}, xout);
  else if (op == CUBE_H) run(xin, xout);
  else run(xin, EpiKX<T, IO_EXT>{ea->k, ea->partial, ea->pstride, -1});
}
template void launch_cube<float>(const Grid&, CubeOp, const float*, float*, const uint32_t*, const Twiddles<float>&,
                                 const EpiArgs<float>*, hipStream_t);
template void launch_cube<double>(const Grid&, CubeOp, const double*, double*, const uint32_t*,
                                  const Twiddles<double>&, const EpiArgs<double>*, hipStream_t);

}  // namespace csipm
