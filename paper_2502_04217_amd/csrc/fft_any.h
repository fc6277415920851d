// Pencil passes at the grid extents 2^a 3^b 5^c 7^d up to 1024 that have no
// instantiated kernels (fft.hip and fft_mixed_f64/f32.hip instantiate the
// powers of two, the paper's non-power-of-two sizes and a few small ones).
// They compute what k_axis12 and k_axis3 compute — the m = 0 plane mixing,
// the fused direction update, the K and refinement epilogues, the axis-3
// c2r / mask / r2c — through the same helpers, with a radix plan computed at
// launch, so that one kernel serves every length.  fft_any_f64.hip and
// fft_any_f32.hip instantiate them.
//
// A workgroup holds TM pencils with NT threads each; the pencils sit in LDS
// between the stages, element e of pencil p at e ES + p (pencils in
// consecutive lanes: free of bank conflicts).  The transform runs in place.
// With radices R_0 .. R_{S-1} and B_s = L / (R_0 .. R_{s-1}):
//   decimation in frequency: stage s takes, in each block of B_s values, the
//     elements j + q B_s/R_s (j < B_s/R_s), writes their DFT times w^(jp) back
//     to j + p B_s/R_s; natural order in, and the value of frequency
//     k = p_0 + R_0 (p_1 + R_1 (p_2 + ..)) ends in slot ((p_0 R_1 + p_1) R_2 +
//     p_2) ..;
//   decimation in time: the same stages from the last to the first with the
//     twiddles on the inputs; that slot order in, natural order out.
// So no stage reads what another butterfly of the stage writes (one barrier
// between stages, one butterfly in registers at a time), the strided passes
// go from global memory into the first stage and from the last stage, which
// knows each output's frequency, to global memory, and an axis-3 pass ends
// its inverse transform with the butterflies its forward transform starts
// with: the mask is applied between the two in registers.
//
// These passes are bound by memory and the latency of its pipeline: the
// transform costs two or three LDS round trips per element (five or six in
// an axis-3 pass), and a run of TM pencils is one 128-byte line (less over few
// pencils, any_few), so that no two workgroups share the lines of an aligned row
// (xcd_tile: nor two XCDs those of any other).  Against passes that kept
// the pencil in LDS through Stockham stages of radix 8, 4, 2, 3, 5, 7 (two
// barriers per stage, 64-byte runs at these lengths), a K-apply takes, in us:
//   300 x 400 x 400 FP32  1224 -> 705 (2.9 GB: 4.1 TB/s)
//   500 x 300 x 200 FP64  1535 -> 768
//   240^3 FP32 305 -> 221, FP64 550 -> 369; 100^3 FP32 60 -> 54
#pragma once

#include "fft_kernels.h"

#include <algorithm>

namespace csipm {
namespace fftk {

namespace any {

constexpr int kMaxThreads = 512;

// n / d for n < 65536, 2 <= d <= 1024, from m = ceil(2^32 / d)
__device__ __forceinline__ int div_m(int n, unsigned m) { return (int)__umulhi((unsigned)n, m); }

// cos and sin of 2 pi m / 9
__device__ constexpr double cos9(int m) {
  const int k = m % 9, a = 2 * k <= 9 ? k : 9 - k;
  return a == 0 ? 1.0
                : (a == 1 ? 0.76604444311897803520
                          : (a == 2 ? 0.17364817766693034885 : (a == 3 ? -0.5 : -0.93969262078590838405)));
}
__device__ constexpr double sin9(int m) {
  const int k = m % 9;
  const bool neg = 2 * k > 9;
  const int a = neg ? 9 - k : k;
  const double v = a == 0 ? 0.0
                          : (a == 1 ? 0.64278760968653932632
                                    : (a == 2 ? 0.98480775301220805937
                                              : (a == 3 ? 0.86602540378443864676 : 0.34202014332566873304)));
  return neg ? -v : v;
}

template <int R, int DIR, typename T>
__device__ __forceinline__ void dft_r(cx<T>* v);

// In-register DFT of size A B with coprime A, B in natural order by the
// prime-factor map: input n = B i + A j, output k with k = i' mod A, j' mod B
// (both mod A B), no twiddles between the two.
template <int A, int B, int DIR, typename T>
__device__ __forceinline__ void dft_pfa(cx<T>* v) {
  constexpr int R = A * B;
  cx<T> u[R];
#pragma unroll
  for (int j = 0; j < B; ++j) {
    cx<T> x[A];
#pragma unroll
    for (int i = 0; i < A; ++i) x[i] = v[(B * i + A * j) % R];
    dft_r<A, DIR, T>(x);
#pragma unroll
    for (int i = 0; i < A; ++i) u[i * B + j] = x[i];
  }
#pragma unroll
  for (int i = 0; i < A; ++i) {
    dft_r<B, DIR, T>(&u[i * B]);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      int k = 0;
      for (int c = 0; c < R; ++c)
        if (c % A == i && c % B == j) k = c;
      v[k] = u[i * B + j];
    }
  }
}

// In-register DFT of size 9 as 3 x 3 with twiddles exp(DIR 2 pi i m / 9).
template <int DIR, typename T>
__device__ __forceinline__ void dft9(cx<T>* v) {
  cx<T> u[9];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    cx<T> x[3] = {v[j], v[j + 3], v[j + 6]};
    dft_odd<3, DIR, T>(x);
    u[j] = x[0];
#pragma unroll
    for (int p = 1; p < 3; ++p)
      u[3 * p + j] = j == 0 ? x[p] : cmul(x[p], cx<T>{T(cos9(j * p)), T(DIR * sin9(j * p))});
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    dft_odd<3, DIR, T>(&u[3 * p]);
#pragma unroll
    for (int k = 0; k < 3; ++k) v[p + 3 * k] = u[3 * p + k];
  }
}

template <int R, int DIR, typename T>
__device__ __forceinline__ void dft_r(cx<T>* v) {
  if constexpr (R == 1) return;
  else if constexpr ((R & (R - 1)) == 0) dft_reg<R, DIR, T>(v);
  else if constexpr (R == 6) dft_pfa<2, 3, DIR, T>(v);
  else if constexpr (R == 9) dft9<DIR, T>(v);
  else if constexpr (R == 10) dft_pfa<2, 5, DIR, T>(v);
  else dft_odd<R, DIR, T>(v);
}

// v[q] *= exp(SGN 2 pi i q at / L), q = 1 .. R-1, from the length-L table in
// LDS (q at < L).  One read per power: the lanes of a wave share 4 (FP32) or 8
// (FP64) addresses, so the reads cost 1 % of a K-apply over products of the
// first power, whose roundings would make the FP32 passes 7 % less exact.
template <int R, int SGN, typename T>
__device__ __forceinline__ void twiddle_powers(cx<T>* v, const cx<T>* twl, int at) {
#pragma unroll
  for (int q = 1; q < R; ++q) v[q] = cmul(v[q], twiddle<T>(twl, q * at, SGN));
}

// Calls f(std::integral_constant<int, R>) for the runtime radix r.  10 is the
// largest: with 12, 15 and 16 the FP32 kernels take 82-103 registers instead
// of 54-73 (4-5 instead of 6-8 waves per SIMD), and the FP32 K-apply at
// 300 x 400 x 400, which needs none of them, takes 769 instead of 702 us (at
// 240^3 = (16 15)^3, with one LDS round trip less, 219 and 221).
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
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    default: f(std::integral_constant<int, 10>{}); break;
  }
}

// frequency of the first slot of block b of the last stage (b < L / R_{S-1})
__device__ __forceinline__ int block_freq(int b, const AnyPlan& pl) {
  int f = 0;
  for (int s = pl.nst - 2; s >= 1; --s) {
    const int q = div_m(b, pl.rm[s]);
    f = (b - q * pl.r[s]) + pl.r[s] * f;
    b = q;
  }
  return pl.nst >= 2 ? b + pl.r[0] * f : 0;
}
// slot of natural index n
__device__ __forceinline__ int slot_of(int n, const AnyPlan& pl) {
  int o = 0;
  for (int s = 0; s + 1 < pl.nst; ++s) {
    const int q = pl.r[s] == 1 ? n : div_m(n, pl.rm[s]);
    o = o * pl.r[s] + (n - q * pl.r[s]);
    n = q;
  }
  return o * pl.r[pl.nst - 1] + n;
}

// Stages lo .. hi - 1 of the in-place transform of the pencil at a (element e
// at a[e es]), decimation in frequency (SGN: sign of the exponent) or in time
// (TIME: from stage hi - 1 down to lo); a barrier before each.
template <typename T, int SGN, bool TIME>
__device__ __forceinline__ void stages(cx<T>* a, int es, const AnyPlan& pl, int lo, int hi, int t,
                                       const cx<T>* twl) {
  for (int i = lo; i < hi; ++i) {
    const int s = TIME ? hi - 1 - (i - lo) : i;
    __syncthreads();
    const int ms = pl.ms[s];          // B_s / R_s
    const unsigned mm = pl.mm[s];
    const int step = pl.step[s];      // L / B_s
    with_radix(pl.r[s], [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      const int nbf = pl.L / R;
      for (int b = t; b < nbf; b += pl.nt) {
        const int blk = s == 0 ? 0 : (ms == 1 ? b : div_m(b, mm));
        const int j = b - blk * ms;
        cx<T>* const x = a + (blk * ms * R + j) * es;
        cx<T> v[R];
#pragma unroll
        for (int q = 0; q < R; ++q) v[q] = x[q * ms * es];
        if constexpr (TIME) twiddle_powers<R, SGN, T>(v, twl, j * step);
        dft_r<R, SGN, T>(v);
        if constexpr (!TIME) twiddle_powers<R, SGN, T>(v, twl, j * step);
#pragma unroll
        for (int q = 0; q < R; ++q) x[q * ms * es] = v[q];
      }
    });
  }
}

// block_sums_store for a workgroup of runtime size
template <int NQ, int NMAX>
__device__ __forceinline__ void block_sums_rt(const double* v, double* out, int stride, double* red) {
  const int nw = blockDim.x >> 6, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double w[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) w[q] = q >= NQ - NMAX ? wave_max(v[q]) : wave_sum(v[q]);
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < NQ; ++q) red[q * nw + wv] = w[q];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      double a = 0.0;
      for (int i = 0; i < nw; ++i) a = q >= NQ - NMAX ? fmax(a, red[q * nw + i]) : a + red[q * nw + i];
      out[q * stride + blockIdx.x] = a;
    }
}

// Strided pass (axis 1 or 2) of k_axis12.  The partner rows of the m = 0
// lanes (one lane in M) are read where they are mixed: the loads go out with
// the lane's own.
template <typename T, int AX, int DIR, class Epi>
__global__ void __launch_bounds__(kMaxThreads)
k_axis12_any(const cx<T>* src, cx<T>* dst, StridedGeom<T> geo, const cx<T>* __restrict__ tw, int m, Plane0 pl0,
             Epi epi, const int* skip, AnyPlan pl) {
  if (skip && *skip) return;
  constexpr bool MIX = AX == 1 && Epi::IO != IO_ODD;
  const int L = pl.L, TM = 1 << pl.tmlog;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* const tile = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* const twl = tile + (size_t)L * TM;
  const int p = threadIdx.x & (TM - 1), t = threadIdx.x >> pl.tmlog;
  const Lane12 ln = lane12<AX, DIR, Epi::IO>(p, TM, geo, m, pl0);
  XLane xl{};
  if constexpr (Epi::IO != IO_INT) xl = xlane<Epi::IO>(ln, m, pl0.n2);
  cx<T>* const a = tile + p;
  for (int i = threadIdx.x; i < L; i += blockDim.x) twl[i] = tw[i];
  bool upd = false;
  T be = T(0);
  if constexpr (Epi::PRO) {
    upd = epi.z != nullptr;
    if (upd) be = (T)*epi.beta;
  }
  __syncthreads();
  // first stage: global memory to LDS (element j + q L/R)
  with_radix(pl.r[0], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int nbf = L / R;
    for (int j = t; j < nbf; j += pl.nt) {
      cx<T> v[R];
#pragma unroll
      for (int q = 0; q < R; ++q)
        v[q] = read_input<T, DIR>(src, j + q * nbf, L, geo, ln, xl, pl0.n2, upd, be, epi, AX == 1 && ln.m0);
      if constexpr (MIX) {
        if (ln.m0 && ln.active) {
          const int prow = ln.k2 ? pl0.n2 - ln.k2 : 0;
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int e = j + q * nbf;
            const cx<T> y = partner_value<T, DIR>(src, prow, e ? L - e : 0, geo, m, pl0.n2, epi, upd, be);
            v[q] = plane0_mix<T, DIR>(v[q], y, e, ln, L, pl0.n2);
          }
        }
      }
      dft_r<R, DIR, T>(v);
      twiddle_powers<R, DIR, T>(v, twl, j);
#pragma unroll
      for (int q = 0; q < R; ++q) a[(j + q * nbf) * TM] = v[q];
    }
  });
  stages<T, DIR, false>(a, TM, pl, 1, pl.nst - 1, t, twl);
  __syncthreads();
  constexpr int NQ = Epi::NRED > 0 ? Epi::NRED : 1;
  double acc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
  // last stage: LDS to global memory or the epilogue (frequency f + q L/R)
  with_radix(pl.r[pl.nst - 1], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int nbf = L / R;
    if (!ln.active) return;
    for (int b = t; b < nbf; b += pl.nt) {
      cx<T> v[R];
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = a[(b * R + q) * TM];
      dft_r<R, DIR, T>(v);
      const int f = block_freq(b, pl);
#pragma unroll
      for (int q = 0; q < R; ++q)
        write_output<T, AX, DIR>(dst, f + q * nbf, v[q], L, geo, ln, xl, pl0.n2, epi, acc);
    }
  });
  extra_output<T, DIR>(epi, acc);
  if constexpr (Epi::NRED > 0)
    block_sums_rt<Epi::NRED, Epi::NMAX>(acc, epi.partial, epi.pstride, reinterpret_cast<double*>(smem_raw));
}

// Axis-3 pass of k_axis3 (half length L = N3/2): the workgroup's TM pencils
// are one contiguous run of memory.  The c2r packing and the r2c unpacking
// take X_e and X_{L-e} together, on the way from and to global memory.
template <typename T, int MODE>
__global__ void __launch_bounds__(kMaxThreads)
k_axis3_any(const cx<T>* src, cx<T>* dst, const uint32_t* __restrict__ mask, const cx<T>* __restrict__ twm,
            const cx<T>* __restrict__ tw3, int npencils, T sc_c2r, T sc_r2c_dc, T sc_r2c, const int* skip,
            AnyPlan pl) {
  if (skip && *skip) return;
  const int L = pl.L, TM = 1 << pl.tmlog, ES = TM + 1, H = L / 2 + 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* const tile = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* const twl = tile + (size_t)L * ES;
  uint32_t* const mw = reinterpret_cast<uint32_t*>(twl + L);
  const int p = threadIdx.x & (TM - 1), t = threadIdx.x >> pl.tmlog;
  cx<T>* const a = tile + p;
  for (int i = threadIdx.x; i < L; i += blockDim.x) twl[i] = twm[i];
  const int tl = xcd_tile(blockIdx.x, gridDim.x);
  const long long run = (long long)tl * TM * L;
  const int np = min(TM, npencils - tl * TM);   // pencils of this workgroup
  const long long bit0 = 2 * run, word0 = bit0 >> 5;
  if constexpr (MODE == A3_FULL) {
    // the mask words of the run (bits bit0 .. bit0 + 2 np L)
    const int nw = (int)(((bit0 + 2 * (long long)np * L - 1) >> 5) - word0) + 1;
    for (int i = threadIdx.x; i < nw; i += blockDim.x) mw[i] = mask[word0 + i];
  }
  if constexpr ((MODE & A3_C2R) != 0) {
    // Z_e and Z_{L-e} from X_e and X_{L-e} (w_{L-e} = -conj w_e)
    for (int i = threadIdx.x; i < TM * H; i += blockDim.x) {
      const int pp = H == 1 ? i : div_m(i, pl.hm), e = i - pp * H;
      cx<T> x{T(0), T(0)}, y{T(0), T(0)};
      if (pp < np) {
        x = src[run + pp * L + e];
        if (e > 0) y = src[run + pp * L + (L - e)];
      }
      if (e == 0) {
        tile[pp] = c2r_dc(x);
      } else {
        const cx<T> b = cconj(y), sm = cadd(x, b), d = csub(x, b);
        const cx<T> it = cmul_i<1>(cmul(cconj(tw3[e]), d));
        tile[e * ES + pp] = cadd(sm, it);
        tile[(L - e) * ES + pp] = cconj(csub(sm, it));
      }
    }
    stages<T, +1, false>(a, ES, pl, 0, pl.nst - 1, t, twl);
    __syncthreads();
    // the last inverse stage and, in a full pass, the mask and the first
    // forward stage on the same values
    with_radix(pl.r[pl.nst - 1], [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      const int nbf = L / R;
      for (int b = t; b < nbf; b += pl.nt) {
        cx<T>* const x = a + b * R * ES;
        cx<T> v[R];
#pragma unroll
        for (int q = 0; q < R; ++q) v[q] = x[q * ES];
        dft_r<R, +1, T>(v);
        if constexpr (MODE == A3_FULL) {
          const int off = (int)(bit0 & 31) + 2 * (p * L + block_freq(b, pl));
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int bit = off + 2 * q * nbf;
            v[q] = mask_pair(v[q], p < np ? mw[bit >> 5] : 0u, bit & 31);
          }
          dft_r<R, -1, T>(v);
        }
#pragma unroll
        for (int q = 0; q < R; ++q) x[q * ES] = v[q];
      }
    });
    if constexpr (MODE == A3_C2R) {
      __syncthreads();
      for (int i = threadIdx.x; i < np * L; i += blockDim.x) {
        const int pp = L == 1 ? i : div_m(i, pl.lm), e = i - pp * L;
        dst[run + i] = cscale(tile[slot_of(e, pl) * ES + pp], sc_c2r);
      }
      return;
    }
    stages<T, -1, true>(a, ES, pl, 0, pl.nst - 1, t, twl);
  } else {
    for (int i = threadIdx.x; i < TM * L; i += blockDim.x) {
      const int pp = L == 1 ? i : div_m(i, pl.lm), e = i - pp * L;
      tile[slot_of(e, pl) * ES + pp] = pp < np ? src[run + i] : cx<T>{T(0), T(0)};
    }
    stages<T, -1, true>(a, ES, pl, 0, pl.nst, t, twl);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < np * H; i += blockDim.x) {
    const int pp = H == 1 ? i : div_m(i, pl.hm), e = i - pp * H;
    const cx<T> x = tile[e * ES + pp];
    if (e == 0) {
      dst[run + pp * L] = r2c_dc(x, sc_r2c_dc);
    } else {
      const cx<T> b = cconj(tile[(L - e) * ES + pp]), sm = cadd(x, b);
      const cx<T> it = cmul_i<-1>(cmul(tw3[e], csub(x, b)));
      dst[run + pp * L + e] = cscale(cadd(sm, it), sc_r2c);
      if (2 * e != L) dst[run + pp * L + (L - e)] = cscale(cconj(csub(sm, it)), sc_r2c);
    }
  }
}

// Axis-3 pass of an odd N3 = L: two real rows a and b share one complex
// transform of length L, z = a + i b.  Its inverse starts from Z_e = A_e + i B_e
// and Z_{L-e} = conj(A_e) + i conj(B_e) (e < M = (L + 1) / 2; the half spectra
// carry the sqrt2 of the real parametrisation, the value of e = 0 does not
// and is real), the mask acts on a and b, and the forward transform Y splits
// into A_e = (Y_e + conj(Y_{L-e})) / 2 and B_e = (Y_e - conj(Y_{L-e})) / 2i.
// A workgroup holds TM pairs: 2 TM rows, one run of memory on either side.
// (Complex transforms of the whole Hermitian spectrum along all three axes,
// with passes of their own for the map, the mask and the parametrisation,
// moved twice the bytes: apply_At at 105 x 135 x 75 in FP64 69 us, now 33.)
// Factors are left to the launch's scales as in k_axis3.
template <typename T, int MODE>
__global__ void __launch_bounds__(kMaxThreads)
k_axis3_odd(const T* src_, T* dst_, const uint32_t* __restrict__ mask, const cx<T>* __restrict__ tw, int npencils,
            T sc_c2r, T sc_dc, T sc_ac, const int* skip, AnyPlan pl) {
  if (skip && *skip) return;
  const int L = pl.L, TM = 1 << pl.tmlog, ES = TM + 1, M = (L + 1) / 2;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* const tile = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* const twl = tile + (size_t)L * ES;
  uint32_t* const mw = reinterpret_cast<uint32_t*>(twl + L);
  const int p = threadIdx.x & (TM - 1), t = threadIdx.x >> pl.tmlog;
  cx<T>* const a = tile + p;
  for (int i = threadIdx.x; i < L; i += blockDim.x) twl[i] = tw[i];
  const long long row0 = 2ll * xcd_tile(blockIdx.x, gridDim.x) * TM;
  const int nrow = (int)min((long long)2 * TM, npencils - row0);   // rows of this workgroup
  const long long bit0 = row0 * L, word0 = bit0 >> 5;
  if constexpr (MODE == A3_FULL) {
    const int nw = (int)(((bit0 + (long long)nrow * L - 1) >> 5) - word0) + 1;
    for (int i = threadIdx.x; i < nw; i += blockDim.x) mw[i] = mask[word0 + i];
  }
  if constexpr ((MODE & A3_C2R) != 0) {
    const cx<T>* const src = reinterpret_cast<const cx<T>*>(src_) + row0 * M;
    for (int i = threadIdx.x; i < TM * M; i += blockDim.x) {
      const int pp = div_m(i, pl.hm), e = i - pp * M;
      cx<T> x{T(0), T(0)}, y{T(0), T(0)};
      if (2 * pp < nrow) x = src[2 * pp * M + e];
      if (2 * pp + 1 < nrow) y = src[(2 * pp + 1) * M + e];
      if (e == 0) {
        const T s2 = T(1.41421356237309504880);
        tile[pp] = {s2 * x.re, s2 * y.re};
      } else {
        tile[e * ES + pp] = {x.re - y.im, x.im + y.re};
        tile[(L - e) * ES + pp] = {x.re + y.im, y.re - x.im};
      }
    }
    stages<T, +1, false>(a, ES, pl, 0, pl.nst - 1, t, twl);
    __syncthreads();
    with_radix(pl.r[pl.nst - 1], [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      const int nbf = L / R;
      for (int b = t; b < nbf; b += pl.nt) {
        cx<T>* const x = a + b * R * ES;
        cx<T> v[R];
#pragma unroll
        for (int q = 0; q < R; ++q) v[q] = x[q * ES];
        dft_r<R, +1, T>(v);
        if constexpr (MODE == A3_FULL) {
          const int off = (int)(bit0 & 31) + 2 * p * L + block_freq(b, pl);
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const int ba = off + q * nbf, bb = ba + L;
            if (!(2 * p < nrow && ((mw[ba >> 5] >> (ba & 31)) & 1u))) v[q].re = T(0);
            if (!(2 * p + 1 < nrow && ((mw[bb >> 5] >> (bb & 31)) & 1u))) v[q].im = T(0);
          }
          dft_r<R, -1, T>(v);
        }
#pragma unroll
        for (int q = 0; q < R; ++q) x[q * ES] = v[q];
      }
    });
    if constexpr (MODE == A3_C2R) {
      __syncthreads();
      for (int i = threadIdx.x; i < nrow * L; i += blockDim.x) {
        const int r = div_m(i, pl.lm), e = i - r * L;
        const cx<T> z = tile[slot_of(e, pl) * ES + (r >> 1)];
        dst_[row0 * L + i] = ((r & 1) ? z.im : z.re) * sc_c2r;
      }
      return;
    }
    stages<T, -1, true>(a, ES, pl, 0, pl.nst - 1, t, twl);
  } else {
    const T* const src = src_ + row0 * L;
    for (int i = threadIdx.x; i < TM * L; i += blockDim.x) {
      const int pp = div_m(i, pl.lm), e = i - pp * L;
      tile[slot_of(e, pl) * ES + pp] = {2 * pp < nrow ? src[2 * pp * L + e] : T(0),
                                        2 * pp + 1 < nrow ? src[(2 * pp + 1) * L + e] : T(0)};
    }
    stages<T, -1, true>(a, ES, pl, 0, pl.nst, t, twl);
  }
  __syncthreads();
  cx<T>* const dst = reinterpret_cast<cx<T>*>(dst_) + row0 * M;
  for (int i = threadIdx.x; i < TM * M; i += blockDim.x) {
    const int pp = div_m(i, pl.hm), e = i - pp * M;
    if (2 * pp >= nrow) continue;
    const cx<T> y = tile[e * ES + pp];
    cx<T> x0, x1;
    if (e == 0) {
      x0 = {y.re * sc_dc, T(0)};
      x1 = {y.im * sc_dc, T(0)};
    } else {
      const cx<T> z = tile[(L - e) * ES + pp];
      x0 = cscale(cx<T>{y.re + z.re, y.im - z.im}, sc_ac);
      x1 = cscale(cx<T>{y.im + z.im, z.re - y.re}, sc_ac);
    }
    dst[2 * pp * M + e] = x0;
    if (2 * pp + 1 < nrow) dst[(2 * pp + 1) * M + e] = x1;
  }
}

}  // namespace any

template <typename T, int AX, int DIR, class Epi>
bool launch_axis12_any(int L, dim3 grid, const cx<T>* src, cx<T>* dst, StridedGeom<T> geo, const cx<T>* tw, int m,
                       int n2, Epi epi, const int* skip, hipStream_t s) {
  AnyPlan plan;
  if (!any_plan(L, (int)sizeof(cx<T>), plan)) return false;
  any_few(plan, geo.batch, kStridedLowest);
  const int tm = 1 << plan.tmlog;
  const Plane0 pl{n2, AX == 1 && Epi::IO != IO_ODD ? plane0_groups(DIR) : 0};
  const size_t shm = (size_t)(tm + 1) * L * sizeof(cx<T>);   // (the tile and the twiddles)
  auto kern = any::k_axis12_any<T, AX, DIR, Epi>;
  if (shm > 65536)
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  hipLaunchKernelGGL(kern, dim3(grid.x + pl.ndedicated), dim3(tm * plan.nt), shm, s, src, dst, geo, tw, m, pl, epi,
                     skip, plan);
  return true;
}

template <typename T>
bool launch_axis3_any(int L, int mode, int np, const cx<T>* cs, cx<T>* cd, const uint32_t* maskbits,
                      const cx<T>* twm, const cx<T>* tw3, T sc_c2r, T sc_dc, T sc_ac, const int* skip,
                      hipStream_t s) {
  AnyPlan plan;
  if (!any_plan(L, (int)sizeof(cx<T>), plan)) return false;
  const int tm = 1 << plan.tmlog;
  // the tile (rows of tm + 1), the twiddles and the mask words of the run
  const size_t shm = (size_t)L * (tm + 2) * sizeof(cx<T>) + 4 * ((size_t)(2 * tm * L) / 32 + 2);
  const dim3 grid((np + tm - 1) / tm), block(tm * plan.nt);
  auto go = [&](auto kern) {
    if (shm > 65536)
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    hipLaunchKernelGGL(kern, grid, block, shm, s, cs, cd, maskbits, twm, tw3, np, sc_c2r, sc_dc, sc_ac, skip, plan);
  };
  if (mode == A3_FULL) go(any::k_axis3_any<T, A3_FULL>);
  else if (mode == A3_C2R) go(any::k_axis3_any<T, A3_C2R>);
  else go(any::k_axis3_any<T, A3_R2C>);
  return true;
}

template <typename T>
bool launch_axis3_odd(int L, int mode, int np, const T* src, T* dst, const uint32_t* maskbits, const cx<T>* tw3,
                      T sc_c2r, T sc_dc, T sc_ac, const int* skip, hipStream_t s) {
  AnyPlan plan;
  if (L % 2 == 0 || L < 3 || !any_plan(L, (int)sizeof(cx<T>), plan)) return false;
  any_few(plan, (np + 1) / 2, 0);
  const int tm = 1 << plan.tmlog;
  const size_t shm = (size_t)L * (tm + 2) * sizeof(cx<T>) + 4 * ((size_t)(2 * tm * L) / 32 + 2);
  const dim3 grid((np + 2 * tm - 1) / (2 * tm)), block(tm * plan.nt);
  auto go = [&](auto kern) {
    if (shm > 65536)
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    hipLaunchKernelGGL(kern, grid, block, shm, s, src, dst, maskbits, tw3, np, sc_c2r, sc_dc, sc_ac, skip, plan);
  };
  if (mode == A3_FULL) go(any::k_axis3_odd<T, A3_FULL>);
  else if (mode == A3_C2R) go(any::k_axis3_odd<T, A3_C2R>);
  else go(any::k_axis3_odd<T, A3_R2C>);
  return true;
}

#define CSIPM_ANY12(T, AX, DIR, EPI)                                                                       \
  template bool launch_axis12_any<T, AX, DIR, EPI>(int, dim3, const cx<T>*, cx<T>*, StridedGeom<T>,        \
                                                   const cx<T>*, int, int, EPI, const int*, hipStream_t);
#define CSIPM_ANY(T)                                                                                        \
  CSIPM_ANY12(T, 1, +1, EpiP<T>)                                                                            \
  CSIPM_ANY12(T, 1, -1, EpiNone)                                                                            \
  CSIPM_ANY12(T, 1, -1, EpiK<T>)                                                                            \
  CSIPM_ANY12(T, 1, +1, CSIPM_IO(EpiIn, T, IO_EXT))                                                         \
  CSIPM_ANY12(T, 1, -1, CSIPM_IO(EpiOut, T, IO_EXT))                                                        \
  CSIPM_ANY12(T, 1, -1, CSIPM_IO(EpiKX, T, IO_EXT))                                                         \
  CSIPM_ANY12(T, 1, +1, CSIPM_IO(EpiIn, T, IO_ODD))                                                         \
  CSIPM_ANY12(T, 1, -1, CSIPM_IO(EpiOut, T, IO_ODD))                                                        \
  CSIPM_ANY12(T, 1, -1, CSIPM_IO(EpiKX, T, IO_ODD))                                                         \
  CSIPM_ANY12(T, 2, +1, EpiNone)                                                                            \
  CSIPM_ANY12(T, 2, -1, EpiNone)                                                                            \
  template bool launch_axis3_any<T>(int, int, int, const cx<T>*, cx<T>*, const uint32_t*, const cx<T>*,     \
                                    const cx<T>*, T, T, T, const int*, hipStream_t);                       \
  template bool launch_axis3_odd<T>(int, int, int, const T*, T*, const uint32_t*, const cx<T>*, T, T, T,   \
                                    const int*, hipStream_t);

}  // namespace fftk
}  // namespace csipm
