// Hartree potential on the periodic grid, V = FFT^-1[ v(G) FFT[rho] ],
// v(G) = scale * 4 pi / |G|^2, v(0) = 0 (the integral kernel of Eq. 3, read
// as the periodic Coulomb kernel of a cubic cell).
//
// Two real fields are packed into one complex field (exact because v(G) is
// real and even, so each real field maps to a real potential).  Grids whose
// edges are among the line lengths of fft_plane.hip, and whose yz planes fit in
// a CU's LDS, take its three in-place passes.  The rest are here: three passes
// with a plane and its ping-pong copy in LDS (edges of 162, 192, 216, 243 or
// 256 points beside short ones),
//   yz forward (+ pack, + sum of GEMM partials) ->
//   x forward, multiply by v(G)/N, x inverse -> yz inverse (+ unpack),
// with the spectrum in between stored y-major (X[ky][x][kz]) so that the x
// pass reads and writes contiguous (x, kz) slabs;
// otherwise (planes too large for either) five passes of batched 1-D transforms:
//   z forward (+ pack) -> y forward -> x (as above) -> y inverse -> z inverse.
// The 1-D transforms are mixed-radix (2, 3, 4, 8) Stockham autosort passes
// with ping-pong LDS buffers (Govindaraju et al., SC'08 formulation); the
// inverse uses conj(FFT(conj(x))).
#include "common.h"
#include "kernels.h"

namespace gwl {

namespace {

template <typename T>
__device__ inline cplx<T> cmul(cplx<T> a, cplx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ inline cplx<T> cadd(cplx<T> a, cplx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ inline cplx<T> csub(cplx<T> a, cplx<T> b) { return {a.x - b.x, a.y - b.y}; }
// -i * a
template <typename T>
__device__ inline cplx<T> mul_mi(cplx<T> a) { return {a.y, -a.x}; }

template <typename T>
__device__ inline void dft2(cplx<T>* v) {
  cplx<T> t = v[0];
  v[0] = cadd(t, v[1]);
  v[1] = csub(t, v[1]);
}

template <typename T>
__device__ inline void dft3(cplx<T>* v) {
  const T c3 = (T)0.86602540378443864676;  // sin(2 pi / 3)
  cplx<T> s = cadd(v[1], v[2]);
  cplx<T> d = csub(v[1], v[2]);
  cplx<T> m = {v[0].x - (T)0.5 * s.x, v[0].y - (T)0.5 * s.y};
  v[0] = cadd(v[0], s);
  v[1] = {m.x + c3 * d.y, m.y - c3 * d.x};
  v[2] = {m.x - c3 * d.y, m.y + c3 * d.x};
}

template <typename T>
__device__ inline void dft4(cplx<T>* v) {
  cplx<T> a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
  cplx<T> c = cadd(v[1], v[3]), d = mul_mi(csub(v[1], v[3]));
  v[0] = cadd(a, c);
  v[2] = csub(a, c);
  v[1] = cadd(b, d);
  v[3] = csub(b, d);
}

template <typename T>
__device__ inline void dft8(cplx<T>* v) {
  const T h = (T)0.70710678118654752440;
  cplx<T> e[4] = {v[0], v[2], v[4], v[6]};
  cplx<T> o[4] = {v[1], v[3], v[5], v[7]};
  dft4(e);
  dft4(o);
  // twiddles W8^k = exp(-i pi k / 4)
  cplx<T> o1 = {h * (o[1].x + o[1].y), h * (o[1].y - o[1].x)};
  cplx<T> o2 = mul_mi(o[2]);
  cplx<T> o3 = {h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y)};
  v[0] = cadd(e[0], o[0]);
  v[4] = csub(e[0], o[0]);
  v[1] = cadd(e[1], o1);
  v[5] = csub(e[1], o1);
  v[2] = cadd(e[2], o2);
  v[6] = csub(e[2], o2);
  v[3] = cadd(e[3], o3);
  v[7] = csub(e[3], o3);
}

// One Stockham radix-R stage over nl lines from in to out.  Element i of line
// l sits at l * ls + i * es.  LINE_FAST: consecutive threads take consecutive
// lines (for lines whose elements are strided in LDS, so that a wave's
// accesses stay on consecutive addresses); otherwise consecutive butterflies
// of one line.
template <typename T, int R, bool LINE_FAST>
__device__ inline void fft_stage(const cplx<T>* __restrict__ in, cplx<T>* __restrict__ out,
                                 int nl, int n, int ls, int es, int ns,
                                 const cplx<T>* __restrict__ tw) {
  const int m = n / R;
  const int tstride = n / (ns * R);
  const int total = nl * m;
  for (int bf = threadIdx.x; bf < total; bf += blockDim.x) {
    int line, j;
    if (LINE_FAST) {
      j = bf / nl;
      line = bf - j * nl;
    } else {
      line = bf / m;
      j = bf - line * m;
    }
    const int jq = j / ns;
    const int k = j - jq * ns;
    cplx<T> v[R];
    const cplx<T>* src = in + line * ls + j * es;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[r * m * es];
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[r * k * tstride]);
    if constexpr (R == 2) dft2(v);
    if constexpr (R == 3) dft3(v);
    if constexpr (R == 4) dft4(v);
    if constexpr (R == 8) dft8(v);
    cplx<T>* dst = out + line * ls + (jq * ns * R + k) * es;
#pragma unroll
    for (int r = 0; r < R; ++r) dst[r * ns * es] = v[r];
  }
}

// The same stage with the line length, the line count and the span of the
// stage known at compile time (index arithmetic by shifts and masks); the
// first stage's twiddles are all 1 and are skipped.  For the 64 x 64 planes of
// grids with a long x edge: 64 fields of 192 x 64 x 64 in FP32 646 us per solve,
// 732 without it.
template <typename T, int R, int N, int NL, int NS>
__device__ inline void fft_stage_c(const cplx<T>* __restrict__ in, cplx<T>* __restrict__ out,
                                   int ls, int es, const cplx<T>* __restrict__ tw) {
  constexpr int m = N / R;
  constexpr int tstride = N / (NS * R);
  constexpr int total = NL * m;
  for (int bf = threadIdx.x; bf < total; bf += blockDim.x) {
    const int j = bf / NL;
    const int line = bf - j * NL;
    const int jq = j / NS;
    const int k = j - jq * NS;
    cplx<T> v[R];
    const cplx<T>* src = in + line * ls + j * es;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[r * m * es];
    if constexpr (NS > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[r * k * tstride]);
    }
    if constexpr (R == 8) dft8(v);
    cplx<T>* dst = out + line * ls + (jq * NS * R + k) * es;
#pragma unroll
    for (int r = 0; r < R; ++r) dst[r * NS * es] = v[r];
  }
}

// Transform nl lines of length n held in LDS at buf0 (line stride ls,
// element stride es).  Returns the buffer that holds the result.  All
// threads of the block call it.
template <typename T, bool LINE_FAST = false>
__device__ cplx<T>* fft_lines(cplx<T>* buf0, cplx<T>* buf1, int nl, int n, int ls,
                              const FftPlan& plan, const cplx<T>* __restrict__ tw, int es = 1) {
  if (LINE_FAST && n == 64 && nl == 64 && plan.nstages == 2 && plan.radix[0] == 8 &&
      plan.radix[1] == 8) {
    // 64 lines of 64 points, consecutive threads on consecutive lines
    fft_stage_c<T, 8, 64, 64, 1>(buf0, buf1, ls, es, tw);
    __syncthreads();
    fft_stage_c<T, 8, 64, 64, 8>(buf1, buf0, ls, es, tw);
    __syncthreads();
    return buf0;
  }
  cplx<T>* in = buf0;
  cplx<T>* out = buf1;
  int ns = 1;
  for (int s = 0; s < plan.nstages; ++s) {
    const int R = plan.radix[s];
    switch (R) {
      case 2: fft_stage<T, 2, LINE_FAST>(in, out, nl, n, ls, es, ns, tw); break;
      case 3: fft_stage<T, 3, LINE_FAST>(in, out, nl, n, ls, es, ns, tw); break;
      case 4: fft_stage<T, 4, LINE_FAST>(in, out, nl, n, ls, es, ns, tw); break;
      default: fft_stage<T, 8, LINE_FAST>(in, out, nl, n, ls, es, ns, tw); break;
    }
    __syncthreads();
    cplx<T>* t = in;
    in = out;
    out = t;
    ns *= R;
  }
  return in;
}

// Moves cnt elements, e = threadIdx.x + k NT, from ld(e) to put(e, v), PER
// per thread at a time: every load of a batch is issued before the first of
// them is consumed, so a thread keeps PER loads in flight instead of one.
template <int NT, int PER, typename V, typename Load, typename Put>
__device__ inline void batched_copy(int cnt, Load ld, Put put) {
  for (int e0 = threadIdx.x; e0 < cnt; e0 += PER * NT) {
    V v[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = e0 + i * NT;
      if (e < cnt) v[i] = ld(e);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = e0 + i * NT;
      if (e < cnt) put(e, v[i]);
    }
  }
}

// Copies a twiddle table (n entries) into LDS; the first __syncthreads of the
// caller publishes it.
template <typename T>
__device__ inline void stage_twiddles(cplx<T>* dst, const cplx<T>* __restrict__ src, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

// Largest |value| over the block, one atomic maximum (float bits:
// non-negative floats order like their bit patterns, so the result does not
// depend on the order of the atomics).
template <typename T>
__device__ inline void block_max_atomic(T m, unsigned* dst) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  __shared__ float wm[16];  // up to 1024 threads
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) wm[wid] = (float)m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float a = 0.0f;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) a = fmaxf(a, wm[i]);
    atomicMax(dst, __float_as_uint(a));
  }
}

// Threads of the yz-plane pass: two blocks share a CU (up to 80 KB of LDS
// each); 16 waves each keep enough loads in flight.
constexpr int kYzThreads = 1024;

// Optional output scaling of the mixed product (FP16 operands downstream):
// the x pass records xmax[p] = max(|Re X|, |Im X|) over its output for the
// field pair p; the rest of the transform is an unnormalised inverse DFT over
// the ny nz (y, z) frequencies, so every potential value obeys
// |V| <= 2 ny nz xmax[p] (|X| <= sqrt 2 max(|Re|, |Im|)), and the last pass
// multiplies both fields by 2^e, e = f16_operand_exp(2 ny nz xmax[p], pexp),
// recording e in vexp[f].  The first pass clears xmax.
struct VScale {
  unsigned* xmax;  // [npairs] float bits, or nullptr (no scaling)
  int* vexp;       // [nf]
  int pexp;
  f16_t* out16;    // scaled output rounded to FP16 (instead of the real output)
};

// One value of an output field: FP16 (scaled) when the solve feeds the mixed
// product, else in the working precision.
template <typename T>
__device__ inline void put_v(T* rout, f16_t* out16, long i, T v) {
  if (out16) out16[i] = f32_to_f16((float)v);
  else rout[i] = v;
}

// Transform of whole yz planes (fixed x, contiguous in memory): the z lines,
// then the y lines, both in LDS, so the plane crosses HBM once each way.
// Forward: builds the complex field from the real fields 2p and 2p+1 (summing
// nparts GEMM partial densities) and clears xmax.  Inverse (conj(FFT(conj)),
// y lines then z lines): writes the real part to field 2p and the imaginary
// part to field 2p+1.  The spectrum between the passes is stored y-major,
// X[p][ky][x][kz], so that the x pass reads whole contiguous (x, kz) slabs;
// a plane's 64 rows of kz go out as 512-byte runs.  LDS: the plane and its
// ping-pong copy (rows padded by one), then the y and z twiddles.
template <typename T, bool INVERSE>
__global__ void __launch_bounds__(kYzThreads)
fft_pass_yz(cplx<T>* __restrict__ X, const T* __restrict__ rin, T* __restrict__ rout, int nf,
            long ld_real, long part_stride, int nparts, int nx, int ny, int nz, long nr,
            FftPlan py, FftPlan pz, const cplx<T>* __restrict__ twy,
            const cplx<T>* __restrict__ twz, VScale vs) {
  extern __shared__ unsigned char smem_raw[];
  const int ls = nz + 1;
  cplx<T>* buf0 = reinterpret_cast<cplx<T>*>(smem_raw);
  cplx<T>* buf1 = buf0 + ny * ls;
  cplx<T>* twy_s = buf1 + ny * ls;
  cplx<T>* twz_s = twy_s + ny;
  stage_twiddles(twy_s, twy, ny);
  stage_twiddles(twz_s, twz, nz);
  const int pair = blockIdx.y;
  const int x = blockIdx.x;
  const int f0 = 2 * pair, f1 = 2 * pair + 1;
  const long base = (long)x * ny * nz;     // plane x of a real field
  cplx<T>* Xp = X + (long)pair * nr;
  const long yrow = (long)nx * nz;         // spectrum: row ky of plane x at (ky nx + x) nz
  const int cnt = ny * nz;
  if (!INVERSE) {
    batched_copy<kYzThreads, 4, cplx<T>>(
        cnt,
        [&](int e) {
          T a = 0, b = 0;
          for (int q = 0; q < nparts; ++q) {
            const T* src = rin + (long)q * part_stride;
            a += src[(long)f0 * ld_real + base + e];
            if (f1 < nf) b += src[(long)f1 * ld_real + base + e];
          }
          return cplx<T>{a, b};
        },
        [&](int e, cplx<T> v) {
          const int y = e / nz, z = e - y * nz;
          buf0[y * ls + z] = v;
        });
  } else {
    batched_copy<kYzThreads, 4, cplx<T>>(
        cnt,
        [&](int e) {
          const int y = e / nz, z = e - y * nz;
          return Xp[y * yrow + (long)x * nz + z];
        },
        [&](int e, cplx<T> v) {
          const int y = e / nz, z = e - y * nz;
          buf0[y * ls + z] = {v.x, -v.y};
        });
  }
  __syncthreads();
  cplx<T>* res;
  if (!INVERSE) {
    res = fft_lines<T, true>(buf0, buf1, ny, nz, ls, pz, twz_s);
    cplx<T>* oth = (res == buf0) ? buf1 : buf0;
    res = fft_lines<T, true>(res, oth, nz, ny, 1, py, twy_s, ls);
  } else {
    res = fft_lines<T, true>(buf0, buf1, nz, ny, 1, py, twy_s, ls);
    cplx<T>* oth = (res == buf0) ? buf1 : buf0;
    res = fft_lines<T, true>(res, oth, ny, nz, ls, pz, twz_s);
  }
  T sc = 1;
  if (INVERSE && vs.xmax) {
    const int e = f16_operand_exp(__uint_as_float(vs.xmax[pair]) * (float)(2 * ny * nz), vs.pexp);
    sc = (T)ldexpf(1.0f, e);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      vs.vexp[f0] = e;
      if (f1 < nf) vs.vexp[f1] = e;
    }
  }
  if (!INVERSE && vs.xmax && blockIdx.x == 0 && threadIdx.x == 0) vs.xmax[pair] = 0u;
  for (int e = threadIdx.x; e < cnt; e += kYzThreads) {
    const int y = e / nz, z = e - y * nz;
    const cplx<T> v = res[y * ls + z];
    if (!INVERSE) {
      Xp[y * yrow + (long)x * nz + z] = v;
    } else {
      put_v(rout, vs.out16, (long)f0 * ld_real + base + e, sc * v.x);
      if (f1 < nf) put_v(rout, vs.out16, (long)f1 * ld_real + base + e, -(sc * v.y));
    }
  }
}

// Pass along z (contiguous lines).  Forward: builds the complex field from the
// real fields 2p and 2p+1, summing nparts GEMM partial densities.  Inverse:
// writes the real part to field 2p and the imaginary part to field 2p+1.
// LDS: lpb lines and their ping-pong copy (padded by one), then the twiddles.
template <typename T, bool INVERSE>
__global__ void __launch_bounds__(256)
fft_pass_z(cplx<T>* __restrict__ X, const T* __restrict__ rin, T* __restrict__ rout,
           int nf, long ld_real, long part_stride, int nparts, int nlines, int nz,
           long nr, int lpb, FftPlan plan, const cplx<T>* __restrict__ tw, VScale vs,
           int nyz) {
  extern __shared__ unsigned char smem_raw[];
  cplx<T>* buf0 = reinterpret_cast<cplx<T>*>(smem_raw);
  const int ls = nz + 1;
  cplx<T>* buf1 = buf0 + lpb * ls;
  cplx<T>* tws = buf1 + lpb * ls;
  stage_twiddles(tws, tw, nz);
  const int pair = blockIdx.y;
  const int f0 = 2 * pair, f1 = 2 * pair + 1;
  const int line0 = blockIdx.x * lpb;
  const int nl = min(lpb, nlines - line0);
  cplx<T>* Xp = X + (long)pair * nr;
  const long base = (long)line0 * nz;
  const int cnt = nl * nz;
  auto put = [&](int e, cplx<T> v) {
    const int l = e / nz, p = e - l * nz;
    buf0[l * ls + p] = v;
  };
  if (!INVERSE) {
    batched_copy<256, 4, cplx<T>>(
        cnt,
        [&](int e) {
          T a = 0, b = 0;
          for (int q = 0; q < nparts; ++q) {
            const T* src = rin + (long)q * part_stride;
            a += src[(long)f0 * ld_real + base + e];
            if (f1 < nf) b += src[(long)f1 * ld_real + base + e];
          }
          return cplx<T>{a, b};
        },
        put);
  } else {
    batched_copy<256, 4, cplx<T>>(
        cnt,
        [&](int e) {
          const cplx<T> v = Xp[base + e];
          return cplx<T>{v.x, -v.y};
        },
        put);
  }
  __syncthreads();
  cplx<T>* res = fft_lines<T, true>(buf0, buf1, nl, nz, ls, plan, tws);
  T sc = 1;
  if (INVERSE && vs.xmax) {
    const int e = f16_operand_exp(__uint_as_float(vs.xmax[pair]) * (float)(2 * nyz), vs.pexp);
    sc = (T)ldexpf(1.0f, e);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      vs.vexp[f0] = e;
      if (f1 < nf) vs.vexp[f1] = e;
    }
  }
  if (!INVERSE && vs.xmax && blockIdx.x == 0 && threadIdx.x == 0) vs.xmax[pair] = 0u;
  for (int e = threadIdx.x; e < cnt; e += blockDim.x) {
    const int l = e / nz, p = e - l * nz;
    cplx<T> v = res[l * ls + p];
    if (!INVERSE) {
      Xp[base + e] = v;
    } else {
      put_v(rout, vs.out16, (long)f0 * ld_real + base + e, sc * v.x);
      if (f1 < nf) put_v(rout, vs.out16, (long)f1 * ld_real + base + e, -(sc * v.y));
    }
  }
}

// Pass along a strided axis: element p of line l sits at p * pstride + l
// from the block's corner, which is outer * outer_stride + iz0; a block takes
// lpb consecutive lines (columns along the fastest index), so a row of its
// tile is one contiguous run.  MODE 0: forward, 1: inverse, 2: forward,
// multiply by the Coulomb kernel, inverse (x axis; outer is then ky and the
// lines are kz).  LDS holds the tile element-major (element p of line l at
// p (lpb + 1) + l), so consecutive threads touch consecutive words both when
// loading rows and inside the butterflies, and the ping-pong copy and the
// twiddles follow it.
template <typename T, int MODE, int NT>
__global__ void __launch_bounds__(NT)
fft_pass_strided(cplx<T>* __restrict__ X, int n, long pstride, long outer_stride,
                 int nzb, int nz, long nr, int lpb, FftPlan plan,
                 const cplx<T>* __restrict__ tw, const T* __restrict__ g2x,
                 const T* __restrict__ g2y, const T* __restrict__ g2z, T vscale,
                 unsigned* __restrict__ xmax) {
  extern __shared__ unsigned char smem_raw[];
  const int es = lpb + 1;
  cplx<T>* buf0 = reinterpret_cast<cplx<T>*>(smem_raw);
  cplx<T>* buf1 = buf0 + n * es;
  cplx<T>* tws = buf1 + n * es;
  stage_twiddles(tws, tw, n);
  const int pair = blockIdx.y;
  const int outer = blockIdx.x / nzb;
  const int iz0 = (blockIdx.x - outer * nzb) * lpb;
  const int nl = min(lpb, nz - iz0);
  cplx<T>* Xp = X + (long)pair * nr + (long)outer * outer_stride + iz0;
  const int cnt = nl * n;
  batched_copy<NT, 4, cplx<T>>(
      cnt,
      [&](int e) {
        const int p = e / nl, l = e - p * nl;
        return Xp[(long)p * pstride + l];
      },
      [&](int e, cplx<T> v) {
        const int p = e / nl, l = e - p * nl;
        if (MODE == 1) v.y = -v.y;
        buf0[p * es + l] = v;
      });
  __syncthreads();
  cplx<T>* res = fft_lines<T, true>(buf0, buf1, nl, n, 1, plan, tws, es);
  if (MODE == 2) {
    // res holds X(kx = p, ky = outer, kz = iz0 + l); multiply by v(G)/N and
    // conjugate for the inverse transform.
    cplx<T>* other = (res == buf0) ? buf1 : buf0;
    const T gyz = g2y[outer];
    for (int e = threadIdx.x; e < cnt; e += NT) {
      const int p = e / nl, l = e - p * nl;
      const T g2 = g2x[p] + gyz + g2z[iz0 + l];
      const T k = (g2 > (T)0) ? vscale / g2 : (T)0;
      const cplx<T> v = res[p * es + l];
      other[p * es + l] = {k * v.x, -k * v.y};
    }
    __syncthreads();
    res = fft_lines<T, true>(other, res, nl, n, 1, plan, tws, es);
  }
  T mx = 0;
  for (int e = threadIdx.x; e < cnt; e += NT) {
    const int p = e / nl, l = e - p * nl;
    cplx<T> v = res[p * es + l];
    if (MODE == 1 || MODE == 2) v.y = -v.y;
    Xp[(long)p * pstride + l] = v;
    mx = fmax(mx, fmax(fabs(v.x), fabs(v.y)));
  }
  if (MODE == 2 && xmax) block_max_atomic(mx, &xmax[pair]);
}

// LDS of the yz-plane pass (two planes); larger planes take the five-pass route
constexpr size_t kYzLdsMax = 80 * 1024;

// Lines per block of the contiguous (z) pass: about 16 KB of complex data per
// LDS buffer, between 4 and 32 lines.
template <typename T>
int lines_per_block(int n) {
  int l = (int)(16384 / sizeof(cplx<T>)) / n;
  if (l < 4) l = 4;
  if (l > 32) l = 32;
  return l;
}

}  // namespace

void poisson_prepare_device() {
  // dynamic LDS beyond 64 KB must be allowed per kernel, on the current device
  const int lim = (int)kYzLdsMax;
  GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&fft_pass_yz<float, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&fft_pass_yz<float, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&fft_pass_yz<double, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&fft_pass_yz<double, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  GWL_HIP(hipFuncSetAttribute(
      reinterpret_cast<const void*>(&fft_pass_strided<float, 2, kYzThreads>),
      hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  GWL_HIP(hipFuncSetAttribute(
      reinterpret_cast<const void*>(&fft_pass_strided<double, 2, kYzThreads>),
      hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  plane_prepare_device();
}

FftPlan make_plan(int n) {
  FftPlan p{};
  int m = n;
  while (m % 8 == 0 && m > 1) { p.radix[p.nstages++] = 8; m /= 8; }
  while (m % 4 == 0 && m > 1) { p.radix[p.nstages++] = 4; m /= 4; }
  while (m % 2 == 0 && m > 1) { p.radix[p.nstages++] = 2; m /= 2; }
  while (m % 3 == 0 && m > 1) { p.radix[p.nstages++] = 3; m /= 3; }
  p.ok = (m == 1) && p.nstages <= 8;
  return p;
}

// LDS of the strided pass: the tile, its copy and the twiddles
template <typename T>
size_t strided_lds(int n, int lpb) {
  return (2 * (size_t)n * (lpb + 1) + n) * sizeof(cplx<T>);
}

template <typename T>
void poisson_launch(const PoissonGeom<T>& g, const T* rin, long ld_in, long part_stride,
                    int nparts, T* rout, long ld_out, int nf, cplx<T>* scratch,
                    hipStream_t st, unsigned* xmax, int* vexp, int pexp, f16_t* rout16) {
  const VScale vs{vexp ? xmax : nullptr, vexp, pexp, vexp ? rout16 : nullptr};
  unsigned* xm = vs.xmax;
  const int nyz = g.ny * g.nz;
  if (nf <= 0) return;
  const int npairs = (nf + 1) / 2;
  const long nr = (long)g.nx * g.ny * g.nz;
  const int nmax = g.nx > g.ny ? g.nx : g.ny;
  int lpb = 1024 / nmax;
  if (lpb > 16) lpb = 16;
  if (lpb < 2) lpb = 2;
  if (lpb > g.nz) lpb = g.nz;
  const int nzb = ceil_div(g.nz, lpb);
  if (poisson_planes<T>(g, rin, ld_in, part_stride, nparts, rout, ld_out, nf, scratch, st, xm,
                        vs.vexp, pexp, vs.out16))
    return;
  // Three HBM round trips when a yz plane and its ping-pong copy fit in LDS:
  // yz forward (+ pack), x forward / kernel / x inverse over (x, kz) slabs of
  // the y-major spectrum, yz inverse (+ unpack)
  const size_t sm_yz = (2 * (size_t)g.ny * (g.nz + 1) + g.ny + g.nz) * sizeof(cplx<T>);
  int lx = g.nz;  // kz columns per block of the x pass
  while (lx > 1 && strided_lds<T>(g.nx, lx) > kYzLdsMax) lx = (lx + 1) / 2;
  if (sm_yz <= kYzLdsMax && strided_lds<T>(g.nx, lx) <= kYzLdsMax) {
    dim3 gyz(g.nx, npairs);
    fft_pass_yz<T, false><<<gyz, kYzThreads, sm_yz, st>>>(
        scratch, rin, nullptr, nf, ld_in, part_stride, nparts, g.nx, g.ny, g.nz, nr, g.py, g.pz,
        g.twy, g.twz, vs);
    const int nzbx = ceil_div(g.nz, lx);
    dim3 gx(g.ny * nzbx, npairs);
    fft_pass_strided<T, 2, kYzThreads><<<gx, kYzThreads, strided_lds<T>(g.nx, lx), st>>>(
        scratch, g.nx, g.nz, (long)g.nx * g.nz, nzbx, g.nz, nr, lx, g.px, g.twx, g.g2x, g.g2y,
        g.g2z, g.vscale, xm);
    fft_pass_yz<T, true><<<gyz, kYzThreads, sm_yz, st>>>(
        scratch, nullptr, rout, nf, ld_out, 0, 1, g.nx, g.ny, g.nz, nr, g.py, g.pz, g.twy, g.twz,
        vs);
    GWL_HIP(hipGetLastError());
    return;
  }
  // otherwise five: z forward + pack
  {
    const int lpbz = lines_per_block<T>(g.nz);
    const int nlines = g.nx * g.ny;
    dim3 grid(ceil_div(nlines, lpbz), npairs);
    size_t sm = (2 * (size_t)lpbz * (g.nz + 1) + g.nz) * sizeof(cplx<T>);
    fft_pass_z<T, false><<<grid, 256, sm, st>>>(scratch, rin, nullptr, nf, ld_in,
                                                part_stride, nparts, nlines, g.nz, nr,
                                                lpbz, g.pz, g.twz, vs, nyz);
  }
  // y forward
  {
    dim3 grid(g.nx * nzb, npairs);
    fft_pass_strided<T, 0, 256><<<grid, 256, strided_lds<T>(g.ny, lpb), st>>>(
        scratch, g.ny, g.nz, (long)g.ny * g.nz, nzb, g.nz, nr, lpb, g.py, g.twy, nullptr,
        nullptr, nullptr, (T)0, nullptr);
  }
  // x forward, kernel, x inverse
  {
    dim3 grid(g.ny * nzb, npairs);
    fft_pass_strided<T, 2, 256><<<grid, 256, strided_lds<T>(g.nx, lpb), st>>>(
        scratch, g.nx, (long)g.ny * g.nz, g.nz, nzb, g.nz, nr, lpb, g.px, g.twx, g.g2x, g.g2y,
        g.g2z, g.vscale, xm);
  }
  // y inverse
  {
    dim3 grid(g.nx * nzb, npairs);
    fft_pass_strided<T, 1, 256><<<grid, 256, strided_lds<T>(g.ny, lpb), st>>>(
        scratch, g.ny, g.nz, (long)g.ny * g.nz, nzb, g.nz, nr, lpb, g.py, g.twy, nullptr,
        nullptr, nullptr, (T)0, nullptr);
  }
  // z inverse + unpack
  {
    const int lpbz = lines_per_block<T>(g.nz);
    const int nlines = g.nx * g.ny;
    dim3 grid(ceil_div(nlines, lpbz), npairs);
    size_t sm = (2 * (size_t)lpbz * (g.nz + 1) + g.nz) * sizeof(cplx<T>);
    fft_pass_z<T, true><<<grid, 256, sm, st>>>(scratch, nullptr, rout, nf, ld_out, 0, 1,
                                               nlines, g.nz, nr, lpbz, g.pz, g.twz, vs, nyz);
  }
  GWL_HIP(hipGetLastError());
}

template void poisson_launch<float>(const PoissonGeom<float>&, const float*, long, long, int,
                                    float*, long, int, cplx<float>*, hipStream_t, unsigned*,
                                    int*, int, f16_t*);
template void poisson_launch<double>(const PoissonGeom<double>&, const double*, long, long,
                                     int, double*, long, int, cplx<double>*, hipStream_t,
                                     unsigned*, int*, int, f16_t*);

}  // namespace gwl
