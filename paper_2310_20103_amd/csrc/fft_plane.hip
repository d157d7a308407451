// Hartree solve in three passes of in-place transforms (see fft_poisson.hip
// for the solve, its packing of two real fields into one complex field and the
// y-major spectrum X[ky][x][kz] between the passes), for edges of 2 to 81 points
// and 96, 108, 128 and 144 whose yz planes fit in 160 KB: in FP32 all but 144 x
// 144, in FP64 up to 96 x 96 (128 x 72, 144 x 64):
//   forward plane pass (fixed x): z lines, then y lines
//   x pass (fixed ky):            x lines, v(G)/N, x lines back
//   inverse plane pass:           y lines, then z lines
//
// A line of N = R1 R2 points takes two steps in registers: R1-point transforms
// over n = j + R2 a (a < R1), then R2-point ones over j that give the
// frequencies k = r + R1 k2 (Cooley and Tukey; a step is one or two of the
// radix-2, 3, 4 and 8 stages of fft_poisson.hip, with the same twiddles in the
// same order, so values equal those of the stage-by-stage transform but for
// which of their products are rounded by themselves).
// Both steps write where they read (slot j + R2 r, then k2 + R2 r): one barrier
// each, no second buffer, no limit on butterflies per thread; the order of the
// slots is left to the addresses of whoever reads them next.  The inverse is
// conj(FFT(conj(x))).
//
// The first step of a pass reads global memory straight into its butterflies
// and the last one writes from them: consecutive threads on consecutive
// addresses along z in the y and x steps, runs of R2 (read) or R1 (written)
// points in the z steps.
//
// Bound by HBM from a few hundred planes on (64 fields of 64^3 in FP64: 177 us
// per call for 1.07 GB over the three passes), by latency below; small planes
// run in blocks of one to a few waves, so many share a CU.  Against stage-by-
// stage transforms with ping-pong buffers and line lengths known at run time: 32
// fields of 128^3 in FP32 (then five passes) 1,055 -> 488 us per call, 128 of
// 48^3 in FP32 320 -> 107, 64 of 32^3 in FP64 92 -> 52, two of 24^3 in FP64
// 34.5 -> 28.2; against in-place radix-8 stages of 64^3 with load and store
// phases of their own, 128 fields in FP32 211 -> 186.  Cutting the batch into runs
// whose spectrum stays in the 256 MB cache gained nothing at 140 MB and lost
// 9 % at 70 MB.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace gwl {
namespace {

__device__ inline float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
// (which products are rounded is spelt out: left to the compiler's contraction
// it changes from use to use, and the results with it)
template <typename T>
__device__ inline cplx<T> cmul(cplx<T> a, cplx<T> b) {
  return {fma_(a.x, b.x, -(a.y * b.y)), fma_(a.y, b.x, a.x * b.y)};
}
template <typename T>
__device__ inline cplx<T> cadd(cplx<T> a, cplx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ inline cplx<T> csub(cplx<T> a, cplx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ inline cplx<T> mul_mi(cplx<T> a) { return {a.y, -a.x}; }  // -i a

template <typename T, int R>
__device__ inline void dft(cplx<T>* v) {
  if constexpr (R == 2) {
    const cplx<T> t = v[0];
    v[0] = cadd(t, v[1]);
    v[1] = csub(t, v[1]);
  } else if constexpr (R == 3) {
    const T c3 = (T)0.86602540378443864676;  // sin(2 pi / 3)
    const cplx<T> s = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const cplx<T> m = {v[0].x - (T)0.5 * s.x, v[0].y - (T)0.5 * s.y};
    v[0] = cadd(v[0], s);
    v[1] = {fma_(c3, d.y, m.x), fma_(-c3, d.x, m.y)};
    v[2] = {fma_(-c3, d.y, m.x), fma_(c3, d.x, m.y)};
  } else if constexpr (R == 4) {
    const cplx<T> a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
    const cplx<T> c = cadd(v[1], v[3]), d = mul_mi(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[2] = csub(a, c);
    v[1] = cadd(b, d);
    v[3] = csub(b, d);
  } else if constexpr (R == 8) {
    const T h = (T)0.70710678118654752440;
    cplx<T> e[4] = {v[0], v[2], v[4], v[6]};
    cplx<T> o[4] = {v[1], v[3], v[5], v[7]};
    dft<T, 4>(e);
    dft<T, 4>(o);
    // twiddles W8^k = exp(-i pi k / 4) (h in the sums below)
    const cplx<T> o1 = {o[1].x + o[1].y, o[1].y - o[1].x};
    const cplx<T> o2 = mul_mi(o[2]);
    const cplx<T> o3 = {o[3].y - o[3].x, -(o[3].x + o[3].y)};
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = {fma_(h, o1.x, e[1].x), fma_(h, o1.y, e[1].y)};
    v[5] = {fma_(-h, o1.x, e[1].x), fma_(-h, o1.y, e[1].y)};
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = {fma_(h, o3.x, e[3].x), fma_(h, o3.y, e[3].y)};
    v[7] = {fma_(-h, o3.x, e[3].x), fma_(-h, o3.y, e[3].y)};
  } else {
    static_assert(R == 1, "radix");
  }
}

// Line lengths and the radices of their two steps, R1 = A1 A2 and R2 = B1 B2,
// in the order in which make_plan factors the length.  The long ones live in
// kernels of their own (12- and 16-point steps need twice the registers).
#define GWL_FFT_SHORT(X)                                                            \
  X(2, 2, 1, 1, 1) X(3, 3, 1, 1, 1) X(4, 4, 1, 1, 1) X(6, 2, 1, 3, 1) X(8, 8, 1, 1, 1) \
  X(9, 3, 1, 3, 1) X(12, 4, 1, 3, 1) X(16, 8, 1, 2, 1) X(18, 2, 3, 3, 1)            \
  X(24, 8, 1, 3, 1) X(27, 3, 3, 3, 1) X(32, 8, 1, 4, 1) X(36, 4, 1, 3, 3)           \
  X(48, 8, 1, 2, 3) X(54, 2, 3, 3, 3) X(64, 8, 1, 8, 1) X(72, 8, 1, 3, 3)           \
  X(81, 3, 3, 3, 3)
#define GWL_FFT_LONG(X) \
  X(96, 8, 1, 4, 3) X(108, 4, 3, 3, 3) X(128, 8, 1, 8, 2) X(144, 8, 2, 3, 3)

bool fft_split(int n, int& r1, int& r2, bool& is_long) {
  is_long = false;
  switch (n) {
#define X(N, A, B, C, D) case N: r1 = A * B; r2 = C * D; return true;
    GWL_FFT_SHORT(X)
#undef X
#define X(N, A, B, C, D) case N: r1 = A * B; r2 = C * D; is_long = true; return true;
    GWL_FFT_LONG(X)
#undef X
  }
  return false;
}

template <int A, int B, int C, int D>
struct Rad {
  static constexpr int A1 = A, A2 = B, B1 = C, B2 = D, R1 = A * B, R2 = C * D;
};
// fn(radices) for the line length n
template <bool LONG, typename F>
__device__ inline void with_length(int n, F fn) {
  switch (n) {
#define X(N, A, B, C, D) case N: fn(Rad<A, B, C, D>{}); return;
    GWL_FFT_SHORT(X)
#undef X
  }
  if constexpr (LONG) {
    switch (n) {
#define X(N, A, B, C, D) case N: fn(Rad<A, B, C, D>{}); return;
      GWL_FFT_LONG(X)
#undef X
    }
  }
}

// First step: v[a] (input j + R2 a) -> v[r]; tw[k] = exp(-2 pi i k / N).
template <typename R, typename T>
__device__ inline void step1(cplx<T>* v, const cplx<T>* __restrict__ tw) {
  if constexpr (R::A2 == 1) {
    dft<T, R::A1>(v);
  } else {
    cplx<T> y[R::A2][R::A1];
#pragma unroll
    for (int al = 0; al < R::A2; ++al) {
#pragma unroll
      for (int i = 0; i < R::A1; ++i) y[al][i] = v[al + R::A2 * i];
      dft<T, R::A1>(y[al]);
    }
#pragma unroll
    for (int i = 0; i < R::A1; ++i) {
      cplx<T> z[R::A2];
#pragma unroll
      for (int al = 0; al < R::A2; ++al)
        z[al] = al * i ? cmul(y[al][i], tw[al * i * R::R2]) : y[al][i];
      dft<T, R::A2>(z);
#pragma unroll
      for (int k = 0; k < R::A2; ++k) v[i + R::A1 * k] = z[k];
    }
  }
}

// Second step: v[j] (from the first steps' output r) -> v[k2] (frequency r + R1 k2).
template <typename R, typename T>
__device__ inline void step2(cplx<T>* v, const cplx<T>* __restrict__ tw, int r) {
  if constexpr (R::B2 == 1) {
#pragma unroll
    for (int j = 1; j < R::B1; ++j) v[j] = cmul(v[j], tw[j * r]);
    dft<T, R::B1>(v);
  } else {
    cplx<T> y[R::B2][R::B1];
#pragma unroll
    for (int be = 0; be < R::B2; ++be) {
#pragma unroll
      for (int i = 0; i < R::B1; ++i) {
        y[be][i] = v[be + R::B2 * i];
        if (i) y[be][i] = cmul(y[be][i], tw[i * r * R::B2]);
      }
      dft<T, R::B1>(y[be]);
    }
#pragma unroll
    for (int i = 0; i < R::B1; ++i) {
      cplx<T> z[R::B2];
#pragma unroll
      for (int be = 0; be < R::B2; ++be)
        z[be] = be ? cmul(y[be][i], tw[be * (r + R::R1 * i)]) : y[be][i];
      dft<T, R::B2>(z);
#pragma unroll
      for (int k = 0; k < R::B2; ++k) v[i + R::B1 * k] = z[k];
    }
  }
}

// e / d for e < 2^16, d <= 256 (m = ceil(2^32 / d): the error stays below 1/d)
struct FastDiv {
  unsigned d, m;
  __device__ int div(int e) const { return d == 1 ? e : (int)__umulhi((unsigned)e, m); }
};
FastDiv fast_div(int d) { return {(unsigned)d, (unsigned)(((1ull << 32) + d - 1) / d)}; }

template <typename T>
__device__ inline cplx<T> conj_(cplx<T> a) { return {a.x, -a.y}; }

// Largest |value| over the block, one atomic maximum (non-negative floats
// order like their bit patterns).  blockDim.x is a multiple of 64.
template <typename T>
__device__ inline void block_max(T m, unsigned* dst) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  __shared__ float wm[16];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) wm[wid] = (float)m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float a = 0.0f;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) a = fmaxf(a, wm[i]);
    atomicMax(dst, __float_as_uint(a));
  }
}

// A grid's plane passes: everything the kernels need besides the fields.
template <typename T>
struct PlaneGeom {
  int nx, ny, nz;
  int r1y, r2y, r1z, r2z;          // slot k2 + R2 r of a line holds r + R1 k2
  long nr;
  FastDiv dy, dz, d2y, d1z;        // by ny, nz, r2y, r1z
  const cplx<T>*twy, *twz;
  __device__ int y_of(int slot) const {
    const int r = d2y.div(slot);
    return r + r1y * (slot - r * r2y);
  }
  __device__ int z_slot(int z) const {
    const int k2 = d1z.div(z);
    return k2 + r2z * (z - k2 * r1z);
  }
};

// Output of the inverse pass: the potentials, or (vexp set: the mixed product)
// FP16 values scaled by the power of two that the x pass's maximum allows.
template <typename T>
struct PlaneOut {
  T* v;
  f16_t* v16;
  long ld;
  const unsigned* xmax;
  int* vexp;
  int pexp;
};

// waves per SIMD the plane passes' registers must allow (FP32 short lines: 80
// registers hold a radix-9 butterfly; eight waves would spill it)
constexpr int min_waves(bool is_long, size_t real) {
  return real == 8 ? (is_long ? 2 : 4) : (is_long ? 4 : 6);
}

template <typename T>
__device__ inline void stage_tables(cplx<T>* tw, const PlaneGeom<T>& g) {
  for (int i = threadIdx.x; i < g.ny + g.nz; i += blockDim.x)
    tw[i] = i < g.ny ? g.twy[i] : g.twz[i - g.ny];
}

// threads per block at most: 16 waves where a butterfly fits 128 registers, 8
// for long lines in FP64
constexpr int max_threads(bool is_long, size_t real) { return is_long && real == 8 ? 512 : 1024; }

// Fields in, for the forward plane pass: sums of nparts GEMM partial densities,
template <typename T>
struct FieldSums {
  const T* in;
  long ld, part_stride;
  int nparts, nf;
  __device__ bool has(int f) const { return f < nf; }
  // v[i] = value e0 + step i of field f
  template <int R, typename V>
  __device__ void load(int f, long e0, int step, V set) const {
    const T* p = in + f * ld + e0;
    T v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = p[step * i];
    for (int q = 1; q < nparts; ++q)
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] += p[q * part_stride + step * i];
#pragma unroll
    for (int i = 0; i < R; ++i) set(i, v[i]);
  }
};
// or products of two orbital rows (n[f] < 0: no field).
struct RowProducts {
  const double* psi;
  long ld;
  const int *m, *n;
  int nf;
  __device__ bool has(int f) const { return f < nf && n[f] >= 0; }
  template <int R, typename V>
  __device__ void load(int f, long e0, int step, V set) const {
    const double* a = psi + m[f] * ld + e0;
    const double* b = psi + n[f] * ld + e0;
    double v[R], w[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = a[step * i], w[i] = b[step * i];
#pragma unroll
    for (int i = 0; i < R; ++i) set(i, v[i] * w[i]);
  }
};

// Forward plane pass: fields 2p and 2p + 1 packed, z lines then y lines of the
// plane at x.
template <typename T, bool LONG, typename In>
__global__ void __launch_bounds__(max_threads(LONG, sizeof(T)))
__attribute__((amdgpu_waves_per_eu(min_waves(LONG, sizeof(T)))))
plane_forward(PlaneGeom<T> g, In in, cplx<T>* __restrict__ X, unsigned* __restrict__ xmax) {
  extern __shared__ unsigned char smem_raw[];
  const int P = g.nz | 1;  // LDS row: odd, for the steps with consecutive threads on consecutive rows
  cplx<T>* buf = reinterpret_cast<cplx<T>*>(smem_raw);
  cplx<T>* twy = buf + g.ny * P;
  cplx<T>* twz = twy + g.ny;
  stage_tables(twy, g);
  const int x = blockIdx.x, pair = blockIdx.y, t = threadIdx.x, nt = blockDim.x;
  const bool two = in.has(2 * pair + 1);
  const long plane = (long)x * g.ny * g.nz;
  if (xmax && x == 0 && t == 0) xmax[pair] = 0u;
  __syncthreads();
  with_length<LONG>(g.nz, [&](auto R_) {
    typedef decltype(R_) R;
    constexpr int R1 = R::R1, R2 = R::R2;
    for (int b = t; b < g.ny * R2; b += nt) {
      const int y = b / R2, j = b - y * R2;
      const long e0 = plane + y * g.nz + j;
      cplx<T> v[R1];
      in.template load<R1>(2 * pair, e0, R2, [&](int i, T a) { v[i].x = a; });
      if (two)
        in.template load<R1>(2 * pair + 1, e0, R2, [&](int i, T a) { v[i].y = a; });
      else
#pragma unroll
        for (int i = 0; i < R1; ++i) v[i].y = 0;
      step1<R>(v, twz);
      cplx<T>* row = buf + y * P + j;
#pragma unroll
      for (int r = 0; r < R1; ++r) row[R2 * r] = v[r];
    }
    __syncthreads();
    if constexpr (R2 > 1) {
      for (int b = t; b < g.ny * R1; b += nt) {
        const int r = g.dy.div(b);
        cplx<T>* row = buf + (b - r * g.ny) * P + R2 * r;
        cplx<T> v[R2];
#pragma unroll
        for (int j = 0; j < R2; ++j) v[j] = row[j];
        step2<R>(v, twz, r);
#pragma unroll
        for (int k = 0; k < R2; ++k) row[k] = v[k];
      }
      __syncthreads();
    }
  });
  cplx<T>* Xp = X + (long)pair * g.nr + (long)x * g.nz;
  with_length<LONG>(g.ny, [&](auto R_) {
    typedef decltype(R_) R;
    constexpr int R1 = R::R1, R2 = R::R2;
    for (int b = t; b < g.nz * R2; b += nt) {
      const int j = g.dz.div(b);
      cplx<T>* col = buf + j * P + (b - j * g.nz);
      cplx<T> v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) v[a] = col[R2 * a * P];
      step1<R>(v, twy);
#pragma unroll
      for (int r = 0; r < R1; ++r) col[R2 * r * P] = v[r];
    }
    __syncthreads();
    for (int b = t; b < g.nz * R1; b += nt) {
      const int r = g.dz.div(b), z = b - r * g.nz;
      const cplx<T>* col = buf + R2 * r * P + g.z_slot(z);
      cplx<T> v[R2];
#pragma unroll
      for (int j = 0; j < R2; ++j) v[j] = col[j * P];
      step2<R>(v, twy, r);
#pragma unroll
      for (int k = 0; k < R2; ++k) Xp[(long)(r + R1 * k) * g.nx * g.nz + z] = v[k];
    }
  });
}

// Inverse plane pass: y lines then z lines back, real and imaginary parts to
// the fields 2p and 2p + 1.
template <typename T, bool LONG>
__global__ void __launch_bounds__(max_threads(LONG, sizeof(T)))
__attribute__((amdgpu_waves_per_eu(min_waves(LONG, sizeof(T)))))
plane_inverse(PlaneGeom<T> g, const cplx<T>* __restrict__ X, int nf, PlaneOut<T> out) {
  extern __shared__ unsigned char smem_raw[];
  const int P = g.nz | 1;
  cplx<T>* buf = reinterpret_cast<cplx<T>*>(smem_raw);
  cplx<T>* twy = buf + g.ny * P;
  cplx<T>* twz = twy + g.ny;
  stage_tables(twy, g);
  const int x = blockIdx.x, pair = blockIdx.y, t = threadIdx.x, nt = blockDim.x;
  const bool two = 2 * pair + 1 < nf;
  T sc = 1;
  if (out.vexp) {
    // every value of the transform is at most 2 ny nz times the x pass's maximum
    const int e = f16_operand_exp(__uint_as_float(out.xmax[pair]) * (float)(2 * g.ny * g.nz), out.pexp);
    sc = (T)ldexpf(1.0f, e);
    if (x == 0 && t == 0) {
      out.vexp[2 * pair] = e;
      if (two) out.vexp[2 * pair + 1] = e;
    }
  }
  __syncthreads();
  const cplx<T>* Xp = X + (long)pair * g.nr + (long)x * g.nz;
  with_length<LONG>(g.ny, [&](auto R_) {
    typedef decltype(R_) R;
    constexpr int R1 = R::R1, R2 = R::R2;
    for (int b = t; b < g.nz * R2; b += nt) {
      const int j = g.dz.div(b), z = b - j * g.nz;
      cplx<T> v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) v[a] = conj_(Xp[(long)(j + R2 * a) * g.nx * g.nz + z]);
      step1<R>(v, twy);
      cplx<T>* col = buf + j * P + z;
#pragma unroll
      for (int r = 0; r < R1; ++r) col[R2 * r * P] = v[r];
    }
    __syncthreads();
    if constexpr (R2 > 1) {
      for (int b = t; b < g.nz * R1; b += nt) {
        const int r = g.dz.div(b);
        cplx<T>* col = buf + R2 * r * P + (b - r * g.nz);
        cplx<T> v[R2];
#pragma unroll
        for (int j = 0; j < R2; ++j) v[j] = col[j * P];
        step2<R>(v, twy, r);
#pragma unroll
        for (int k = 0; k < R2; ++k) col[k * P] = v[k];
      }
      __syncthreads();
    }
  });
  const long o0 = (long)(2 * pair) * out.ld + (long)x * g.ny * g.nz;
  with_length<LONG>(g.nz, [&](auto R_) {
    typedef decltype(R_) R;
    constexpr int R1 = R::R1, R2 = R::R2;
    for (int b = t; b < g.ny * R2; b += nt) {
      const int j = g.dy.div(b);
      cplx<T>* row = buf + (b - j * g.ny) * P + j;
      cplx<T> v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) v[a] = row[R2 * a];
      step1<R>(v, twz);
#pragma unroll
      for (int r = 0; r < R1; ++r) row[R2 * r] = v[r];
    }
    __syncthreads();
    for (int b = t; b < g.ny * R1; b += nt) {
      const int slot = b / R1, r = b - slot * R1;
      const cplx<T>* row = buf + slot * P + R2 * r;
      cplx<T> v[R2];
#pragma unroll
      for (int j = 0; j < R2; ++j) v[j] = row[j];
      step2<R>(v, twz, r);
      const long o1 = o0 + g.y_of(slot) * g.nz + r;
#pragma unroll
      for (int k = 0; k < R2; ++k) {
        const long o = o1 + R1 * k;
        const T re = sc * v[k].x, im = -(sc * v[k].y);
        if (out.v16) {
          out.v16[o] = f32_to_f16((float)re);
          if (two) out.v16[o + out.ld] = f32_to_f16((float)im);
        } else {
          out.v[o] = re;
          if (two) out.v[o + out.ld] = im;
        }
      }
    }
  });
}

// x pass over lx kz columns of the slab at ky (blockIdx.x = ky nzb + block of
// columns): forward along x, v(G)/N, back; records max(|Re|, |Im|) per pair.
template <typename T, bool LONG>
__global__ void __launch_bounds__(max_threads(LONG, sizeof(T)))
x_pass(cplx<T>* __restrict__ X, int nx, int nz, int lx, int nzb, long nr, FastDiv dlx,
       const cplx<T>* __restrict__ twx, const T* __restrict__ g2x, const T* __restrict__ g2y,
       const T* __restrict__ g2z, T vscale, unsigned* __restrict__ xmax) {
  extern __shared__ unsigned char smem_raw[];
  cplx<T>* buf = reinterpret_cast<cplx<T>*>(smem_raw);  // [x slot][lx]
  cplx<T>* tw = buf + nx * lx;
  T* g2s = reinterpret_cast<T*>(tw + nx);
  const int t = threadIdx.x, nt = blockDim.x, pair = blockIdx.y;
  for (int i = t; i < nx; i += nt) {
    tw[i] = twx[i];
    g2s[i] = g2x[i];
  }
  const int ky = blockIdx.x / nzb, z0 = (blockIdx.x - ky * nzb) * lx;
  const int nl = min(lx, nz - z0);  // (columns past the end repeat column z0)
  cplx<T>* Xp = X + (long)pair * nr + (long)ky * nx * nz + z0;
  const T gy = g2y[ky];
  T mx = 0;
  __syncthreads();
  with_length<LONG>(nx, [&](auto R_) {
    typedef decltype(R_) R;
    constexpr int R1 = R::R1, R2 = R::R2;
    // slot of index n = r + R1 k2 after a second step
    auto slot = [](int n) { return n / R1 + R2 * (n % R1); };
    for (int b = t; b < lx * R2; b += nt) {
      const int j = dlx.div(b), c = b - j * lx;
      const cplx<T>* i = Xp + (c < nl ? c : 0);
      cplx<T> v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) v[a] = i[(j + R2 * a) * nz];
      step1<R>(v, tw);
#pragma unroll
      for (int r = 0; r < R1; ++r) buf[(j + R2 * r) * lx + c] = v[r];
    }
    __syncthreads();
    for (int b = t; b < lx * R1; b += nt) {
      const int r = dlx.div(b), c = b - r * lx;
      const T gz = g2z[z0 + (c < nl ? c : 0)];
      cplx<T>* col = buf + R2 * r * lx + c;
      cplx<T> v[R2];
#pragma unroll
      for (int j = 0; j < R2; ++j) v[j] = col[j * lx];
      step2<R>(v, tw, r);
#pragma unroll
      for (int k = 0; k < R2; ++k) {
        const T g2 = g2s[r + R1 * k] + gy + gz;
        const T f = g2 > (T)0 ? vscale / g2 : (T)0;
        col[k * lx] = {f * v[k].x, -f * v[k].y};  // conjugated for the way back
      }
    }
    __syncthreads();
    for (int b = t; b < lx * R2; b += nt) {
      const int j = dlx.div(b), c = b - j * lx;
      cplx<T> v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) v[a] = buf[slot(j + R2 * a) * lx + c];
      step1<R>(v, tw);
#pragma unroll
      for (int r = 0; r < R1; ++r) buf[slot(j + R2 * r) * lx + c] = v[r];
    }
    __syncthreads();
    for (int b = t; b < lx * R1; b += nt) {
      const int r = dlx.div(b), c = b - r * lx;
      cplx<T> v[R2];
#pragma unroll
      for (int j = 0; j < R2; ++j) v[j] = buf[slot(j + R2 * r) * lx + c];
      step2<R>(v, tw, r);
      if (c >= nl) continue;
#pragma unroll
      for (int k = 0; k < R2; ++k) {
        Xp[(r + R1 * k) * nz + c] = conj_(v[k]);
        mx = fmax(mx, fmax(fabs(v[k].x), fabs(v[k].y)));
      }
    }
  });
  if (xmax) block_max(mx, &xmax[pair]);
}

// The forward half of the x pass for the energies dV sum_r rho V = dV sum_k
// (v(G)/N) |rho_k|^2: part[pair][block] = this block's share of the sum of both
// fields' energies (the cross terms of the packed spectrum cancel between k
// and -k), nothing is written back.  HBM-bound: with the products formed in the
// forward pass, 1,024 products of 64^3 cross memory as orbital rows in, spectrum
// out and in (8.6 GB): 1.48 ms, against 12.3 ms for product, whole solve and a
// grid sum with one block per field.
template <bool LONG>
__global__ void __launch_bounds__(max_threads(LONG, 8))
x_energy(const cplx<double>* __restrict__ X, int nx, int nz, int lx, int nzb, long nr, FastDiv dlx,
         const cplx<double>* __restrict__ twx, const double* __restrict__ g2x,
         const double* __restrict__ g2y, const double* __restrict__ g2z, double vscale,
         double* __restrict__ part) {
  extern __shared__ unsigned char smem_raw[];
  cplx<double>* buf = reinterpret_cast<cplx<double>*>(smem_raw);
  cplx<double>* tw = buf + nx * lx;
  double* g2s = reinterpret_cast<double*>(tw + nx);
  const int t = threadIdx.x, nt = blockDim.x, pair = blockIdx.y;
  for (int i = t; i < nx; i += nt) {
    tw[i] = twx[i];
    g2s[i] = g2x[i];
  }
  const int ky = blockIdx.x / nzb, z0 = (blockIdx.x - ky * nzb) * lx;
  const int nl = min(lx, nz - z0);
  const cplx<double>* Xp = X + (long)pair * nr + (long)ky * nx * nz + z0;
  const double gy = g2y[ky];
  double sum = 0.0;
  __syncthreads();
  with_length<LONG>(nx, [&](auto R_) {
    typedef decltype(R_) R;
    constexpr int R1 = R::R1, R2 = R::R2;
    for (int b = t; b < lx * R2; b += nt) {
      const int j = dlx.div(b), c = b - j * lx;
      const cplx<double>* i = Xp + (c < nl ? c : 0);
      cplx<double> v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) v[a] = i[(j + R2 * a) * nz];
      step1<R>(v, tw);
#pragma unroll
      for (int r = 0; r < R1; ++r) buf[(j + R2 * r) * lx + c] = v[r];
    }
    __syncthreads();
    for (int b = t; b < lx * R1; b += nt) {
      const int r = dlx.div(b), c = b - r * lx;
      if (c >= nl) continue;
      const double gz = g2z[z0 + c];
      cplx<double> v[R2];
#pragma unroll
      for (int j = 0; j < R2; ++j) v[j] = buf[(j + R2 * r) * lx + c];
      step2<R>(v, tw, r);
#pragma unroll
      for (int k = 0; k < R2; ++k) {
        const double g2 = g2s[r + R1 * k] + gy + gz;
        const double f = g2 > 0.0 ? vscale / g2 : 0.0;
        sum += f * (v[k].x * v[k].x + v[k].y * v[k].y);
      }
    }
  });
  // fixed order: lanes of a wave, then the waves
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  __shared__ double ws[16];
  if ((t & 63) == 0) ws[t >> 6] = sum;
  __syncthreads();
  if (t == 0) {
    double a = 0.0;
    for (int i = 0; i < nt >> 6; ++i) a += ws[i];
    part[(long)pair * gridDim.x + blockIdx.x] = a;
  }
}

constexpr size_t kLdsMax = 160 * 1024;  // one CU's LDS
// LDS of an x-pass block at most: two blocks share a CU
constexpr size_t kXLds = 72 * 1024;

template <typename T>
int threads_for(int work, bool is_long) {
  return std::min((int)round_up(work, 64), max_threads(is_long, sizeof(T)));
}

template <typename T>
size_t plane_lds(int ny, int nz) { return ((size_t)ny * (nz | 1) + ny + nz) * sizeof(cplx<T>); }
template <typename T>
size_t x_lds(int nx, int lx) { return ((size_t)nx * lx + nx) * sizeof(cplx<T>) + nx * sizeof(T); }

template <typename T, bool LONG>
void allow_lds() {
  const int lim = (int)kLdsMax;
  GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&plane_forward<T, LONG, FieldSums<T>>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  if constexpr (sizeof(T) == 8) {
    GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&plane_forward<T, LONG, RowProducts>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lim));
    GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&x_energy<LONG>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kXLds));
  }
  GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&plane_inverse<T, LONG>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lim));
  GWL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&x_pass<T, LONG>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kXLds));
}

}  // namespace

void plane_prepare_device() {
  allow_lds<float, false>();
  allow_lds<float, true>();
  allow_lds<double, false>();
  allow_lds<double, true>();
}

namespace {

// Launch shapes of a grid's passes.
template <typename T>
struct Plan {
  PlaneGeom<T> p;
  bool ok, lg, lgx;      // covered; long y or z lines; long x lines
  int nt, ntx, lx, nzb;  // threads, kz columns per x block and blocks per slab
  size_t sm, smx;
};

template <typename T>
Plan<T> plan_for(const PoissonGeom<T>& g) {
  Plan<T> q{};
  int r1x, r2x, r1y, r2y, r1z, r2z;
  bool lgy, lgz;
  if (!fft_split(g.nx, r1x, r2x, q.lgx) || !fft_split(g.ny, r1y, r2y, lgy) ||
      !fft_split(g.nz, r1z, r2z, lgz) || plane_lds<T>(g.ny, g.nz) > kLdsMax)
    return q;
  q.ok = true;
  q.lg = lgy || lgz;
  PlaneGeom<T>& p = q.p;
  p.nx = g.nx;
  p.ny = g.ny;
  p.nz = g.nz;
  p.r1y = r1y;
  p.r2y = r2y;
  p.r1z = r1z;
  p.r2z = r2z;
  p.nr = (long)g.nx * g.ny * g.nz;
  p.dy = fast_div(g.ny);
  p.dz = fast_div(g.nz);
  p.d2y = fast_div(r2y);
  p.d1z = fast_div(r1z);
  p.twy = g.twy;
  p.twz = g.twz;
  q.nt = threads_for<T>(std::max(g.nz * std::max(r1y, r2y), g.ny * std::max(r1z, r2z)), q.lg);
  q.sm = plane_lds<T>(g.ny, g.nz);
  q.lx = g.nz;
  while (q.lx > 8 && x_lds<T>(g.nx, q.lx) > kXLds) q.lx = (q.lx + 1) / 2;
  q.nzb = ceil_div(g.nz, q.lx);
  q.ntx = threads_for<T>(q.lx * std::max(r1x, r2x), q.lgx);
  q.smx = x_lds<T>(g.nx, q.lx);
  return q;
}

template <typename T, typename In>
void forward(const Plan<T>& q, const In& in, int npairs, cplx<T>* X, unsigned* xmax,
             hipStream_t st) {
  const dim3 grid(q.p.nx, npairs);
  if (q.lg)
    plane_forward<T, true, In><<<grid, q.nt, q.sm, st>>>(q.p, in, X, xmax);
  else
    plane_forward<T, false, In><<<grid, q.nt, q.sm, st>>>(q.p, in, X, xmax);
}

template <typename T>
void rest(const PoissonGeom<T>& g, const Plan<T>& q, int nf, cplx<T>* X, const PlaneOut<T>& out,
          unsigned* xmax, hipStream_t st) {
  const int npairs = (nf + 1) / 2;
  const dim3 gx(g.ny * q.nzb, npairs), gp(g.nx, npairs);
  if (q.lgx)
    x_pass<T, true><<<gx, q.ntx, q.smx, st>>>(X, g.nx, g.nz, q.lx, q.nzb, q.p.nr, fast_div(q.lx),
                                              g.twx, g.g2x, g.g2y, g.g2z, g.vscale, xmax);
  else
    x_pass<T, false><<<gx, q.ntx, q.smx, st>>>(X, g.nx, g.nz, q.lx, q.nzb, q.p.nr, fast_div(q.lx),
                                               g.twx, g.g2x, g.g2y, g.g2z, g.vscale, xmax);
  if (q.lg)
    plane_inverse<T, true><<<gp, q.nt, q.sm, st>>>(q.p, X, nf, out);
  else
    plane_inverse<T, false><<<gp, q.nt, q.sm, st>>>(q.p, X, nf, out);
  GWL_HIP(hipGetLastError());
}

}  // namespace

template <typename T>
bool poisson_planes(const PoissonGeom<T>& g, const T* rin, long ld_in, long part_stride, int nparts,
                    T* rout, long ld_out, int nf, cplx<T>* scratch, hipStream_t st, unsigned* xmax,
                    int* vexp, int pexp, f16_t* rout16) {
  const Plan<T> q = plan_for<T>(g);
  if (!q.ok) return false;
  unsigned* xm = vexp ? xmax : nullptr;
  forward(q, FieldSums<T>{rin, ld_in, part_stride, nparts, nf}, (nf + 1) / 2, scratch, xm, st);
  rest(g, q, nf, scratch, PlaneOut<T>{rout, vexp ? rout16 : nullptr, ld_out, xmax, vexp, pexp}, xm,
       st);
  return true;
}

bool poisson_products(const PoissonGeom<double>& g, const double* psi, long ld, const int* m,
                      const int* n, double* rout, long ld_out, int nf, cplx<double>* scratch,
                      hipStream_t st) {
  const Plan<double> q = plan_for<double>(g);
  if (!q.ok) return false;
  forward(q, RowProducts{psi, ld, m, n, nf}, (nf + 1) / 2, scratch, (unsigned*)nullptr, st);
  rest(g, q, nf, scratch, PlaneOut<double>{rout, nullptr, ld_out, nullptr, nullptr, 0},
       (unsigned*)nullptr, st);
  return true;
}

int product_energy_blocks(const PoissonGeom<double>& g) {
  const Plan<double> q = plan_for<double>(g);
  return q.ok ? g.ny * q.nzb : 0;
}

void product_energies(const PoissonGeom<double>& g, const double* psi, long ld, const int* m,
                      const int* n, int npairs, double* part, cplx<double>* scratch,
                      hipStream_t st) {
  if (npairs <= 0) return;
  const Plan<double> q = plan_for<double>(g);
  forward(q, RowProducts{psi, ld, m, n, 2 * npairs}, npairs, scratch, (unsigned*)nullptr, st);
  const dim3 gx(g.ny * q.nzb, npairs);
  if (q.lgx)
    x_energy<true><<<gx, q.ntx, q.smx, st>>>(scratch, g.nx, g.nz, q.lx, q.nzb, q.p.nr,
                                             fast_div(q.lx), g.twx, g.g2x, g.g2y, g.g2z, g.vscale,
                                             part);
  else
    x_energy<false><<<gx, q.ntx, q.smx, st>>>(scratch, g.nx, g.nz, q.lx, q.nzb, q.p.nr,
                                              fast_div(q.lx), g.twx, g.g2x, g.g2y, g.g2z, g.vscale,
                                              part);
  GWL_HIP(hipGetLastError());
}

template bool poisson_planes<float>(const PoissonGeom<float>&, const float*, long, long, int, float*,
                                    long, int, cplx<float>*, hipStream_t, unsigned*, int*, int, f16_t*);
template bool poisson_planes<double>(const PoissonGeom<double>&, const double*, long, long, int,
                                     double*, long, int, cplx<double>*, hipStream_t, unsigned*, int*,
                                     int, f16_t*);

}  // namespace gwl
