// Continued fraction (Haydock, Eq. 14) and assembly of Sigma(w, n) (Eq. 12):
//   R(zeta) = ||P||^2 / (zeta - a_0 - b_1^2 / (zeta - a_1 - ...)),
//   Sigma(w, n) = [R(-eta_n z_n) - R(0)] / z_n,  z_n = w - e_n - i eta_n delta.
// Tamm-Dancoff (B = 0 in the Casida matrix, Lanczos on A from (nm|vc)):
//   Sigma(w, n) = -eta_n R_A(-eta_n z_n).
// FP64 complex.  One thread per (pair, frequency); the pair's coefficients are
// staged in LDS.  Both evaluation points are off the spectrum (Im = +delta, or
// 0 below the positive spectrum of D), so the backward recurrence never
// divides by zero.
#include "common.h"
#include "kernels.h"

namespace gwl {
namespace {

constexpr int CF_MAXL = 4000;

// Bound by the chain of dependent FP64 divisions: the LDS holds the pair's
// ld coefficients, not the longest recurrence's 4,000 (64 KB: two blocks per
// CU), so that eight blocks hide each other's chains, and the real fraction
// R(0) is wave 0's affair while the other waves are under way (640 pairs x 2,000
// frequencies, L up to 200: 244 -> 173 us).
__global__ void __launch_bounds__(256)
cfrac_kernel(const double* __restrict__ ca, const double* __restrict__ cb,
             const int* __restrict__ lens, const double* __restrict__ norm2, int ld,
             const double* __restrict__ e_n, const double* __restrict__ eta_n,
             const double* __restrict__ omega, int nomega, double delta, int tda,
             double* __restrict__ sig) {
  extern __shared__ double coef[];
  __shared__ double r0_sh;
  double* const sa = coef;
  double* const sb2 = coef + ld;
  const int p = blockIdx.y;
  const int L = lens[p];
  const double n2 = norm2[p];
  for (int k = threadIdx.x; k < L; k += blockDim.x) {
    sa[k] = ca[(long)p * ld + k];
    const double b = (k + 1 < L) ? cb[(long)p * ld + k] : 0.0;  // b_{k+1}
    sb2[k] = b * b;
  }
  __syncthreads();
  const bool run = L > 0 && n2 > 0.0;
  if (threadIdx.x < 64) {
    double r0 = 0.0;
    if (run && !tda) {
      double t = -sa[L - 1];
      for (int k = L - 2; k >= 0; --k) t = -sa[k] - sb2[k] / t;
      r0 = n2 / t;
    }
    if (threadIdx.x == 0) r0_sh = r0;
  }
  const double en = e_n[p], eta = eta_n[p];
  const int w = blockIdx.x * blockDim.x + threadIdx.x;  // (one frequency per thread)
  const double om = omega[w < nomega ? w : 0];
  const double zr = om - en, zi = -eta * delta;
  double rr = 0.0, ri = 0.0;
  if (run) {
    // zeta = -eta z
    const double xr = -eta * zr, xi = -eta * zi;
    double tr = xr - sa[L - 1], ti = xi;
    for (int k = L - 2; k >= 0; --k) {
      const double inv = sb2[k] / (tr * tr + ti * ti);
      // t = zeta - a_k - b^2 / t ;  b^2 / t = b^2 conj(t) / |t|^2
      tr = xr - sa[k] - inv * tr;
      ti = xi + inv * ti;
    }
    // R(zeta) = n2 / t
    const double d = 1.0 / (tr * tr + ti * ti);
    rr = n2 * tr * d;
    ri = -n2 * ti * d;
  }
  __syncthreads();
  if (w >= nomega) return;
  double sr = 0.0, si = 0.0;
  if (run) {
    if (tda) {
      sr = -eta * rr;
      si = -eta * ri;
    } else {
      // (R - r0) / z
      const double nr = rr - r0_sh, ni = ri;
      const double dz = 1.0 / (zr * zr + zi * zi);
      sr = (nr * zr + ni * zi) * dz;
      si = (ni * zr - nr * zi) * dz;
    }
  }
  double2* const o = reinterpret_cast<double2*>(sig) + (long)p * nomega + w;
  *o = double2{sr * kHartreeEv, si * kHartreeEv};
}

// ---------------------------------------------------------------- interval check
// Number of eigenvalues of the L x L tridiagonal T below tau: the negative
// pivots of T - tau I = L D L^T (Sylvester's law of inertia).  A zero pivot
// is replaced by a tiny negative one, as in bisection codes.
__device__ inline int sturm_below(const double* __restrict__ a, const double* __restrict__ b,
                                  int L, double tau) {
  int cnt = 0;
  double d = 1.0;
  for (int i = 0; i < L; ++i) {
    d = (a[i] - tau) - (i > 0 ? b[i - 1] * b[i - 1] / d : 0.0);
    if (fabs(d) < 1e-280) d = -1e-280;
    cnt += d < 0.0;
  }
  return cnt;
}

__global__ void __launch_bounds__(256)
interval_check_kernel(int npairs, const double* __restrict__ ca, const double* __restrict__ cb,
                      const int* __restrict__ lens, int ld, double t_lo, double t_hi,
                      int* __restrict__ bad) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npairs) return;
  const int L = lens[p];
  const double* a = ca + (long)p * ld;
  const double* b = cb + (long)p * ld;
  int out = 0;
  if (L > 0) out = sturm_below(a, b, L, t_lo) > 0 || sturm_below(a, b, L, t_hi) < L;
  bad[p] = out;
}

// ---------------------------------------------------------------- quadrature
// Lanczos on C + Gauss quadrature: the eigenvalues theta_k of each pair's
// tridiagonal T and the first components u_k(0) of its eigenvectors, by the
// implicit QL iteration with shifts (Bowdler, Martin, Reinsch and Wilkinson)
// applying each plane rotation to the first row of the eigenvector matrix
// only (Golub and Welsch).  One thread per pair: a serial chain of rotations
// over d, e and z (FP64), which live in LDS ([k][thread], stride = blockDim.x)
// where those of all pairs fit there (quad_sigma), and in the pair's rows of the
// scratch arrays otherwise (80 pairs, L = 30: 1,257 us in the
// scratch rows with 64 lanes per wave, 617 us as it is).  On return qd = theta, qz = ||P||^2 u(0)^2.
// status[p] = 1 if an eigenvalue needed more than 60 sweeps.
template <typename T>
struct Strided {
  T* p;
  int s;
  __device__ T& operator[](int i) const { return p[(long)i * s]; }
};
template <bool LDS>
__global__ void quad_eig_kernel(int npairs, const double* __restrict__ ca,
                                const double* __restrict__ cb, const int* __restrict__ lens,
                                const double* __restrict__ norm2, int ld, double* __restrict__ qd,
                                double* __restrict__ qe, double* __restrict__ qz,
                                int* __restrict__ status) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npairs) return;
  const int n = lens[p];
  extern __shared__ double tri[];
  const int s = LDS ? (int)blockDim.x : 1;
  Strided<double> d, e, z;
  if constexpr (LDS) {
    d = {tri + threadIdx.x, s};
    e = {d.p + (long)ld * s, s};
    z = {e.p + (long)ld * s, s};
  } else {
    d = {qd + (long)p * ld, s};
    e = {qe + (long)p * ld, s};
    z = {qz + (long)p * ld, s};
  }
  for (int i = 0; i < n; ++i) {
    d[i] = ca[(long)p * ld + i];
    e[i] = (i + 1 < n) ? cb[(long)p * ld + i] : 0.0;  // e[i] couples i and i + 1
    z[i] = (i == 0) ? 1.0 : 0.0;
  }
  int bad = 0;
  for (int l = 0; l < n; ++l) {
    int sweeps = 0;
    while (true) {
      int m = l;
      for (; m < n - 1; ++m) {
        const double dd = fabs(d[m]) + fabs(d[m + 1]);
        if (fabs(e[m]) <= 2.220446049250313e-16 * dd) break;  // below one ulp of the diagonal
      }
      if (m == l) break;
      if (++sweeps > 60) {
        bad = 1;
        break;
      }
      // shift from the leading 2 x 2 block
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = hypot(g, 1.0);
      g = d[m] - d[l] + e[l] / (g + (g >= 0.0 ? r : -r));
      double sn = 1.0, c = 1.0, pp = 0.0;
      int i = m - 1;
      bool underflow = false;
      for (; i >= l; --i) {
        const double f = sn * e[i], b = c * e[i];
        r = hypot(f, g);
        e[i + 1] = r;
        if (r == 0.0) {
          d[i + 1] -= pp;
          e[m] = 0.0;
          underflow = true;
          break;
        }
        sn = f / r;
        c = g / r;
        g = d[i + 1] - pp;
        r = (d[i] - g) * sn + 2.0 * c * b;
        pp = sn * r;
        d[i + 1] = g + pp;
        g = c * r - b;
        const double zf = z[i + 1];
        z[i + 1] = sn * z[i] + c * zf;
        z[i] = c * z[i] - sn * zf;
      }
      if (underflow) continue;
      d[l] -= pp;
      e[l] = g;
      e[m] = 0.0;
    }
  }
  const double n2 = norm2[p];
  for (int i = 0; i < n; ++i) {
    const double w = n2 * z[i] * z[i];
    qz[(long)p * ld + i] = w;
    if constexpr (LDS) qd[(long)p * ld + i] = d[i];
  }
  status[p] = bad;
}

// Sigma(w, n) = sum_k w_k [1/sqrt(theta_k) - 1/(sqrt(theta_k) + eta z)] / z.
__global__ void __launch_bounds__(256)
quad_sigma_kernel(const double* __restrict__ qd, const double* __restrict__ qz,
                  const int* __restrict__ lens, int ld, const double* __restrict__ e_n,
                  const double* __restrict__ eta_n, const double* __restrict__ omega, int nomega,
                  double delta, double* __restrict__ sig) {
  extern __shared__ double coef[];  // (as many as ld: see cfrac_kernel)
  double* const so = coef;
  double* const sw = coef + ld;
  const int p = blockIdx.y;
  const int L = lens[p];
  for (int k = threadIdx.x; k < L; k += blockDim.x) {
    so[k] = sqrt(fmax(qd[(long)p * ld + k], 0.0));
    sw[k] = qz[(long)p * ld + k];
  }
  __syncthreads();
  const double en = e_n[p], eta = eta_n[p];
  for (int w = blockIdx.x * blockDim.x + threadIdx.x; w < nomega; w += gridDim.x * blockDim.x) {
    const double zr = omega[w] - en, zi = -eta * delta;
    double ar = 0.0, ai = 0.0;  // sum_k w_k [1/O_k - 1/(O_k + eta z)]
    for (int k = 0; k < L; ++k) {
      const double o = so[k];
      if (o <= 0.0 || sw[k] == 0.0) continue;
      const double dr = o + eta * zr, di = eta * zi;
      const double inv = 1.0 / (dr * dr + di * di);
      ar += sw[k] * (1.0 / o - dr * inv);
      ai += sw[k] * (di * inv);
    }
    const double dz = 1.0 / (zr * zr + zi * zi);
    const double sr = (ar * zr + ai * zi) * dz;
    const double si = (ai * zr - ar * zi) * dz;
    sig[((long)p * nomega + w) * 2] = sr * kHartreeEv;
    sig[((long)p * nomega + w) * 2 + 1] = si * kHartreeEv;
  }
}

__global__ void sum_groups_kernel(const double* __restrict__ sig, int per, int nomega,
                                  double* __restrict__ out) {
  const int q = blockIdx.y;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < 2 * nomega; e += gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int i = 0; i < per; ++i) s += sig[((long)(q * per + i) * nomega) * 2 + e];
    out[(long)q * nomega * 2 + e] = s;
  }
}

// out[e] = (sum_n sig[2n][e] - sig[2n+1][e]) / 4, n in order: the
// polarisation identity over runs from P_nm + P_nm' (even pairs) and
// P_nm - P_nm' (odd pairs)
__global__ void sum_polar_kernel(const double* __restrict__ sig, int nn, int nomega,
                                 double* __restrict__ out) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < 2 * nomega; e += gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int n = 0; n < nn; ++n)
      s += sig[((long)(2 * n) * nomega) * 2 + e] - sig[((long)(2 * n + 1) * nomega) * 2 + e];
    out[e] = 0.25 * s;
  }
}

}  // namespace

void cfrac_sigma(int npairs, const double* coef_a, const double* coef_b, const int* lens,
                 const double* norm2, int ld, const double* e_n, const double* eta_n,
                 const double* omega_ha, int nomega, double delta_ha, int tda, double* sig,
                 hipStream_t st) {
  if (npairs <= 0 || nomega <= 0) return;
  GWL_CHECK(ld <= CF_MAXL, GWL_EINVAL, "Lanczos length exceeds 4000");
  dim3 grid(ceil_div(nomega, 256), npairs);
  cfrac_kernel<<<grid, 256, 2 * sizeof(double) * ld, st>>>(coef_a, coef_b, lens, norm2, ld, e_n, eta_n, omega_ha,
                                     nomega, delta_ha, tda, sig);
  GWL_HIP(hipGetLastError());
}

void quad_sigma(int npairs, const double* coef_a, const double* coef_b, const int* lens,
                const double* norm2, int ld, const double* e_n, const double* eta_n,
                const double* omega_ha, int nomega, double delta_ha, double* qd, double* qe,
                double* qz, int* status, double* sig, hipStream_t st) {
  if (npairs <= 0 || nomega <= 0) return;
  GWL_CHECK(ld <= CF_MAXL, GWL_EINVAL, "Lanczos length exceeds 4000");
  // In LDS where every block is resident at once: blocks that wait for others to
  // end cost more than LDS saves (20,000 pairs of 600: 2.58 s in ten rounds, 0.67 s
  // in the scratch rows; of 200: 112 and 72 ms; 6,400 of 200, all resident, 53 and
  // 57 ms).  Threads per block: as few as give no more than a wave per SIMD (lanes
  // of a wave wait for the longest of their sweeps), else as many as fit.
  auto lds_of = [&](int nt) { return (size_t)nt * 3 * ld * sizeof(double); };
  int nt = 0;
  for (int t = 1; t <= 64 && lds_of(t) <= 65536; t *= 2) {
    const long blocks = ceil_div(npairs, t);
    const long per_cu = std::min<long>(32, 160 * 1024 / round_up(lds_of(t), 1280));
    if (blocks > 256 * per_cu) continue;
    nt = t;
    if (blocks <= 1024) break;
  }
  const size_t lds = lds_of(nt);
  if (nt > 0)
    quad_eig_kernel<true><<<ceil_div(npairs, nt), nt, lds, st>>>(npairs, coef_a, coef_b, lens,
                                                                 norm2, ld, qd, qe, qz, status);
  else
    quad_eig_kernel<false><<<ceil_div(npairs, 64), 64, 0, st>>>(npairs, coef_a, coef_b, lens, norm2,
                                                                ld, qd, qe, qz, status);
  GWL_HIP(hipGetLastError());
  dim3 grid(ceil_div(nomega, 256), npairs);
  quad_sigma_kernel<<<grid, 256, 2 * sizeof(double) * ld, st>>>(qd, qz, lens, ld, e_n, eta_n, omega_ha, nomega,
                                          delta_ha, sig);
  GWL_HIP(hipGetLastError());
}

void sum_groups(const double* sig, int ngroups, int per, int nomega, double* out,
                hipStream_t st) {
  if (ngroups <= 0) return;
  dim3 grid(ceil_div(2 * nomega, 256), ngroups);
  sum_groups_kernel<<<grid, 256, 0, st>>>(sig, per, nomega, out);
  GWL_HIP(hipGetLastError());
}

void sum_polar(const double* sig, int nn, int nomega, double* out, hipStream_t st) {
  if (nn <= 0 || nomega <= 0) return;
  sum_polar_kernel<<<ceil_div(2 * nomega, 256), 256, 0, st>>>(sig, nn, nomega, out);
  GWL_HIP(hipGetLastError());
}

void lz_interval_check(int npairs, const double* coef_a, const double* coef_b, const int* lens,
                       int ld, double t_lo, double t_hi, int* bad, hipStream_t st) {
  if (npairs <= 0) return;
  interval_check_kernel<<<(npairs + 255) / 256, 256, 0, st>>>(npairs, coef_a, coef_b, lens, ld,
                                                              t_lo, t_hi, bad);
  GWL_HIP(hipGetLastError());
}

}  // namespace gwl
