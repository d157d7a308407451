// FP64 K product with the pair densities as the GEMM operand.
//
//   first   rho_b(r) = sum_vc u_b,vc [phi_v phi_c](r)        M = b, N = r,  K = vc
//   second  y_b,vc   = sum_r  V_b(r) [phi_v phi_c](r)        M = b, N = vc, K = r (split)
//
// (the two halves of K x, Eqs. 2-4).  The (b, v)-row kernels of gemm_mfma.hip
// pad N_v to 64 and N_c to 64 or 128: with 8 + 32 orbitals 15 of 16 of their
// matrix instructions work on padding.  Here the pair index is flat, the
// products phi_v phi_c are formed while the operand is staged into LDS (one
// multiplication per element and M tile, against 2 * 16 MI flop on the matrix
// cores) and only the batch is padded, to 16.  Operands u, y are compact
// [b][N_v N_c]; no row-dot epilogue and a single density per vector.
//
// v_mfma_f64_16x16x4f64 takes 64 cycles, so one wave per column block of 16
// (NJ = 1) or 32 (NJ = 2) against all 16 MI rows of the M tile keeps the
// matrix cores fed from one or two LDS reads per instruction; the K steps are
// double-buffered in LDS with the next step's loads in registers.  Where the
// tiles are too few for the chip (small grids or few pairs) a block's four
// waves take KG = 2 or 4 shares of every K step of a tile 32 or 16 columns
// wide instead of four column blocks, and add their sums through LDS in a
// fixed order.
//
// Bound by the matrix cores once a CU holds two blocks.  Rows and pairs on one
// card: 64 vectors, 32^3, 32 + 128 orbitals 572 and 322 us (53 TFLOP/s), 492 and
// 280 (61); 80 vectors, 24^3, 8 + 32: 211 and 24 us, 279 and 27.  Few points and
// many pairs are the rows' (gwl_ctx::pd): 64 vectors on 640 points, 35 + 248
// orbitals, 84 and 318 us for both.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace gwl {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));

constexpr int NT = 256;

// M tiles: as few as hold the batch with at most 128 rows each, evenly filled.
inline int pd_mt(int nb) { return (nb + 127) / 128; }
inline int pd_mi(int nb) { return (int)((ceil_div(nb, pd_mt(nb)) + 15) / 16); }

// Block to work item: each XCD takes a contiguous run of the items, so that
// neighbours (M tiles of one N tile, tiles of one split) share its L2.
__device__ inline int pd_item(int bid, int total) {
  const int per = (total + 7) / 8;
  const int i = (bid & 7) * per + (bid >> 3);
  return (bid >> 3) < per && i < total ? i : -1;
}
inline int pd_grid(long total) { return (int)(8 * ((total + 7) / 8)); }

// Block tile: 16 MI rows x NB columns, KB deep (at most KMAX): the fewer matrix
// instructions 16 of K take, the deeper the step, so that a barrier and a
// load's latency are spread over enough of them, while two blocks fit a CU (one
// C product of one vector, 24^3, 8 + 32 orbitals: 54.3 -> 50.1 us; 32-deep steps
// gained nothing at 64 or 80 vectors).
constexpr int pd_kb(int mi, int nj, int kg, int kmax) {
  const int mt = 16 * mi, nb = 64 * nj / kg;
  int kb = mi * nj <= 2 ? 64 : 16;
  if (kb > kmax) kb = kmax;
  while (kb > 16 && 16 * (mt * (kb + 2) + (nb + 16) * (kb + 2)) > 80 * 1024) kb /= 2;
  return kb;
}
template <int MI, int NJ, int KG, int KMAX>
struct PdTile {
  static_assert(KG == 1 || NJ == 1, "K shares only with one column block per wave");
  static constexpr int MT = 16 * MI, NB = 64 * NJ / KG;
  static constexpr int WC = 4 / KG;       // waves side by side
  static constexpr int KB = pd_kb(MI, NJ, KG, KMAX);
  // LDS row of an operand stored row by row: the 16 rows times two k of a
  // half-wave's fragment read cover every bank once
  static constexpr int ALD = KB + (MI > 2 ? 1 : 2);
  static constexpr int BLD1 = NB + 16;    // first GEMM: LDS row of the B tile [KB][BLD1]
  // two register stages (the loads of step s + 2 in flight while step s
  // computes and step s + 1 goes to LDS) up to the size of tile whose K step
  // is too short to hide a load; beyond it they would spill
  static constexpr bool DEEP = MI * NJ <= 8;
};

// acc += the wave's share of one K step.  a: row (l & 15) + 16 i, k = 4 ks +
// (l >> 4) of [MT][ALD]; b: element (k, column) at k * brow + column * bcol.
template <typename T, int MI, int NJ, int KG>
__device__ inline void pd_mma(const double* as, const double* bs, int bcol, int brow, int wc,
                              int kg, d4 (&acc)[MI][NJ]) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int k4 = 0; k4 < T::KB / 4 / KG; ++k4) {
    const int kk = 4 * (k4 * KG + kg) + (l >> 4);
    double b[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[j] = bs[kk * brow + (16 * (wc * NJ + j) + (l & 15)) * bcol];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const double a = as[(16 * i + (l & 15)) * T::ALD + kk];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[j], acc[i][j], 0, 0, 0);
    }
  }
}

// Sum of the KG shares into the waves of share 0 (the K loop has ended with a
// barrier; sh is the block's staging memory, 512 MI doubles of it): the
// upper half of the shares hands over to the lower half.
template <int MI, int KG, int WC>
__device__ inline void pd_reduce(double* sh, int wc, int kg, d4 (&acc)[MI][1]) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int half = KG / 2; half > 0; half >>= 1) {
    if (kg >= half && kg < 2 * half) {
      double* o = sh + ((kg - half) * WC + wc) * (MI * 256) + l;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) o[(4 * i + q) * 64] = acc[i][0][q];
    }
    __syncthreads();
    if (kg < half) {
      const double* o = sh + (kg * WC + wc) * (MI * 256) + l;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[i][0][q] += o[(4 * i + q) * 64];
    }
    __syncthreads();
  }
}

template <int MI, int NJ, int KG>
__global__ void __launch_bounds__(NT, 2)
gemm1_pd_kernel(GemmDims d, long nvc, int nb, int mt, const double* __restrict__ psi_v_t,
                const double* __restrict__ psi_c_t, const double* __restrict__ u,
                double* __restrict__ rho) {
  typedef PdTile<MI, NJ, KG, 32> T;  // (deeper ones than N_c would miss the path below)
  constexpr int NB = T::NB, BLD = T::BLD1, KB = T::KB, ALD = T::ALD;
  constexpr int AR = NT / KB, QA = T::MT / AR;  // A rows staged per pass, passes
  constexpr int SB = NB < 64 ? NB : 64;   // columns of a staged row segment
  constexpr int RK = KB * SB / NT;        // consecutive K rows staged by one thread
  constexpr int SA1 = T::MT * ALD, SB1 = KB * BLD;
  __shared__ double sh[2 * (SA1 + SB1)];
  double* const As = sh;
  double* const Bs = sh + 2 * SA1;
  const int item = pd_item(blockIdx.x, mt * (d.nrp / NB));
  if (item < 0) return;
  const int ni = item / mt, mi = item - ni * mt;
  const int t = threadIdx.x, l = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wc = w % T::WC, kg = w / T::WC;
  const int m0 = mi * T::MT, n0 = ni * NB;
  d4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = d4{0, 0, 0, 0};
  // A: element e = t + 256 q of the tile is row e / KB, k = e % KB
  const int ak = t % KB, ar = t / KB;
  // B: column t % SB (+ 64 j), K rows RK (t / SB) + [0, RK)
  const int bc = t % SB, br = KG == 1 ? RK * w : RK * (t / SB);
  // Every load is unconditional (a guarded one made the compiler wait for it
  // before it issued the next): u has room past its last row (gemm_pd_u_size),
  // steps past the end read some other pairs, and the A operand is zeroed
  // there as it is stored.
  const double* const ap = u + (long)(m0 + ar) * nvc + ak;
  const double* const pvb = psi_v_t + n0 + bc;
  const double* const pcb = psi_c_t + n0 + bc;
  auto lstore_a = [&](int buf, const double* a, bool ok) {
#pragma unroll
    for (int q = 0; q < QA; ++q) As[buf * SA1 + (ar + AR * q) * ALD + ak] = ok ? a[q] : 0.0;
  };

  // Whole blocks of KB conduction orbitals: a block's values stay in registers
  // while all occupied orbitals go by, so a K step reads one orbital row
  // besides u (against KB; 396 -> 333 us at 32^3, 32 + 128 orbitals, 64 vectors).
  const int ncf = d.nv > 1 ? d.nc / KB * KB : 0;
  if (ncf > 0) {
    struct Stage {
      double a[QA], v[NJ];
    } x0, x1;
    double cn[RK][NJ], cc[RK][NJ];
    int v = 0, c0 = 0, lv = 0;  // next step to load, occupied orbital of the next to store
    auto gload = [&](Stage& x) {
      const double* p = ap + (long)v * d.nc + c0;
#pragma unroll
      for (int q = 0; q < QA; ++q) x.a[q] = p[AR * q * nvc];
#pragma unroll
      for (int j = 0; j < NJ; ++j) x.v[j] = pvb[(long)v * d.nrp + 64 * j];
      if (v == 0) {
#pragma unroll
        for (int i = 0; i < RK; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) cn[i][j] = pcb[(long)(c0 + br + i) * d.nrp + 64 * j];
      }
      if (++v == d.nv) {
        v = 0;
        c0 += KB;
        if (c0 == ncf) c0 = 0;
      }
    };
    auto lstore = [&](int buf, const Stage& x, bool ok) {
      lstore_a(buf, x.a, ok);
      if (lv == 0) {
#pragma unroll
        for (int i = 0; i < RK; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) cc[i][j] = cn[i][j];
      }
      if (++lv == d.nv) lv = 0;
#pragma unroll
      for (int i = 0; i < RK; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          Bs[buf * SB1 + (br + i) * BLD + bc + 64 * j] = x.v[j] * cc[i][j];
    };
    const int steps = ncf / KB * d.nv;
    gload(x0);
    if constexpr (T::DEEP) gload(x1);
    lstore(0, x0, true);
    __syncthreads();
    for (int s = 0; s < steps; s += 2) {
      gload(x0);
      pd_mma<T, MI, NJ, KG>(As, Bs, 1, BLD, wc, kg, acc);
      lstore(1, T::DEEP ? x1 : x0, s + 1 < steps);
      __syncthreads();
      gload(T::DEEP ? x1 : x0);
      pd_mma<T, MI, NJ, KG>(As + SA1, Bs + SB1, 1, BLD, wc, kg, acc);
      lstore(0, x0, s + 2 < steps);
      __syncthreads();
    }
  }
  // The remaining (fewer than KB) conduction orbitals, or all pairs when there
  // is one occupied orbital: flat over (v, c), a K step may span several v.
  const int tw = d.nc - ncf;
  if (tw > 0) {
    double xa[QA], xv[RK][NJ], xc[RK][NJ];
    const int nflat = d.nv * tw;
    const int dv = KB / tw, dc = KB - dv * tw;  // pair step of KB
    int av = ak / tw, ac = ak - av * tw;        // pair of the thread's A column
    int v = br / tw, c = br - v * tw;           // pair of the thread's first B row
    auto advance = [&](int& vi, int& ci) {
      vi += dv;
      ci += dc;
      const bool wrap = ci >= tw;
      ci -= wrap ? tw : 0;
      vi += wrap;
    };
    auto gload = [&]() {
      const double* p = ap - ak + (long)min(av, d.nv - 1) * d.nc + ncf + ac;
#pragma unroll
      for (int q = 0; q < QA; ++q) xa[q] = p[AR * q * nvc];
      int vi = v, ci = c;
#pragma unroll
      for (int i = 0; i < RK; ++i) {
        const double* pv = pvb + (long)min(vi, d.nv - 1) * d.nrp;
        const double* pc = pcb + (long)(ncf + ci) * d.nrp;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          xv[i][j] = pv[64 * j];
          xc[i][j] = pc[64 * j];
        }
        const bool wrap = ++ci == tw;
        ci = wrap ? 0 : ci;
        vi += wrap;
      }
      advance(av, ac);
      advance(v, c);
    };
    auto lstore = [&](int buf, int k0) {
      lstore_a(buf, xa, k0 + ak < nflat);
#pragma unroll
      for (int i = 0; i < RK; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          Bs[buf * SB1 + (br + i) * BLD + bc + 64 * j] = xv[i][j] * xc[i][j];
    };
    gload();
    lstore(0, 0);
    __syncthreads();
    for (int k0 = 0; k0 < nflat; k0 += KB) {
      const int cur = (k0 / KB) & 1;
      gload();
      pd_mma<T, MI, NJ, KG>(As + cur * SA1, Bs + cur * SB1, 1, BLD, wc, kg, acc);
      lstore(cur ^ 1, k0 + KB);
      __syncthreads();
    }
  }
  if constexpr (KG > 1) {
    pd_reduce<MI, KG, T::WC>(sh, wc, kg, acc);
    if (kg > 0) return;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int b = m0 + 16 * i + (l >> 4) + 4 * q;
      if (b >= nb) continue;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        rho[(long)b * d.nrp + n0 + 16 * (wc * NJ + j) + (l & 15)] = acc[i][j][q];
    }
}

template <int MI, int NJ, int KG>
__global__ void __launch_bounds__(NT, 2)
gemm2_pd_kernel(GemmDims d, long nvc, int nb, int mt, int nt, int splitk, int kchunk,
                const double* __restrict__ psi_v_t, const double* __restrict__ psi_c_t,
                const double* __restrict__ vpot, double* __restrict__ ypart) {
  typedef PdTile<MI, NJ, KG, 64> T;
  constexpr int NB = T::NB, MT = T::MT, KB = T::KB, ALD = T::ALD;
  // 4 grid points of a row per thread and pass (A), CW of them (B)
  constexpr int AT = KB / 4, AR = NT / AT, QA = (MT + AR - 1) / AR;
  constexpr int CW = NB * KB >= 4 * NT ? 4 : NB * KB / NT;
  constexpr int BT = KB / CW, BR = NT / BT, QB = NB / BR;
  static_assert(CW >= 1 && QB * BR == NB, "B staging");
  constexpr int SA1 = MT * ALD, SB1 = NB * ALD;
  __shared__ double sh[2 * (SA1 + SB1)];
  double* const As = sh;
  double* const Bs = sh + 2 * SA1;
  const int item = pd_item(blockIdx.x, mt * nt * splitk);
  if (item < 0) return;
  const int si = item / (mt * nt), mi = item - si * (mt * nt);
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const int wc = w % T::WC, kg = w / T::WC;
  const int m0 = (mi % mt) * MT, n0 = (mi / mt) * NB;
  const int kb = si * kchunk, ke = min(d.nrp, kb + kchunk);
  d4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = d4{0, 0, 0, 0};
  const int row = t / AT, col = 4 * (t % AT);
  const int brow = t / BT, bcol = CW * (t % BT);
  const double *pv[QB], *pc[QB];
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    const long n = min((long)n0 + brow + BR * j, nvc - 1);  // (columns past the end: dropped)
    const int v = (int)(n / d.nc), c = (int)(n - (long)v * d.nc);
    pv[j] = psi_v_t + (long)v * d.nrp + bcol;
    pc[j] = psi_c_t + (long)c * d.nrp + bcol;
  }
  const double* pa[QA];
#pragma unroll
  for (int q = 0; q < QA; ++q)
    pa[q] = vpot + (long)min(m0 + row + AR * q, nb - 1) * d.nrp + col;
  struct Stage {  // (loads unconditional: as in the first GEMM)
    d2v a[QA][2];
    double v[QB][CW], c[QB][CW];
  } x0, x1;
  auto gload = [&](Stage& x, int k) {
    const int k0 = min(k, ke - KB);
#pragma unroll
    for (int q = 0; q < QA; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h) x.a[q][h] = *reinterpret_cast<const d2v*>(pa[q] + k0 + 2 * h);
#pragma unroll
    for (int j = 0; j < QB; ++j) {
      if constexpr (CW > 1) {
#pragma unroll
        for (int h = 0; h < CW; h += 2) {
          const d2v a = *reinterpret_cast<const d2v*>(pv[j] + k0 + h);
          const d2v b = *reinterpret_cast<const d2v*>(pc[j] + k0 + h);
          x.v[j][h] = a[0];
          x.v[j][h + 1] = a[1];
          x.c[j][h] = b[0];
          x.c[j][h + 1] = b[1];
        }
      } else {
        x.v[j][0] = pv[j][k0];
        x.c[j][0] = pc[j][k0];
      }
    }
  };
  auto lstore = [&](int buf, const Stage& x) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int m = row + AR * q;
      if (m < MT)
#pragma unroll
        for (int e = 0; e < 4; ++e) As[buf * SA1 + m * ALD + col + e] = x.a[q][e >> 1][e & 1];
    }
#pragma unroll
    for (int j = 0; j < QB; ++j)
#pragma unroll
      for (int e = 0; e < CW; ++e)
        Bs[buf * SB1 + (brow + BR * j) * ALD + bcol + e] = x.v[j][e] * x.c[j][e];
  };
  if (kb < ke) {  // (N_rp and kchunk are multiples of 128)
    gload(x0, kb);
    if constexpr (T::DEEP) gload(x1, kb + KB);
    lstore(0, x0);
  }
  __syncthreads();
  for (int k0 = kb; k0 < ke; k0 += 2 * KB) {
    gload(x0, T::DEEP ? k0 + 2 * KB : k0 + KB);
    pd_mma<T, MI, NJ, KG>(As, Bs, ALD, 1, wc, kg, acc);
    lstore(1, T::DEEP ? x1 : x0);
    __syncthreads();
    gload(T::DEEP ? x1 : x0, T::DEEP ? k0 + 3 * KB : k0 + 2 * KB);
    pd_mma<T, MI, NJ, KG>(As + SA1, Bs + SB1, ALD, 1, wc, kg, acc);
    lstore(0, x0);
    __syncthreads();
  }
  if constexpr (KG > 1) {
    pd_reduce<MI, KG, T::WC>(sh, wc, kg, acc);
    if (kg > 0) return;
  }
  double* out = ypart + (long)si * nb * nvc;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int b = m0 + 16 * i + (l >> 4) + 4 * q;
      if (b >= nb) continue;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const long n = (long)n0 + 16 * (wc * NJ + j) + (l & 15);
        if (n < nvc) out[(long)b * nvc + n] = acc[i][j][q];
      }
    }
}

}  // namespace

size_t gemm_pd_u_size(int nb, long nvc) {
  return (size_t)(nb + 16 * pd_mt(nb)) * nvc;  // whole M tiles
}

namespace {

// Blocks of the second GEMM aimed at: two per CU.  K shares inside the block
// while 32 splits of the grid sum cannot give them.
int pd2_shares(const GemmDims& d, int nb) {
  const long nvc = (long)d.nv * d.nc, smax = std::min<long>(32, std::max(1, d.nrp / 128));
  for (int kg : {1, 2})
    if ((long)pd_mt(nb) * ceil_div(nvc, 64 / kg) * smax >= 384) return kg;
  return 4;
}

// Column blocks per wave and K shares of a launch: PdTile's NJ and KG.
struct PdShape {
  int nj, kg;
  int columns() const { return 64 * nj / kg; }
};
PdShape pd1_shape(const GemmDims& d, int nb) {
  const long blocks = (long)pd_mt(nb) * (d.nrp / 64);
  if (blocks >= 1024) return {2, 1};
  return {1, blocks >= 384 ? 1 : blocks >= 192 ? 2 : 4};
}
// (one column block per wave: two were 5 to 30 % slower from 33 vectors on, 8 to
// 12 % faster up to 16; 40 vectors, 24^3, 300 + 300 orbitals: 2,351 and 2,939 us)
PdShape pd2_shape(const GemmDims& d, int nb) { return {1, pd2_shares(d, nb)}; }

// Time (us) of `blocks` blocks of K steps of kb on 256 CUs, two to a CU: the CU
// is busy with both blocks' matrix instructions (`mma` each, per wave), or a block
// waits for its own chain of barrier and loads, `lat` a step.
double pd_us(long blocks, const PdShape& s, int mi, int kb, double steps, double mma, double lat) {
  const double per_cu = ceil_div(blocks, 256), both = std::min(per_cu, 2.0);
  const double m = mma * mi * s.nj * (kb / 4) / s.kg;
  return per_cu / both * steps * std::max(both * m, m + lat);
}

}  // namespace

// Times of both GEMMs, fitted like those of the row GEMMs (9 and 11 % rms).  The
// first has no split of K: its chain of N_v N_c / KB steps is what few columns
// and many pairs wait for (640 points, 30 + 120 orbitals, 64 vectors: 123 us, the
// row GEMM 30).  From 2^18 points on, rows 2 MB apart, the second is 10 to 40 %
// slower than its blocks say.
double gemm1_pd_us(const GemmDims& d, int nb) {
  const PdShape s = pd1_shape(d, nb);
  const int mi = pd_mi(nb), kb = pd_kb(mi, s.nj, s.kg, 32);
  const double mma = s.nj == 2 ? 0.034 : s.kg == 1 ? 0.038 : s.kg == 2 ? 0.044 : 0.0545;
  const long blocks = (long)pd_mt(nb) * (d.nrp / s.columns());
  const int ncf = d.nv > 1 ? d.nc / kb * kb : 0;
  return 5.0 + pd_us(blocks, s, mi, kb, round_up((long)ncf / kb * d.nv, 2), mma, 0.32) +
         pd_us(blocks, s, mi, kb, ceil_div((long)d.nv * (d.nc - ncf), kb), mma, 0.49);
}
double gemm2_pd_us(const GemmDims& d, int nb) {
  const int splitk = gemm2_pd_split(d, nb);
  const PdShape s = pd2_shape(d, nb);
  const int mi = pd_mi(nb), kb = pd_kb(mi, s.nj, s.kg, 64);
  const long blocks = (long)pd_mt(nb) * ceil_div((long)d.nv * d.nc, s.columns()) * splitk;
  return (6.0 + pd_us(blocks, s, mi, kb, split_chunk(d.nrp, splitk, kUnitPd) / kb, 0.035,
                      0.32 + 0.16 * kb / 16)) *
         (d.nrp >= 1 << 18 ? 1.1 : 1.0);
}

int gemm2_pd_split(const GemmDims& d, int nb) {
  const long nvc = (long)d.nv * d.nc;
  const long tiles = (long)pd_mt(nb) * ceil_div(nvc, 64 / pd2_shares(d, nb));
  const long most = std::max<long>(1, std::min<long>({512 / tiles, 32, d.nrp / 128}));
  return full_splits(d.nrp, (int)most, kUnitPd);
}

#define GWL_PD_MI(NJV, KGV)                               \
  switch (pd_mi(nb)) {                                    \
    case 1: GWL_PD(1, NJV, KGV); break;                   \
    case 2: GWL_PD(2, NJV, KGV); break;                   \
    case 3: GWL_PD(3, NJV, KGV); break;                   \
    case 4: GWL_PD(4, NJV, KGV); break;                   \
    case 5: GWL_PD(5, NJV, KGV); break;                   \
    case 6: GWL_PD(6, NJV, KGV); break;                   \
    case 7: GWL_PD(7, NJV, KGV); break;                   \
    default: GWL_PD(8, NJV, KGV); break;                  \
  }

void gemm1_pd(const GemmDims& d, int nb, const double* psi_v_t, const double* psi_c_t,
              const double* u, double* rho, hipStream_t st) {
  if (nb <= 0) return;
  const long nvc = (long)d.nv * d.nc;
  const int mt = pd_mt(nb);
#define GWL_PD(MIV, NJV, KGV)                                                              \
  gemm1_pd_kernel<MIV, NJV, KGV>                                                           \
      <<<pd_grid((long)mt * (d.nrp / (64 * NJV / KGV))), NT, 0, st>>>(            \
          d, nvc, nb, mt, psi_v_t, psi_c_t, u, rho)
  const PdShape s = pd1_shape(d, nb);
  if (s.nj == 2) {
    GWL_PD_MI(2, 1)
  } else if (s.kg == 1) {
    GWL_PD_MI(1, 1)
  } else if (s.kg == 2) {
    GWL_PD_MI(1, 2)
  } else {
    GWL_PD_MI(1, 4)
  }
#undef GWL_PD
  GWL_HIP(hipGetLastError());
}

void gemm2_pd(const GemmDims& d, int nb, int splitk, const double* psi_v_t,
              const double* psi_c_t, const double* vpot, double* ypart, hipStream_t st) {
  if (nb <= 0) return;
  const long nvc = (long)d.nv * d.nc;
  const int mt = pd_mt(nb);
  const int kchunk = split_chunk(d.nrp, splitk, kUnitPd);
#define GWL_PD(MIV, NJV, KGV)                                                              \
  do {                                                                                     \
    const int nt = ceil_div(nvc, (64 * NJV / KGV));                               \
    gemm2_pd_kernel<MIV, NJV, KGV><<<pd_grid((long)mt * nt * splitk), NT, 0, st>>>(        \
        d, nvc, nb, mt, nt, splitk, kchunk, psi_v_t, psi_c_t, vpot, ypart);                \
  } while (0)
  const PdShape s = pd2_shape(d, nb);
  if (s.kg == 1) {
    GWL_PD_MI(1, 1)
  } else if (s.kg == 2) {
    GWL_PD_MI(1, 2)
  } else {
    GWL_PD_MI(1, 4)
  }
#undef GWL_PD
  GWL_HIP(hipGetLastError());
}

}  // namespace gwl
