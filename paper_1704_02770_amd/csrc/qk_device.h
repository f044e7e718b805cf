// Device-side helpers shared by the HIP kernels of libqkrylov: complex
// vector types, ranking in the sorted basis, the model rows of Eq. (1),
// the XCD-aware tile walk and deterministic block reductions.
#pragma once

#include "qk_internal.h"

namespace qk {

template <typename T> struct Cx;
template <> struct Cx<double> { using V = double2; };
template <> struct Cx<float> { using V = float2; };

// ------------------------------------------------------------------ ranking
__device__ __forceinline__ int popc(uint32_t s) { return __popc(s); }
__device__ __forceinline__ int popc(uint64_t s) { return __popcll(s); }
__device__ __forceinline__ int ctz(uint32_t s) { return __builtin_ctz(s); }
__device__ __forceinline__ int ctz(uint64_t s) { return __builtin_ctzll(s); }

// Position of a state in the sorted basis: with set bits at p_1 < ... < p_N,
// the number of sector states below it is sum_k C(p_k, k) (the counting that
// the sorted order of Sec. 2 implies; the paper finds it by binary lookup).
template <typename S>
__device__ __forceinline__ uint32_t cns_rank(S s, const uint32_t* tab) {
  constexpr int K = StateT<S>::kStride;
  uint32_t r = 0;
  int k = 1;
  while (s) {
    const int p = ctz(s);
    r += tab[p * K + k];
    ++k;
    s &= s - (S)1;
  }
  return r;
}

// The r-th state of the sorted basis (Algorithm 3's first_int()).
template <typename S>
__device__ __forceinline__ S cns_unrank(uint32_t r, int L, int N, const uint32_t* tab) {
  constexpr int K = StateT<S>::kStride;
  S s = 0;
  int k = N;
  for (int p = L - 1; p >= 0 && k > 0; --p) {
    const uint32_t c = tab[p * K + k];
    if (r >= c) {
      s |= (S)1 << p;
      r -= c;
      --k;
    }
  }
  return s;
}

// Next larger integer with the same popcount (Algorithm 2).  The paper's
// exact division of two powers of two is a right shift by ctz(v).
template <typename S>
__device__ __forceinline__ S next_perm(S v) {
  const S t = (v | (v - (S)1)) + (S)1;
  return t | ((((t & ((S)0 - t)) >> ctz(v)) >> 1) - (S)1);
}

// ------------------------------------------------------------- model rows
template <typename S>
__device__ __forceinline__ int anti_bonds(S s, const ModelArgs& a) {
  const S mask = (S)a.lmask;
  if (a.pbc) {
    const S rot = ((s >> 1) | (s << (a.L - 1))) & mask;
    return popc((S)((s ^ rot) & mask));
  }
  return popc((S)((s ^ (s >> 1)) & (mask >> 1)));
}

// Diagonal of Eq. (1): jz/4 * (aligned - anti-aligned bonds) + sum_i h_i (bit_i - 1/2).
template <typename S>
__device__ __forceinline__ double diag_value(S s, const ModelArgs& a, const double* f, double hhalf) {
  const int nb = a.pbc ? a.L : a.L - 1;
  double d = 0.25 * a.jz * (double)(nb - 2 * anti_bonds(s, a)) - hhalf;
  S t = s;
  while (t) {
    d += f[ctz(t)];
    t &= t - (S)1;
  }
  return d;
}

// Calls f(column) for every bond whose bits differ.  A particle hopping
// p -> p+1 raises the rank by C(p, #set bits below p); p+1 -> p lowers it by
// the same amount.  The ring bond (L-1, 0) renumbers every particle and is
// ranked in full.
template <typename S, class F>
__device__ __forceinline__ void for_each_hop(S s, uint32_t r, const ModelArgs& a, const uint32_t* tab, F&& f) {
  constexpr int K = StateT<S>::kStride;
  int pc = 0;
  for (int p = 0; p < a.L - 1; ++p) {
    const uint32_t b0 = (uint32_t)(s >> p) & 1u;
    const uint32_t b1 = (uint32_t)(s >> (p + 1)) & 1u;
    if (b0 != b1) {
      const uint32_t c = tab[p * K + pc];
      f(b0 ? r + c : r - c);
    }
    pc += (int)b0;
  }
  if (a.pbc) {
    const uint32_t b0 = (uint32_t)s & 1u, b1 = (uint32_t)(s >> (a.L - 1)) & 1u;
    if (b0 != b1) f(cns_rank<S>(s ^ ((S)1 | ((S)1 << (a.L - 1))), tab));
  }
}

// Per-block LDS copies of the small tables every row kernel needs.
template <typename S>
struct RowShared {
  uint32_t tab[StateT<S>::kStride * StateT<S>::kStride];
  double fld[kFldCap];
  double hhalf[QK_MAX_BATCH];
};

template <typename S>
__device__ __forceinline__ void load_row_shared(RowShared<S>& sh, const ModelArgs& a, const uint32_t* gtab,
                                                const double* gfields) {
  constexpr int K = StateT<S>::kStride;
  for (int i = threadIdx.x; i < K * K; i += blockDim.x) sh.tab[i] = gtab[i];
  for (int i = threadIdx.x; i < a.B * a.L; i += blockDim.x) sh.fld[i] = gfields[i];
  __syncthreads();
  for (int b = threadIdx.x; b < a.B; b += blockDim.x) {
    double t = 0.0;
    for (int i = 0; i < a.L; ++i) t += sh.fld[b * a.L + i];
    sh.hhalf[b] = 0.5 * t;
  }
  __syncthreads();
}

template <typename S>
struct HamView {
  const S* states;
  const uint32_t* rowptr;
  const uint32_t* cols;
  const double* diag;
  uint32_t D;
};

// (H x)[r, b] and x[r, b].
template <typename T, bool CSR, typename S>
__device__ __forceinline__ typename Cx<T>::V h_row(uint32_t r, int b, const ModelArgs& a, const RowShared<S>& sh,
                                                   const HamView<S>& hv, const typename Cx<T>::V* __restrict__ x,
                                                   typename Cx<T>::V& xr) {
  using V = typename Cx<T>::V;
  const int B = a.B;
  xr = x[(size_t)r * B + b];
  const T g = (T)a.half_jxy;
  V acc;
  if (CSR) {
    const T d = (T)hv.diag[(size_t)r * B + b];
    acc.x = d * xr.x;
    acc.y = d * xr.y;
    V hs = {0, 0};
    for (uint32_t k = hv.rowptr[r]; k < hv.rowptr[r + 1]; ++k) {
      const V xc = x[(size_t)hv.cols[k] * B + b];
      hs.x += xc.x;
      hs.y += xc.y;
    }
    acc.x += g * hs.x;
    acc.y += g * hs.y;
  } else {
    const S s = hv.states[r];
    const T d = (T)diag_value<S>(s, a, sh.fld + b * a.L, sh.hhalf[b]);
    acc.x = d * xr.x;
    acc.y = d * xr.y;
    V hs = {0, 0};
    for_each_hop<S>(s, r, a, sh.tab, [&](uint32_t c) {
      const V xc = x[(size_t)c * B + b];
      hs.x += xc.x;
      hs.y += xc.y;
    });
    acc.x += g * hs.x;
    acc.y += g * hs.y;
  }
  return acc;
}

// The block index and block count a kernel body works with.
struct VGrid {
  uint32_t id, n;
};
__device__ __forceinline__ VGrid hw_grid() { return VGrid{blockIdx.x, gridDim.x}; }

// A run of consecutive virtual blocks v0 .. v1-1 of a grid of n, taken by one
// work-group one after another: what a block's results depend on (tables,
// the scalars reduced from the previous pass) is set up once for the run,
// then each virtual block does its own rows and writes its own partial sums.
// Every launch gives a work-group one.  The loop over them stays because the
// bodies compile to slower code without it: the update pass of the open 24-site
// chain 24.13 against 24.40 us, of L = 22 with three phases 33.07 against 33.37.
struct VRange {
  uint32_t v0, v1, n;
};
__device__ __forceinline__ VRange hw_range() { return VRange{blockIdx.x, blockIdx.x + 1, gridDim.x}; }

// XCD-aware tile walk: work-groups are dealt round-robin to the 8 XCDs, so
// block i runs on XCD i % 8.  Each XCD gets one contiguous eighth of the row
// tiles, and its blocks stride through that eighth together, which keeps the
// rows being read on one XCD close together in that XCD's L2.
struct TileWalk {
  uint32_t t, t_end, step;
  __device__ TileWalk(uint32_t ntiles, VGrid g) {
    if (g.n % kNumXcd) {   // a grid that does not split evenly over the XCDs: plain grid stride
      t = g.id;
      t_end = ntiles;
      step = g.n;
      return;
    }
    const uint32_t x = g.id % kNumXcd, k = g.id / kNumXcd, per = g.n / kNumXcd;
    const uint32_t t0 = (uint32_t)(((uint64_t)ntiles * x) / kNumXcd);
    t_end = (uint32_t)(((uint64_t)ntiles * (x + 1)) / kNumXcd);
    t = t0 + k;
    step = per;
  }
};

// ------------------------------------------------------ block reductions
// Sums each of Q values over the threads of the block that share a batch
// column (threadIdx % B; blockDim = B * 2^k) by a fixed tree in LDS and
// writes the Q * B column sums to out_block.
template <int Q>
__device__ __forceinline__ void block_partials(const double (&v)[Q], int B, double* red, double* out_block) {
  // red: LDS scratch of Q * blockDim doubles
  for (int q = 0; q < Q; ++q) red[q * blockDim.x + threadIdx.x] = v[q];
  __syncthreads();
  for (int s = blockDim.x / 2; s >= B; s >>= 1) {
    if (threadIdx.x < (unsigned)s)
      for (int q = 0; q < Q; ++q) red[q * blockDim.x + threadIdx.x] += red[q * blockDim.x + threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < (unsigned)B)
    for (int q = 0; q < Q; ++q) out_block[q * B + threadIdx.x] = red[q * blockDim.x + threadIdx.x];
}

// Totals of partials part[g][c] over g < G for cols = Q * B columns in a fixed
// order; every block computes identical totals.  out[q * B + b] in LDS, valid
// after return; red: LDS scratch of blockDim doubles.  The pass that waits for
// these totals is bound by latency, so the rows are read as one contiguous
// array with four loads in flight per thread, and the lanes of a column are
// added by shuffles inside a wave and one short sum over the waves.  (A serial
// sum of a column's 64 to 256 lanes by one thread before: a step of the L = 16
// chain went from 755 to 599 us, of L = 24 from 2.94 to 2.67 ms, with the
// running maximum of lanczos_h_scalars in the place of a loop over all earlier
// coefficients.)  Column counts that are no power of two, or above 32, and
// blocks that are no whole number of waves take the tree in LDS.
__device__ __forceinline__ void reduce_partials(const double* __restrict__ part, int G, int Q, int B, double* red,
                                                double* out) {
  const int cols = Q * B, tid = threadIdx.x, nt = blockDim.x;
  const int n = G * cols;
  if (cols <= 32 && (cols & (cols - 1)) == 0 && nt % 64 == 0) {
    double acc = 0.0;
    int i = tid;
    for (; i + 3 * nt < n; i += 4 * nt) {
      const double v0 = part[i], v1 = part[i + nt], v2 = part[i + 2 * nt], v3 = part[i + 3 * nt];
      acc += (v0 + v1) + (v2 + v3);
    }
    for (; i < n; i += nt) acc += part[i];
    for (int s = 32; s >= cols; s >>= 1) acc += __shfl_xor(acc, s);
    const int lane = tid & 63, wave = tid >> 6, waves = nt >> 6;
    if (lane < cols) red[wave * cols + lane] = acc;
    __syncthreads();
    if (tid < cols) {
      double t = 0.0;
      for (int w = 0; w < waves; ++w) t += red[w * cols + tid];
      out[tid] = t;
    }
    __syncthreads();
    return;
  }
  // any column count: lanes of a column (lpc of them) by a tree in LDS
  const int lpc = nt / cols > 0 ? nt / cols : 1;
  for (int c0 = 0; c0 < cols; c0 += nt) {
    const int c = c0 + (lpc > 1 ? tid % cols : tid), l = lpc > 1 ? tid / cols : 0;
    double acc = 0.0;
    if (c < cols && l < lpc)
      for (int g = l; g < G; g += lpc) acc += part[(size_t)g * cols + c];
    if (lpc > 1) {
      red[tid] = acc;
      __syncthreads();
      for (int k = lpc; k > 1;) {
        const int h = (k + 1) / 2;
        if (l < k - h) red[tid] += red[tid + h * cols];
        k = h;
        __syncthreads();
      }
      if (tid < cols) out[tid] = red[tid];
    } else if (c < cols) {
      out[c] = acc;
    }
  }
  __syncthreads();
}
// ------------------------------------------------------- Lanczos passes
// Stored vectors u_j are unnormalised: v_j = sigma_j u_j.  Iteration j:
//   pass A:  w = a_j H u_j - b_j u_{j-1}      (= H v_j - beta_{j-1} v_{j-1}, or H u_0 at j = 0)
//            partials  Re<u_j, w>, |u_j|^2
//   pass B:  u_{j+1} = c_j (w - d_j u_j)       (= w - alpha_j v_j in v-units)
//            partial   |u_{j+1}|^2  -> beta_j
// The scalars come from the previous pass's partials, reduced in each block.
struct LanczosArgs {
  int j, m;
  double breakdown_rtol;
  int reorth;   // 1: the update pass also removes the component along v_{j-1}
};

// Partial sums of the H-pass per batch column: Re<u_j, w>, |u_j|^2 and the
// complex <u_{j-1}, w> used by the local reorthogonalisation.
constexpr int kQA = 4;



// v of the lane below (UP) or above, zero past the ends of the wave.
template <bool UP>
__device__ __forceinline__ double wave_next(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  constexpr int ctrl = UP ? 0x138 : 0x130;   // the wave shifted by one lane
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, ctrl, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), ctrl, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// (exp(-i tau T) e_1)_i in lane i of one wavefront, for the real symmetric
// tridiagonal T with diagonal al (lane i), coupling be to component i+1 and bl
// to component i-1 (zero outside the used dimension; `on` marks used lanes).
// With the centre mu and the radius R of T's Gershgorin interval, X = (T - mu)
// / R and z = |tau| R, the Chebyshev series exp(-i tau (T - mu)) = J_0(z) + 2
// sum_k (-+i)^k J_k(z) T_k(X) is summed from its last term down (Clenshaw), the
// same order in which Miller's recurrence gives J_k(z) up to a common factor;
// J_0 + 2 (J_2 + J_4 + ...) = 1 fixes that at the end.  One serial chain of
// about z + 11 z^(1/3) + 10 short steps, whose neighbours come by whole-wave
// shifts (a Taylor series in substeps of |tau| R <= 1/2, with its test for the
// end, had three to six times as many, each with 16 shuffles).  The kernel of
// the 20-site ring's step took 20 us, now 4.9; the step-size control of an
// adaptive step of the 19-site chain 76, the nodes of a gradient step 26, now
// 8.6.  Rounding errors against a longer type (root mean square over random T
// of 8 to 40 rows) are 0.9e-16 against 0.8e-16 at |tau| R = 0.2 and 2.2e-16
// against 4.9e-16 at |tau| R = 4.  All 64 lanes must call
// it.
__device__ __forceinline__ void tri_expm_e1(double al, double be, double bl, bool on, int i, double tau, double& er,
                                            double& ei) {
  double lo = on ? al - be - bl : INFINITY, hi = on ? al + be + bl : -INFINITY;
  for (int s = 32; s > 0; s >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, s));
    hi = fmax(hi, __shfl_xor(hi, s));
  }
  const double mu_shift = 0.5 * (lo + hi);
  const double radius = 0.5 * (hi - lo);
  const double ad = on ? al - mu_shift : 0.0;
  const double z = fabs(tau) * radius;
  double vr, vi;
  if (!(z >= 1e-20)) {
    // two terms of the exponential (also passes on what is not a number)
    vr = i == 0 ? 1.0 : 0.0;
    vi = i == 0 ? -tau * ad : i == 1 ? -tau * bl : 0.0;
  } else {
    // bounded number of terms: a non-finite or huge norm cannot stall the wave
    const double zb = fmin(z, 1e6);
    const int n = ((int)(zb + 11.0 * cbrt(zb) + 10.0) + 4) & ~3;   // whole groups of four
    const double q = 2.0 / radius, rz = 2.0 / z;
    const double x0 = ad * q, xu = bl * q, xd = (on ? be : 0.0) * q;   // 2 X
    const double e1 = i == 0 ? 2.0 : 0.0, e1s = tau >= 0.0 ? e1 : -e1;
    double j1 = 1e-30, j2 = 0.0, even = 0.0;            // J_k, J_{k+1} and the sum of the even ones
    double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;      // b_{k+1} and b_{k+2}
    // b_k = a_k + 2 X b_{k+1} - b_{k+2}, a_k = 2 (-+i)^k J_k e_1
    auto down = [&](int k, int phase) {
      double r = fma(x0, ar, fma(xu, wave_next<true>(ar), fma(xd, wave_next<false>(ar), -br)));
      double c = fma(x0, ai, fma(xu, wave_next<true>(ai), fma(xd, wave_next<false>(ai), -bi)));
      if (phase == 0) r = fma(e1, j1, r);
      if (phase == 1) c = fma(-e1s, j1, c);
      if (phase == 2) r = fma(-e1, j1, r);
      if (phase == 3) c = fma(e1s, j1, c);
      if ((phase & 1) == 0) even += j1;
      br = ar;
      bi = ai;
      ar = r;
      ai = c;
      const double j0 = fma((double)k * rz, j1, -j2);
      j2 = j1;
      j1 = j0;
    };
    for (int k = n; k > 0; k -= 4) {
      down(k, 0);
      down(k - 1, 3);
      down(k - 2, 2);
      down(k - 3, 1);
    }
    const double norm = 1.0 / fma(2.0, even, j1);
    vr = 0.5 * fma(x0, ar, fma(xu, wave_next<true>(ar), xd * wave_next<false>(ar))) - br + 0.5 * e1 * j1;
    vi = 0.5 * fma(x0, ai, fma(xu, wave_next<true>(ai), xd * wave_next<false>(ai))) - bi;
    vr *= norm;
    vi *= norm;
  }
  const double cr = cos(tau * mu_shift), ci = -sin(tau * mu_shift);
  er = vr * cr - vi * ci;
  ei = vr * ci + vi * cr;
}

// Largest v >= 0 of the wave, in every lane.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
  return fmax(v, __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max<0x111, 0xf>(v);   // from the lane 1, 2, 4, 8 below in a row of 16
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);   // the last lane of row 0 (2) to row 1 (3)
  v = dpp_max<0x143, 0xc>(v);   // the last lane of the first half to the second
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// The same by a Taylor series in substeps of |tau| R <= 1/2 that end where the
// terms fall below 1e-18 of the sum.  Components smaller than that come out
// smaller than they are, or zero; the step-size rule, whose estimate is such a
// component after a short step, keeps the steps that follow from it.  Neighbours
// and maxima go through the data-parallel moves of the vector unit (by shuffles
// a call took 100 us).
__device__ __forceinline__ void tri_expm_e1_taylor(double al, double be, double bl, bool on, int i, double tau, double& er,
                                                   double& ei) {
  double lo = on ? al - be - bl : INFINITY, hi = on ? al + be + bl : -INFINITY;
  for (int s = 32; s > 0; s >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, s));
    hi = fmax(hi, __shfl_xor(hi, s));
  }
  const double mu_shift = 0.5 * (lo + hi);
  const double radius = 0.5 * (hi - lo);
  const double ad = on ? al - mu_shift : 0.0;
  // bounded substep count (a non-finite or huge norm cannot stall the wave)
  const double nsd = ceil(fabs(tau) * radius / 0.5);
  const int nsub = (nsd >= 1.0 && nsd <= 100000.0) ? (int)nsd : (nsd > 100000.0 ? 100000 : 1);
  const double ts = tau / nsub;
  double vr = (i == 0) ? 1.0 : 0.0, vi = 0.0;
  for (int sub = 0; sub < nsub; ++sub) {
    double sr = vr, si = vi, tr = vr, ti = vi;
    for (int k = 1; k <= 40; ++k) {
      // t <- (-i ts / k) (T - mu) t
      const double up_r = wave_next<true>(tr), up_i = wave_next<true>(ti);
      const double dn_r = wave_next<false>(tr), dn_i = wave_next<false>(ti);
      double yr = ad * tr + (i > 0 ? bl * up_r : 0.0) + (i < 63 ? be * dn_r : 0.0);
      double yi = ad * ti + (i > 0 ? bl * up_i : 0.0) + (i < 63 ? be * dn_i : 0.0);
      if (!on) yr = yi = 0.0;
      const double f = ts / k;
      tr = f * yi;    // (-i f) (yr + i yi) = f yi - i f yr
      ti = -f * yr;
      sr += tr;
      si += ti;
      const double tn = wave_max(fabs(tr) + fabs(ti)), sn = wave_max(fabs(sr) + fabs(si));
      if (tn <= 1e-18 * sn) break;
    }
    vr = sr;
    vi = si;
  }
  const double cr = cos(tau * mu_shift), ci = -sin(tau * mu_shift);
  er = vr * cr - vi * ci;
  ei = vr * ci + vi * cr;
}

// A workspace whose step has given up (resident_verdict): its state stays behind.
__device__ __forceinline__ bool left_behind(const uint32_t* __restrict__ gave_up) {
  return gave_up && *gave_up == kResGaveUp;
}

// Scalars of the H-pass of Lanczos iteration j for every batch column b,
// from the update pass of iteration j-1 (its partial sums |u_j|^2):
//   sa[b] = sigma_j, sb[b] = beta_{j-1} sigma_{j-1}, act[b] = column still running.
// Block 0 (of the virtual grid g) records beta_{j-1}, sigma_j, and m_used / status on breakdown or a
// non-finite norm.  Every block reduces the same partials in the same order,
// so all blocks reach the same decisions.
__device__ __forceinline__ void lanczos_h_scalars(int B, const KState& st, const LanczosArgs& la,
                                                  const double* __restrict__ partB, int Gp, double* red, double* tot,
                                                  double* sa, double* sb, int* act, VGrid g) {
  const int j = la.j;
  const bool first = g.id == 0;   // the block that records the shared results
  const int b = threadIdx.x;      // B <= QK_MAX_BATCH <= blockDim
  if (j == 0) {
    if (b < B) {
      sa[b] = 1.0;
      sb[b] = 0.0;
      act[b] = 1;
      if (first) {
        st.mused[b] = la.m;
        st.status[b] = QK_OK;
        st.smax[b] = 0.0;
      }
    }
    __syncthreads();
    return;
  }
  // the column's earlier scalars are fetched while the partials are in flight
  int mused = 0;
  double sig = 0.0, scale = 0.0;
  if (b < B) {
    mused = st.mused[b];
    sig = st.sigma[(j - 1) * B + b];
    // largest coefficient so far: of the iterations before j - 1, and alpha_{j-1}
    scale = fmax(st.smax[(j - 1) * B + b], fabs(st.alpha[(j - 1) * B + b]));
  }
  reduce_partials(partB, Gp, 1, B, red, tot);
  if (b < B) {
    int active = mused > j;
    const double beta = sqrt(tot[b]);
    if (active) {
      scale = fmax(scale, beta);
      if (!isfinite(beta)) {
        active = 0;
        if (first) {
          st.status[b] = QK_ENUMERIC;
          st.mused[b] = j;
        }
      } else if (beta <= la.breakdown_rtol * scale) {
        active = 0;  // invariant subspace: the Krylov space stops at dimension j
        if (first) st.mused[b] = j;
      }
      if (first) {
        st.beta[(j - 1) * B + b] = beta;
        st.smax[j * B + b] = scale;
      }
    }
    if (active) {
      sa[b] = 1.0 / beta;
      sb[b] = beta * sig;
      if (first) st.sigma[j * B + b] = 1.0 / beta;
    }
    act[b] = active;
  }
  __syncthreads();
}


qk_status launch_tile_lanczos_h(const TilePlan& P, int dtype, const void* uj, const void* ujm1, void* w,
                                const KState& st, const LanczosArgs& la, const double* partB, int Gp, double* partA,
                                int* grid_out, int wgs, hipStream_t s);

// Two-pass split iteration (qk_split.hip): the pre-pass partials |x|^2 and
// Re<x, H_lo x> of a step's initial vector, the high pass
// z = sigma_j H_hi u_j - beta_{j-1} sigma_{j-1} u_{j-1}, and the low pass
// u_{j+1} = c (z + s H_lo u_j - d u_j) with the partials of the next iteration.
qk_status launch_split_form(const qk_ham* H, int dtype, const void* x, double* partB, double* partQ, int* grid,
                            hipStream_t s);
qk_status launch_split_hi(const qk_ham* H, int dtype, const void* uj, const void* ujm1, void* z, const KState& st,
                          const LanczosArgs& la, const double* partB, int GB, double* partA, int* grid, int wgs,
                          hipStream_t s);
qk_status launch_split_lo(const qk_ham* H, int dtype, const void* uj, const void* z, void* out, const KState& st,
                          const LanczosArgs& la, const double* partA, int GA, const double* partBin,
                          const double* partQin, int GB, double* partBout, double* partQout, int store, int* grid,
                          hipStream_t s);
qk_status launch_split_combine(const qk_ham* H, int dtype, void* psi, const void* U, const KState& st, hipStream_t s);

}  // namespace qk
