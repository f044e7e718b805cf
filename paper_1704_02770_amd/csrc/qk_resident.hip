// One launch for the whole Lanczos recurrence of a small sector (Sec. 2
// "Krylov subspace methods"), with a row per thread.
//
// Below about 200,000 elements a Krylov step is a chain of 2 m short kernels:
// each starts by fetching what the previous one left in memory and ends by
// flushing what the next one needs, 7 to 20 us an iteration for vectors of
// 0.2 to 3 MB.  Here a thread keeps its row for the whole step -- the current
// and the previous Lanczos vector and the current vector's values at the
// row's neighbours, in registers -- and an iteration exchanges two things:
//   A  w = a H u_j - b u_{j-1} is published; Re<u_j, w> is totalled (alpha_j);
//      every thread reads w at its neighbours and forms u_{j+1} there as well
//      as on its own row, the same expression in both places, so the same bits;
//   B  |u_{j+1}|^2 is totalled (beta_j); no vector is exchanged.
// u_{j+1} goes to the basis slot for the combination that follows.
//
// Totals and waiting are one thing: a work-group publishes its partial sums as
// 8-byte words that hold 32 bits of the value and the number of the exchange,
// and reads the words of all work-groups until every number matches; then it
// adds them in slot order, so all work-groups (and all runs) get the same bits.
// Words of consecutive exchanges alternate between two arrays: a work-group
// can be at most one exchange ahead of the slowest.  Vectors are published
// with agent-scope stores and waited for before the words are written; reads
// are agent-scope too, so no cache is flushed.
//
// Waiting needs every waited-for work-group to be running.  The work-groups
// register first; the first one closes the list when all have come, or, with
// other kernels holding the chip, after kJoinTicks with those that have.  Only
// registered work-groups take part (late ones leave at once), and if some are
// missing the rows are dealt out to the others, which then keep their vectors
// in memory: slower, the same arithmetic, and no wait for a work-group that
// may never run beside them.
//
// What bounds it: the two exchanges of an iteration, 3.0 us at 924 rows and
// 8 us at 184,756 (a store to the agent's point of coherence and the read that
// sees it are about 0.7 us each, the rest is the sum over a work-group and the
// neighbours' 20 gathers).  A step of 30 vectors, complex128, one phase, against
// the passes: L = 12 (open, m = 20) 105 against 244 us, L = 16 184 against 420,
// L = 18 237, L = 20 329 against 690.
#include <algorithm>
#include <type_traits>

#include "qk_tile.h"

namespace qk {

constexpr int kResMaxThreads = 768;
constexpr int kResMaxSites = 20;
constexpr int kResMaxGroups = 256;
constexpr int kResMaxLanes = 8;                    // columns of a batch, rounded up to a power of two
constexpr long long kJoinTicks = 100000;           // 1 ms of the 100 MHz wall clock
constexpr long long kGiveUpTicks = 500000000ll;    // 5 s: ends a wait that cannot end otherwise

struct ResCtl {
  uint32_t epoch;     // launches' exchanges so far: the next one's first number is epoch + 1
  uint32_t arrived;   // work-groups that have come, and kClosed
  uint32_t left;      // work-groups that have ended
  uint32_t pad;
  uint64_t joined;    // number of the launch's first exchange << 32 | registered work-groups
};
constexpr uint32_t kClosed = 0x80000000u;

struct ResArgs {
  int L, pbc, B, lbp, m, olo, nbonds;
  uint32_t D;
  int join_max;                    // work-groups that may register (all of them, or fewer in tests)
  double half_jxy, jz, rtol;
  const uint32_t* states;
  const uint32_t* bn;
  const double* fields;
  uint64_t stride;                 // elements of a basis slot
  uint64_t* words;                 // [2][groups][2][lanes per row] pairs of words
  ResCtl* ctl;
  double* norm2;                   // [B] |u_m|^2
};

constexpr int kSc1 = 16;   // agent scope
constexpr int kResLoads = 7;

template <typename V>
struct ResBuf {
  using S = decltype(V{}.x);
  typedef uint32_t W __attribute__((ext_vector_type(sizeof(V) / 4)));
  typedef S E __attribute__((ext_vector_type(2)));
  __amdgpu_buffer_rsrc_t r;
  __device__ ResBuf(const void* p, uint64_t n) {
    r = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)(uint32_t)(n * sizeof(V)), 0x00027000);
  }
  template <int AUX>
  __device__ __forceinline__ V ld(uint32_t off) const {
    W w;
    if constexpr (sizeof(V) == 16) w = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX);
    else w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
    const E e = __builtin_bit_cast(E, w);
    return V{e.x, e.y};
  }
  template <int AUX>
  __device__ __forceinline__ void st(uint32_t off, V v) const {
    const E e = {v.x, v.y};
    const W w = __builtin_bit_cast(W, e);
    if constexpr (sizeof(V) == 16) __builtin_amdgcn_raw_buffer_store_b128(w, r, off, 0, AUX);
    else __builtin_amdgcn_raw_buffer_store_b64(w, r, off, 0, AUX);
  }
};
constexpr uint32_t kNoRow = 0xfffffff0u;   // an offset past every buffer: reads zeros, writes nothing

__device__ __forceinline__ uint64_t word_ld(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void word_st(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct ResShared {
  double red[2 * kResMaxThreads / 64 * kResMaxLanes];
  double sa[kResMaxLanes], sb[kResMaxLanes], sc[kResMaxLanes], sd[kResMaxLanes];
  int act[kResMaxLanes];
  uint32_t tab[kBinomStride * kBinomStride];
  uint32_t ticket, joined, epoch, dead, go;
};

// v added over the lanes of a wave that share a column (lane % Bp): the totals
// are in the lanes below Bp.  One column takes the data-parallel moves of the
// vector unit, a few cycles each where a shuffle through LDS takes about 60.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
  return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double res_wave_sum(double v, int Bp) {
  if (Bp == 1) {
    v = dpp_add<0x111, 0xf>(v);   // from the lane 1, 2, 4, 8 below in a row of 16
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);   // the last lane of row 0 (2) to row 1 (3)
    v = dpp_add<0x143, 0xc>(v);   // the last lane of the first half to the second
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
  }
  for (int s = 32; s >= Bp; s >>= 1) v += __shfl_xor(v, s);
  return v;
}

// Partial sums of a work-group's columns into LDS; with ROWS, all vectors the
// waves have published are out when the barrier that follows is passed.
template <int Q, bool ROWS>
__device__ __forceinline__ void res_partials(ResShared& sh, const ResArgs& ra, const double (&v)[Q]) {
  const int Bp = 1 << ra.lbp, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = (int)blockDim.x >> 6;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const double t = res_wave_sum(v[q], Bp);
    if (lane < Bp) sh.red[(q * waves + wave) * Bp + lane] = t;
  }
  if (ROWS) __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// By the first wave: the partial sums as slot `slot` of exchange `no`.
__device__ __forceinline__ void res_publish(ResShared& sh, const ResArgs& ra, int Q, uint32_t no, uint32_t nslots,
                                            uint32_t slot) {
  const int Bp = 1 << ra.lbp, tid = threadIdx.x, waves = (int)blockDim.x >> 6;
  if (tid < Q * Bp) {
    const int q = tid >> ra.lbp, p = tid & (Bp - 1);
    double t = 0.0;
    for (int w = 0; w < waves; ++w) t += sh.red[(q * waves + w) * Bp + p];
    const uint64_t b = __builtin_bit_cast(uint64_t, t), tag = (uint64_t)no << 32;
    uint64_t* w = ra.words + (((size_t)(no & 1u) * nslots + slot) * (size_t)(2 * Bp) + (size_t)tid) * 2;
    word_st(w, tag | (uint32_t)b);
    word_st(w + 1, tag | (b >> 32));
  }
}

// By the first wave: waits for exchange `no` of all slots.  Lane q * Bp + p
// returns the total of quantity q, column p.
__device__ __forceinline__ double res_collect(ResShared& sh, const ResArgs& ra, int Q, uint32_t no, uint32_t nslots) {
  const int Bp = 1 << ra.lbp, cols = Q * Bp, lane = threadIdx.x;
  const uint32_t n = nslots * (uint32_t)cols;
  const uint64_t* base = ra.words + (size_t)(no & 1u) * nslots * (size_t)(2 * Bp) * 2;
  // lane l adds the entries l, l + 64, ..., four at a time, then the lanes of a
  // column are added in a fixed order
  double acc = 0.0;
  long long t0 = 0;
  for (uint32_t i0 = 0; i0 < n; i0 += 256) {
    uint64_t a[4], b[4];
    bool ok;
    uint32_t tries = 0;
    do {
      ok = true;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t i = i0 + 64u * e + (uint32_t)lane, slot = i / (uint32_t)cols, c = i & (uint32_t)(cols - 1);
        const uint64_t* w = base + ((size_t)(i < n ? slot : 0u) * (2 * Bp) + c) * 2;
        a[e] = word_ld(w);
        b[e] = word_ld(w + 1);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i0 + 64u * e + (uint32_t)lane < n) ok = ok && (uint32_t)(a[e] >> 32) == no && (uint32_t)(b[e] >> 32) == no;
      if (!ok && (++tries & 1023u) == 0u) {
        const long long now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 > kGiveUpTicks) {
          sh.dead = 1;
          ok = true;
        }
      }
    } while (!ok);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (i0 + 64u * e + (uint32_t)lane < n) acc += __builtin_bit_cast(double, (b[e] << 32) | (uint32_t)a[e]);
  }
  return res_wave_sum(acc, cols);
}

// The sum over a row's hops, bond by bond in ascending order with the ring bond
// last, x zero for an inactive bond, in the order that the pass's plain kernels
// use (TileArgs::order): complex64 gives the same bits as they do.
// BLOCKED: that of a block decomposition (complex64 from 18 sites on);
// otherwise one by one.  flush: bit k set where the hop on bond k ends a group
// of four.
template <typename T, bool BLOCKED>
struct HopSum {
  using V = typename Cx<T>::V;
  V hs = {0, 0}, ac = {0, 0}, vd = {0, 0}, vw = {0, 0};
  __device__ __forceinline__ void add(const ResArgs& ra, int k, V x, uint32_t flush) {
    if (!BLOCKED || k < ra.olo - 1) {
      hs.x += x.x;
      hs.y += x.y;
    } else if (k == ra.L - 1) {
      vw = x;
    } else if (k == ra.olo - 1) {
      vd = x;
    } else {
      ac.x += x.x;
      ac.y += x.y;
      const bool f = ((flush >> k) & 1u) != 0u;
      hs.x += f ? ac.x : (T)0;
      hs.y += f ? ac.y : (T)0;
      ac.x = f ? (T)0 : ac.x;
      ac.y = f ? (T)0 : ac.y;
    }
  }
  __device__ __forceinline__ V total() const {
    if (!BLOCKED) return hs;
    V t = {hs.x + ac.x, hs.y + ac.y};
    t.x += vd.x + vw.x;
    t.y += vd.y + vw.y;
    return t;
  }
};

template <typename T, bool BLOCKED>
__device__ __forceinline__ typename Cx<T>::V res_w(double d, T g, T ca, T cb,
                                                   typename Cx<T>::V u, typename Cx<T>::V um, typename Cx<T>::V hs) {
  typename Cx<T>::V h, w;
  if (!BLOCKED) {
    const T dd = (T)d;
    h.x = dd * u.x;
    h.y = dd * u.y;
    h.x += g * hs.x;
    h.y += g * hs.y;
    w.x = ca * h.x;
    w.y = ca * h.y;
    w.x -= cb * um.x;
    w.y -= cb * um.y;
  } else {
    h.x = (T)d * u.x + g * hs.x;
    h.y = (T)d * u.y + g * hs.y;
    w.x = ca * h.x - cb * um.x;
    w.y = ca * h.y - cb * um.y;
  }
  return w;
}

// u_{j+1} of one row, as the update pass forms it.
template <typename T>
__device__ __forceinline__ typename Cx<T>::V res_next(double c, double d, typename Cx<T>::V w, typename Cx<T>::V u) {
  typename Cx<T>::V o;
  o.x = (T)(c * ((double)w.x - d * (double)u.x));
  o.y = (T)(c * ((double)w.y - d * (double)u.y));
  return o;
}

// What lane b < B of the first wave keeps of column b over the iterations.
struct ResCol {
  double sigma = 0.0, smax = 0.0, alpha = 0.0;   // sigma_j, the largest coefficient so far, alpha_j
};

// By the first wave, after exchange A of iteration j (lane q * Bp + b holds S_q
// of column b): alpha_j and the factors of the update.  `first`: the work-group
// that records the shared results.
__device__ __forceinline__ void res_alpha(ResShared& sh, const ResArgs& ra, const KState& st, int j, bool first,
                                          double S, ResCol& col) {
  const int b = threadIdx.x, B = ra.B, Bp = 1 << ra.lbp;
  const double S2 = j == 0 ? __shfl(S, b + Bp) : 0.0;
  if (b >= B) return;
  int active = sh.act[b];
  if (active) {
    double c, d;
    if (j == 0) {
      const double n0 = sqrt(S2);
      col.alpha = S / S2;
      c = 1.0 / n0;
      d = col.alpha;
      col.sigma = c;
      if (first) {
        st.n0[b] = n0;
        st.sigma[b] = c;
      }
      if (!(n0 > 0.0)) {
        active = 0;   // zero vector: nothing to propagate
        if (first) {
          st.mused[b] = 0;
          if (!isfinite(S2)) st.status[b] = QK_ENUMERIC;
        }
      }
    } else {
      col.alpha = col.sigma * S;
      c = 1.0;
      d = col.alpha * col.sigma;
    }
    if (active && !isfinite(col.alpha)) {
      active = 0;
      if (first) {
        st.status[b] = QK_ENUMERIC;
        st.mused[b] = j;
      }
    }
    if (active && first) st.alpha[j * B + b] = col.alpha;
    sh.sc[b] = c;
    sh.sd[b] = d;
  }
  sh.act[b] = active;
}

// By the first wave, after exchange B of iteration j (lane b holds |u_{j+1}|^2):
// beta_j, the breakdown test, the factors of the next H-pass.
__device__ __forceinline__ void res_beta(ResShared& sh, const ResArgs& ra, const KState& st, int j, bool first,
                                         double norm2, ResCol& col) {
  const int b = threadIdx.x, B = ra.B;
  if (b < B) {
    int active = sh.act[b];
    const double beta = sqrt(norm2);
    if (j + 1 == ra.m) {
      if (first) ra.norm2[b] = norm2;
    } else {
      if (active) {
        col.smax = fmax(fmax(col.smax, fabs(col.alpha)), beta);
        if (!isfinite(beta)) {
          active = 0;
          if (first) {
            st.status[b] = QK_ENUMERIC;
            st.mused[b] = j + 1;
          }
        } else if (beta <= ra.rtol * col.smax) {
          active = 0;   // invariant subspace
          if (first) st.mused[b] = j + 1;
        }
        if (first) st.beta[j * B + b] = beta;
      }
      if (active) {
        sh.sa[b] = 1.0 / beta;
        sh.sb[b] = beta * col.sigma;
        col.sigma = 1.0 / beta;
        if (first) st.sigma[(j + 1) * B + b] = col.sigma;
      }
      sh.act[b] = active;
    }
  }
  const bool any = __any(b < B && sh.act[b] != 0);
  if (b == 0) sh.go = any && !sh.dead && j + 1 < ra.m;
}

template <typename T, int KMAX, bool BLOCKED>
__global__ void __launch_bounds__(kResMaxThreads, 3)
k_resident(ResArgs ra, typename Cx<T>::V* __restrict__ psi, typename Cx<T>::V* __restrict__ U,
           typename Cx<T>::V* __restrict__ X, KState st) {
  using V = typename Cx<T>::V;
  __shared__ ResShared sh;
  const int tid = threadIdx.x, nt = blockDim.x, B = ra.B, Bp = 1 << ra.lbp, p = tid & (Bp - 1);
  const uint32_t G = gridDim.x;
  const uint64_t nel = (uint64_t)ra.D * B;
  // register
  if (tid == 0) {
    sh.dead = 0;
    sh.epoch = __hip_atomic_load(&ra.ctl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;   // the cleared words hold 0
    sh.ticket = __hip_atomic_fetch_add(&ra.ctl->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (int i = tid; i < kBinomStride * kBinomStride; i += nt) sh.tab[i] = ra.bn[i];
  __syncthreads();
  const uint32_t epoch = sh.epoch, ticket = sh.ticket;
  const double* f = ra.fields + (size_t)(p < B ? p : 0) * ra.L;
  const T g = (T)ra.half_jxy;
  double hh = 0.0;
  for (int i = 0; i < ra.L; ++i) hh += f[i];
  ModelArgs ma;
  ma.L = ra.L;
  ma.pbc = ra.pbc;
  ma.jz = ra.jz;
  ma.lmask = (1ull << ra.L) - 1ull;
  // offset of the partner of state s (row r) across bond k, kNoRow if the
  // bond's bits agree; pc: set bits below k
  auto partner = [&](uint32_t s, uint32_t r, int k, int pc) -> uint32_t {
    uint32_t q;
    if (k < ra.L - 1) {
      const uint32_t b0 = (s >> k) & 1u;
      const uint32_t c = sh.tab[k * kBinomStride + pc];
      if (b0 == ((s >> (k + 1)) & 1u)) return kNoRow;
      q = b0 ? r + c : r - c;
    } else {
      if (((s ^ (s >> (ra.L - 1))) & 1u) == 0u) return kNoRow;
      q = cns_rank<uint32_t>(s ^ (1u | (1u << (ra.L - 1))), sh.tab);
    }
    return (q * (uint32_t)B + p) * (uint32_t)sizeof(V);
  };
  // this thread's row
  const uint32_t row = (blockIdx.x * (uint32_t)nt + (uint32_t)tid) >> ra.lbp;
  const bool has = row < ra.D && p < B;
  const uint32_t eo = has ? (row * (uint32_t)B + p) * (uint32_t)sizeof(V) : kNoRow;
  const uint32_t state = has ? ra.states[row] : 0u;
  uint32_t off[KMAX];
  {
    int pc = 0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      off[k] = kNoRow;
      if (k < ra.nbonds) off[k] = partner(state, row, k, pc);
      pc += (int)((state >> k) & 1u);
    }
  }
  // where the groups of four hops of a state end (HopSum)
  auto flushes = [&](uint32_t s) -> uint32_t {
    uint32_t m = 0;
    int n = 0;
    if (BLOCKED)
      for (int k = ra.olo; k < ra.L - 1; ++k)
        if (((s >> k) ^ (s >> (k + 1))) & 1u)
          if ((++n & 3) == 0) m |= 1u << k;
    return m;
  };
  uint32_t flush = flushes(state);
  const double d = has ? diag_value<uint32_t>(state, ma, f, 0.5 * hh) : 0.0;
  const ResBuf<V> bpsi(psi, nel);
  V u = bpsi.template ld<0>(eo), um = {0, 0};
  V un[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) un[k] = bpsi.template ld<0>(off[k]);
  if (tid == 0) {
    if ((ticket & kClosed) || ticket >= (uint32_t)ra.join_max) {
      sh.joined = 0;   // too late
    } else if (ticket == 0) {
      const long long t0 = wall_clock64();
      uint32_t n = 0;
      for (;;) {
        n = __hip_atomic_load(&ra.ctl->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n >= (uint32_t)ra.join_max || wall_clock64() - t0 > kJoinTicks) break;
        __builtin_amdgcn_s_sleep(1);
      }
      n = __hip_atomic_fetch_or(&ra.ctl->arrived, kClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (n > (uint32_t)ra.join_max) n = (uint32_t)ra.join_max;
      sh.joined = n;
      word_st(&ra.ctl->joined, ((uint64_t)epoch << 32) | n);
    } else {
      uint64_t w;
      const long long t0 = wall_clock64();
      do {
        w = word_ld(&ra.ctl->joined);
        if (wall_clock64() - t0 > kGiveUpTicks) {
          sh.dead = 1;
          break;
        }
      } while ((uint32_t)(w >> 32) != epoch || (uint32_t)w == 0u);
      sh.joined = (uint32_t)w;
    }
  }
  if (tid < B) {
    sh.sa[tid] = 1.0;
    sh.sb[tid] = 0.0;
    sh.act[tid] = 1;
  }
  __syncthreads();
  const uint32_t R = sh.joined;
  const bool member = R != 0 && (ticket & ~kClosed) < R;
  const bool first = member && ticket == 0;
  if (first && tid < B) {
    st.mused[tid] = ra.m;
    st.status[tid] = QK_OK;
  }
  ResCol col;
  const bool wave0 = tid < 64;
  uint32_t no = epoch;
  if (member && R == G) {
    // every row has its thread: vectors in registers
    for (int j = 0; j < ra.m; ++j) {
      const bool mine = p < B && sh.act[p] != 0;
      const T ca = mine ? (T)sh.sa[p] : (T)0, cb = mine ? (T)sh.sb[p] : (T)0;
      HopSum<T, BLOCKED> sum;
      if (BLOCKED) __asm__ volatile("" : "+v"(flush));   // its bits as lane masks would not fit the scalar registers
#pragma unroll
      for (int k = 0; k < KMAX; ++k)
        if (!BLOCKED || k < ra.nbonds) sum.add(ra, k, un[k], flush);
      const V w = res_w<T, BLOCKED>(d, g, ca, cb, u, um, sum.total());
      const ResBuf<V> bx(X + (size_t)(j & 1) * nel, nel);
      if (mine) bx.template st<kSc1>(eo, w);
      const bool on = mine && has;
      const double s1 = on ? (double)u.x * (double)w.x + (double)u.y * (double)w.y : 0.0;
      if (j == 0) {
        const double v[2] = {s1, on ? (double)u.x * (double)u.x + (double)u.y * (double)u.y : 0.0};
        res_partials<2, true>(sh, ra, v);
      } else {
        const double v[1] = {s1};
        res_partials<1, true>(sh, ra, v);
      }
      if (wave0) {
        const int Q = j == 0 ? 2 : 1;
        res_publish(sh, ra, Q, no, G, blockIdx.x);
        res_alpha(sh, ra, st, j, first, res_collect(sh, ra, Q, no, G), col);
      }
      __syncthreads();
      const bool live = p < B && sh.act[p] != 0;
      const double c = live ? sh.sc[p] : 0.0, dd = live ? sh.sd[p] : 0.0;
      const V o = res_next<T>(c, dd, w, u);
      const double v[1] = {live && has ? (double)o.x * (double)o.x + (double)o.y * (double)o.y : 0.0};
      res_partials<1, false>(sh, ra, v);
      if (wave0) res_publish(sh, ra, 1, no + 1, G, blockIdx.x);
      if (j + 1 < ra.m) {
        if (live) ResBuf<V>(U + (size_t)j * ra.stride, nel).template st<0>(eo, o);
        // w at the neighbours, while the sums are under way
#pragma unroll
        for (int k0 = 0; k0 < KMAX; k0 += kResLoads) {
          V x[kResLoads];
#pragma unroll
          for (int i = 0; i < kResLoads; ++i)
            if (k0 + i < KMAX) x[i] = bx.template ld<kSc1>(off[k0 + i]);
#pragma unroll
          for (int i = 0; i < kResLoads; ++i)
            if (k0 + i < KMAX) un[k0 + i] = res_next<T>(c, dd, x[i], un[k0 + i]);
          __asm__ volatile("" ::: "memory");   // no more loads in flight than registers hold
        }
      }
      um = u;
      u = o;
      if (wave0) res_beta(sh, ra, st, j, first, res_collect(sh, ra, 1, no + 1, G), col);
      no += 2;
      __syncthreads();
      if (!sh.go) break;
    }
  } else if (member) {
    // rows of missing work-groups are dealt out: vectors in memory
    for (int j = 0; j < ra.m; ++j) {
      const ResBuf<V> bu(j == 0 ? psi : U + (size_t)(j - 1) * ra.stride, nel);
      const ResBuf<V> bm(j <= 1 ? psi : U + (size_t)(j - 2) * ra.stride, nel);
      const ResBuf<V> bx(X, nel), bo(U + (size_t)j * ra.stride, nel);
      const bool mine = p < B && sh.act[p] != 0;
      const T ca = mine ? (T)sh.sa[p] : (T)0, cb = mine ? (T)sh.sb[p] : (T)0;
      const int Q = j == 0 ? 2 : 1;
      for (uint32_t ch = ticket; ch < G; ch += R) {
        const uint32_t r = (ch * (uint32_t)nt + (uint32_t)tid) >> ra.lbp;
        const bool on = r < ra.D && mine;
        const uint32_t e = on ? (r * (uint32_t)B + p) * (uint32_t)sizeof(V) : kNoRow;
        const uint32_t s = on ? ra.states[r] : 0u;
        const V x = bu.template ld<kSc1>(e);
        V xm = {0, 0};
        if (j > 0) xm = bm.template ld<kSc1>(e);
        HopSum<T, BLOCKED> sum;
        const uint32_t fl = flushes(s);
        int pc = 0;
        for (int k = 0; k < ra.nbonds; ++k) {
          sum.add(ra, k, bu.template ld<kSc1>(partner(s, r, k, pc)), fl);
          pc += (int)((s >> k) & 1u);
        }
        const V w = res_w<T, BLOCKED>(on ? diag_value<uint32_t>(s, ma, f, 0.5 * hh) : 0.0, g, ca, cb, x, xm, sum.total());
        bx.template st<kSc1>(e, w);
        const double v[2] = {on ? (double)x.x * (double)w.x + (double)x.y * (double)w.y : 0.0,
                             on ? (double)x.x * (double)x.x + (double)x.y * (double)x.y : 0.0};
        res_partials<2, true>(sh, ra, v);
        if (wave0) res_publish(sh, ra, Q, no, G, ch);
        __syncthreads();
      }
      if (wave0) res_alpha(sh, ra, st, j, first, res_collect(sh, ra, Q, no, G), col);
      __syncthreads();
      const bool live = p < B && sh.act[p] != 0;
      const double c = live ? sh.sc[p] : 0.0, dd = live ? sh.sd[p] : 0.0;
      for (uint32_t ch = ticket; ch < G; ch += R) {
        const uint32_t r = (ch * (uint32_t)nt + (uint32_t)tid) >> ra.lbp;
        const bool on = r < ra.D && live;
        const uint32_t e = on ? (r * (uint32_t)B + p) * (uint32_t)sizeof(V) : kNoRow;
        const V o = res_next<T>(c, dd, bx.template ld<kSc1>(e), bu.template ld<kSc1>(e));
        if (j + 1 < ra.m) bo.template st<kSc1>(e, o);
        const double v[1] = {on ? (double)o.x * (double)o.x + (double)o.y * (double)o.y : 0.0};
        res_partials<1, true>(sh, ra, v);
        if (wave0) res_publish(sh, ra, 1, no + 1, G, ch);
        __syncthreads();
      }
      if (wave0) res_beta(sh, ra, st, j, first, res_collect(sh, ra, 1, no + 1, G), col);
      no += 2;
      __syncthreads();
      if (!sh.go) break;
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (sh.dead)
      for (int b = 0; b < B; ++b) st.status[b] = QK_ENUMERIC;
    // the last work-group, late ones included, makes room for the next launch
    if (__hip_atomic_fetch_add(&ra.ctl->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == G - 1) {
      __hip_atomic_store(&ra.ctl->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&ra.ctl->left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      word_st(&ra.ctl->joined, 0ull);
      __hip_atomic_store(&ra.ctl->epoch, epoch - 1u + 2u * (uint32_t)ra.m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ------------------------------------------------------------------- host
// Lanes of a workspace's rows, 0 if the resident recurrence does not cover it
// (that of the two-pass split has no d_res either).
static uint64_t resident_lanes(const qk_krylov* k) {
  const qk_ham* H = k->H;
  if (H->p.mode != QK_MATFREE || H->basis->L > kResMaxSites || k->reorth != 0) return 0;
  uint64_t Bp = 1;
  while (Bp < (uint64_t)k->batch) Bp *= 2;
  const uint64_t lanes = (uint64_t)k->D * Bp;
  return Bp <= (uint64_t)kResMaxLanes && lanes <= (uint64_t)kResMaxThreads * kResMaxGroups ? lanes : 0;
}

// Threads per work-group and work-groups: 256 threads up to 256 work-groups,
// then larger work-groups.
static void resident_grid(uint64_t lanes, int* threads, int* groups) {
  int nt = 256;
  if (lanes > (uint64_t)nt * kResMaxGroups) nt = (int)((lanes + kResMaxGroups * 64 - 1) / (kResMaxGroups * 64)) * 64;
  *threads = nt;
  *groups = (int)((lanes + nt - 1) / nt);
}

static size_t resident_words(int groups, int lanes_per_row) { return (size_t)2 * groups * 2 * lanes_per_row * 2; }

void resident_bytes(const qk_krylov* k, size_t* head, size_t* body) {
  *head = *body = 0;
  const uint64_t lanes = resident_lanes(k);
  if (!lanes) return;
  int nt, G;
  resident_grid(lanes, &nt, &G);
  *head = sizeof(ResCtl) + sizeof(uint64_t) * resident_words(G, (int)(lanes / (uint64_t)k->D));
  *body = 2 * (size_t)k->D * k->batch * (k->dtype == QK_C128 ? 16 : 8);
}

template <typename T, int KMAX, bool BLOCKED>
static void resident_launch(const ResArgs& ra, int G, int nt, void* psi, void* U, void* X, const KState& st,
                            hipStream_t s) {
  using V = typename Cx<T>::V;
  hipLaunchKernelGGL((k_resident<T, KMAX, BLOCKED>), dim3(G), dim3(nt), 0, s, ra, (V*)psi, (V*)U, (V*)X, st);
}

qk_status launch_resident(qk_krylov* k, void* psi, double rtol, hipStream_t s) {
  const qk_ham* H = k->H;
  const uint64_t lanes = resident_lanes(k);
  int nt, G;
  resident_grid(lanes, &nt, &G);
  ResArgs ra{};
  ra.L = H->basis->L;
  ra.pbc = H->p.pbc;
  ra.B = k->batch;
  while ((1 << ra.lbp) < k->batch) ++ra.lbp;
  ra.m = k->m;
  ra.olo = H->llo > 0 ? H->llo : ra.L + 1;
  ra.nbonds = ra.pbc ? ra.L : ra.L - 1;
  ra.D = (uint32_t)k->D;
  ra.join_max = k->res_join > 0 ? std::min(G, k->res_join) : G;
  ra.half_jxy = 0.5 * H->p.jxy;
  ra.jz = H->p.jz;
  ra.rtol = rtol;
  ra.states = (const uint32_t*)H->basis->d_states;
  ra.bn = H->basis->d_binom;
  ra.fields = H->d_fields;
  ra.stride = k->ustride;
  ra.ctl = (ResCtl*)k->d_res;
  ra.words = (uint64_t*)((char*)k->d_res + sizeof(ResCtl));
  ra.norm2 = k->d_partB;
  void* X = k->d_X;
  const KState st = make_kstate(k);
  // the bonds that a thread keeps registers for: 14, 17 or 20
  if (k->dtype == QK_C128) {
    if (ra.nbonds <= 14) resident_launch<double, 14, false>(ra, G, nt, psi, k->d_U, X, st, s);
    else if (ra.nbonds <= 17) resident_launch<double, 17, false>(ra, G, nt, psi, k->d_U, X, st, s);
    else resident_launch<double, 20, false>(ra, G, nt, psi, k->d_U, X, st, s);
  } else if (ra.olo > ra.L) {
    if (ra.nbonds <= 14) resident_launch<float, 14, false>(ra, G, nt, psi, k->d_U, X, st, s);
    else if (ra.nbonds <= 17) resident_launch<float, 17, false>(ra, G, nt, psi, k->d_U, X, st, s);
    else resident_launch<float, 20, false>(ra, G, nt, psi, k->d_U, X, st, s);
  } else {
    resident_launch<float, 20, true>(ra, G, nt, psi, k->d_U, X, st, s);
  }
  QK_HIP(hipGetLastError());
  return QK_OK;
}

}  // namespace qk
