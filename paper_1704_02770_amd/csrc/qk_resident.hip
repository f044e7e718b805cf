// One launch for a whole Krylov step of a small sector (Sec. 2 "Krylov subspace
// methods"), with a row per thread.
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
// u_{j+1} goes to the basis slot.  At the end every work-group computes the
// small exponential for itself and combines its own rows of the basis.
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
// may never run beside them.  A wait has a limit all the same, counted in polls
// (a clock would go on while the queue is not on the device), and a launch of
// which a wait gives up leaves psi as it was, in all its rows, and reports
// QK_ENUMERIC, as every later one of the workspace does.  For that a work-group
// at its limit first raises a doubt and polls once more.  One that has passed
// exchange A of the last iteration looks for a doubt before it combines.  If
// there is none, whoever raises one later finds everything that it waits for,
// as all had published it before the other looked.  If there is one, the first
// to say decides (ResCtl::verdict); work-groups that have passed say "go", and
// a wait after that ends by itself.  Without doubts a step costs one load
// more, beside the coefficients (L = 16, m = 30: 176.2 us before, 173.9 now).
//
// Sectors of up to 1,024 rows (over all columns) take one work-group, which
// keeps u_j in LDS and exchanges nothing (k_resident_one).
//
// What bounds it: the two exchanges of an iteration, 1.4 to 3 us for the first
// (all must have stored w) and 1.1 us for the second, a load that sees another
// work-group's store taking 0.7 us; the neighbours, 1.0 to 1.3 us (3 us at
// L = 20); three barriers and the scalars between them, 1.5 us.  In one
// work-group 1.4 us an iteration, the gathers from LDS and the sums over the
// waves.  A step of 30 vectors, complex128, one phase, against the passes:
// L = 12 (open, 20 vectors) 51 against 244 us, L = 16 173 against 420, L = 18
// 219, L = 20 333 against 690; of four phases at L = 12 in complex64 182.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "qk_step_bodies.h"
#include "qk_tile.h"

namespace qk {

constexpr int kResMaxThreads = 768;
constexpr int kResMaxSites = 20;
constexpr int kResMaxGroups = 256;
constexpr int kResMaxLanes = 8;                    // columns of a batch, rounded up to a power of two
constexpr long long kJoinTicks = 100000;           // 1 ms of the 100 MHz wall clock

struct ResCtl {
  uint32_t epoch;     // launches' exchanges so far: the next one's first number is epoch + 1
  uint32_t arrived;   // work-groups that have come, and kClosed
  uint32_t left;      // work-groups that have ended
  uint32_t pad;
  uint64_t joined;    // number of the launch's first exchange << 32 | registered work-groups
  uint32_t verdict;   // kResGaveUp, the (odd) number of a launch's first exchange if it went on in spite of a doubt
  uint32_t doubt;     // that number of the last launch in which a doubt was raised; with verdict one 8-byte word
};
static_assert(sizeof(ResCtl) == 32, "verdict and doubt on an 8-byte boundary");
constexpr uint32_t kClosed = 0x80000000u;
enum { kTailNone = 0, kTailStep = 1, kTailAdaptive = 2 };

struct ResArgs {
  int L, pbc, B, lbp, m, nbonds, reorth;
  int qcap;                        // quantities of a slot of words
  uint32_t D;
  int groups;                      // work-groups that the rows take
  int join_max;                    // work-groups that may register (all of them, or fewer in tests)
  uint32_t polls;                  // of a wait before it gives up, 0: at once
  uint32_t check;                  // mask of the polls after which a wait looks at that
  double half_jxy, jz, rtol;
  const uint32_t* states;
  const uint32_t* bn;
  const double* fields;
  uint64_t stride;                 // elements of a basis slot
  uint64_t* words;                 // [2][groups][2, reorth: 4][lanes per row] pairs of words
  ResCtl* ctl;
  int tail;                        // what follows the recurrence (kTail*)
  double* norm2;                   // [B] |u_m|^2
  double tau, tol;                 // the step, or the largest one and the tolerance of an adaptive step
};

constexpr int kSc1 = 16;   // agent scope

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

// The verdict of launch `epoch` where there is a doubt: `go`, unless another
// work-group was first.
__device__ __forceinline__ bool res_settle(ResCtl* ctl, uint32_t epoch, bool go) {
  uint32_t cur = __hip_atomic_load(&ctl->verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  while (cur != kResGaveUp && cur != epoch)   // a verdict of this launch is final
    if (__hip_atomic_compare_exchange_strong(&ctl->verdict, &cur, go ? epoch : kResGaveUp, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return go;
  return cur == epoch;
}
// Whether a wait goes on after its tries-th poll without success; passed: this
// work-group has been through exchange A of the last iteration.
__device__ __forceinline__ bool res_wait_on(const ResArgs& ra, uint32_t epoch, uint32_t tries, bool passed) {
  if (tries < ra.polls) {
    if ((tries & 0xffffu) != 0u) return true;
    return __hip_atomic_load(&ra.ctl->verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kResGaveUp;
  }
  if (tries == ra.polls && tries != 0u) {
    // at the memory before the next poll
    const uint32_t was = __hip_atomic_exchange(&ra.ctl->doubt, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __asm__ volatile("s_waitcnt vmcnt(0)" ::"v"(was) : "memory");
    return true;
  }
  return res_settle(ra.ctl, epoch, passed);
}
// What a work-group does that has been through its last wait; word: verdict and
// doubt, read after it.
__device__ __forceinline__ bool res_goes_on(const ResArgs& ra, uint32_t epoch, uint64_t word) {
  if ((uint32_t)word == kResGaveUp) return false;
  return (uint32_t)(word >> 32) != epoch || res_settle(ra.ctl, epoch, true);
}

struct ResShared {
  double red[4 * kResMaxThreads / 64 * kResMaxLanes];
  double sa[kResMaxLanes], sb[kResMaxLanes], sc[kResMaxLanes], sd[kResMaxLanes], ser[kResMaxLanes], sei[kResMaxLanes];
  int act[kResMaxLanes];
  // per column: coefficients and scales, then the combination's coefficients in al and be
  double al[kResMaxLanes * 64], be[kResMaxLanes * 64], sg[kResMaxLanes * 64];
  double n0[kResMaxLanes], last[kResMaxLanes];   // |psi|, |u_m|
  int mu[kResMaxLanes], ok[kResMaxLanes];
  uint32_t tab[kBinomStride * kBinomStride];
  uint32_t ticket, joined, epoch, dead, go, combine;
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
    uint64_t* w = ra.words + (((size_t)(no & 1u) * nslots + slot) * (size_t)ra.qcap * Bp + (size_t)tid) * 2;
    word_st(w, tag | (uint32_t)b);
    word_st(w + 1, tag | (b >> 32));
  }
}

// By the first wave: waits for exchange `no` of all slots.  Lane q * Bp + p
// returns the total of quantity q, column p.  passed: as in res_wait_on.
__device__ __forceinline__ double res_collect(ResShared& sh, const ResArgs& ra, int Q, uint32_t no, uint32_t nslots,
                                              bool passed = false) {
  const int Bp = 1 << ra.lbp, cols = Q * Bp, lane = threadIdx.x;
  const uint32_t n = nslots * (uint32_t)cols;
  const uint64_t* base = ra.words + (size_t)(no & 1u) * nslots * (size_t)ra.qcap * Bp * 2;
  // lane l adds the entries l, l + 64, ..., four at a time, then the lanes of a
  // column are added in a fixed order
  double acc = 0.0;
  if (ra.polls == 0u && !res_wait_on(ra, sh.epoch, 0u, passed)) {
    sh.dead = 1;
    return 0.0;
  }
  for (uint32_t i0 = 0; i0 < n; i0 += 256) {
    uint64_t a[4], b[4];
    bool ok;
    uint32_t tries = 0;
    do {
      ok = true;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t i = i0 + 64u * e + (uint32_t)lane, slot = i / (uint32_t)cols, c = i & (uint32_t)(cols - 1);
        const uint64_t* w = base + ((size_t)(i < n ? slot : 0u) * (ra.qcap * Bp) + c) * 2;
        a[e] = word_ld(w);
        b[e] = word_ld(w + 1);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i0 + 64u * e + (uint32_t)lane < n) ok = ok && (uint32_t)(a[e] >> 32) == no && (uint32_t)(b[e] >> 32) == no;
      if (!ok && __builtin_expect((++tries & ra.check) == 0u, 0) && !res_wait_on(ra, sh.epoch, tries, passed)) {
        sh.dead = 1;
        ok = true;
      }
    } while (!ok);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (i0 + 64u * e + (uint32_t)lane < n) acc += __builtin_bit_cast(double, (b[e] << 32) | (uint32_t)a[e]);
  }
  return res_wave_sum(acc, cols);
}

// The sum over a row's hops, slot by slot, x zero where there is none, in the
// order that the pass's plain kernels use (TileArgs::order): complex64 gives
// the same bits as they do.
// OLO = 0: one by one; slot k is bond k.
// OLO > 0: that of a block decomposition (complex64 from 18 sites on) -- bonds
// below OLO - 1 one by one (slot k is bond k), the active ones of the bonds
// from OLO on in groups of four (the next slots in turn, so that a group ends
// at the same slot in every lane), and bond OLO - 1 with the ring bond (the
// last two slots).
template <typename T, int KMAX, int OLO>
struct HopSum {
  using V = typename Cx<T>::V;
  V hs = {0, 0}, ac = {0, 0}, vd = {0, 0}, vw = {0, 0};
  __device__ __forceinline__ void add(int k, V x) {
    if (OLO == 0 || k < OLO - 1) {
      hs.x += x.x;
      hs.y += x.y;
    } else if (k == KMAX - 1) {
      vw = x;
    } else if (k == KMAX - 2) {
      vd = x;
    } else {
      ac.x += x.x;
      ac.y += x.y;
      if (((k - (OLO - 1)) & 3) == 3) {
        hs.x += ac.x;
        hs.y += ac.y;
        ac.x = ac.y = (T)0;
      }
    }
  }
  __device__ __forceinline__ V total() const {
    if (OLO == 0) return hs;
    V t = {hs.x + ac.x, hs.y + ac.y};
    t.x += vd.x + vw.x;
    t.y += vd.y + vw.y;
    return t;
  }
};

// Rows of the sector as a thread sees them.
struct ResRows {
  const ResArgs& ra;
  const uint32_t* tab;   // binomials, in LDS
  int p;                 // column
  uint32_t size;         // bytes of an element
  // the partner of state s (row r) across bond k, kNoRow if the bond's bits
  // agree; pc: set bits below k
  __device__ __forceinline__ uint32_t partner(uint32_t s, uint32_t r, int k, int pc) const {
    uint32_t q;
    if (k < ra.L - 1) {
      const uint32_t b0 = (s >> k) & 1u;
      const uint32_t c = tab[k * kBinomStride + pc];
      if (b0 == ((s >> (k + 1)) & 1u)) return kNoRow;
      q = b0 ? r + c : r - c;
    } else {
      if (((s ^ (s >> (ra.L - 1))) & 1u) == 0u) return kNoRow;
      q = cns_rank<uint32_t>(s ^ (1u | (1u << (ra.L - 1))), tab);
    }
    return (q * (uint32_t)ra.B + p) * size;
  }
  // offsets of the neighbours by slot (HopSum), kNoRow where there is none:
  // slot k at lo[k * pitch], in LDS, this thread's own
  template <int KMAX, int OLO>
  __device__ __forceinline__ void slots(uint32_t s, uint32_t r, uint32_t* lo, int pitch) const {
    for (int k = 0; k < KMAX; ++k) lo[k * pitch] = kNoRow;
    int pc = 0, n = OLO - 1;
    for (int k = 0; k < ra.nbonds; ++k) {
      const uint32_t o = partner(s, r, k, pc);
      pc += (int)((s >> k) & 1u);
      if (o == kNoRow) continue;
      lo[(OLO == 0 || k < OLO - 1 ? k : k == OLO - 1 ? KMAX - 2 : k == ra.L - 1 ? KMAX - 1 : n++) * pitch] = o;
    }
  }
};

template <typename T, int OLO>
__device__ __forceinline__ typename Cx<T>::V res_w(double d, T g, T ca, T cb,
                                                   typename Cx<T>::V u, typename Cx<T>::V um, typename Cx<T>::V hs) {
  typename Cx<T>::V h, w;
  if (OLO == 0) {
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

// After the recurrence: every work-group computes the step's length and the
// combination's coefficients of all columns for itself, a wave a column (the
// values are the same in all of them).
__device__ __forceinline__ void res_coefs(ResShared& sh, const ResArgs& ra, const KState& st, bool first) {
  const int B = ra.B, m = ra.m, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = (int)blockDim.x >> 6;
  auto tri = [&](int b, int mu) {
    TriLane t;
    t.on = lane < mu;
    t.al = t.on ? sh.al[b * 64 + lane] : 0.0;
    t.be = lane + 1 < mu ? sh.be[b * 64 + lane] : 0.0;
    t.bl = t.on && lane > 0 ? sh.be[b * 64 + lane - 1] : 0.0;
    return t;
  };
  double tau = ra.tau;
  if (ra.tail == kTailAdaptive) {
    for (int b = wave; b < B; b += waves) {
      double next = sh.ok[b] ? ra.tau : NAN, own = ra.tau;
      if (sh.ok[b] && sh.mu[b] == m && m > 1) own = step_size(tri(b, m), m, lane, sh.n0[b] * sh.last[b], ra.tau, ra.tol, next);
      if (lane == 0) {
        sh.sa[b] = own;
        if (first) {
          st.tau[b] = own;
          st.tau[B + b] = next;
        }
      }
    }
    __syncthreads();
    tau = sh.sa[0];
    for (int c = 1; c < B; ++c) tau = fmin(tau, sh.sa[c]);
  }
  for (int b = wave; b < B; b += waves) {
    const int mu = sh.mu[b];
    if (!sh.ok[b] || mu <= 0) {
      if (first && lane == 0) st.err[b] = 0.0;
      continue;
    }
    const TriLane t = tri(b, mu);
    double er, ei;
    tri_expm_e1(t.al, t.be, t.bl, t.on, lane, tau, er, ei);
    const double n0 = sh.n0[b], g = t.on ? n0 * sh.sg[b * 64 + lane] : 0.0;
    sh.al[b * 64 + lane] = g * er;
    sh.be[b * 64 + lane] = g * ei;
    const double end = __shfl(sqrt(er * er + ei * ei), mu - 1);
    if (first && lane == 0) st.err[b] = mu == m ? n0 * sh.last[b] * end : 0.0;
  }
  __syncthreads();
}

// psi of one element i of column p: the combination of the element's own
// entries, which the same thread wrote.
template <typename V>
__device__ __forceinline__ void res_combine(const ResShared& sh, const ResArgs& ra, int p, V* psi, const V* U, size_t i) {
  using T = decltype(V{}.x);
  const int mu = sh.mu[p];
  if (!sh.ok[p] || mu <= 0) return;
  const double* gr = sh.al + p * 64;
  const double* gi = sh.be + p * 64;
  const V x0 = psi[i];
  double ar = gr[0] * (double)x0.x - gi[0] * (double)x0.y;
  double ai = gr[0] * (double)x0.y + gi[0] * (double)x0.x;
  for (int j0 = 1; j0 < mu; j0 += 8) {
    V x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      x[k] = V{0, 0};
      if (j0 + k < mu) x[k] = U[(size_t)(j0 + k - 1) * ra.stride + i];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (j0 + k < mu) {
        const double cr = gr[j0 + k], ci = gi[j0 + k];
        ar += cr * (double)x[k].x - ci * (double)x[k].y;
        ai += cr * (double)x[k].y + ci * (double)x[k].x;
      }
  }
  psi[i] = V{(T)ar, (T)ai};
}

// u_{j+1} of one row, as the update pass forms it; with the component along
// v_{j-1} taken out (er, ei: <v_{j-1}, w> sigma_{j-1}).
template <typename T>
__device__ __forceinline__ typename Cx<T>::V res_next(double c, double d, double er, double ei, typename Cx<T>::V w,
                                                      typename Cx<T>::V u, typename Cx<T>::V um) {
  double nx = c * ((double)w.x - d * (double)u.x);
  double ny = c * ((double)w.y - d * (double)u.y);
  nx -= er * (double)um.x - ei * (double)um.y;
  ny -= er * (double)um.y + ei * (double)um.x;
  typename Cx<T>::V o;
  o.x = (T)nx;
  o.y = (T)ny;
  return o;
}
template <typename T>
__device__ __forceinline__ typename Cx<T>::V res_next(double c, double d, typename Cx<T>::V w, typename Cx<T>::V u) {
  typename Cx<T>::V o;
  o.x = (T)(c * ((double)w.x - d * (double)u.x));
  o.y = (T)(c * ((double)w.y - d * (double)u.y));
  return o;
}

// What lane b < B of the first wave keeps of column b over the iterations.
struct ResCol {
  double sigma = 0.0, before = 0.0;              // sigma_j, sigma_{j-1}
  double smax = 0.0, alpha = 0.0;                // the largest coefficient so far, alpha_j
};

// By the first wave, after exchange A of iteration j (lane q * Bp + b holds S_q
// of column b): alpha_j and the factors of the update.  `first`: the work-group
// that records the shared results.
__device__ __forceinline__ void res_alpha(ResShared& sh, const ResArgs& ra, const KState& st, int j, bool first,
                                          double S, ResCol& col) {
  const int b = threadIdx.x, B = ra.B, Bp = 1 << ra.lbp;
  // second and third quantity: |u_0|^2, or <u_{j-1}, w> to reorthogonalise
  const double S2 = __shfl(S, (b + Bp) & 63), S3 = __shfl(S, (b + 2 * Bp) & 63);
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
      sh.n0[b] = n0;
      sh.sg[b * 64] = c;
      if (first) {
        st.n0[b] = n0;
        st.sigma[b] = c;
      }
      if (!(n0 > 0.0)) {
        active = 0;   // zero vector: nothing to propagate
        sh.mu[b] = 0;
        if (!isfinite(S2)) sh.ok[b] = 0;
        if (first) {
          st.mused[b] = 0;
          if (!isfinite(S2)) st.status[b] = QK_ENUMERIC;
        }
      }
    } else {
      col.alpha = col.sigma * S;
      c = 1.0;
      d = col.alpha * col.sigma;
      sh.ser[b] = col.before * col.before * S2;
      sh.sei[b] = col.before * col.before * S3;
    }
    if (active && !isfinite(col.alpha)) {
      active = 0;
      sh.ok[b] = 0;
      if (first) {
        st.status[b] = QK_ENUMERIC;
        st.mused[b] = j;
      }
    }
    sh.al[b * 64 + j] = col.alpha;
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
      sh.last[b] = beta;
      if (first) ra.norm2[b] = norm2;
      if (first && sh.ok[b] && sh.mu[b] == ra.m) st.beta[j * B + b] = beta;
    } else {
      if (active) {
        col.smax = fmax(fmax(col.smax, fabs(col.alpha)), beta);
        if (!isfinite(beta)) {
          active = 0;
          sh.ok[b] = 0;
          if (first) {
            st.status[b] = QK_ENUMERIC;
            st.mused[b] = j + 1;
          }
        } else if (beta <= ra.rtol * col.smax) {
          active = 0;   // invariant subspace
          sh.mu[b] = j + 1;
          if (first) st.mused[b] = j + 1;
        }
        sh.be[b * 64 + j] = beta;
        if (first) st.beta[j * B + b] = beta;
      }
      if (active) {
        sh.sa[b] = 1.0 / beta;
        sh.sb[b] = beta * col.sigma;
        col.before = col.sigma;
        col.sigma = 1.0 / beta;
        sh.sg[b * 64 + j + 1] = col.sigma;
        if (first) st.sigma[(j + 1) * B + b] = col.sigma;
      }
      sh.act[b] = active;
    }
  }
  const bool any = __any(b < B && sh.act[b] != 0);
  if (b == 0) sh.go = any && !sh.dead && j + 1 < ra.m;
}

// Diagonal of state s in column p.
__device__ __forceinline__ double res_diag(const ResArgs& ra, uint32_t s, const double* f) {
  double hh = 0.0;
  for (int i = 0; i < ra.L; ++i) hh += f[i];
  ModelArgs ma;
  ma.L = ra.L;
  ma.pbc = ra.pbc;
  ma.jz = ra.jz;
  ma.lmask = (1ull << ra.L) - 1ull;
  return diag_value<uint32_t>(s, ma, f, 0.5 * hh);
}

// Whether the form of NT threads goes on to the exponential and the combination.
// Their code costs the largest complex128 work-groups registers in the loop:
// the step of the 20-site ring took 337 us with them, 325 us with the kernels
// that the passes use.
template <typename T, int NT>
constexpr bool resident_tail = !(NT > 512 && std::is_same<T, double>::value);

// Loads of LOADS neighbours are in flight at a time, as many as the registers of
// a thread hold beside everything else: all of them with two waves a SIMD
// (L = 18: 3.7 us an iteration in three batches, 1.2 at once), seven with three.
// LATE: u_{j+1} itself is published, with the second exchange, and gathered
// after it.  Local reorthogonalisation takes it: the other form would need
// u_{j-1} at the neighbours as well.  The gather no longer runs beside the
// exchange (L = 20, 330 against 410 us a step), so nothing else does.
template <typename T, int KMAX, int OLO, int NT, int LOADS, bool LATE>
__global__ void __launch_bounds__(NT, NT / 256)
k_resident(ResArgs ra, typename Cx<T>::V* psi, typename Cx<T>::V* U, typename Cx<T>::V* X, KState st) {
  using V = typename Cx<T>::V;
  __shared__ ResShared sh;
  // offsets of the neighbours: three waves a SIMD leave no registers for them
  constexpr bool LDSOFF = NT > 512;
  constexpr bool TAIL = resident_tail<T, NT>;
  __shared__ uint32_t lo[KMAX * NT];
  const int tid = threadIdx.x, nt = blockDim.x, B = ra.B, Bp = 1 << ra.lbp, p = tid & (Bp - 1);
  const uint32_t G = ra.groups;
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
  const bool late = (ticket & kClosed) != 0 || ticket >= (uint32_t)ra.join_max;
  uint32_t R = 0;
  if (!late) {
    const double* f = ra.fields + (size_t)(p < B ? p : 0) * ra.L;
    const T g = (T)ra.half_jxy;
    const ResRows rows{ra, sh.tab, p, (uint32_t)sizeof(V)};
    // this thread's row
    const uint32_t row = (ticket * (uint32_t)nt + (uint32_t)tid) >> ra.lbp;
    const bool has = row < ra.D && p < B;
    const uint32_t eo = has ? (row * (uint32_t)B + p) * (uint32_t)sizeof(V) : kNoRow;
    const uint32_t state = has ? ra.states[row] : 0u;
    rows.template slots<KMAX, OLO>(state, row, lo + tid, NT);
    const double d = has ? res_diag(ra, state, f) : 0.0;
    const ResBuf<V> bpsi(psi, nel);
    V u = bpsi.template ld<0>(eo), um = {0, 0};
    V un[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) un[k] = bpsi.template ld<0>(lo[k * NT + tid]);
    uint32_t off[LDSOFF ? 1 : KMAX];
#pragma unroll
    for (int k = 0; k < (LDSOFF ? 0 : KMAX); ++k) off[k] = lo[k * NT + tid];
    if (tid == 0) {
      if (ticket == 0) {
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
        uint32_t tries = 0;
        for (;;) {
          w = word_ld(&ra.ctl->joined);
          if ((uint32_t)(w >> 32) == epoch && (uint32_t)w != 0u) break;
          if (!res_wait_on(ra, epoch, ++tries, false)) {
            sh.dead = 1;
            w = 0;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
        sh.joined = (uint32_t)w;
      }
    }
    if (tid < B) {
      sh.sa[tid] = 1.0;
      sh.sb[tid] = 0.0;
      sh.act[tid] = 1;
      sh.mu[tid] = ra.m;
      sh.ok[tid] = 1;
    }
    __syncthreads();
    R = ticket < sh.joined ? sh.joined : 0u;   // 0: not among the registered
    const bool first = ticket == 0;
    if (first && tid < B) {
      st.mused[tid] = ra.m;
      st.status[tid] = QK_OK;
    }
    ResCol col;
    const bool wave0 = tid < 64;
    uint32_t no = epoch;
    if (R == G) {
      // every row has its thread: vectors in registers
      for (int j = 0; j < ra.m; ++j) {
        const bool mine = p < B && sh.act[p] != 0;
        const T ca = mine ? (T)sh.sa[p] : (T)0, cb = mine ? (T)sh.sb[p] : (T)0;
        HopSum<T, KMAX, OLO> sum;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) sum.add(k, un[k]);
        const V w = res_w<T, OLO>(d, g, ca, cb, u, um, sum.total());
        const ResBuf<V> bx(X + (size_t)(j & 1) * nel, nel);
        const bool ro = LATE && ra.reorth && j > 0;
        if (!LATE && mine) bx.template st<kSc1>(eo, w);
        const bool on = mine && has;
        const double s1 = on ? (double)u.x * (double)w.x + (double)u.y * (double)w.y : 0.0;
        if (j == 0) {
          const double v[2] = {s1, on ? (double)u.x * (double)u.x + (double)u.y * (double)u.y : 0.0};
          res_partials<2, !LATE>(sh, ra, v);
        } else if (ro) {
          const double v[4] = {s1, on ? (double)um.x * (double)w.x + (double)um.y * (double)w.y : 0.0,
                               on ? (double)um.x * (double)w.y - (double)um.y * (double)w.x : 0.0, 0.0};
          res_partials<4, false>(sh, ra, v);
        } else {
          const double v[1] = {s1};
          res_partials<1, !LATE>(sh, ra, v);
        }
        if (wave0) {
          const int Q = j == 0 ? 2 : ro ? 4 : 1;
          res_publish(sh, ra, Q, no, G, ticket);
          res_alpha(sh, ra, st, j, first, res_collect(sh, ra, Q, no, G), col);
        }
        __syncthreads();
        const bool live = p < B && sh.act[p] != 0;
        const double c = live ? sh.sc[p] : 0.0, dd = live ? sh.sd[p] : 0.0;
        V o;
        if (ro) o = res_next<T>(c, dd, live ? sh.ser[p] : 0.0, live ? sh.sei[p] : 0.0, w, u, um);
        else o = res_next<T>(c, dd, w, u);
        if (LATE && live && j + 1 < ra.m) bx.template st<kSc1>(eo, o);
        const double v[1] = {live && has ? (double)o.x * (double)o.x + (double)o.y * (double)o.y : 0.0};
        res_partials<1, LATE>(sh, ra, v);
        if (wave0) res_publish(sh, ra, 1, no + 1, G, ticket);
        if (j + 1 < ra.m) {
          if (live) ResBuf<V>(U + (size_t)j * ra.stride, nel).template st<0>(eo, o);
          // w at the neighbours, while the sums are under way
#pragma unroll
          for (int k0 = 0; k0 < (LATE ? 0 : KMAX); k0 += LATE ? 1 : LOADS) {
            V x[LATE ? 1 : LOADS];
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
              if (k0 + i < KMAX) x[i] = bx.template ld<kSc1>(LDSOFF ? lo[(k0 + i) * NT + tid] : off[LDSOFF ? 0 : k0 + i]);
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
              if (k0 + i < KMAX) un[k0 + i] = res_next<T>(c, dd, x[i], un[k0 + i]);
            __asm__ volatile("" ::: "memory");   // no more loads in flight than that
          }
        }
        um = u;
        u = o;
        // |u_m| is needed for the error estimate only
        if (wave0)
          res_beta(sh, ra, st, j, first,
                   j + 1 < ra.m || first || ra.tail == kTailAdaptive ? res_collect(sh, ra, 1, no + 1, G, j + 1 == ra.m)
                                                                     : 0.0,
                   col);
        no += 2;
        __syncthreads();
        if (!sh.go) break;
        if (LATE)
#pragma unroll
          for (int k = 0; k < KMAX; ++k) un[k] = bx.template ld<kSc1>(LDSOFF ? lo[k * NT + tid] : off[LDSOFF ? 0 : k]);
      }
    } else if (R != 0) {
      // rows of missing work-groups are dealt out: vectors in memory, agent scope
      for (int j = 0; j < ra.m; ++j) {
        const ResBuf<V> bu(j == 0 ? psi : U + (size_t)(j - 1) * ra.stride, nel);
        const ResBuf<V> bm(j <= 1 ? psi : U + (size_t)(j - 2) * ra.stride, nel);
        const ResBuf<V> bx(X, nel), bo(U + (size_t)j * ra.stride, nel);
        const bool mine = p < B && sh.act[p] != 0;
        const T ca = mine ? (T)sh.sa[p] : (T)0, cb = mine ? (T)sh.sb[p] : (T)0;
        const bool ro = LATE && ra.reorth && j > 0;
        const int Q = j == 0 ? 2 : ro ? 4 : 1;
        for (uint32_t ch = ticket; ch < G; ch += R) {
          const uint32_t r = (ch * (uint32_t)nt + (uint32_t)tid) >> ra.lbp;
          const bool on = r < ra.D && mine;
          const uint32_t e = on ? (r * (uint32_t)B + p) * (uint32_t)sizeof(V) : kNoRow;
          const uint32_t s = on ? ra.states[r] : 0u;
          const V x = bu.template ld<kSc1>(e);
          V xm = {0, 0};
          if (j > 0) xm = bm.template ld<kSc1>(e);
          HopSum<T, KMAX, OLO> sum;
          rows.template slots<KMAX, OLO>(s, r, lo + tid, NT);
#pragma unroll 1
          for (int k = 0; k < KMAX; ++k) sum.add(k, bu.template ld<kSc1>(lo[k * NT + tid]));
          const V w = res_w<T, OLO>(on ? res_diag(ra, s, f) : 0.0, g, ca, cb, x, xm, sum.total());
          bx.template st<kSc1>(e, w);
          const double s1 = on ? (double)x.x * (double)w.x + (double)x.y * (double)w.y : 0.0;
          if (ro) {
            const double v[4] = {s1, on ? (double)xm.x * (double)w.x + (double)xm.y * (double)w.y : 0.0,
                                 on ? (double)xm.x * (double)w.y - (double)xm.y * (double)w.x : 0.0, 0.0};
            res_partials<4, true>(sh, ra, v);
          } else {
            const double v[2] = {s1, on ? (double)x.x * (double)x.x + (double)x.y * (double)x.y : 0.0};
            res_partials<2, true>(sh, ra, v);
          }
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
          const V w = bx.template ld<kSc1>(e), x = bu.template ld<kSc1>(e);
          V o;
          if (ro) o = res_next<T>(c, dd, live ? sh.ser[p] : 0.0, live ? sh.sei[p] : 0.0, w, x, bm.template ld<kSc1>(e));
          else o = res_next<T>(c, dd, w, x);
          if (j + 1 < ra.m) bo.template st<kSc1>(e, o);
          const double v[1] = {on ? (double)o.x * (double)o.x + (double)o.y * (double)o.y : 0.0};
          res_partials<1, true>(sh, ra, v);
          if (wave0) res_publish(sh, ra, 1, no + 1, G, ch);
          __syncthreads();
        }
        if (wave0)
          res_beta(sh, ra, st, j, first,
                   j + 1 < ra.m || first || ra.tail == kTailAdaptive ? res_collect(sh, ra, 1, no + 1, G, j + 1 == ra.m)
                                                                     : 0.0,
                   col);
        no += 2;
        __syncthreads();
        if (!sh.go) break;
      }
    }
    if (R != 0) {
      // read by the last thread, whose wave has no column unless there are as many as waves,
      // while the coefficients are computed
      const bool tail = TAIL && ra.tail != kTailNone;
      uint64_t word = 0;
      if (tid == nt - 1) word = word_ld((const uint64_t*)&ra.ctl->verdict);
      if (tail && !sh.dead) res_coefs(sh, ra, st, first);
      if (tid == nt - 1) sh.combine = !sh.dead && res_goes_on(ra, epoch, word);
      __syncthreads();
      const bool go = sh.combine != 0;
      for (uint32_t ch = tail && go ? ticket : G; ch < G; ch += R) {   // its own row only where R == G
        const uint32_t r = (ch * (uint32_t)nt + (uint32_t)tid) >> ra.lbp;
        if (r < ra.D && p < B) res_combine(sh, ra, p, psi, U, (size_t)r * B + p);
      }
      if (first && !go && tid < B) {
        st.status[tid] = QK_ENUMERIC;
        st.err[tid] = 0.0;
        st.tau[tid] = st.tau[B + tid] = NAN;
      }
    }
  }
  // the last work-group, late ones included, makes room for the next launch
  if (tid == 0 &&
      __hip_atomic_fetch_add(&ra.ctl->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == G - 1) {
    __hip_atomic_store(&ra.ctl->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&ra.ctl->left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word_st(&ra.ctl->joined, 0ull);
    __hip_atomic_store(&ra.ctl->epoch, epoch - 1u + 2u * (uint32_t)ra.m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Rows that fit one work-group: nothing leaves it but the basis.  The current
// vector lies in LDS; sums go through LDS once, and every thread computes its
// column's scalars for itself, so an iteration has two barriers.
constexpr int kOneThreads = 1024;
template <typename T, int KMAX, int OLO>
__global__ void __launch_bounds__(kOneThreads)
k_resident_one(ResArgs ra, typename Cx<T>::V* psi, typename Cx<T>::V* U, KState st) {
  using V = typename Cx<T>::V;
  __shared__ ResShared sh;
  __shared__ uint32_t lo[KMAX * kOneThreads];
  __shared__ V ul[kOneThreads + 1];                        // u_j of the rows, and a zero
  __shared__ double red[2][3 * kOneThreads / 64 * kResMaxLanes];   // of the two sums in turn
  const int tid = threadIdx.x, nt = blockDim.x, B = ra.B, Bp = 1 << ra.lbp, p = tid & (Bp - 1);
  const int lane = tid & 63, wave = tid >> 6, waves = nt >> 6;
  for (int i = tid; i < kBinomStride * kBinomStride; i += nt) sh.tab[i] = ra.bn[i];
  const uint32_t row = (uint32_t)tid >> ra.lbp;
  const bool has = row < ra.D && p < B;
  const size_t e = (size_t)row * B + p;
  const uint32_t state = has ? ra.states[row] : 0u;
  V u = has ? psi[e] : V{0, 0}, um = {0, 0};
  ul[tid] = u;
  if (tid == 0) {
    ul[nt] = V{0, 0};
    sh.dead = 0;
  }
  __syncthreads();
  const double* f = ra.fields + (size_t)(p < B ? p : 0) * ra.L;
  const T g = (T)ra.half_jxy;
  uint32_t off[KMAX];   // places in ul
  {
    ResArgs one = ra;
    one.B = Bp;   // columns of ul
    ResRows{one, sh.tab, p, 1u}.template slots<KMAX, OLO>(state, row, lo + tid, kOneThreads);
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      off[k] = lo[k * kOneThreads + tid];
      if (off[k] == kNoRow) off[k] = (uint32_t)nt;
    }
  }
  const double d = has ? res_diag(ra, state, f) : 0.0;
  // the sum over the work-group of one quantity of a column, its per-wave sums
  // in r[wave * Bp + column]
  auto total = [&](const double* r) -> double {
    if (Bp == 1) {
      double v = lane < waves ? r[lane] : 0.0;   // at most 16
      v = dpp_add<0x111, 0xf>(v);
      v = dpp_add<0x112, 0xf>(v);
      v = dpp_add<0x114, 0xf>(v);
      v = dpp_add<0x118, 0xf>(v);
      const uint64_t b = __builtin_bit_cast(uint64_t, v);
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 15);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 15);
      return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    }
    double t = 0.0;
    for (int w = 0; w < waves; ++w) t += r[w * Bp + p];
    return t;
  };
  const bool rec = tid < B;   // records its column's results
  bool act = p < B, ok = true;
  int mu = ra.m;
  double sa = 1.0, sb = 0.0, sigma = 0.0, before = 0.0, smax = 0.0, n0 = 0.0, last = 0.0;
  for (int j = 0; j < ra.m; ++j) {
    const T ca = act ? (T)sa : (T)0, cb = act ? (T)sb : (T)0;
    HopSum<T, KMAX, OLO> sum;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) sum.add(k, ul[off[k]]);
    const V w = res_w<T, OLO>(d, g, ca, cb, u, um, sum.total());
    const bool on = act && has;
    const double t1 = res_wave_sum(on ? (double)u.x * (double)w.x + (double)u.y * (double)w.y : 0.0, Bp);
    if (lane < Bp) red[0][wave * Bp + lane] = t1;
    if (j == 0) {
      const double t2 = res_wave_sum(on ? (double)u.x * (double)u.x + (double)u.y * (double)u.y : 0.0, Bp);
      if (lane < Bp) red[0][(waves + wave) * Bp + lane] = t2;
    }
    const bool ro = ra.reorth && j > 0;
    if (ro) {
      const double t3r = res_wave_sum(on ? (double)um.x * (double)w.x + (double)um.y * (double)w.y : 0.0, Bp);
      const double t3i = res_wave_sum(on ? (double)um.x * (double)w.y - (double)um.y * (double)w.x : 0.0, Bp);
      if (lane < Bp) {
        red[0][(waves + wave) * Bp + lane] = t3r;
        red[0][(2 * waves + wave) * Bp + lane] = t3i;
      }
    }
    __syncthreads();
    const double S = total(red[0]);
    double c = 1.0, dd, alpha;
    if (j == 0) {
      const double S2 = total(red[0] + waves * Bp);
      n0 = sqrt(S2);
      alpha = S / S2;
      c = 1.0 / n0;
      dd = alpha;
      sigma = c;
      if (act && !(n0 > 0.0)) {
        act = false;   // zero vector: nothing to propagate
        mu = 0;
        if (!isfinite(S2)) ok = false;
      }
    } else {
      alpha = sigma * S;
      dd = alpha * sigma;
    }
    if (act && !isfinite(alpha)) {
      act = false;
      ok = false;
      mu = j;
    }
    const double sj = sigma;
    V o = {0, 0};
    if (ro) {
      const double er = before * before * total(red[0] + waves * Bp), ei = before * before * total(red[0] + 2 * waves * Bp);
      if (act) o = res_next<T>(c, dd, er, ei, w, u, um);
    } else if (act) {
      o = res_next<T>(c, dd, w, u);
    }
    ul[tid] = o;
    if (act && has && j + 1 < ra.m) U[(size_t)j * ra.stride + e] = o;
    const double t3 = res_wave_sum(act && has ? (double)o.x * (double)o.x + (double)o.y * (double)o.y : 0.0, Bp);
    if (lane < Bp) red[1][wave * Bp + lane] = t3;
    if (rec && act) {
      sh.al[tid * 64 + j] = alpha;
      sh.sg[tid * 64 + j] = sj;
    }
    __syncthreads();
    um = u;
    u = o;
    const double beta = sqrt(total(red[1]));
    if (j + 1 == ra.m) {
      last = beta;
    } else if (act) {
      smax = fmax(fmax(smax, fabs(alpha)), beta);
      if (rec) sh.be[tid * 64 + j] = beta;
      if (!isfinite(beta)) {
        act = false;
        ok = false;
        mu = j + 1;
      } else if (beta <= ra.rtol * smax) {
        act = false;   // invariant subspace
        mu = j + 1;
      } else {
        sb = beta * sigma;
        sa = 1.0 / beta;
        before = sigma;
        sigma = sa;
      }
    }
    // every wave holds every column: the same answer in all of them
    if (!__any(act)) break;
  }
  if (rec) {
    const int b = tid;
    sh.mu[b] = mu;
    sh.ok[b] = ok ? 1 : 0;
    sh.n0[b] = n0;
    sh.last[b] = last;
    st.mused[b] = mu;
    st.status[b] = ok ? QK_OK : QK_ENUMERIC;
    st.n0[b] = n0;
    if (ok && mu == ra.m) sh.be[b * 64 + ra.m - 1] = last;
  }
  __syncthreads();
  for (int i = tid; i < B * 64; i += nt) {
    const int b = i >> 6, j = i & 63, n = sh.mu[b];
    if (j < n) {
      st.alpha[j * B + b] = sh.al[i];
      st.sigma[j * B + b] = sh.sg[i];
      if (j + 1 < n || (sh.ok[b] && n == ra.m)) st.beta[j * B + b] = sh.be[i];
    }
  }
  if (ra.tail == kTailNone) return;
  __syncthreads();
  res_coefs(sh, ra, st, true);
  if (has) res_combine(sh, ra, p, psi, U, e);
}

// ------------------------------------------------------------------- host
// Lanes of a workspace's rows, 0 if the resident recurrence does not cover it
// (that of the two-pass split has no d_res either).
static uint64_t resident_lanes(const qk_krylov* k) {
  const qk_ham* H = k->H;
  if (H->p.mode != QK_MATFREE || H->basis->L > kResMaxSites || k->reorth > 1) return 0;
  uint64_t Bp = 1;
  while (Bp < (uint64_t)k->batch) Bp *= 2;
  const uint64_t lanes = (uint64_t)k->D * Bp;
  return Bp <= (uint64_t)kResMaxLanes && lanes <= (uint64_t)kResMaxThreads * kResMaxGroups ? lanes : 0;
}

// Threads per work-group and work-groups for a number of lanes; one work-group
// is the form of its own.  Otherwise 256 threads up to 256 work-groups, then
// larger work-groups.
struct ResShape {
  int threads, groups;
};

static ResShape resident_shape(uint64_t lanes, uint64_t per_row) {
  if (lanes <= (uint64_t)kOneThreads) return {(int)((lanes + 63) / 64) * 64, 1};
  int nt = 256;
  while (nt < 512 && (lanes + nt - 1) / nt * per_row > 256) nt += 64;   // one round of the wave that collects
  if (lanes > (uint64_t)nt * kResMaxGroups) nt = (int)((lanes + kResMaxGroups * 64 - 1) / (kResMaxGroups * 64)) * 64;
  return {nt, (int)((lanes + nt - 1) / nt)};
}

void resident_bytes(const qk_krylov* k, size_t* head, size_t* body) {
  *head = *body = 0;
  const uint64_t lanes = resident_lanes(k);
  if (!lanes) return;
  const size_t per_row = (size_t)(lanes / (uint64_t)k->D);
  const ResShape sp = resident_shape(lanes, per_row);
  *head = sizeof(ResCtl);
  if (sp.groups == 1) return;
  *head += sizeof(uint64_t) * (size_t)2 * sp.groups * (k->reorth ? 4 : 2) * per_row * 2;
  *body = (size_t)2 * k->D * k->batch * (k->dtype == QK_C128 ? 16 : 8);
}

struct ResLaunch {
  ResArgs ra;
  ResShape sp;
  void *psi, *U, *X;
  KState st;
  hipStream_t s;
  int* occupancy = nullptr;   // not NULL: receives the work-groups that a compute unit holds, instead of a launch
  template <typename T, int KMAX, int OLO>
  void one() const {
    using V = typename Cx<T>::V;
    hipLaunchKernelGGL((k_resident_one<T, KMAX, OLO>), dim3(1), dim3(sp.threads), 0, s, ra, (V*)psi, (V*)U, st);
  }
  template <typename T, int KMAX, int OLO, int NT, int LOADS>
  void many() const {
    using V = typename Cx<T>::V;
    if (occupancy) {
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(occupancy, k_resident<T, KMAX, OLO, NT, LOADS, LOADS == 0>,
                                                       sp.threads, 0) != hipSuccess)
        *occupancy = 1;
      return;
    }
    hipLaunchKernelGGL((k_resident<T, KMAX, OLO, NT, LOADS, LOADS == 0>), dim3(sp.groups), dim3(sp.threads), 0, s, ra,
                       (V*)psi, (V*)U, (V*)X, st);
  }
  // the bonds that a thread keeps registers for: 14, 17 or 20; no loads beside
  // the neighbours' values where they are gathered late
  template <typename T, int OLO>
  void go() const {
    constexpr int LOADS = std::is_same<T, double>::value ? 7 : 20;   // of the largest work-groups
    const bool late = ra.reorth != 0;
    if (sp.groups == 1) {
      if (OLO == 0 && ra.nbonds <= 14) one<T, 14, 0>();
      else one<T, 20, OLO>();
    } else if (sp.threads <= 512) {
      if (OLO == 0 && ra.nbonds <= 17 && late) many<T, 17, 0, 512, 0>();
      else if (late) many<T, 20, OLO, 512, 0>();
      else if (OLO == 0 && ra.nbonds <= 14) many<T, 14, 0, 512, 14>();
      else if (OLO == 0 && ra.nbonds <= 17) many<T, 17, 0, 512, 17>();
      else many<T, 20, OLO, 512, 20>();
    } else {
      if (late) many<T, 20, OLO, kResMaxThreads, 0>();
      else many<T, 20, OLO, kResMaxThreads, LOADS>();
    }
  }
};

// Low bits of the decomposition whose order complex64 follows, 0: none.
static int resident_olo(const qk_krylov* k) { return k->dtype == QK_C128 || k->H->llo <= 0 ? 0 : k->H->llo; }

// Whether the next step takes it: a decomposition that the caller has chosen
// (qk_launch_shape) may ask for an order of summation that it has no form for.
bool resident_covers(const qk_krylov* k) {
  const int olo = resident_olo(k);
  return k->d_res && (olo == 0 || olo == 9 || olo == 10);
}

const uint32_t* resident_verdict(const qk_krylov* k) { return k->d_res ? &((const ResCtl*)k->d_res)->verdict : nullptr; }

bool resident_gave_up(const qk_krylov* k) {
  uint32_t v = 0;
  return k->d_res && hipMemcpy(&v, resident_verdict(k), sizeof v, hipMemcpyDeviceToHost) == hipSuccess && v == kResGaveUp;
}

int resident_groups(const qk_krylov* k) {
  if (!resident_covers(k)) return 0;
  const uint64_t lanes = resident_lanes(k);
  return resident_shape(lanes, lanes / (uint64_t)k->D).groups;
}

// Steps on several streams.  Two launches that find no place together on the
// compute units and come at the same time get a part of their work-groups in
// each: both wait for the rest (kJoinTicks), then run dealt out.  Three streams
// with the 19-site ring took 4.5 ms for a step each that way, four with 20 sites
// 6 to 7 ms; one after another they take 0.79 and 1.33 ms (by the passes of an
// earlier version, side by side, 1.03 and 1.19 ms).  So a launch waits, on the
// device, for those on other streams that it does not fit beside, the latest
// ones first in the places: of the others a second chipful is waited for,
// which has itself waited for what came before.  Workspaces that all fit, or
// are used on one stream, pay nothing, nor do the members of a batch among
// themselves and other batches on the same stream: their streams are forked from
// it, and batch_beside has seen to their places (with an event each they took
// 0.43 ms a step instead of 0.41: 15 sites with 8 phases beside 14, 10 and 12).
// A captured launch is not ordered (its replays come when they come), nor are
// other processes.
static std::mutex g_order_mu;
static qk_krylov* g_order_head = nullptr;   // latest launch first

static void order_unlink(qk_krylov* k) {
  if (k->res_prev) k->res_prev->res_next = k->res_next;
  else if (g_order_head == k) g_order_head = k->res_next;
  if (k->res_next) k->res_next->res_prev = k->res_prev;
  k->res_prev = k->res_next = nullptr;
}

static void order_front(qk_krylov* k) {
  k->res_next = g_order_head;
  if (g_order_head) g_order_head->res_prev = k;
  g_order_head = k;
}

void resident_register(qk_krylov* k) {
  if (!k->d_res || resident_groups(k) <= 1) return;
  std::lock_guard<std::mutex> lk(g_order_mu);
  order_front(k);
}

void resident_unregister(qk_krylov* k) {
  std::lock_guard<std::mutex> lk(g_order_mu);
  order_unlink(k);
  if (k->res_event) (void)hipEventDestroy(k->res_event);
  k->res_event = nullptr;
}

// Under the mutex, before a launch on s (forked from `from`): the waits; returns
// whether an event is to be recorded after it.
static bool resident_order(qk_krylov* k, hipStream_t s, hipStream_t from) {
  const int cus = qk_num_cus();
  auto beside = [&](const qk_krylov* o) {   // may run while this launch does
    return o != k && o->res_launched && o->device == k->device && o->res_stream != from;
  };
  int all = k->res_share;
  for (const qk_krylov* o = g_order_head; o; o = o->res_next)
    if (beside(o)) all += o->res_share;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  const bool several = all > cus;
  if (several && (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone)) {
    (void)hipGetLastError();
    return false;
  }
  int with = k->res_share, after = 0;
  for (const qk_krylov* o = several ? g_order_head : nullptr; o && after <= cus; o = o->res_next) {
    if (!beside(o)) continue;
    if (with + o->res_share <= cus) {
      with += o->res_share;
    } else {
      after += o->res_share;
      if (o->res_event && hipStreamWaitEvent(s, o->res_event, 0) != hipSuccess) (void)hipGetLastError();
    }
  }
  k->res_stream = from;
  k->res_launched = true;
  order_unlink(k);
  order_front(k);
  return several;
}

qk_status launch_resident(qk_krylov* k, void* psi, double rtol, double tau, StepUpTo upto, const AdaptiveStep* ad,
                          hipStream_t s, hipStream_t from, bool* done) {
  const qk_ham* H = k->H;
  ResLaunch rl{};
  const uint64_t lanes = resident_lanes(k);
  rl.sp = resident_shape(lanes, lanes / (uint64_t)k->D);
  ResArgs& ra = rl.ra;
  ra.L = H->basis->L;
  ra.pbc = H->p.pbc;
  ra.B = k->batch;
  while ((1 << ra.lbp) < k->batch) ++ra.lbp;
  ra.m = k->m;
  ra.reorth = k->reorth;
  ra.qcap = k->reorth ? 4 : 2;
  ra.nbonds = ra.pbc ? ra.L : ra.L - 1;
  ra.D = (uint32_t)k->D;
  ra.groups = rl.sp.groups;
  ra.join_max = k->res_join > 0 ? std::min(ra.groups, k->res_join) : ra.groups;
  // a wait looks at its limit when the count of its polls is a multiple of check + 1, so the limit is one
  ra.check = k->res_polls >= 1024u ? 1023u : 0u;
  ra.polls = k->res_polls & ~ra.check;
  ra.half_jxy = 0.5 * H->p.jxy;
  ra.jz = H->p.jz;
  ra.rtol = rtol;
  ra.states = (const uint32_t*)H->basis->d_states;
  ra.bn = H->basis->d_binom;
  ra.fields = H->d_fields;
  ra.stride = k->ustride;
  ra.ctl = (ResCtl*)k->d_res;
  ra.words = (uint64_t*)((char*)k->d_res + sizeof(ResCtl));
  const bool whole = k->dtype != QK_C128 || rl.sp.threads <= 512 || rl.sp.groups == 1;   // resident_tail
  ra.tail = !whole || upto == StepUpTo::basis ? kTailNone : ad ? kTailAdaptive : kTailStep;
  ra.norm2 = k->d_partB;
  *done = whole || upto == StepUpTo::basis;
  ra.tau = tau;
  ra.tol = ad ? ad->tol : 0.0;
  rl.psi = psi;
  rl.U = k->d_U;
  rl.X = k->d_X;
  rl.st = make_kstate(k);
  rl.s = s;
  const int olo = resident_olo(k);
  auto go = [&] {
    if (k->dtype == QK_C128) rl.go<double, 0>();
    else if (olo == 0) rl.go<float, 0>();
    else if (olo == 9) rl.go<float, 9>();
    else rl.go<float, 10>();
  };
  if (ra.groups == 1) {
    go();
    QK_HIP(hipGetLastError());
    return QK_OK;
  }
  std::lock_guard<std::mutex> lk(g_order_mu);
  if (k->res_share == 0) {
    int occ = 1;
    rl.occupancy = &occ;
    go();
    rl.occupancy = nullptr;
    k->res_share = (ra.groups + std::max(1, occ) - 1) / std::max(1, occ);
  }
  const bool record = resident_order(k, s, from);
  go();
  QK_HIP(hipGetLastError());
  if (record) {
    if (!k->res_event) QK_HIP(hipEventCreateWithFlags(&k->res_event, hipEventDisableTiming));
    QK_HIP(hipEventRecord(k->res_event, s));
  }
  return QK_OK;
}

}  // namespace qk
