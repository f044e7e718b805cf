// Tiled matrix-free H x (Sec. 3 "Hamiltonian matrix construction", Eq. (1)),
// used by qk_ham_apply and the H-pass of every Lanczos iteration.
//
// A state splits into top, middle and low bits (T, M, l of them).  The sorted
// basis lists the states of one top and middle pattern as one block of
// consecutive rows, the low states of one popcount in ascending order.  A tile
// is the C(M, km) blocks of one top pattern with km middle and kl low
// particles; all tiles of a class (kl, km) have the same size and the same
// hops inside:
//   * a hop on a low bond stays in the block, at a rank that depends only on
//     the low state: each lane of a work-group keeps one low state for the
//     whole class, with the LDS offsets of its (at most l - 1) low partners in
//     registers, so a row costs one LDS read and two adds per low hop and no
//     index arithmetic;
//   * a hop on a middle bond goes to another block of the tile at the same
//     rank: one LDS read at a uniform distance;
//   * a hop on a top bond goes to another tile of the same class at the same
//     position: one uniform row shift per hop, a contiguous run of x;
//   * the bonds joining low and middle, middle and top, and the ring bond go
//     to blocks whose positions are uniform, at a rank fixed per lane.
// A work-group (512 lanes) takes one item: a tile of a large class, or several
// tiles of a small one.  It stages the item's rows in LDS, then walks its
// blocks; the records that a block's waves share are read with scalar loads,
// the next block's ahead of time, and vectors through buffer descriptors
// (uniform offset in a scalar register, 32-bit lane offset).  Items of a class
// have equal work, classes come in the order of their items' cost, and
// work-group w takes items w, w + G, ...: the work-groups end together.
//
// What bounds it: reads that miss the L2.  At L = 28 (complex128) a row still
// gathers about 5.7 top partners and the joining and ring partners, 4.7 GB per
// H x of 1.28 GB algorithmic, at 7.2 TB/s out of the last-level cache and HBM
// (a copy in the last-level cache reaches 7.2).  Instructions per row and wave:
// 100 vector, 120 scalar.  Against the kernel that it took the place of (blocks
// of 2^11 low states, one LDS lookup of every bond's rank per row): H x of
// L = 28 0.94 -> 0.74 ms in complex128, 0.48 -> 0.39 ms in complex64 (1.7 and
// 1.6 TB/s algorithmic); L = 20 with 64 columns in complex64 0.131 -> 0.099 ms.
// Measured and not kept: tops in ascending order with the classes of a top
// pattern together (0.89 ms: the class order leaves all partners of a class in
// the last-level cache), a soft barrier per item that keeps the work-groups of
// an XCD on the same middle pattern (10 % fewer misses, 0.98 ms), 17 bits per
// tile in complex128 (one work-group per CU, 0.78 ms).
#include <algorithm>
#include <cstdlib>
#include <new>
#include <type_traits>

#include "qk_tile.h"

namespace qk {

// ------------------------------------------------------------------ kernel
template <typename X>
using ConstAs = const __attribute__((address_space(4))) X;
template <typename X>
__device__ __forceinline__ ConstAs<X>* as_const(const X* p) {
  return (ConstAs<X>*)(uintptr_t)p;
}

// Vector accesses go through buffer descriptors: a uniform byte offset in a
// scalar register plus one 32-bit offset per lane, and a lane whose offset is
// kNoLane reads zeros without any access (past the descriptor's range).
constexpr uint32_t kNoLane = 0xfffffff0u;
constexpr int kBufNt = 2;   // non-temporal
constexpr int kBufFlags = 0x00027000;

template <typename V, bool W64>
struct TileBuf {
  using S = decltype(V{}.x);
  typedef uint32_t W __attribute__((ext_vector_type(sizeof(V) / 4)));
  typedef S E __attribute__((ext_vector_type(2)));
  __amdgpu_buffer_rsrc_t r;
  const char* base;
  uint32_t unit;
  __device__ TileBuf(const V* p, uint64_t n, uint32_t unit) : base(reinterpret_cast<const char*>(p)), unit(unit) {
    r = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, W64 ? 0x7fffffff : (int)(uint32_t)(n * sizeof(V)), kBufFlags);
  }
  // W64: a descriptor at the position itself; lane offsets stay inside one block
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t at(uint32_t pos) const {
    return W64 ? __builtin_amdgcn_make_buffer_rsrc((void*)(base + (uint64_t)pos * unit), 0, 0x7fffffff, kBufFlags) : r;
  }
  template <int AUX = 0>
  __device__ __forceinline__ V ld(uint32_t pos, uint32_t lane) const {
    W w;
    if constexpr (sizeof(V) == 16) w = __builtin_amdgcn_raw_buffer_load_b128(at(pos), lane, W64 ? 0u : pos, AUX);
    else w = __builtin_amdgcn_raw_buffer_load_b64(at(pos), lane, W64 ? 0u : pos, AUX);
    const E e = __builtin_bit_cast(E, w);
    return V{e.x, e.y};
  }
  __device__ __forceinline__ void st_nt(uint32_t pos, uint32_t lane, V v) const {
    const E e = {v.x, v.y};
    const W w = __builtin_bit_cast(W, e);
    if constexpr (sizeof(V) == 16) __builtin_amdgcn_raw_buffer_store_b128(w, at(pos), lane, W64 ? 0u : pos, kBufNt);
    else __builtin_amdgcn_raw_buffer_store_b64(w, at(pos), lane, W64 ? 0u : pos, kBufNt);
  }
};

typedef uint32_t U32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t U32x4 __attribute__((ext_vector_type(4)));
template <typename X>
__device__ __forceinline__ U32x8 sload8(const X* p) {
  static_assert(sizeof(X) % 32 == 0, "32-byte records");
  return *(const __attribute__((address_space(4))) U32x8*)(uintptr_t)p;
}

// MODE 0: y = H x; 1: H-pass; 2: H-pass with the sums of the local
// reorthogonalisation.  NLOW: low hops read per row (at least l - 1).
template <typename T, int MODE, int NLOW, int ORDER, bool W64>
__global__ void __launch_bounds__(kTileThreads, 4)
k_tile(TileArgs ta, uint64_t nel, const typename Cx<T>::V* __restrict__ x, typename Cx<T>::V* __restrict__ y,
       const typename Cx<T>::V* __restrict__ ujm1, KState st, LanczosArgs la, const double* __restrict__ partB, int Gp,
       double* __restrict__ partA) {
  using V = typename Cx<T>::V;
  constexpr bool LANCZOS = MODE > 0;
  constexpr int kQ = 8;   // top gathers in flight
  constexpr int kU = 5;   // rows per lane staged at a time
  extern __shared__ unsigned char smem[];
  const int tid = threadIdx.x;
  const int B = ta.B, Bp = 1 << ta.lbp;
  const int p = tid & (Bp - 1);
  T ca = (T)1, cb = (T)0;
  bool mine = p < B;   // and, after the scalars, the column is still running
  const bool prev = LANCZOS && la.j > 0;
  const bool pbc = ta.pbc != 0;
  const T g = (T)ta.half_jxy;
  const double hjz = ta.hjz;
  const int l = ta.l, M = ta.M;
  const uint32_t mtop = 1u << (M - 1), ttopbit = 1u << (ta.T - 1);
  const uint32_t rowb = (uint32_t)B * (uint32_t)sizeof(V);   // bytes of a row
  const TileBuf<V, W64> bx(x, nel, ta.unit), by(y, nel, ta.unit), bu(ujm1, nel, ta.unit);
  const double* dmid = ta.dmid + (p < B ? p : 0);
  const double* dtop = ta.dtop + (p < B ? p : 0);
  double s1 = 0.0, s2 = 0.0, s3r = 0.0, s3i = 0.0;
  // lane constants of the current class
  uint32_t cls = ~0u;
  uint32_t slot = 0, strideb = 0;
  bool on = false;
  uint32_t eo = 0, ojoin = 0, oring = 0;   // byte offsets of the own row and of the two partners' rows in their blocks
  uint32_t nb[NLOW];
  bool b0 = false, bl = false;
  double dlow = 0.0;
#pragma unroll
  for (int i = 0; i < NLOW; ++i) nb[i] = 0;

  // the current item: its tiles' records, and the lanes' constants of its class
  uint32_t t0 = 0, nmid = 0, nblk = 0, magic = 0, nslots = 0;
  const TileMid* mids = nullptr;
  const TileTop* tops = nullptr;
  auto take = [&](int it) {
    const U32x8 item = sload8(ta.items + it);
    const uint32_t icls = item[0];
    t0 = item[1];
    nmid = item[3];
    nblk = item[4];
    magic = item[5];
    nslots = (uint32_t)kTileThreads >> item[6];
    mids = ta.mid + item[2];
    tops = ta.top + t0;
    if (icls != cls) {
      cls = icls;
      const int kl = (int)(icls & 255u);
      const uint32_t base = ta.low_base[kl], len = ta.low_base[kl + 1] - base;
      strideb = (len + 1) * rowb;
      slot = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> item[6]);
      const uint32_t j = ((uint32_t)tid & ((1u << item[6]) - 1u)) >> ta.lbp;
      on = j < len && mine;
      if (on) {
        const TileLow lo = ta.low[base + j];
        dlow = ta.dlow[(size_t)(base + j) * B + p];
        eo = (j * B + p) * (uint32_t)sizeof(V);
        ojoin = (lo.join * (uint32_t)B + p) * (uint32_t)sizeof(V);
        oring = (lo.ring * (uint32_t)B + p) * (uint32_t)sizeof(V);
#pragma unroll
        for (int i = 0; i < NLOW; ++i) nb[i] = (lo.nbr[i] * (uint32_t)B + p) * (uint32_t)sizeof(V);
        b0 = (lo.bits & 1u) != 0;
        bl = ((lo.bits >> (l - 1)) & 1u) != 0;
      }
    }
    // stage: kU blocks per lane at a time (past the end the last block again)
    if (on) {
      for (uint32_t q0 = slot; q0 < nblk; q0 += kU * nslots) {
        uint32_t pos[kU], qq[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const uint32_t qn = q0 + u * nslots;
          qq[u] = qn < nblk ? qn : nblk - 1;
          const uint32_t ti = (qq[u] * magic) >> 20;
          pos[u] = as_const(tops + ti)->off + as_const(mids + (qq[u] - ti * nmid))->off;
        }
        V v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = bx.ld(pos[u], eo);
#pragma unroll
        for (int u = 0; u < kU; ++u) *reinterpret_cast<V*>(smem + qq[u] * strideb + eo) = v[u];
      }
      if (eo < rowb)   // the row of zeros behind every block
        for (uint32_t q = slot; q < nblk; q += nslots)
          *reinterpret_cast<V*>(smem + (q + 1) * strideb - rowb + eo) = V{0, 0};
    }
  };

  // the first item's rows are on their way while the scalars are reduced
  int it = blockIdx.x;
  if (it < ta.nitems) take(it);
  if (LANCZOS) {
    double* sa = reinterpret_cast<double*>(smem + ta.scratch);
    double *sb = sa + B, *tot = sb + B, *red = tot + B;
    int* act = reinterpret_cast<int*>(red + ta.nred);
    lanczos_h_scalars(B, st, la, partB, Gp, red, tot, sa, sb, act, hw_grid());
    if (mine) {
      ca = (T)sa[p];
      cb = (T)sb[p];
      mine = act[p] != 0;
    }
    on = on && mine;
    bool any = false;
    for (int b = 0; b < B; ++b) any = any || act[b] != 0;
    if (!any) it = ta.nitems;   // every column has stopped
  } else {
    __syncthreads();
  }
  while (it < ta.nitems) {
    if (on && slot < nblk) {
      uint32_t ti = (slot * magic) >> 20, mi = slot - ti * nmid;
      uint32_t ob = slot * strideb;   // LDS offset of the block
      U32x8 mv = sload8(mids + mi);
      U32x8 tv0 = sload8(tops + ti), tv1 = sload8((const TileItem*)(tops + ti) + 1);
      double dt = dtop[(size_t)(t0 + ti) * B];
      for (uint32_t q = slot; q < nblk; q += nslots) {
        const uint32_t tb = tv0[3];
        const int nact = (int)(tb >> 24);
        const uint32_t mu = mv[5] & 255u;
        const int nseq = (int)((mv[5] >> 8) & 255u), ngroup = (int)((mv[5] >> 16) & 255u);
        const uint32_t last = (mv[7] >> 16) & 255u;
        const uint32_t pos = tv0[0] + mv[0];
        const V z = {0, 0};
        // bonds leaving the tile: the ones joining low and middle and middle
        // and top, the ring bond, and the top hops (uniform shifts)
        const bool cj = bl != ((mu & 1u) != 0);
        const V vj = bx.ld(tv0[0] + mv[1], cj ? ojoin : kNoLane);
        const bool ct = ((mu & mtop) != 0) != ((tb & 1u) != 0);
        V vt = z;
        if (ct) vt = bx.ld(tv0[1] + mv[2], eo);
        const bool ttop = (tb & ttopbit) != 0;
        const bool cw = pbc && b0 != ttop;
        V vw = z;
        if (pbc) vw = bx.ld(tv0[2] + (ttop ? mv[3] : mv[4]), cw ? oring : kNoLane);
        V um = z;
        if (prev) um = bu.template ld<kBufNt>(pos, eo);
        V qv[kQ];
#pragma unroll
        for (int k = 0; k < kQ; ++k) {
          if (k >= nact) break;
          qv[k] = bx.ld(pos + (k < 4 ? tv0[4 + k] : tv1[k - 4]), eo);
        }
        double d = dlow + dmid[(size_t)mu * B];
        // hops inside the tile, from LDS
        const V xr = *reinterpret_cast<const V*>(smem + ob + eo);
        V hs = {0, 0}, ac = {0, 0}, vd = {0, 0};
#pragma unroll
        for (int k = 0; k < NLOW; ++k) {
          const V v = *reinterpret_cast<const V*>(smem + ob + nb[k]);
          hs.x += v.x;
          hs.y += v.y;
        }
        // the next block's record
        const uint32_t qn = q + nslots < nblk ? q + nslots : q;
        const uint32_t tin = (qn * magic) >> 20;
        const uint32_t min_ = qn - tin * nmid;
        const U32x8 mn = sload8(mids + min_);
        auto add = [&](const V& v) {
          hs.x += v.x;
          hs.y += v.y;
        };
        int n = 0;   // hops in the current group of four
        auto group = [&](const V& v) {
          if constexpr (ORDER == kOrderFree) {
            add(v);
          } else {
            ac.x += v.x;
            ac.y += v.y;
            if ((++n & 3) == 0) {
              add(ac);
              ac = z;
            }
          }
        };
        const uint32_t tq = ob - mi * strideb + eo;
        auto part = [&](uint32_t k) { return *reinterpret_cast<const V*>(smem + tq + k * strideb); };
        auto partk = [&](int k) {
          return part((k < 4 ? mv[6] >> (8 * k) : mv[7] >> (8 * (k - 4))) & 255u);
        };
        if (ORDER == kOrderFree || ta.join_kind == kHopSeq) add(vj);
        else vd = vj;
        if constexpr (ORDER == kOrderAny) {
#pragma unroll
          for (int k = 0; k < kTileMaxMid - 1; ++k) {
            if (k >= nseq + ngroup) break;
            if (k < nseq) add(partk(k));
            else group(partk(k));
          }
        } else {
#pragma unroll
          for (int k = 0; k < kTileMaxMid - 1; ++k) {
            if (k >= ngroup) break;
            group(partk(k));   // n == k: flushed at fixed places
          }
          n = ngroup;
        }
        if (ORDER != kOrderFree && last != kTileNone) vd = part(last);
        if (ct) {
          if (ORDER != kOrderAny || ta.mt_kind == kHopGroup) group(vt);
          else if (ta.mt_kind == kHopDeferred) vd = vt;
          else add(vt);
        }
        auto top_hop = [&](int k) {
          return bx.ld(pos + (uint32_t)as_const(tops + ti)->delta[k], eo);
        };
        if constexpr (ORDER == kOrderFree) {
#pragma unroll
          for (int k = 0; k < kQ; ++k) {
            if (k >= nact) break;
            add(qv[k]);
          }
          for (int k = kQ; k < nact; ++k) add(top_hop(k));
        } else if (ORDER == kOrderAny && ta.top_kind == kHopSeq) {
#pragma unroll
          for (int k = 0; k < kQ; ++k) {
            if (k >= nact) break;
            add(qv[k]);
          }
          for (int k = kQ; k < nact; ++k) add(top_hop(k));
        } else {
          auto tops_from = [&](auto n0) {   // n % 4 == n0: flushes at fixed places
#pragma unroll
            for (int k = 0; k < kQ; ++k) {
              if (k >= nact) break;
              ac.x += qv[k].x;
              ac.y += qv[k].y;
              if ((n0 + k) % 4 == 3) {
                add(ac);
                ac = z;
              }
            }
          };
          switch (n & 3) {
            case 0: tops_from(std::integral_constant<int, 0>{}); break;
            case 1: tops_from(std::integral_constant<int, 1>{}); break;
            case 2: tops_from(std::integral_constant<int, 2>{}); break;
            default: tops_from(std::integral_constant<int, 3>{}); break;
          }
          n += kQ;
          for (int k = kQ; k < nact; ++k) group(top_hop(k));
          add(ac);
        }
        hs.x += vd.x + vw.x;
        hs.y += vd.y + vw.y;
        d += dt;
        d -= (cj ? hjz : 0.0) + ((ct ? hjz : 0.0) + (cw ? hjz : 0.0));
        V h;
        if (ORDER == kOrderAny && ta.rows) {
          const T dd = (T)d;
          h.x = dd * xr.x;
          h.y = dd * xr.y;
          h.x += g * hs.x;
          h.y += g * hs.y;
        } else {
          h.x = (T)d * xr.x + g * hs.x;
          h.y = (T)d * xr.y + g * hs.y;
        }
        if (LANCZOS) {
          V wv;
          if (ORDER == kOrderAny && ta.rows) {
            wv.x = ca * h.x;
            wv.y = ca * h.y;
            wv.x -= cb * um.x;
            wv.y -= cb * um.y;
          } else {
            wv.x = ca * h.x - cb * um.x;
            wv.y = ca * h.y - cb * um.y;
          }
          by.st_nt(pos, eo, wv);
          s1 += (double)xr.x * (double)wv.x + (double)xr.y * (double)wv.y;
          s2 += (double)xr.x * (double)xr.x + (double)xr.y * (double)xr.y;
          if (MODE == 2) {
            s3r += (double)um.x * (double)wv.x + (double)um.y * (double)wv.y;
            s3i += (double)um.x * (double)wv.y - (double)um.y * (double)wv.x;
          }
        } else {
          by.st_nt(pos, eo, h);
        }
        if (tin != ti) {
          ti = tin;
          tv0 = sload8(tops + ti);
          tv1 = sload8((const TileItem*)(tops + ti) + 1);
          dt = dtop[(size_t)(t0 + ti) * B];
        }
        mv = mn;
        mi = min_;
        ob += nslots * strideb;
      }
    }
    it += gridDim.x;
    if (it >= ta.nitems) break;
    __syncthreads();   // the item's rows are no longer read
    take(it);
    __syncthreads();
  }
  if (LANCZOS) {
    // per batch column: lanes of a wave by a fixed tree, then the waves in order
    double v[kQA] = {s1, s2, s3r, s3i};
    double* red = reinterpret_cast<double*>(smem);
    __syncthreads();
    for (int q = 0; q < kQA; ++q) {
      for (int s = 32; s >= Bp; s >>= 1) v[q] += __shfl_xor(v[q], s);
      if ((tid & 63) < Bp) red[(q * (kTileThreads / 64) + (tid >> 6)) * Bp + p] = v[q];
    }
    __syncthreads();
    for (int c = tid; c < kQA * B; c += kTileThreads) {
      const int q = c / B, b = c % B;
      double t = 0.0;
      for (int w = 0; w < kTileThreads / 64; ++w) t += red[(q * (kTileThreads / 64) + w) * Bp + b];
      partA[(size_t)blockIdx.x * kQA * B + c] = t;
    }
  }
}

// Diagonal parts of Eq. (1) per batch column: the low states (their fields and
// zz bonds), the middle patterns, and the top patterns with the constant.
__global__ void __launch_bounds__(256)
k_tile_diag(TileArgs ta, const double* __restrict__ fields, double zz0, int ntop, double* __restrict__ dlow,
            double* __restrict__ dmid, double* __restrict__ dtop) {
  const int B = ta.B;
  const int64_t n0 = (int64_t)(1 << ta.l) * B, n1 = n0 + (int64_t)(1 << ta.M) * B, n2 = n1 + (int64_t)ntop * B;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n2) return;
  const int64_t e = i < n0 ? i : i < n1 ? i - n0 : i - n1;
  const int b = (int)(e % B);
  const uint32_t k = (uint32_t)(e / B);
  uint32_t bits;
  int nbits, first;
  double d = 0.0;
  if (i < n0) {
    bits = ta.low[k].bits;
    nbits = ta.l;
    first = 0;
  } else if (i < n1) {
    bits = k;
    nbits = ta.M;
    first = ta.l;
  } else {
    bits = ta.top[k].bits & 0xffffffu;
    nbits = ta.T;
    first = ta.l + ta.M;
    d = zz0;
  }
  const double* f = fields + (size_t)b * ta.L + first;
  for (int q = 0; q < nbits; ++q) d += ((bits >> q) & 1u) ? 0.5 * f[q] : -0.5 * f[q];
  d -= ta.hjz * (double)__popc((bits ^ (bits >> 1)) & ((1u << (nbits - 1)) - 1u));
  (i < n0 ? dlow : i < n1 ? dmid : dtop)[e] = d;
}

// ------------------------------------------------------------------ tables
static uint64_t bin(int n, int k) {
  if (k < 0 || k > n) return 0;
  uint64_t r = 1;
  for (int i = 1; i <= k; ++i) r = r * (uint64_t)(n - k + i) / (uint64_t)i;
  return r;
}

struct TileChoice {
  int l, M, blocks;   // blocks: blocks per slot of an item (rows of work per lane)
  size_t maxel;       // elements an item may stage
};

constexpr size_t kTileLds = 160 * 1024;   // per CU

// Doubles of the scalars' reduction scratch, and bytes of LDS behind the rows.
static int tile_nred(int B) { return B <= 32 && (B & (B - 1)) == 0 ? kTileThreads / 64 * B : kTileThreads; }
static size_t tile_scratch(int B) { return sizeof(double) * (3 * (size_t)B + tile_nred(B)) + sizeof(int) * B + 16; }

// The decomposition for B columns of vbytes-byte elements; `fewer` middle bits
// less than the rule gives (launch shapes).  Low bits above olo would mix hops
// that complex64 adds in another order (TileArgs::order).
//
// l: a block takes one row of lanes of a slot, so C(l, l/2) * B lanes (B rounded
// up to a power of two) must fit the work-group.  Every low or middle bit more
// keeps half a gather per row in LDS; the share of lanes that hold a row falls
// with blocks just above a power of two.  The best product of the two is taken:
// l = 10 for one column (252 of 256 lanes), 6 for 8 (H-pass of L = 26 in
// complex64 1.20 ms, as l = 7 with a third more idle lanes), 4 for 64 (L = 20:
// 117 us, l = 3 125 us).
// M: as many bits as two work-groups per CU can stage and as leave enough items
// to fill 256 CUs evenly.  H-pass, complex128 / complex64, us, by M:
//   L = 20: M = 2 13.0 / 12.6, 4 13.4 / 12.7, 5 15.6 / 14.8
//   L = 22: M = 3 22.4 / 20.6, 5 22.3 / 18.7, 6 25 / 22.4
//   L = 24: M = 4 54.7 / 43.2, 5 54.4 / 37.4, 6 59.6 / 39.4
//   L = 26: M = 4 198 / 139, 5 196 / 122, 6 204 / 112, 7 - / 122
//   L = 28: M = 4 891 / 597, 5 856 / 520, 6 864 / 488, 7 - / 476
static TileChoice tile_choice(int L, int N, int B, int vbytes, int fewer, int olo) {
  TileChoice c{0, 1, 1, (kTileLds / 2 - tile_scratch(B)) / vbytes};
  int Bp = 1;
  while (Bp < B) Bp *= 2;
  double best = -1.0;
  for (int l = 2; l <= kTileMaxLow && l <= L - 2 && (olo == 0 || l <= olo); ++l) {
    if (bin(l, l / 2) * Bp > kTileThreads) break;
    double lanes = 0.0;   // lanes taken for all low states of every popcount, per low state
    for (int k = 0; k <= l; ++k) {
      int slot = 64;
      while (slot < (int)bin(l, k) * Bp) slot *= 2;
      lanes += (double)slot * (double)bin(l, k) / (double)(1 << l) / ((double)bin(l, k) * B);
    }
    const double score = (1.0 + 0.1 * l) / lanes;
    if (score > best) {
      best = score;
      c.l = l;
    }
  }
  const double rows = (double)bin(L, N) / (double)bin(c.l, c.l / 2);   // blocks, if all were of the largest size
  const int mmax = vbytes == 16 ? 5 : kTileMaxMid;
  for (int M = 2; M <= mmax && c.l + M < L; ++M) {
    const double items = rows / (double)bin(M, M / 2);
    if (items < (M >= 7 ? 2000 : M == 6 ? 1000 : 250)) break;
    if ((bin(c.l, c.l / 2) + 1) * B * bin(M, M / 2) > c.maxel) break;
    c.M = M;
  }
  if (c.M - fewer >= 1 && c.M - fewer <= kTileMaxMid && c.l + c.M - fewer < L &&
      L - c.l - (c.M - fewer) <= kTileMaxTop)
    c.M -= fewer;
  // an item of the largest class is one tile
  int slot = 64;
  while (slot < (int)bin(c.l, c.l / 2) * Bp) slot *= 2;
  c.blocks = (int)((bin(c.M, c.M / 2) * slot + kTileThreads - 1) / kTileThreads);
  return c;
}

// What the tables of one decomposition are built from.
constexpr int kTileMaxCls = (kTileMaxLow + 1) * (kTileMaxMid + 1);
struct TileBuild {
  int L, N, l, M, T, lbp;
  int olo;                         // low-bit count whose order of summation the hops follow (L + 1: the row form's;
                                   // 0: any order)
  uint32_t unit;                   // bytes of a row to premultiply the positions with, or 1
  int ncls, nitems, ntop;
  uint32_t top0[kTileMaxTop + 2];  // first TileTop of each popcount
  // classes in the order of their items: the costliest item first, so that the
  // work-groups, which take every G-th item, end together
  struct Cls {
    uint8_t kl, km;
    uint16_t per;                  // top patterns per item
    uint32_t item0;                // first item
  } cls[kTileMaxCls];
};

__host__ __device__ inline int tile_kind(int olo, int bond) {
  return bond < olo - 1 ? kHopSeq : bond == olo - 1 ? kHopDeferred : kHopGroup;
}
__host__ __device__ inline int tile_slot_log2(uint32_t lanes) {
  return lanes <= 64 ? 6 : lanes <= 128 ? 7 : lanes <= 256 ? 8 : 9;
}
// Rank of a state among the states of its popcount (bn: C(n, k) with stride kBinomStride).
__host__ __device__ inline uint32_t tile_rank(uint32_t s, const uint32_t* bn) {
  uint32_t r = 0;
  for (int k = 1; s; ++k) {
    r += bn[__builtin_ctz(s) * kBinomStride + k];
    s &= s - 1;
  }
  return r;
}
__host__ __device__ inline uint32_t tile_binom(int n, int k, const uint32_t* bn) {
  return k < 0 || k > n ? 0u : bn[n * kBinomStride + k];
}
// First row, among the rows of `bits` states with K particles, whose bits above
// the lowest n are `high`; 0 where there is none.
__host__ __device__ inline uint32_t tile_first(uint32_t high, int n, int K, const uint32_t* bn) {
  const int k = K - __builtin_popcount(high);
  return k < 0 || k > n ? 0u : tile_rank((high << n) | ((1u << k) - 1u), bn);
}

__host__ __device__ inline TileLow tile_low(const TileBuild& tb, uint32_t b, const uint32_t* bn) {
  TileLow e{};
  const uint32_t len = bn[tb.l * kBinomStride + __builtin_popcount(b)];
  int n = 0;
  for (int q = 0; q + 1 < tb.l; ++q)
    if (((b >> q) ^ (b >> (q + 1))) & 1u) e.nbr[n++] = (uint16_t)tile_rank(b ^ (3u << q), bn);
  e.anti = (uint16_t)n;
  for (; n < kTileMaxLow - 1; ++n) e.nbr[n] = (uint16_t)len;
  e.join = (uint16_t)tile_rank(b ^ (1u << (tb.l - 1)), bn);
  e.ring = (uint16_t)tile_rank(b ^ 1u, bn);
  e.bits = (uint16_t)b;
  return e;
}

// Middle pattern mu below which kl particles are left.
__host__ __device__ inline TileMid tile_mid(const TileBuild& tb, int kl, uint32_t mu, const uint32_t* bn) {
  TileMid e{};
  const int l = tb.l, M = tb.M, K = kl + __builtin_popcount(mu);
  const uint32_t hb = 1u << (M - 1);
  e.off = tile_first(mu, l, K, bn) * tb.unit;
  e.off_join = tile_first(mu ^ 1u, l, K, bn) * tb.unit;
  e.off_top = tile_first(mu ^ hb, l, (mu & hb) ? K - 1 : K + 1, bn) * tb.unit;
  e.off_up = tile_first(mu, l, K + 1, bn) * tb.unit;
  e.off_dn = tile_first(mu, l, K - 1, bn) * tb.unit;
  e.bits = (uint8_t)mu;
  e.last = kTileNone;
  int n = 0;
  for (int q = 0; q + 1 < M; ++q)
    if (((mu >> q) ^ (mu >> (q + 1))) & 1u) {
      const uint8_t to = (uint8_t)tile_rank(mu ^ (3u << q), bn);
      ++e.anti;
      const int kd = tb.olo == 0 ? (int)kHopGroup : tile_kind(tb.olo, l + q);
      if (kd == kHopDeferred) {
        e.last = to;
        continue;
      }
      e.part[n++] = to;
      ++(kd == kHopSeq ? e.nseq : e.ngroup);
    }
  return e;
}

__host__ __device__ inline TileTop tile_top(const TileBuild& tb, uint32_t t, const uint32_t* bn) {
  TileTop e{};
  const int lm = tb.l + tb.M, K = tb.N - __builtin_popcount(t);
  e.off = tile_first(t, lm, tb.N, bn) * tb.unit;
  e.off_join = tile_first(t ^ 1u, lm, tb.N, bn) * tb.unit;
  e.off_ring = tile_first(t ^ (1u << (tb.T - 1)), lm, tb.N, bn) * tb.unit;
  uint32_t n = 0;
  for (int q = 0; q + 1 < tb.T; ++q)
    if (((t >> q) ^ (t >> (q + 1))) & 1u) {
      const uint32_t c = bn[(lm + q) * kBinomStride + K + __builtin_popcount(t & ((1u << q) - 1u))];
      e.delta[n++] = (int32_t)((((t >> q) & 1u) ? c : 0u - c) * tb.unit);
    }
  e.bits = t | (n << 24);
  return e;
}

__host__ __device__ inline TileItem tile_item(const TileBuild& tb, uint32_t idx, const uint32_t* bn) {
  int c = 0;
  while (c + 1 < tb.ncls && tb.cls[c + 1].item0 <= idx) ++c;
  const int kl = tb.cls[c].kl, km = tb.cls[c].km, kt = tb.N - kl - km;
  const uint32_t per = tb.cls[c].per, item0 = tb.cls[c].item0, q = idx - item0;
  const uint32_t n = bn[tb.T * kBinomStride + kt], ni = (n + per - 1) / per;
  // item idx runs on XCD idx % 8: each XCD takes a contiguous part of the
  // class's top patterns, so that the nearest top hops stay in its L2
  const uint32_t x = idx % kNumXcd;
  uint32_t first = 0;
  for (uint32_t y = 0; y < x; ++y) {
    const uint32_t r = (y - item0) % kNumXcd;   // items of XCD y: q = r, r + 8, ...
    if (r < ni) first += (ni - r + kNumXcd - 1) / kNumXcd;
  }
  const uint32_t k = first + q / kNumXcd;
  TileItem e{};
  e.cls = (uint32_t)kl | ((uint32_t)km << 8);
  e.t0 = tb.top0[kt] + k * per;
  e.mid0 = ((uint32_t)kl << tb.M);
  for (int m = 0; m < km; ++m) e.mid0 += bn[tb.M * kBinomStride + m];
  e.nmid = bn[tb.M * kBinomStride + km];
  const uint32_t left = n - k * per;
  e.nblk = (left < per ? left : per) * e.nmid;
  e.magic = (1u << 20) / e.nmid + 1;
  e.slot_log2 = (uint32_t)tile_slot_log2(bn[tb.l * kBinomStride + kl] << tb.lbp);
  return e;
}

// Table positions: low states by popcount and rank, middle patterns by (kl,
// popcount, rank), top patterns by popcount and rank.
__host__ __device__ inline uint32_t tile_low_at(const TileBuild& tb, uint32_t b, const uint32_t* bn) {
  uint32_t i = tile_rank(b, bn);
  for (int k = 0; k < __builtin_popcount(b); ++k) i += bn[tb.l * kBinomStride + k];
  return i;
}
__host__ __device__ inline uint32_t tile_mid_at(const TileBuild& tb, int kl, uint32_t mu, const uint32_t* bn) {
  uint32_t i = ((uint32_t)kl << tb.M) + tile_rank(mu, bn);
  for (int k = 0; k < __builtin_popcount(mu); ++k) i += bn[tb.M * kBinomStride + k];
  return i;
}

// One thread per entry.
__global__ void __launch_bounds__(256)
k_tile_tables(TileBuild tb, const uint32_t* __restrict__ bn, TileLow* __restrict__ low, TileMid* __restrict__ mid,
              TileTop* __restrict__ top, TileItem* __restrict__ items) {
  const uint32_t n0 = 1u << tb.l, n1 = n0 + ((uint32_t)(tb.l + 1) << tb.M), n2 = n1 + (1u << tb.T);
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n0) {
    low[tile_low_at(tb, i, bn)] = tile_low(tb, i, bn);
  } else if (i < n1) {
    const uint32_t e = i - n0, mu = e & ((1u << tb.M) - 1u);
    const int kl = (int)(e >> tb.M);
    mid[tile_mid_at(tb, kl, mu, bn)] = tile_mid(tb, kl, mu, bn);
  } else if (i < n2) {
    const uint32_t t = i - n1;
    const int kt = __popc(t), K = tb.N - kt;
    if (K >= 0 && K <= tb.l + tb.M) top[tb.top0[kt] + tile_rank(t, bn)] = tile_top(tb, t, bn);
  } else if (i - n2 < (uint32_t)tb.nitems) {
    items[i - n2] = tile_item(tb, i - n2, bn);
  }
}

// Sizes, classes and items of one decomposition (host).
static void tile_layout(int L, int N, int B, const TileChoice& ch, int olo, uint32_t unit, TileArgs& a, TileBuild& tb,
                        size_t* maxel) {
  const int l = ch.l, M = ch.M, T = L - l - M, lm = l + M;
  a.L = tb.L = L;
  a.l = tb.l = l;
  a.M = tb.M = M;
  a.T = tb.T = T;
  a.B = B;
  a.lbp = 0;
  while ((1 << a.lbp) < B) ++a.lbp;
  tb.lbp = a.lbp;
  tb.N = N;
  tb.olo = olo;
  tb.unit = unit;
  a.rows = olo > L ? 1 : 0;
  a.order = olo == 0 ? kOrderFree : l >= olo - 1 ? kOrderLow : kOrderAny;
  a.join_kind = tile_kind(olo, l - 1);
  a.mt_kind = tile_kind(olo, l + M - 1);
  a.top_kind = tile_kind(olo, l + M);
  uint32_t acc = 0;
  for (int k = 0; k <= l + 1; ++k) {
    a.low_base[k] = (uint16_t)acc;
    acc += (uint32_t)bin(l, k);
  }
  acc = 0;
  for (int k = 0; k <= T; ++k) {
    tb.top0[k] = acc;
    if (N - k >= 0 && N - k <= lm) acc += (uint32_t)bin(T, k);
  }
  tb.ntop = (int)acc;
  struct Cost { int kl, km; uint32_t per; uint64_t cost; };
  Cost cl[kTileMaxCls];
  int n = 0;
  *maxel = 0;
  for (int kl = 0; kl <= l; ++kl)
    for (int km = 0; km <= M; ++km) {
      const int kt = N - kl - km;
      if (kt < 0 || kt > T) continue;
      const uint32_t len = (uint32_t)bin(l, kl), nb = (uint32_t)bin(M, km), nt = (uint32_t)bin(T, kt);
      const uint32_t nslots = (uint32_t)kTileThreads >> tile_slot_log2(len << a.lbp);
      uint32_t per = nslots * (uint32_t)ch.blocks / nb;
      per = std::min<uint32_t>(per, (uint32_t)(ch.maxel / ((size_t)nb * (len + 1) * B)));
      per = std::max(1u, std::min(per, nt));
      *maxel = std::max(*maxel, (size_t)per * nb * (len + 1) * B);
      cl[n++] = {kl, km, per, (uint64_t)((per * nb + nslots - 1) / nslots) * 1000000 + len};
    }
  std::stable_sort(cl, cl + n, [](const Cost& p, const Cost& q) { return p.cost > q.cost; });
  tb.ncls = n;
  acc = 0;
  for (int i = 0; i < n; ++i) {
    const Cost& c = cl[i];
    tb.cls[i] = {(uint8_t)c.kl, (uint8_t)c.km, (uint16_t)c.per, acc};
    acc += ((uint32_t)bin(T, N - c.kl - c.km) + c.per - 1) / c.per;
  }
  tb.nitems = a.nitems = (int)acc;
}

// The diagonal parts from the fields (device, on s).
static qk_status tile_diag(const qk_ham* H, const TilePlan& P, hipStream_t s) {
  const TileArgs& a = P.a;
  const int64_t n = ((int64_t)(1 << a.l) + (1 << a.M) + P.ntop) * a.B;
  const double zz0 = 0.25 * H->p.jz * (H->p.pbc ? a.L : a.L - 1);
  hipLaunchKernelGGL(k_tile_diag, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, H->d_fields, zz0, P.ntop,
                     (double*)a.dlow, (double*)a.dmid, (double*)a.dtop);
  QK_HIP(hipGetLastError());
  return QK_OK;
}

qk_status tile_fields(const qk_ham* H, hipStream_t s) {
  for (const TilePlan* P : H->tile)
    if (P) {
      const qk_status st = tile_diag(H, *P, s);
      if (st != QK_OK) return st;
    }
  return QK_OK;
}

// Order of summation (TileBuild::olo) for the low-bit count llo.
static int tile_olo(int L, int vbytes, int llo) { return vbytes == 16 ? 0 : llo > 0 ? llo : L + 1; }

// Layout of one plan; *bytes receives the device memory it needs.
static void tile_plan_layout(const qk_ham* H, int vbytes, int llo, TilePlan* P, TileBuild* tb, size_t* bytes) {
  const int L = H->basis->L, N = H->basis->N, B = H->batch;
  TileArgs& a = P->a;
  P->nel = (uint64_t)H->basis->D * B;
  P->w64 = P->nel * vbytes >= 0xffffff00ull;
  a.unit = P->w64 ? (uint32_t)(B * vbytes) : 1u;
  const int fewer = llo > 0 ? blocked_llo(L, N, B, H->p.mode) - llo : 0;
  const int olo = tile_olo(L, vbytes, llo);
  size_t maxel = 0;
  tile_layout(L, N, B, tile_choice(L, N, B, vbytes, fewer, olo), olo, P->w64 ? 1u : (uint32_t)(B * vbytes), a, *tb,
              &maxel);
  a.pbc = H->p.pbc;
  a.half_jxy = 0.5 * H->p.jxy;
  a.hjz = 0.5 * H->p.jz;
  // LDS: the rows of the largest item, then the scratch of the scalars
  a.nred = tile_nred(B);
  a.scratch = (uint32_t)((maxel * vbytes + 15) & ~(size_t)15);
  P->lds = a.scratch + sizeof(double) * (3 * (size_t)B + a.nred) + sizeof(int) * B;
  P->lds = std::max(P->lds, sizeof(double) * kQA * (kTileThreads / 64) * ((size_t)1 << a.lbp));
  P->ntop = tb->ntop;
  P->nlow = a.l - 1 <= 3 ? 3 : a.l - 1 <= 6 ? 6 : 9;
  *bytes = sizeof(TileTop) * (size_t)tb->ntop + sizeof(TileLow) * ((size_t)1 << a.l) +
           sizeof(TileMid) * ((size_t)(a.l + 1) << a.M) + sizeof(TileItem) * (size_t)a.nitems +
           sizeof(double) * ((size_t)(1 << a.l) + (1 << a.M) + tb->ntop) * B;
  *bytes = (*bytes + 255) & ~(size_t)255;
}

// The tables in device memory d (on s).
static qk_status tile_plan_fill(const qk_ham* H, TilePlan* P, const TileBuild& tb, unsigned char* d, hipStream_t s) {
  TileArgs& a = P->a;
  TileTop* top = (TileTop*)d;
  TileLow* low = (TileLow*)(top + tb.ntop);
  TileMid* mid = (TileMid*)(low + ((size_t)1 << a.l));
  TileItem* items = (TileItem*)(mid + ((size_t)(a.l + 1) << a.M));
  a.top = top;
  a.low = low;
  a.mid = mid;
  a.items = items;
  a.dlow = (const double*)(items + a.nitems);
  a.dmid = a.dlow + (size_t)(1 << a.l) * a.B;
  a.dtop = a.dmid + (size_t)(1 << a.M) * a.B;
  const uint64_t n = (1ull << a.l) + ((uint64_t)(a.l + 1) << a.M) + (1ull << a.T) + (uint64_t)a.nitems;
  hipLaunchKernelGGL(k_tile_tables, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, tb, H->basis->d_binom, low, mid,
                     top, items);
  QK_HIP(hipGetLastError());
  return tile_diag(H, *P, s);
}

static void plans_free(const qk_allocator& al, TilePlan* (&P)[2]) {
  for (TilePlan*& p : P) {
    if (p) dev_free(al, p->d_mem);
    delete p;
    p = nullptr;
  }
}

// Matrix-free chains of kTileMinL to 32 sites take the tiled kernels (below,
// one thread per row fills no more than a few work-groups either), unless the
// table of top patterns would be too long: batches of some GB per column.
constexpr int kTileMinL = 8;

// llo: the low-bit count that the tables are for (complex64 takes no more low
// bits than that: 31 sites with at most four particles have 21 top bits at 9).
static bool tile_covers(const qk_ham* H, int vbytes, int llo) {
  const int L = H->basis->L;
  if (H->p.mode != QK_MATFREE || L < kTileMinL || L > 32) return false;
  const TileChoice c = tile_choice(L, H->basis->N, H->batch, vbytes, 0, tile_olo(L, vbytes, llo));
  return L - c.l - c.M <= kTileMaxTop;
}

// Plans of both element sizes for the low-bit count llo (0: no block tables),
// in one allocation.
static qk_status plans_build(qk_ham* H, int llo, TilePlan* (&P)[2], hipStream_t s) {
  TileBuild tb[2] = {};
  size_t bytes[2] = {0, 0};
  for (int d = 0; d < 2; ++d) {
    if (!tile_covers(H, d ? 16 : 8, llo)) continue;
    P[d] = new (std::nothrow) TilePlan;
    if (!P[d]) {
      plans_free(H->al, P);
      set_error("out of host memory building the tables of the Hamiltonian");
      return QK_ENOMEM;
    }
    tile_plan_layout(H, d ? 16 : 8, llo, P[d], &tb[d], &bytes[d]);
  }
  if (bytes[0] + bytes[1] == 0) return QK_OK;
  void* mem = nullptr;
  const hipError_t e = dev_alloc(H->al, &mem, bytes[0] + bytes[1]);
  if (e != hipSuccess) {
    plans_free(H->al, P);
    return hip_fail(e, "tables of the Hamiltonian");
  }
  P[P[0] ? 0 : 1]->d_mem = mem;   // the first plan owns it
  qk_status st = QK_OK;
  for (int d = 0; d < 2 && st == QK_OK; ++d)
    if (P[d]) st = tile_plan_fill(H, P[d], tb[d], (unsigned char*)mem + (d ? bytes[0] : 0), s);
  if (st != QK_OK) {
    (void)hipStreamSynchronize(s);   // nothing queued may still use what is released
    plans_free(H->al, P);
  }
  return st;
}

qk_status tile_create(qk_ham* H, hipStream_t s) {
  return plans_build(H, H->llo, H->tile, s);
}

void tile_free(qk_ham* H) { plans_free(H->al, H->tile); }

const TilePlan* tile_plan(const qk_ham* H, int dtype) { return H->tile[dtype == QK_C128 ? 1 : 0]; }

bool tile_wide(const TilePlan* P) { return P->w64; }

// -------------------------------------------------- block decomposition knob
static int env_int(const char* name, int dflt) {
  const char* v = getenv(name);
  if (!v || !*v) return dflt;
  const int x = atoi(v);
  return x > 0 ? x : dflt;
}

// Low bits of the block decomposition reported for a Hamiltonian (0: none):
// the blocks whose order of summation complex64 follows (TileArgs::order) and
// the scale that qk_launch_shape.blocked_llo is set on -- one count lower
// takes one middle bit out of the tiles.
int blocked_llo(int L, int N, int B, int mode) {
  (void)N;
  if (mode != QK_MATFREE || L < 18 || L > 32) return 0;
  if (B == 1) {
    int llo = env_int("QK_BLOCKED_LLO", 11);
    if (llo < 9) llo = 9;
    if (llo > 11) llo = 11;
    if (llo > L / 2) llo = L / 2;
    return llo;
  }
  // batches: B a power of two; the largest count whose biggest block of B
  // complex128 phases is at most 32 KB
  if (B < 2 || B > QK_MAX_BATCH || (B & (B - 1)) != 0) return 0;
  for (int llo = (L / 2 < 11 ? L / 2 : 11); llo >= 5; --llo)
    if (bin(llo, llo / 2) * (uint64_t)B * 16u <= 32768u && L - llo <= 20) return llo;
  return 0;
}

bool blocked_llo_valid(const qk_ham* H, int llo) {
  const int L = H->basis->L, B = H->batch;
  if (H->llo <= 0 || H->p.mode != QK_MATFREE || L < 18 || L > 32 || llo > L / 2) return false;
  if (B == 1) return llo >= 9 && llo <= 11;
  return llo >= 5 && llo <= 11 && L - llo <= 20 && bin(llo, llo / 2) * (uint64_t)B * 16u <= 65536u;
}

qk_status blocked_rebuild(qk_ham* H, int llo) {
  if (!blocked_llo_valid(H, llo)) {
    set_error("unsupported low-bit count for this Hamiltonian's block decomposition");
    return QK_EINVAL;
  }
  if (llo == H->llo) return QK_OK;
  TilePlan* P[2] = {nullptr, nullptr};
  const qk_status st = plans_build(H, llo, P, nullptr);
  if (st != QK_OK) return st;   // the previous decomposition stays
  const hipError_t e = hipDeviceSynchronize();   // no queued kernel may still read the old tables
  if (e != hipSuccess) {
    plans_free(H->al, P);
    return hip_fail(e, "block decomposition");
  }
  plans_free(H->al, H->tile);
  H->tile[0] = P[0];
  H->tile[1] = P[1];
  H->llo = llo;
  ++H->tables_gen;
  return QK_OK;
}

// --------------------------------------------------------------- launchers
template <typename T, int MODE, int NLOW, int ORDER, bool W64>
static qk_status launch_tile_k(const TilePlan& P, const void* x, void* y, const void* ujm1, const KState& st,
                               const LanczosArgs& la, const double* partB, int Gp, double* partA, int* grid_out,
                               int wgs_req, hipStream_t s) {
  using V = typename Cx<T>::V;
  static const hipError_t attr = hipFuncSetAttribute((const void*)k_tile<T, MODE, NLOW, ORDER, W64>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTileLds);
  QK_HIP(attr);
  // as many work-groups per CU as the registers (two, or three in complex64)
  // and the LDS hold
  static const int regs = [] {
    int n = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_tile<T, MODE, NLOW, ORDER, W64>, kTileThreads, 0) ==
                       hipSuccess && n > 0 ? n : 2;
  }();
  int occ = std::min<int>(regs, (int)(kTileLds / P.lds));
  if (occ > 3) occ = 3;
  if (occ < 1) occ = 1;
  if (wgs_req < 0) {   // tile_max_wgs
    *grid_out = occ;
    return QK_OK;
  }
  const int req = wgs_req > 0 ? wgs_req : env_int("QK_BLOCKED_WGS_PER_CU", occ);
  if (req < occ) occ = req;
  int G = qk_num_cus() * occ;
  if (G > P.a.nitems) G = P.a.nitems;
  G = (G + kNumXcd - 1) / kNumXcd * kNumXcd;
  hipLaunchKernelGGL((k_tile<T, MODE, NLOW, ORDER, W64>), dim3(G), dim3(kTileThreads), P.lds, s, P.a, P.nel, (const V*)x, (V*)y,
                     (const V*)ujm1, st, la, partB, Gp, partA);
  QK_HIP(hipGetLastError());
  if (grid_out) *grid_out = G;
  return QK_OK;
}

template <typename T, int MODE, int ORDER>
static qk_status launch_tile_o(const TilePlan& P, const void* x, void* y, const void* ujm1, const KState& st,
                               const LanczosArgs& la, const double* partB, int Gp, double* partA, int* grid_out,
                               int wgs, hipStream_t s) {
  // QK_BLOCKED_W64=1 takes the 64-bit form for smaller vectors too (the same
  // arithmetic, so the same bits): their positions are bytes, in units of 1
  const char* fw = getenv("QK_BLOCKED_W64");
  if (P.w64 || (fw && fw[0] == '1'))
    return launch_tile_k<T, MODE, 9, ORDER, true>(P, x, y, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
  switch (P.nlow) {
    case 3: return launch_tile_k<T, MODE, 3, ORDER, false>(P, x, y, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
    case 6: return launch_tile_k<T, MODE, 6, ORDER, false>(P, x, y, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
    default: return launch_tile_k<T, MODE, 9, ORDER, false>(P, x, y, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
  }
}

template <typename T, int MODE>
static qk_status launch_tile_t(const TilePlan& P, const void* x, void* y, const void* ujm1, const KState& st,
                               const LanczosArgs& la, const double* partB, int Gp, double* partA, int* grid_out,
                               int wgs, hipStream_t s) {
  if constexpr (sizeof(T) == 8) {
    return launch_tile_o<T, MODE, kOrderFree>(P, x, y, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
  } else {
    if (P.a.order == kOrderLow)
      return launch_tile_o<T, MODE, kOrderLow>(P, x, y, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
    return launch_tile_o<T, MODE, kOrderAny>(P, x, y, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
  }
}

qk_status launch_tile_apply(const TilePlan& P, int dtype, const void* x, void* y, hipStream_t s) {
  if (dtype == QK_C128)
    return launch_tile_t<double, 0>(P, x, y, nullptr, KState{}, LanczosArgs{}, nullptr, 0, nullptr, nullptr, 0, s);
  return launch_tile_t<float, 0>(P, x, y, nullptr, KState{}, LanczosArgs{}, nullptr, 0, nullptr, nullptr, 0, s);
}

qk_status launch_tile_lanczos_h(const TilePlan& P, int dtype, const void* uj, const void* ujm1, void* w,
                                const KState& st, const LanczosArgs& la, const double* partB, int Gp, double* partA,
                                int* grid_out, int wgs, hipStream_t s) {
  const bool ro = la.reorth && la.j > 0;
  if (dtype == QK_C128)
    return ro ? launch_tile_t<double, 2>(P, uj, w, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s)
              : launch_tile_t<double, 1>(P, uj, w, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
  return ro ? launch_tile_t<float, 2>(P, uj, w, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s)
            : launch_tile_t<float, 1>(P, uj, w, ujm1, st, la, partB, Gp, partA, grid_out, wgs, s);
}

int tile_max_wgs(const TilePlan& P, int dtype) {
  int n = 1;
  const qk_status st = launch_tile_lanczos_h(P, dtype, nullptr, nullptr, nullptr, KState{}, LanczosArgs{}, nullptr, 0,
                                             nullptr, &n, -1, nullptr);
  return st == QK_OK ? n : 1;
}

}  // namespace qk
