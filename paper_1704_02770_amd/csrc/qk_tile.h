// Tiled matrix-free H x (Sec. 3 "Hamiltonian matrix construction", Eq. (1)):
// tables and launch plan of the kernels in qk_tile.hip.
//
// A state splits into top, middle and low bits (T, M and l of them).  For a
// fixed top pattern and fixed popcounts of the low and the middle part (a
// class (kl, km)) the rows are C(M, km) blocks of C(l, kl) consecutive rows
// each: a tile.  Tiles of one class have the same size and the same hops.
#pragma once

#include "qk_device.h"

namespace qk {

constexpr int kTileThreads = 512;
constexpr int kTileMaxLow = 10;    // low bits l
constexpr int kTileMaxMid = 7;     // middle bits M
constexpr int kTileMaxTop = 20;    // top bits T
constexpr int kTileDeltas = 20;    // row shifts of a top pattern (at most T - 1, padded)

// One low state, grouped by popcount, ascending inside a group.
struct TileLow {
  uint16_t nbr[kTileMaxLow - 1];   // ranks of the states one low hop away (ascending bonds), then the group size (a row of zeros)
  uint16_t join;                   // rank of the state with the highest low bit flipped (in its own group)
  uint16_t ring;                   // rank of the state with the lowest bit flipped
  uint16_t bits;                   // the state
  uint16_t anti;                   // number of low hops
  uint16_t pad[3];
};
static_assert(sizeof(TileLow) == 32, "two 16-byte loads");

// Row positions below are in units of TileArgs::unit bytes: the bytes of a row,
// premultiplied, for vectors that 32-bit byte offsets reach, else rows.

// One middle pattern of a class: positions inside the top pattern's rows.
struct TileMid {
  uint32_t off;                    // first row of the block
  uint32_t off_join;               // of the block with the lowest middle bit flipped (same top pattern)
  uint32_t off_top;                // of the block with the highest middle bit flipped, one particle moved to or from the top
  uint32_t off_up, off_dn;         // of this pattern's block with one low particle more / fewer (ring partner)
  uint8_t bits;                    // the pattern
  uint8_t nseq;                    // hops inside the middle bits that are added one by one,
  uint8_t ngroup;                  // and those added in groups of four after them (see HopOrder)
  uint8_t anti;                    // all hops inside the middle bits
  uint8_t part[kTileMaxMid - 1];   // block index in the tile of each of those hops' partners, ascending bonds
  uint8_t last;                    // block index of the deferred hop's partner, or kTileNone
  uint8_t pad;
};
static_assert(sizeof(TileMid) == 32, "one scalar load");
constexpr uint8_t kTileNone = 0xff;

// One top pattern, sorted by popcount, ascending inside a popcount.
struct TileTop {
  uint32_t off;                    // first row with this pattern
  uint32_t off_join;               // first row with its lowest bit flipped
  uint32_t off_ring;               // first row with its highest bit flipped
  uint32_t bits;                   // the pattern | number of hops inside the top bits << 24
  int32_t delta[kTileDeltas];      // shift of each hop, ascending bonds, then zeros
  uint32_t pad[8];
};
static_assert(sizeof(TileTop) == 128, "two scalar cache lines");

// One unit of work: tiles of class (kl, km) with the top patterns t0 .. t0 + nblk / nmid - 1.
struct TileItem {
  uint32_t cls;                    // kl | km << 8
  uint32_t t0;
  uint32_t mid0;                   // first TileMid of the class
  uint32_t nmid;                   // blocks of one tile, C(M, km)
  uint32_t nblk;                   // blocks of the item
  uint32_t magic;                  // q / nmid = q * magic >> 20 for q < nblk
  uint32_t slot_log2;              // lanes that take one block together, a power of two >= its lanes
  uint32_t pad;
};
static_assert(sizeof(TileItem) == 32, "one scalar load");

// The order in which a row's hops are summed.  complex128 takes them as they
// come.  complex64 follows one order whatever the decomposition -- that of
// blocks of H->llo low bits: hops below bond llo - 1 one by one, the hops above
// it in groups of four, then bond llo - 1 and the ring bond together; without
// block tables all one by one -- so that a decomposition does not show in the
// last bit of single precision.
enum : int { kHopSeq = 0, kHopDeferred = 1, kHopGroup = 2 };
enum : int {
  kOrderFree = 0,      // complex128
  kOrderLow = 1,       // no middle or top hop is added one by one (l >= llo - 1)
  kOrderAny = 2
};

struct TileArgs {
  int L, pbc, l, M, T, B, lbp;     // lbp: log2 of the lanes per row (batch rounded up to a power of two)
  int nitems;
  int nred;                        // doubles of the scalars' reduction scratch
  uint32_t scratch;                // its LDS offset, behind the rows
  int join_kind, mt_kind, top_kind;   // of the bonds low-middle and middle-top and of the top bonds
  int order;
  int rows;                        // 1: products of the diagonal and the hops rounded as the row form does
  uint32_t unit;                   // bytes of a row, or 1 (positions premultiplied)
  double half_jxy, hjz;
  const TileLow* low;
  const TileMid* mid;
  const TileTop* top;
  const TileItem* items;
  const double* dlow;              // [2^l][B] diagonal parts of the low states, in TileLow order
  const double* dmid;              // [2^M][B] of the middle patterns, by pattern
  const double* dtop;              // [tops][B] of the top patterns, in TileTop order
  uint16_t low_base[kTileMaxLow + 2];   // first TileLow of each popcount; differences are the group sizes
};

// Host and device tables of one decomposition.
struct TilePlan {
  TileArgs a{};
  void* d_mem = nullptr;           // device memory of both plans of a Hamiltonian (one of them owns it)
  uint64_t nel = 0;                // elements of a vector
  bool w64 = false;                // 32-bit byte offsets do not reach it
  int ntop = 0;                    // top patterns
  int nlow = 0;                    // low hops read per row by the kernel
  size_t lds = 0;                  // bytes of dynamic LDS
};

}  // namespace qk
