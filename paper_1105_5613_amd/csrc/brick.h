// brick.h -- tiles of cells and their LDS neighbourhoods on the brick path
// (the default list path of boxes with at least three cells per side).
//
// A tile is a block of tx x ty x tz home cells; with cells of side >= cutoff +
// skin every partner of a home particle lies in the (tx + 2) x (ty + 2) x
// (tz + 2) cells around them.  The force kernel copies that neighbourhood
// into LDS once per launch and walks 16-bit list entries against it; one
// block per tile.  Cells are stored in z-major order, so a row of the
// neighbourhood (fixed y and z) is one contiguous particle range, or two
// where it wraps around the periodic box.  A slot is a place in that
// neighbourhood: rows follow each other in (z, y) order, inside a row the
// cell at the image -L if there is one (left), the cells inside the box
// (main), and the cell at +L (right).
//
// The rows of every tile change only at list builds; they are tabulated then
// (tile_rows), so that a force launch reads them instead of the cell starts.
//
// A brick is the block of home cells of a tile (1 x 1 x 1 at the
// Lennard-Jones density, up to 2 x 2 x 2 in sparse grids) whose particles one
// wave of the list build searches partners for.
//
// List entry: slot << shift | species bits 14 and 15 (see force_brick.hip);
// shift 3 (the byte offset of an 8-byte LDS word) with up to 2,048 slots, 2
// with up to 3,072.  The highest slot is never filled by a particle: it holds
// a point infinitely far away, and the places of a row past its last entry
// point at it.
#pragma once
#include "md_internal.h"

namespace mdk {

constexpr int32_t kBrickSlots = 2048;           // LDS slots of a tile, the far point included
constexpr int32_t kBrickSlotsBig = 3072;        // ... of contexts whose tiles need more
constexpr int32_t kTileUnits = 4;               // partials of a tile in small replicas,
constexpr int32_t kUnitHomes = 64;              // each of 64 homes (the last one the rest)
constexpr int32_t kTileRows = 36;               // rows of a neighbourhood: (ty + 2)(tz + 2), t <= 4
constexpr int32_t kTileHomeRows = 16;           // rows of home cells: ty * tz
constexpr int32_t kBrickThreads = 1024;         // most threads per block of the force kernel
constexpr int32_t kChunksAhead = 1;             // chunks the force kernel may read past a row
constexpr int32_t kChunkEntries = 8;            // entries per 16-byte list chunk
// Most chunks of a row: its entries are slots of one neighbourhood, and every
// pass of the search (of at least 12 chunks of 64 candidates) ends with a chunk
// that need not be full.
constexpr int32_t kMostChunks =
    kBrickSlotsBig / kChunkEntries + (kBrickSlotsBig + 12 * 64 - 1) / (12 * 64);

struct BrickTile {
  int32_t rep;
  int32_t cx, cy, cz;   // first home cell
  int32_t tx, ty, tz;   // home cells per axis, 1 .. 4
  int32_t units;        // partials of the tile: 1, or kTileUnits of kUnitHomes homes each
  int32_t part;         // its first partial
  int32_t b0, nb;       // its bricks
  int32_t waves, groups;  // list-free search: waves that work, and how many share a brick
};
struct Brick {
  int32_t tile;
  int8_t lx, ly, lz;    // first cell, relative to the tile's
  int8_t hx, hy, hz;    // cells per axis
  int8_t pass;          // candidate chunks per pass of the list search
  int8_t pad;
};
struct TileRow {        // row q = (y + 1) + (z + 1) (ty + 2) of the neighbourhood
  int32_t l0, l1, l2, l3;  // first slot of the left, main and right piece, end of the row
  int32_t gl, gm, gr;      // sorted index of the first particle of each piece
  int32_t pad;
};
struct HomeRow {        // row y + z ty of the home cells
  int32_t g;            // sorted index of its first particle
  int32_t h;            // home particles of the rows before it
  int32_t slot;         // slot of its first particle
  int32_t pad;
};
struct TileHead {
  int32_t total;        // slots in use
  int32_t nh;           // home particles
  int32_t pad[2];
};

// Chunk c of the row of particle i is element list_base(i, capc) + c kSlice of
// the list, in 16-byte units.  kChunksAhead chunks per particle of a slice more
// than the capacity are allocated: the force kernel reads ahead.
inline size_t chunk_elems(int32_t ntot, int32_t capc) {
  return list_elems(ntot, capc) + kChunksAhead * kSlice;
}

// Whether the rows of every tile lie within 4 GiB of list, which the force
// kernel addresses with 32 bits from the tile's first one; layer: the most
// particles that a layer of tiles can hold.
inline bool list_span_fits(int64_t layer, int32_t capc) {
  return ((layer / kSlice + 2) * capc + kChunksAhead) * kSlice * (int64_t)sizeof(uint4) <
         (int64_t)1 << 32;
}

__device__ inline void wrap_cell(int32_t& q, int32_t nc, int32_t& s) {
  s = 0;
  if (q < 0) {
    q += nc;
    s = -1;
  } else if (q >= nc) {
    q -= nc;
    s = 1;
  }
}

__device__ inline int32_t wave_scan(int32_t v, int lane) {  // inclusive
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t y = __shfl_up(v, d, 64);
    if (lane >= d) v += y;
  }
  return v;
}

// Rows of one tile, by one wave (lane q: row q).  cs: cell starts.  Latches
// kErrSlots when the neighbourhood does not fit the slots.
__device__ inline void tile_rows(const BrickTile& T, const RepDesc& R, const int32_t* cs, int lane,
                                 int32_t slots, TileHead* head, TileRow* tr, HomeRow* hr,
                                 DevState* st) {
  const int32_t nc = R.nc, ry = T.ty + 2, nr = ry * (T.tz + 2), nhr = T.ty * T.tz;
  int32_t nl = 0, nm = 0, nrt = 0;
  TileRow row{};
  if (lane < nr) {
    int32_t y = T.cy + lane % ry - 1, z = T.cz + lane / ry - 1, s;
    wrap_cell(y, nc, s);
    wrap_cell(z, nc, s);
    const int32_t* c = cs + R.coff + (z * nc + y) * nc;
    const int32_t lo = T.cx - 1, hi = T.cx + T.tx;  // logical x range, inclusive
    const int32_t mlo = lo < 0 ? 0 : lo, mhi = hi >= nc ? nc - 1 : hi;
    row.gl = c[nc - 1];
    row.gm = c[mlo];
    row.gr = c[0];
    nl = lo < 0 ? c[nc] - row.gl : 0;
    nm = c[mhi + 1] - row.gm;
    nrt = hi >= nc ? c[1] - row.gr : 0;
  }
  const int32_t len = nl + nm + nrt;
  const int32_t end = wave_scan(len, lane);
  row.l0 = end - len;
  row.l1 = row.l0 + nl;
  row.l2 = row.l1 + nm;
  row.l3 = end;
  if (lane < nr) tr[lane] = row;
  // home rows
  int32_t g = 0, hn = 0;
  if (lane < nhr) {
    const int32_t* c =
        cs + R.coff + ((T.cz + lane / T.ty) * nc + T.cy + lane % T.ty) * nc + T.cx;
    g = c[0];
    hn = c[T.tx] - g;
  }
  const int src = lane < nhr ? (lane / T.ty + 1) * ry + lane % T.ty + 1 : 0;
  const int32_t l1s = __shfl(row.l1, src, 64), gms = __shfl(row.gm, src, 64);
  const int32_t he = wave_scan(hn, lane);
  if (lane < nhr) hr[lane] = HomeRow{g, he - hn, l1s + (g - gms), 0};
  const int32_t total = __shfl(end, nr - 1, 64), nh = __shfl(he, nhr - 1, 64);
  if (lane == 0) {
    *head = TileHead{total, nh, {0, 0}};
    if (total >= slots) atomicOr(&st->err, kErrSlots);
  }
}

// Sorted index of home h of a tile with nh home particles, from its home rows;
// places past the last home stand for the first one.  A tile without home
// particles has none: its rows' starts may lie at the end of the particle
// arrays, where nothing is to be read.
__host__ __device__ inline int32_t home_index(const HomeRow* hr, int32_t nhr, int32_t h,
                                              int32_t nh) {
  if (nh <= 0) return -1;
  if (h >= nh) h = 0;
  int32_t r = 0;
  while (r + 1 < nhr && hr[r + 1].h <= h) ++r;
  return hr[r].g + (h - hr[r].h);
}

// brick tables of a context
struct BrickArgs {
  int32_t ntiles, nbricks;
  int32_t rows, hrows;       // table strides: most rows / home rows of a tile
  int32_t slots, shift;      // LDS slots of a tile, place of the slot in an entry
  const BrickTile* tiles;
  const Brick* bricks;
  TileHead* head;            // [ntiles]
  TileRow* row;              // [ntiles][rows]
  HomeRow* hrow;             // [ntiles][hrows]
  uint4* list;               // chunk_elems
  int32_t* nchunk;           // [N] chunks of each row
  int32_t capc;              // chunks per row
  int32_t groups;            // home groups of a brick, as expected
  int32_t split;             // blocks of the force kernel per tile (1, 2 or 4)
};

// Constants of the pair function on the brick path (force_brick.hip).
struct BrickPair {
  // two species: value = p1 + (p0 - p1) for the species whose list entries
  // have bit 14 set, p1 for the other; per home species
  double rc2[4][2], a[4][2], b[4][2], fs[4][2];  // FP64: f(r)/r = (a r^-6 + b) r^-8 + fs / r
  float msig2[4][2], mf12[4][2], mfs[4][2];      // mixed, as force.hip's
  // energies, 12 V* = (a r^-6 + 2 b) r^-6 - 12 f r - v12 with v12 = 12 (vc - rc fs)
  // in FP64, p1 and d as above; mixed keeps (r - rc) fs and 12 vc apart, the
  // values for bit 14 clear and set
  double v12[4][2];
  float mrc[4][2], mv12[4][2];
  double tiny;                                   // far below the last bit of any r^2
  float mk;                                      // f6 = -mk f12
  int32_t flip;                                  // the species with bit 14 set is `flip`
  int32_t four;                                  // 1: use the table of up to four species
};

}  // namespace mdk
