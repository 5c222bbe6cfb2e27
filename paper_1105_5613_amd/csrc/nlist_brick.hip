// nlist_brick.hip -- cut-off neighbour search of the brick path (brick.h):
// the same inclusion test and so the same partners as nlist.hip (FP64, no FMA
// contraction, d = (x_j - x_i) + s L and r^2 = (dx dx + dy dy) + dz dz against
// (r_c,ab + skin)^2; "Grid-search method", Fig. 1), written as 16-bit entries
// for the force kernel's LDS neighbourhoods.
//
// One wave per brick, in two phases per group of at most 32 home particles.
//
// Test phase, on the matrix cores.  The particles of the (hx + 2) x (hy + 2) x
// (hz + 2) cells around the brick, with their periodic shift, are packed 64 to
// a chunk.  With u = x - centre of the brick,
//   r^2 - thr = -2 u_i . u_j + |u_j|^2 - b_i s_j + (|u_i|^2 - a_i),
// thr_ij = a_i + b_i s_j for the species value s_j in {0, 1}, is a product of a
// 32 x 6 and a 6 x 32 matrix for 32 candidates and the 32 homes of a group:
// three v_mfma_f32_32x32x2 (a fourth for the species 2 and 3).  A lane of the
// result holds 16 candidates of one home, and the sign bits are its hits; the
// candidates are dealt to the matrix rows so that they come out in packed
// order, one 32-bit word per home and 32 candidates, written to LDS.  Nothing
// is done per hit.
//
// The inclusion test has to round like the plain FP64 one, so the FP32
// product only decides where it is clear.  For a 1 x 1 x 1 brick, in units of
// the cell side, |u_i| <= 1/2 per axis, thr <= 1, and near the threshold the terms and
// partial sums stay below 8; six additions then err by less than 3e-6 even
// with truncation, and the operands' own rounding moves r^2 by less than
// 1e-6.  Terms grow with the square of the brick's width.  A value within
// kUnclear * (width * side)^2 of zero is decided by the FP64 test of that pair (one
// pair in a dozen bricks at the LJ density).
//
// Write phase: two lanes per home walk the set bits of its words, one from
// the first candidate on and one from the last back, and pack eight entries
// to a 16-byte chunk in registers, stored whole.  The order of a row is not
// specified; it is the same in every launch.  Places of the last chunk past
// the row's end point at the far slot (a search of several passes
// ends each pass like that).
//
// Bound by vector issue (0.69 of the launch; the matrix cores work in 0.26 of
// it): the sign bits, the operands and the walk of the write phase.  Measured
// at 1,048,576 particles (LJ box, list radius 2.8): 290 us; the VALU search of
// nlist.hip writing 32-bit entries takes 491 us (in the first steps of a
// process, at lower clocks, 316 and 530).
#include <type_traits>

#include "brick_device.h"

#pragma clang fp contract(off)

namespace mdk {
namespace {

// Candidate chunks per pass.  A 1 x 1 x 1 brick of cells 2.8 to 3 wide
// (replicas that need the larger LDS layout) has up to 14 chunks of
// candidates: with 12 it took two passes (64 replicas of 1,000 to 65,536, a
// fifth rebuilding: 167 us per launch, 158 with 15).
constexpr int kNbChunks = 12, kNbChunksBig = 15;
static_assert(kNbChunks >= 12 && kNbChunksBig >= 12, "kMostChunks counts on passes of 12");
constexpr int kNbWaves = 4;     // bricks per block
constexpr int kCoopWaves = 8;   // waves per brick (COOP)
constexpr int kCoopBlocks = 1024;  // most blocks of the COOP form
constexpr float kUnclear = 1.0e-5f;

// (This file is compiled with -fno-honor-nans: the results hold no NaN, as
// positions are finite after the wrap, and the minimum needs no quieting of
// its operands.)
__device__ inline float least_magnitude(const f32x16& w) {
  float least = 3.0e38f;
#pragma unroll
  for (int r = 0; r < 16; r += 2)
    least = __builtin_fminf(__builtin_fminf(__builtin_fabsf(w[r]), __builtin_fabsf(w[r + 1])), least);
  return least;
}

__device__ inline uint32_t image_code(int32_t sx, int32_t sy, int32_t sz) {
  return ((uint32_t)(sx & 3) | ((uint32_t)(sy & 3) << 2) | ((uint32_t)(sz & 3) << 4))
         << kIdxBits;
}
// the shift -1 / 0 / 1 of one axis (lsb 26, 28, 30) of an image code
__device__ inline double image(uint32_t code, int lsb) {
  return (double)(((int32_t)(code << (30 - lsb))) >> 30);
}

// NS = 2: at most two species; NS = 4: up to four.
//
// COOP: contexts with few bricks, where the time is the latency of one wave's
// walk (4,000 particles, 125 bricks: 67 to 90 us).  The eight waves of a block share
// a brick: each takes every eighth chunk of the test phase and every
// sixteenth list chunk of a home in the write phase, starting at that chunk's
// rank; a brick's groups of homes go to `groups` blocks.  The rows are the
// same, entry for entry.  15 us in that box (nlist_small.hip: 28 us).
template <int NS, bool COOP, int CH>
__global__ __launch_bounds__(64 * (COOP ? kCoopWaves : kNbWaves))
__attribute__((amdgpu_waves_per_eu(COOP || CH > kNbChunks ? 4 : 5))) void
k_nlist_brick(BrickArgs A, const RepDesc* __restrict__ reps, const int32_t* __restrict__ rebuild,
              const PairTab* __restrict__ tab, const int32_t* __restrict__ cell_start,
              int32_t stride, int32_t cap, int32_t flip, const double4* __restrict__ pos_tmp,
              const double* __restrict__ vel_tmp, const int32_t* __restrict__ id_tmp,
              double4* __restrict__ pos, double* __restrict__ vel, int32_t* __restrict__ id,
              double* __restrict__ xref, int32_t* __restrict__ ncount, DevState* st,
              int32_t spread, int32_t groups) {
  constexpr int kW = COOP ? kCoopWaves : kNbWaves;  // waves per block
  constexpr int kB = COOP ? 1 : kNbWaves;           // bricks per block
  constexpr int kShare = COOP ? kCoopWaves : 1;     // waves per brick
  __shared__ double s_thr[16];
  __shared__ uint32_t s_n[COOP ? kW : 1][64], s_full[COOP ? kW : 1][64];
  __shared__ uint32_t s_kc[kB][CH * 64];  // sorted index | image code
  __shared__ uint16_t s_ent[kB][CH * 64];  // list entry
  // [word][home], a spare row before and after a wave's
  __shared__ uint32_t s_hits[kB][(2 * CH + 2) * kGroup];
  if (!st->any_rebuild) return;  // whole block: one flag load when nothing rebuilds
  if (threadIdx.x < 16) s_thr[threadIdx.x] = tab->thr[threadIdx.x];
  __syncthreads();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int ws = COOP ? wv : 0;  // share of the brick's work
  const int32_t b =
      COOP ? (int32_t)blockIdx.x / groups
           : (spread ? xcd_spread(blockIdx.x, spread) : xcd_block(blockIdx.x, gridDim.x)) *
                     kNbWaves + wv;
  const int32_t grp = COOP ? (int32_t)blockIdx.x % groups : 0;
  auto sync = [&]() {
    if constexpr (COOP)
      __syncthreads();
    else
      wave_lds_sync();
  };
  if (b >= A.nbricks) return;
  const Brick B = A.bricks[b];
  const BrickTile T = A.tiles[B.tile];
  if (!rebuild[T.rep]) return;
  const RepDesc R = reps[T.rep];
  const int32_t nc = R.nc;
  uint32_t* const kc = s_kc[COOP ? 0 : wv];
  uint16_t* const ent = s_ent[COOP ? 0 : wv];
  uint32_t* const hits = s_hits[COOP ? 0 : wv] + kGroup;

  // lane q: row q of the cells around the brick, as up to three pieces
  const int32_t ry = B.hy + 2, nr = ry * (B.hz + 2), nhr = B.hy * B.hz;
  const int32_t X = T.cx + B.lx;
  int32_t kl = 0, km = 0, kr = 0, nl = 0, nm = 0, nrt = 0, dl = 0, dm = 0, dr = 0;
  uint32_t cyz = 0;
  if (lane < nr) {
    const int32_t qy = lane % ry, qz = lane / ry;
    int32_t y = T.cy + B.ly + qy - 1, z = T.cz + B.lz + qz - 1, sy, sz;
    wrap_cell(y, nc, sy);
    wrap_cell(z, nc, sz);
    cyz = image_code(0, sy, sz);
    const int32_t* c = cell_start + R.coff + (z * nc + y) * nc;
    const int32_t lo = X - 1, hi = X + B.hx;
    const int32_t mlo = lo < 0 ? 0 : lo, mhi = hi >= nc ? nc - 1 : hi;
    kl = c[nc - 1];
    nl = lo < 0 ? c[nc] - kl : 0;
    km = c[mlo];
    nm = c[mhi + 1] - km;
    kr = c[0];
    nrt = hi >= nc ? c[1] - kr : 0;
    // slot of a piece's particle j: j + d
    const TileRow tr = A.row[(size_t)B.tile * A.rows + (B.ly + qy) + (B.lz + qz) * (T.ty + 2)];
    dl = tr.l0 - tr.gl;
    dm = tr.l1 - tr.gm;
    dr = tr.l2 - tr.gr;
  }
  const int32_t rend = wave_scan(nl + nm + nrt, lane);
  const int32_t pl = rend - (nl + nm + nrt), pm = pl + nl, pr = pm + nm;  // packed starts
  const int32_t ncand = __builtin_amdgcn_readlane(rend, nr - 1);
  const bool face = __builtin_amdgcn_ballot_w64(cyz != 0u || nl || nrt) != 0;
  // lane r: home row r
  int32_t hg = 0, hn = 0, hv = 0;
  {
    const int src = lane < nhr ? (lane / B.hy + 1) * ry + lane % B.hy + 1 : 0;
    const int32_t pms = __shfl(pm, src, 64), kms = __shfl(km, src, 64);
    if (lane < nhr) {
      const int32_t* c = cell_start + R.coff +
                         ((T.cz + B.lz + lane / B.hy) * nc + T.cy + B.ly + lane % B.hy) * nc + X;
      hg = c[0];
      hn = c[B.hx] - hg;
      hv = pms + (hg - kms);  // packed candidate of its first particle
    }
  }
  const int32_t hend = wave_scan(hn, lane);
  const int32_t nh = __builtin_amdgcn_readlane(hend, nhr - 1);
  const int32_t hpre = hend - hn;
  // sorted index and own packed candidate of home h
  auto home = [&](int32_t h, int32_t& i, int32_t& v) {
    i = 0;
    v = 0;
    for (int r = 0; r < nhr; ++r) {
      const int32_t p = __builtin_amdgcn_readlane(hpre, r);
      if (h >= p) {
        i = __builtin_amdgcn_readlane(hg, r) + (h - p);
        v = __builtin_amdgcn_readlane(hv, r) + (h - p);
      }
    }
  };
  const double ccx = ((double)X + 0.5 * (double)B.hx) * R.cside,
               ccy = ((double)(T.cy + B.ly) + 0.5 * (double)B.hy) * R.cside,
               ccz = ((double)(T.cz + B.lz) + 0.5 * (double)B.hz) * R.cside;
  const int32_t width = max(max((int32_t)B.hx, (int32_t)B.hy), (int32_t)B.hz);
  // in squared lengths from here on
  const float side2 = (float)(R.cside * R.cside);
  const float unclear = kUnclear * (float)(width * width) * side2, no_hit = kNoHit * side2;
  const int hl = lane & (kGroup - 1), seg = lane >> 5;
  const double fsp = (double)flip;
  // the candidate of a chunk that this lane loads: result register r of lane
  // l is matrix row 8 (r / 4) + 4 (l / 32) + r % 4, so that row 8 a + 4 b + c
  // holds candidate 16 b + 4 a + c and a lane's 16 results are 16 candidates
  // in order
  const int cofs = (lane & 32) + ((lane >> 2) & 1) * 16 + ((lane >> 3) & 3) * 4 + (lane & 3);

  // groups of at most kGroup home particles, of equal size
  const int32_t ngrp = (nh + kGroup - 1) / kGroup;
  const int32_t gsz = ngrp ? (nh + ngrp - 1) / ngrp : 1;
  // (the replica's own, not the context's: the order of its rows depends on it)
  const int32_t pass = 64 * (CH > kNbChunks ? min((int32_t)B.pass, CH) : CH);
  int32_t filled = -1;  // the pass whose candidates kc and ent hold
  for (int32_t g0 = grp * gsz; g0 < nh; g0 += gsz * (COOP ? groups : 1)) {
    const int32_t gn = nh - g0 < gsz ? nh - g0 : gsz;
    int32_t ih, vh;  // column hl: its sorted index and own packed candidate
    home(g0 + (hl < gn ? hl : 0), ih, vh);
    int32_t cnt = 0, nch = 0;  // its entries and chunks so far
    uint4* const row = A.list + list_base(ih, A.capc);
    // lanes < 32 hold the rows k = 0, 2, 4 (6) of the operand, the others
    // k = 1, 3, 5 (7)
    float b0, b1, b2, b3 = 0.0f;
    {
      const double4 p = pos_tmp[ih];
      const float ux = (float)(p.x - ccx), uy = (float)(p.y - ccy), uz = (float)(p.z - ccz);
      const double* th = &s_thr[4 * (int32_t)p.w];
      const float a0 = (float)th[0], d1 = (float)(th[1] - th[0]);
      const float uu = __builtin_fmaf(uz, uz, __builtin_fmaf(uy, uy, ux * ux));
      b0 = -2.0f * (seg ? uy : ux);
      b1 = seg ? 1.0f : -2.0f * uz;
      b2 = seg ? (hl < gn ? uu - a0 : no_hit) : -d1;
      if constexpr (NS > 2) b3 = (float)(th[0] - th[seg ? 3 : 2]);
    }
    for (int32_t pb = 0; pb < ncand; pb += pass) {
      const int32_t np = ncand - pb < pass ? ncand - pb : pass;
      const int32_t nwords = 2 * ((np + 63) >> 6);
      if (filled != pb) {
        // index, image and slot of every candidate of the pass
        auto fill = [&](int32_t k, int32_t n, int32_t p, int32_t d, uint32_t code) {
          for (int32_t t = lane; t < n; t += 64) {
            const int32_t v = p + t - pb;
            if (v >= 0 && v < np) {
              kc[v] = (uint32_t)(k + t) | code;
              ent[v] = (uint16_t)((k + t + d) << A.shift);
            }
          }
        };
        for (int q = ws; q < nr; q += kShare) {
#define MDK_RL(x) __builtin_amdgcn_readlane((x), q)
          const uint32_t cq = (uint32_t)MDK_RL((int32_t)cyz);
          fill(MDK_RL(km), MDK_RL(nm), MDK_RL(pm), MDK_RL(dm), cq);
          if (face) {
            fill(MDK_RL(kl), MDK_RL(nl), MDK_RL(pl), MDK_RL(dl), cq | image_code(-1, 0, 0));
            fill(MDK_RL(kr), MDK_RL(nrt), MDK_RL(pr), MDK_RL(dr), cq | image_code(1, 0, 0));
          }
#undef MDK_RL
        }
        sync();
      }
      const bool first = filled != pb;  // the species bits are not in ent yet
      filled = pb;
      int32_t n = 0;  // lane: hits of its words in this pass, then of its home
      // the range of the group's own candidates in the pass
      int32_t own0 = vh - pb, own1 = vh - pb;
#pragma unroll
      for (int d = 16; d >= 1; d >>= 1) {
        own0 = min(own0, __shfl_xor(own0, d, 64));
        own1 = max(own1, __shfl_xor(own1, d, 64));
      }
      own0 = __builtin_amdgcn_readfirstlane(own0);
      own1 = __builtin_amdgcn_readfirstlane(own1);
      uint32_t full = 0u;  // its words that hold hits (bit = word of the pass)
      // ---- test phase ----
      uint32_t kcv = 0u;
      double4 q{};
      auto fetch = [&](int32_t base) {
        const int32_t v = base + cofs;
        kcv = kc[v < np ? v : 0];
        q = pos_tmp[kcv & kIdxMask];
      };
      fetch(ws * 64);
      for (int32_t base = ws * 64; base < np; base += 64 * kShare) {
        const int32_t v = base + cofs;
        const int32_t tj = (int32_t)q.w;
        if (first && v < np) {
          const uint32_t sp = NS > 2 ? (uint32_t)tj << 14 : (q.w == fsp ? 1u << 14 : 0u);
          ent[v] = (uint16_t)(ent[v] | sp);
        }
        double dx = q.x - ccx, dy = q.y - ccy, dz = q.z - ccz;
        if (face) {
          dx += image(kcv, 26) * R.L;
          dy += image(kcv, 28) * R.L;
          dz += image(kcv, 30) * R.L;
        }
        float ax = (float)dx, ay = (float)dy, az = (float)dz;
        float aq = v < np ? __builtin_fmaf(az, az, __builtin_fmaf(ay, ay, ax * ax)) : no_hit;
        float as = NS > 2 ? (tj == 1 ? 1.0f : 0.0f) : (float)q.w, one = 1.0f;
        float s2 = tj == 2 ? 1.0f : 0.0f, s3 = tj == 3 ? 1.0f : 0.0f;
        if (base + 64 * kShare < np) fetch(base + 64 * kShare);  // in flight under the product
        // first 32 candidates in (ax, az, as, s2), last 32 in (ay, aq, one, s3)
        swap_halves(ax, ay);
        swap_halves(az, aq);
        swap_halves(as, one);
        if constexpr (NS > 2) swap_halves(s2, s3);
        f32x16 w0 = {}, w1 = {};
        w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(ax, b0, w0, 0, 0, 0);
        w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ay, b0, w1, 0, 0, 0);
        w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(az, b1, w0, 0, 0, 0);
        w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(aq, b1, w1, 0, 0, 0);
        w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(as, b2, w0, 0, 0, 0);
        w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(one, b2, w1, 0, 0, 0);
        if constexpr (NS > 2) {
          w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(s2, b3, w0, 0, 0, 0);
          w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(s3, b3, w1, 0, 0, 0);
        }
        uint32_t m0 = sign_bits(w0), m1 = sign_bits(w1);
        if (__builtin_amdgcn_ballot_w64(least_magnitude(w0) < unclear ||
                                        least_magnitude(w1) < unclear) != 0) {
          // the FP64 test of the lane's unclear pairs
          uint32_t un = 0u;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            un |= __builtin_fabsf(w0[r]) < unclear ? 1u << r : 0u;
            un |= __builtin_fabsf(w1[r]) < unclear ? 0x10000u << r : 0u;
          }
          uint32_t mm = m0 | (m1 << 16);
          while (un) {
            const int r = __builtin_ctz(un);
            un &= un - 1u;
            const uint32_t cj = kc[base + ((r & 16) << 1) + seg * 16 + (r & 15)];
            const double4 pj = pos_tmp[cj & kIdxMask];
            const double4 pi = pos_tmp[ih];
            const double ex = (pj.x - pi.x) + image(cj, 26) * R.L,
                         ey = (pj.y - pi.y) + image(cj, 28) * R.L,
                         ez = (pj.z - pi.z) + image(cj, 30) * R.L;
            const bool hit =
                (ex * ex + ey * ey) + ez * ez < s_thr[4 * (int32_t)pi.w + (int32_t)pj.w];
            mm = (mm & ~(1u << r)) | (hit ? 1u << r : 0u);
          }
          m0 = mm & 0xffffu;
          m1 = mm >> 16;
        }
        // lane h < 32: the word of home h for the first 32 candidates, lane
        // h + 32: for the last 32
        swap_halves(m0, m1);
        uint32_t word = m0 | (m1 << 16);
        if (base <= own1 && own0 < base + 64) {  // not its own neighbour
          const int32_t self = vh - pb - base - 32 * seg;
          if (self >= 0 && self < 32) word &= ~(1u << self);
        }
        hits[(base >> 6) * 64 + lane] = word;
        n += (int32_t)__popc(word);
        full |= word ? (1u << (base >> 5)) << seg : 0u;
      }
      if constexpr (COOP) {
        s_n[ws][lane] = (uint32_t)n;
        s_full[ws][lane] = full;
        __syncthreads();
        n = 0;
        full = 0u;
#pragma unroll
        for (int q = 0; q < kW; ++q) {
          n += (int32_t)(s_n[q][hl] + s_n[q][hl + 32]);
          full |= s_full[q][hl] | s_full[q][hl + 32];
        }
        n = hl < gn ? n : 0;
      } else {
        n = hl < gn ? n + __shfl_xor(n, 32, 64) : 0;
        full |= (uint32_t)__shfl_xor((int32_t)full, 32, 64);
        wave_lds_sync();
      }
      // ---- write phase ----
      // the first lane of a home takes the first c0 whole chunks, the second
      // the rest of the pass, walking back from the last candidate
      const int32_t c0 = (n + 8) >> 4;
      if constexpr (COOP) {
        // list chunk q of home hl: from its first entry's rank on
        const int32_t nq = (n + kChunkEntries - 1) / kChunkEntries;
        for (int32_t q = threadIdx.x >> 5; q < nq; q += 2 * kW) {
          const bool back = q >= c0;
          int32_t rank = kChunkEntries * (back ? q - c0 : q);
          const int32_t left = back ? n - kChunkEntries * c0 - rank : kChunkEntries;
          uint32_t m = back ? __builtin_bitreverse32(full) >> (32 - nwords) : full;
          int f = 0;
          uint32_t cur = 0u;
          auto next = [&]() {
            f = __builtin_ctz(m);
            m &= m - 1u;
            const uint32_t x = hits[(back ? nwords - 1 - f : f) * kGroup + hl];
            cur = back ? __builtin_bitreverse32(x) : x;
          };
          for (next(); (int32_t)__popc(cur) <= rank; next()) rank -= (int32_t)__popc(cur);
          for (; rank > 0; --rank) cur &= cur - 1u;
          uint32_t e[4];
#pragma unroll
          for (int u = 0; u < kChunkEntries; ++u) {
            uint32_t x = (uint32_t)(A.slots - 1) << A.shift;
            if (u < left) {
              if (cur == 0u) next();
              const int32_t k = f * 32 + __builtin_ctz(cur);
              cur &= cur - 1u;
              x = ent[back ? nwords * 32 - 1 - k : k];
            }
            if (u & 1)
              e[u / 2] |= x << 16;
            else
              e[u / 2] = x;
          }
          if (nch + q < A.capc) row[(size_t)(nch + q) * kSlice] = make_uint4(e[0], e[1], e[2], e[3]);
        }
      } else {
        int32_t left = seg ? n - 8 * c0 : 8 * c0;
        int32_t c = nch + (seg ? c0 : 0);
        // A lane walks the words that hold hits, the second lane from the last
        // one back with their bits reversed.  Byte offsets: the entry of bit b
        // of its f-th word is at ebase + f eword + b estep, the word itself at
        // hbase + f hword; f = -1 when none is left, a spare row of hits.
        if (seg) full = __builtin_bitreverse32(full) >> (32 - nwords);
        const int estep = seg ? -2 : 2, eword = 32 * estep, hword = seg ? -128 : 128;
        const int ebase = seg ? (nwords * 32 - 1) * 2 : 0;
        const int hbase = (seg ? (nwords - 1) * 128 : 0) + hl * 4;
        uint32_t cur = 0u, nxt;
        int f, eat = 0;
        auto ahead = [&]() {
          f = full ? __builtin_ctz(full) : -1;
          full &= full - 1u;
          nxt = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(hits) + hbase +
                                                   __mul24(f, hword));
        };
        ahead();
        // eight entries of every lane with left > 0: the places past the last
        // entry (LAST) take the far slot; the lanes stay in step
        auto chunk = [&](auto last_tag) {
          constexpr bool LAST = decltype(last_tag)::value;
          uint32_t e[4];
  #pragma unroll
          for (int u = 0; u < kChunkEntries; ++u) {
            uint32_t x = (uint32_t)(A.slots - 1) << A.shift;
            if (!LAST || u < left) {
              if (cur == 0u) {
                cur = seg ? __builtin_bitreverse32(nxt) : nxt;
                eat = ebase + __mul24(f, eword);
                ahead();
              }
              x = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(ent) + eat +
                                                     __mul24(__builtin_ctz(cur), estep));
              cur &= cur - 1u;
            }
            if (u & 1)
              e[u / 2] |= x << 16;
            else
              e[u / 2] = x;
          }
          if (c < A.capc) row[(size_t)c * kSlice] = make_uint4(e[0], e[1], e[2], e[3]);
          ++c;
          left -= kChunkEntries;
        };
        for (int32_t t = 0; t < A.capc && __builtin_amdgcn_ballot_w64(left > 0); ++t) {
          if (__builtin_amdgcn_ballot_w64(left > 0 && left < kChunkEntries) == 0) {
            if (left > 0) chunk(std::false_type{});
          } else {
            if (left > 0) chunk(std::true_type{});
          }
        }
      }
      cnt += n;
      nch += (n + kChunkEntries - 1) / kChunkEntries;
      sync();  // the next pass or group rewrites the hits
    }
    if (lane < gn && ws == 0) {
      ncount[ih] = cnt;
      A.nchunk[ih] = nch;
      if (cnt > cap || nch > A.capc) atomicOr(&st->err, kErrOverflow);
    }
  }
  // the new cell order becomes the live state
  if (COOP && grp != 0) return;
  for (int32_t h = ws * 64 + lane; h < ((nh + 63) & ~63); h += 64 * kShare) {
    int32_t i, v;
    home(h < nh ? h : 0, i, v);
    if (h < nh) {
      const double4 p4 = pos_tmp[i];
      pos[i] = p4;
      xref[i] = p4.x;
      xref[stride + i] = p4.y;
      xref[2 * (size_t)stride + i] = p4.z;
      vel[i] = vel_tmp[i];
      vel[stride + i] = vel_tmp[stride + i];
      vel[2 * (size_t)stride + i] = vel_tmp[2 * (size_t)stride + i];
      id[i] = id_tmp[i];
    }
  }
}

// The rows back as sorted indices in the gather layout (neighbour-list parity
// hook): one block per tile, a thread per home particle.
__global__ __launch_bounds__(256) void k_decode_brick(BrickArgs A, int32_t cap,
                                                      const int32_t* __restrict__ ncount,
                                                      uint32_t* __restrict__ out) {
  const BrickTile T = A.tiles[blockIdx.x];
  const int32_t nr = (T.ty + 2) * (T.tz + 2), nhr = T.ty * T.tz;
  const TileRow* tr = A.row + (size_t)blockIdx.x * A.rows;
  const HomeRow* hr = A.hrow + (size_t)blockIdx.x * A.hrows;
  for (int32_t h = threadIdx.x; h < A.head[blockIdx.x].nh; h += blockDim.x) {
    const int32_t i = home_index(hr, nhr, h, A.head[blockIdx.x].nh);
    const int32_t n = min(ncount[i], cap), nch = min(A.nchunk[i], A.capc);
    const uint16_t* e = reinterpret_cast<const uint16_t*>(A.list + list_base(i, A.capc));
    const size_t b = list_base(i, cap);
    int32_t k = 0;
    for (int32_t c = 0; c < nch && k < n; ++c)
      for (int u = 0; u < kChunkEntries && k < n; ++u) {
        const int32_t s = (e[(size_t)c * kSlice * kChunkEntries + u] & 0x3fff) >> A.shift;
        if (s == A.slots - 1) continue;
        int q = 0;
        while (q + 1 < nr && tr[q].l3 <= s) ++q;
        const TileRow w = tr[q];
        const int32_t j = s < w.l1 ? w.gl + (s - w.l0)
                                   : (s < w.l2 ? w.gm + (s - w.l1) : w.gr + (s - w.l2));
        out[b + (size_t)k * kSlice] = (uint32_t)j;
        ++k;
      }
  }
}

}  // namespace

int32_t nlist_brick_pass(bool big) { return big ? kNbChunksBig : kNbChunks; }

void launch_nlist_brick(hipStream_t s, const BrickArgs& A, int32_t ntypes, const RepDesc* reps,
                        const int32_t* rebuild, const PairTab* tab, const int32_t* cell_start,
                        int32_t stride, int32_t cap, const BrickPair& bp,
                        const double4* pos_tmp, const double* vel_tmp, const int32_t* id_tmp,
                        double4* pos, double* vel, int32_t* id, double* xref, int32_t* ncount,
                        DevState* st, int32_t spread) {
  const int32_t nb = (A.nbricks + kNbWaves - 1) / kNbWaves;
  const int32_t g = spread / kNbWaves, grid = g ? spread_grid(nb, g) : nb;
  // entries carry the species as one bit (two-species constants) or as two
  // (the table of up to four)
#define KB(NS, CO, CH, GRID, W)                                                          \
  k_nlist_brick<NS, CO, CH><<<GRID, 64 * W, 0, s>>>(                                     \
      A, reps, rebuild, tab, cell_start, stride, cap, bp.flip, pos_tmp, vel_tmp, id_tmp, \
      pos, vel, id, xref, ncount, st, g, A.groups)
#define KC(NS, CH)                                                          \
  if (A.nbricks * A.groups <= kCoopBlocks)                                  \
    KB(NS, true, CH, A.nbricks * A.groups, kCoopWaves);                     \
  else                                                                      \
    KB(NS, false, CH, grid, kNbWaves)
  const bool four = bp.four || ntypes > 2;
  if (A.slots > kBrickSlots) {
    if (four) { KC(4, kNbChunksBig); } else { KC(2, kNbChunksBig); }
  } else {
    if (four) { KC(4, kNbChunks); } else { KC(2, kNbChunks); }
  }
#undef KC
#undef KB
}

void launch_decode_brick(hipStream_t s, const BrickArgs& A, int32_t cap, const int32_t* ncount,
                         uint32_t* out) {
  k_decode_brick<<<A.ntiles, 256, 0, s>>>(A, cap, ncount, out);
}

}  // namespace mdk
