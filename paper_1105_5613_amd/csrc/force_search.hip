// force_search.hip -- the list-free force evaluation ("Grid-search method",
// Fig. 1) on tiles of cells (brick.h): every launch finds the interacting
// pairs from the cell grid itself, on the matrix cores, and evaluates them
// from LDS.  No neighbour list is kept.  The pair function is that of
// force_brick.hip, displacement, r^2 and the cut-off test in FP64.
//
// One block per tile copies the tile's neighbourhood into LDS as there; a wave
// takes one brick of home cells (1 x 1 x 1 at the Lennard-Jones density) at a
// time, at most 32 home particles together.  LDS allows two blocks per CU, so
// that in tiles of fewer bricks than eight, whose cells are crowded, the groups
// of a brick's homes go to several waves (plan_bricks).
//
// Search.  The candidates of a brick are, per neighbour row, one run of slots;
// the runs are cut into pieces of at most 32 slots, the words of candidates,
// two words to a chunk.  With u = x - centre of the brick,
//   r^2 - rc_ij^2 = -2 u_i . u_j + |u_j|^2 - b_i s_j + (|u_i|^2 - a_i)
// for 32 candidates against the 32 homes is a product of a 32 x 6 and a 6 x 32
// matrix, three v_mfma_f32_32x32x2 (a fourth for the species 2 and 3), as in
// nlist_brick.hip.  The sign bits are the hits.  FP32 errs by less than 4e-6
// of the squared width of the brick; a_i is widened by five times that, so that
// every pair inside the cut-off is among the hits, and the FP64 test of the
// evaluation decides.
//
// Evaluation.  The two lanes of a home walk the set bits of its words, one from
// the first hit on and one from the last back, the same number each; a word
// comes with its first slot and the species bits of its candidates.  The two
// sums of a home are added at the end.
//
// What bounds it: vector issue (in 0.68 of a launch of 1,048,576 particles,
// 400 us) at four waves per SIMD, which LDS allows (62 pairs per particle in
// the evaluation, half of the time at 1 to 2 ns per instruction; the sign bits
// and operands of the search), and the waves' wait for the copy to LDS.  The
// form before this (force_cells.hip: one lane per home, candidates through the
// scalar cache) tests every candidate in FP64, 720 per particle, and stays for
// row tiles asked for and for boxes too dense for the tiles.
// Measured per launch at 262,144 particles FP64: 526 -> 142 us, the search 65
// and the evaluation 38 of it (reading candidates ahead, 4 pairs in flight
// instead of 2, words of two 16-slot pieces: 141 to 148 us).
#include <type_traits>

#include "brick_device.h"

namespace mdk {
namespace {

constexpr float kWiden = 2.0e-5f;  // of the squared width of the brick
constexpr int kWaves = 8;          // waves per block, at most (two blocks fit a CU)
constexpr int kPiece = 32;         // slots per word, at most
constexpr int kUnroll = 2;         // pairs of a lane's walk in flight together

// NS = 2: at most two species, one bit per candidate; NS = 4: two.
template <bool MIXED, int MODE, bool EN, int NS>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(4))) void
k_force_search(BrickArgs A, const RepDesc* __restrict__ reps, const PairTab* __restrict__ tab,
               const BrickPair* __restrict__ bp, const int32_t* __restrict__ cell_start,
               const double4* __restrict__ pos, double* __restrict__ vel,
               void* __restrict__ frc_, int32_t stride, double dt, double* __restrict__ part,
               DevState* st, FuseOut fo) {
  using T = typename std::conditional<MIXED, float, double>::type;
  constexpr int kPadSlot = kBrickSlots - 1, kPlanes = NS > 2 ? 2 : 1;
  // words per pass: three for each of the nine rows at the Lennard-Jones
  // density; two blocks' LDS fits a CU
  constexpr int kWords = NS > 2 ? 24 : 27, kMeta = 1 + kPlanes;
  __shared__ double2 s_xy[kBrickSlots];
  __shared__ double s_z[kBrickSlots];
  __shared__ uint32_t s_sp[kPlanes][kBrickSlots / 32 + 1];  // species bits of the slots
  __shared__ uint32_t s_hits[kWaves][kWords * kGroup];      // [word][home]
  __shared__ uint32_t s_word[kWaves][kMeta * (kWords + 1)];  // first slot | slots << 16, species bits
  __shared__ double s_red[4][kWaves];
  __shared__ typename std::conditional<EN && (NS > 2), EnergyTab<T>, char>::type s_en[1];
  // energy constants by home species and species bit (force_brick.hip): v12, or
  // rc and 12 vc in the mixed form; one read per pair (the form with two species
  // has no registers to spare)
  __shared__ typename std::conditional<MIXED, float2, double>::type s_ev[EN && NS == 2 ? 8 : 1];
  __shared__ PairRow s_pair[NS > 2 ? 16 : 1];
  __shared__ double s_mass[4], s_im[4];
  static_assert(sizeof(TileRow) * kTileRows <= sizeof(s_hits), "rows share the words' LDS");
  TileRow* const s_row = reinterpret_cast<TileRow*>(&s_hits[0][0]);
  const int32_t tb = xcd_block(blockIdx.x, gridDim.x);
  const BrickTile Tl = A.tiles[tb];
  const TileRow* trow = A.row + (size_t)tb * A.rows;
  const int nthr = blockDim.x, nw = nthr / 64;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int32_t ry = Tl.ty + 2, nrow = ry * (Tl.tz + 2);
  if (halted(st)) {  // as in force_brick.hip
    if (blockIdx.x == 0 && threadIdx.x == 0) st->any_rebuild = 0;
    if constexpr (MODE == 2) {
      const HomeRow* hr = A.hrow + (size_t)tb * A.hrows;
      const int32_t nh = A.head[tb].nh, nhr = Tl.ty * Tl.tz;
      for (int32_t h = threadIdx.x; h < nh; h += nthr) {
        const int32_t i = home_index(hr, nhr, h, nh);
        fo.pos_out[i] = pos[i];
      }
    }
    return;
  }
  if constexpr (MODE == 2) {
    const uint32_t gz = blockIdx.x * (uint32_t)nthr + threadIdx.x;  // up to 2^32 (plan_bricks)
    if (gz < (uint32_t)fo.nzero) fo.counts[gz] = 0;
  }
  if ((int)threadIdx.x < nrow) s_row[threadIdx.x] = trow[threadIdx.x];
  for (int k = threadIdx.x; k < kPlanes * (kBrickSlots / 32 + 1); k += nthr) (&s_sp[0][0])[k] = 0u;
  if (threadIdx.x < 4) {
    s_mass[threadIdx.x] = tab->mass[threadIdx.x];
    s_im[threadIdx.x] = tab->inv_mass[threadIdx.x];
  }
  if (threadIdx.x < 16) {
    const int k = threadIdx.x;
    if constexpr (EN && NS == 2) {
      if (k < 8) {
        if constexpr (MIXED)
          s_ev[k] = make_float2(bp->mrc[k >> 1][k & 1], bp->mv12[k >> 1][k & 1]);
        else
          s_ev[k] = __builtin_fma(bp->v12[k >> 1][1], (k & 1) ? 2.0 : 0.0, bp->v12[k >> 1][0]);
      }
    }
    if constexpr (EN && NS > 2) {
      fill_energy(s_en[0], tab, k);
    }
    if constexpr (NS > 2) {
      s_pair[k] = pair_row(tab, k);
    }
  }
  if (threadIdx.x == 0) {
    s_xy[kPadSlot] = make_double2(kFarAway, 0.0);
    s_z[kPadSlot] = 0.0;
  }
  const RepDesc& R = reps[Tl.rep];
  const int32_t nc = R.nc;
  const int32_t flip = bp->flip;
  __syncthreads();
  copy_neighbourhood(Tl, R, s_row, pos, s_xy, s_z, kPadSlot, wv, nw, lane,
                     [&](int32_t v, const double4& c) {
    const int32_t tj = (int32_t)c.w;
    if constexpr (NS > 2) {
      if (tj & 1) atomicOr(&s_sp[0][v >> 5], 1u << (v & 31));
      if (tj & 2) atomicOr(&s_sp[1][v >> 5], 1u << (v & 31));
    } else {
      if (tj == flip) atomicOr(&s_sp[0][v >> 5], 1u << (v & 31));
    }
  });
  __syncthreads();  // the rows' LDS holds words from here on

  uint32_t* const hits = s_hits[wv];
  uint32_t* const meta = s_word[wv];
  const int hl = lane & (kGroup - 1), seg = lane >> 5;
  const uint32_t back = seg ? 31u : 0u;
  // the candidate of a chunk that this lane loads (see nlist_brick.hip)
  const int cofs = (lane & 32) + ((lane >> 2) & 1) * 16 + ((lane >> 3) & 3) * 4 + (lane & 3);
  const T mk = MIXED ? (T)bp->mk : (T)0;
  double sum_pe = 0.0, sum_w = 0.0, sum_ke = 0.0, d2 = 0.0;

  // unit: a brick, or every Tl.groups-th group of its homes
  const int32_t units = wv < Tl.waves ? Tl.nb * Tl.groups : 0;
  for (int32_t un = wv; un < units; un += Tl.waves) {
    const int32_t bi = un / Tl.groups, gfirst = un - bi * Tl.groups;
    const Brick B = A.bricks[Tl.b0 + bi];
    // lane q: the run of neighbour row q
    const int32_t by = B.hy + 2, nr = by * (B.hz + 2), nhr = B.hy * B.hz;
    const int32_t X = Tl.cx + B.lx;
    int32_t rs = 0, rn = 0, ms = 0, mg = 0;  // first slot, slots, main piece's
    if (lane < nr) {
      const int32_t qy = B.ly + lane % by, qz = B.lz + lane / by;  // row of the tile
      int32_t y = Tl.cy + qy - 1, z = Tl.cz + qz - 1, s;
      wrap_cell(y, nc, s);
      wrap_cell(z, nc, s);
      const int32_t* c = cell_start + R.coff + (z * nc + y) * nc;
      const TileRow tr = trow[qy + qz * ry];
      const int32_t lo = X - 1, hi = X + B.hx;
      rs = lo < 0 ? tr.l0 : tr.l1 + (c[lo] - tr.gm);
      rn = (hi >= nc ? tr.l3 : tr.l1 + (c[hi + 1] - tr.gm)) - rs;
      ms = tr.l1;
      mg = tr.gm;
    }
    const int32_t rp = (rn + kPiece - 1) / kPiece;  // pieces of the run
    const int32_t pend = wave_scan(rp, lane);
    const int32_t pbeg = pend - rp;
    const int32_t npiece = __builtin_amdgcn_readlane(pend, nr - 1);
    // lane r: home row r, its sorted index, slot and place among the pieces
    int32_t hg = 0, hn = 0, hs = 0, hp = 0;
    {
      const int src = lane < nhr ? (lane / B.hy + 1) * by + lane % B.hy + 1 : 0;
      const int32_t mss = __shfl(ms, src, 64), mgs = __shfl(mg, src, 64);
      const int32_t rss = __shfl(rs, src, 64), pbs = __shfl(pbeg, src, 64);
      if (lane < nhr) {
        const int32_t* c =
            cell_start + R.coff +
            ((Tl.cz + B.lz + lane / B.hy) * nc + Tl.cy + B.ly + lane % B.hy) * nc + X;
        hg = c[0];
        hn = c[B.hx] - hg;
        hs = mss + (hg - mgs);
        hp = pbs * kPiece + (hs - rss);
      }
    }
    const int32_t hend = wave_scan(hn, lane);
    const int32_t nh = __builtin_amdgcn_readlane(hend, nhr - 1);
    const int32_t hpre = hend - hn;
    const double ccx = ((double)X + 0.5 * (double)B.hx) * R.cside,
                 ccy = ((double)(Tl.cy + B.ly) + 0.5 * (double)B.hy) * R.cside,
                 ccz = ((double)(Tl.cz + B.lz) + 0.5 * (double)B.hz) * R.cside;
    const int32_t width = max(max((int32_t)B.hx, (int32_t)B.hy), (int32_t)B.hz);
    const float side2 = (float)(R.cside * R.cside);
    const float widen = kWiden * (float)(width * width) * side2, no_hit = kNoHit * side2;

    // passes of equal size over the pieces, groups of equal size of the homes
    const int32_t npass = (npiece + kWords - 1) / kWords;
    const int32_t psz = npass ? (npiece + npass - 1) / npass : 1;
    const int32_t ngrp = (nh + kGroup - 1) / kGroup;
    const int32_t gsz = ngrp ? (nh + ngrp - 1) / ngrp : 1;
    int32_t filled = -1;  // the pass whose pieces the tables hold
    for (int32_t g0 = gfirst * gsz; g0 < nh; g0 += gsz * Tl.groups) {
      const int32_t gn = nh - g0 < gsz ? nh - g0 : gsz;
      // column hl: sorted index, slot and own candidate (32 piece + place)
      int32_t i = 0, slot = 0, own = 0;
      {
        const int32_t h = g0 + (hl < gn ? hl : 0);
        for (int r = 0; r < nhr; ++r) {
          const int32_t p = __builtin_amdgcn_readlane(hpre, r);
          if (h >= p) {
            i = __builtin_amdgcn_readlane(hg, r) + (h - p);
            slot = __builtin_amdgcn_readlane(hs, r) + (h - p);
            own = __builtin_amdgcn_readlane(hp, r) + (h - p);
          }
        }
      }
      const double px = s_xy[slot].x, py = s_xy[slot].y, pz = s_z[slot];
      const uint32_t b0s = (s_sp[0][slot >> 5] >> (slot & 31)) & 1u;
      const int32_t ti = NS > 2 ? (int32_t)(b0s | (((s_sp[kPlanes - 1][slot >> 5] >> (slot & 31)) & 1u) << 1))
                                : (b0s ? flip : 1 - flip);
      // constants of the home particle's species against either partner
      // species (force_brick.hip)
      double rc1 = 0, drc = 0;
      T a1 = 0, da = 0, c1 = 0, dc = 0, f1 = 0, df = 0;
      if constexpr (NS == 2) {
        rc1 = bp->rc2[ti][0];
        drc = bp->rc2[ti][1];
        a1 = MIXED ? (T)bp->msig2[ti][0] : (T)bp->a[ti][0];
        da = MIXED ? (T)bp->msig2[ti][1] : (T)bp->a[ti][1];
        c1 = MIXED ? (T)bp->mf12[ti][0] : (T)bp->b[ti][0];
        dc = MIXED ? (T)bp->mf12[ti][1] : (T)bp->b[ti][1];
        f1 = MIXED ? (T)bp->mfs[ti][0] : (T)bp->fs[ti][0];
        df = MIXED ? (T)bp->mfs[ti][1] : (T)bp->fs[ti][1];
      }
      // lanes < 32 hold the rows k = 0, 2, 4 (6) of the operand, the others
      // k = 1, 3, 5 (7)
      float o0, o1, o2, o3 = 0.0f;
      {
        const float ux = (float)(px - ccx), uy = (float)(py - ccy), uz = (float)(pz - ccz);
        const float uu = __builtin_fmaf(uz, uz, __builtin_fmaf(uy, uy, ux * ux));
        float r0, r1;
        if constexpr (NS > 2) {
          r0 = (float)s_pair[4 * ti].rc2;
          r1 = (float)s_pair[4 * ti + 1].rc2;
          o3 = r0 - (float)s_pair[4 * ti + (seg ? 3 : 2)].rc2;
        } else {
          r0 = (float)rc1;
          r1 = (float)__builtin_fma(drc, 2.0, rc1);
        }
        o0 = -2.0f * (seg ? uy : ux);
        o1 = seg ? 1.0f : -2.0f * uz;
        o2 = seg ? (hl < gn ? uu - (r0 + widen) : no_hit) : r0 - r1;
      }
      T fx = 0, fy = 0, fz = 0, pe = 0, vw = 0;
      for (int32_t p0 = 0; p0 < npiece; p0 += psz) {
        const int32_t np = npiece - p0 < psz ? npiece - p0 : psz;
        const int32_t nchunk = (np + 1) >> 1;
        if (filled != p0) {
          filled = p0;
          for (int32_t t = 0; t < rp; ++t) {
            const int32_t k = pbeg + t - p0;
            if (k >= 0 && k < np) {
              const uint32_t x = (uint32_t)(rs + kPiece * t);
              meta[kMeta * k] = x | (uint32_t)min(kPiece, rn - kPiece * t) << 16;
#pragma unroll
              for (int pl = 0; pl < kPlanes; ++pl)
                meta[kMeta * k + 1 + pl] =
                    __builtin_amdgcn_alignbit(s_sp[pl][(x >> 5) + 1], s_sp[pl][x >> 5], x & 31u);
            }
          }
          if (lane < kMeta) meta[kMeta * np + lane] = 0u;  // the odd word of the last chunk
          wave_lds_sync();
        }
        // ---- search ----
        int32_t n = 0;       // hits of the lane's words, then of its home
        uint32_t full = 0u;  // its words that hold hits
        // the lane's candidate of a chunk, read ahead under the product
        bool valid = false;
        double2 xy{};
        double zz = 0.0;
        uint32_t sb = 0u, sb1 = 0u;
        auto fetch = [&](int32_t ch) {
          const uint32_t* m = meta + kMeta * (2 * ch + (cofs >> 5));
          const uint32_t pw = m[0];
          const int32_t in = cofs & 31;
          valid = in < (int32_t)(pw >> 16);
          const int32_t v = (int32_t)(pw & 0xffffu) + (valid ? in : 0);
          xy = s_xy[v];
          zz = s_z[v];
          sb = m[1] >> in;
          if constexpr (NS > 2) sb1 = m[kPlanes] >> in;
        };
        fetch(0);
        for (int32_t ch = 0; ch < nchunk; ++ch) {
          float ax = (float)(xy.x - ccx), ay = (float)(xy.y - ccy), az = (float)(zz - ccz);
          float aq = valid ? __builtin_fmaf(az, az, __builtin_fmaf(ay, ay, ax * ax)) : no_hit;
          float as, one = 1.0f, s2 = 0.0f, s3 = 0.0f;
          if constexpr (NS > 2) {
            const uint32_t tj = (sb & 1u) | ((sb1 & 1u) << 1);
            as = tj == 1u ? 1.0f : 0.0f;
            s2 = tj == 2u ? 1.0f : 0.0f;
            s3 = tj == 3u ? 1.0f : 0.0f;
          } else {
            as = (float)(sb & 1u);
          }
          if (ch + 1 < nchunk) fetch(ch + 1);
          swap_halves(ax, ay);
          swap_halves(az, aq);
          swap_halves(as, one);
          if constexpr (NS > 2) swap_halves(s2, s3);
          f32x16 w0 = {}, w1 = {};
          w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(ax, o0, w0, 0, 0, 0);
          w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ay, o0, w1, 0, 0, 0);
          w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(az, o1, w0, 0, 0, 0);
          w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(aq, o1, w1, 0, 0, 0);
          w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(as, o2, w0, 0, 0, 0);
          w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(one, o2, w1, 0, 0, 0);
          if constexpr (NS > 2) {
            w0 = __builtin_amdgcn_mfma_f32_32x32x2f32(s2, o3, w0, 0, 0, 0);
            w1 = __builtin_amdgcn_mfma_f32_32x32x2f32(s3, o3, w1, 0, 0, 0);
          }
          uint32_t m0 = sign_bits(w0), m1 = sign_bits(w1);
          swap_halves(m0, m1);
          // lane h < 32: the word of home h for the first 32 candidates, lane
          // h + 32: for the last 32; places past the word's end never count
          const int32_t word = 2 * ch + seg;
          const uint32_t nv = meta[kMeta * word] >> 16;
          uint32_t hit = (m0 | (m1 << 16)) & (uint32_t)((1ull << nv) - 1ull);
          const uint32_t self = (uint32_t)(own - kPiece * (p0 + word));
          if (self < 32u) hit &= ~(1u << self);  // not its own neighbour
          if (word < np) {
            hits[word * kGroup + hl] = hit;
            n += (int32_t)__popc(hit);
            full |= hit ? 1u << word : 0u;
          }
        }
        n += __shfl_xor(n, 32, 64);
        full |= (uint32_t)__shfl_xor((int32_t)full, 32, 64);
        wave_lds_sync();
        // ---- evaluation ----
        int32_t left = seg ? n >> 1 : (n + 1) >> 1;
        if (seg) full = __builtin_bitreverse32(full) >> (32 - np);
        // word f from the lane's end: byte offsets base + f stride
        const int hstr = (seg ? -kGroup : kGroup) * 4, mstr = (seg ? -kMeta : kMeta) * 4;
        const char* const hbase =
            reinterpret_cast<const char*>(hits + (seg ? (np - 1) * kGroup : 0) + hl);
        const char* const mbase =
            reinterpret_cast<const char*>(meta + (seg ? (np - 1) * kMeta : 0));
        uint32_t cur = 0u, nxt, nsl, nsp[kPlanes], csl = 0u, csp[kPlanes] = {};
        auto ahead = [&]() {
          const int f = full ? __builtin_ctz(full) : 0;
          full &= full - 1u;
          nxt = *reinterpret_cast<const uint32_t*>(hbase + __mul24(f, hstr));
          const uint32_t* m = reinterpret_cast<const uint32_t*>(mbase + __mul24(f, mstr));
          nsl = m[0];
#pragma unroll
          for (int pl = 0; pl < kPlanes; ++pl) nsp[pl] = m[1 + pl];
        };
        ahead();
        while (__builtin_amdgcn_ballot_w64(left > 0) != 0) {
          uint32_t at[kUnroll], sp[kUnroll];
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) {
            at[u] = kPadSlot;
            sp[u] = 0u;
            if (u < left) {
              if (cur == 0u) {
                cur = seg ? __builtin_bitreverse32(nxt) : nxt;
                csl = nsl & 0xffffu;
#pragma unroll
                for (int pl = 0; pl < kPlanes; ++pl) csp[pl] = nsp[pl];
                ahead();
              }
              const uint32_t k = (uint32_t)__builtin_ctz(cur) ^ back;
              cur &= cur - 1u;
              at[u] = csl + k;
              sp[u] = (csp[0] >> k) & 1u;
              if constexpr (NS > 2) sp[u] |= ((csp[kPlanes - 1] >> k) & 1u) << 1;
            }
          }
          left -= kUnroll;
          double qx[kUnroll], qy[kUnroll], qz[kUnroll];
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) {
            const double2 v = s_xy[at[u]];
            qx[u] = v.x;
            qy[u] = v.y;
            qz[u] = s_z[at[u]];
          }
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) {
            const double ex = px - qx[u], ey = py - qy[u], ez = pz - qz[u];
            const double r2d = __builtin_fma(ez, ez, __builtin_fma(ey, ey, ex * ex));
            // 2.0 or 0.0 from the species bit
            const double sel = __hiloint2double((int)(sp[u] << 30), 0);
            const int32_t ab = NS > 2 ? 4 * ti + (int32_t)sp[u] : 0;
            double rc2;
            if constexpr (NS == 2)
              rc2 = __builtin_fma(drc, sel, rc1);
            else
              rc2 = s_pair[ab].rc2;
            if (r2d < rc2) {
              T a, b, f, fr, rinv, r2i, x6;  // x6: (s/r)^6 (mixed) or r^-6
              if constexpr (NS == 2) {
                const T sl = MIXED ? (T)__int_as_float((int)(sp[u] << 30)) : (T)sel;
                a = fma_t(da, sl, a1);
                b = fma_t(dc, sl, c1);
                f = fma_t(df, sl, f1);
              } else {
                const PairRow& w = s_pair[ab];
                a = MIXED ? (T)w.sig2 : (T)w.a;
                b = MIXED ? (T)w.f12 : (T)w.b;
                f = MIXED ? (T)w.mfs : (T)w.fs;
              }
              const T r2 = (T)r2d, dx = (T)ex, dy = (T)ey, dz = (T)ez;
              if constexpr (MIXED) {
                rinv = __builtin_amdgcn_rsqf(r2);
                r2i = rinv * rinv;
                const float q2 = a * r2i;
                x6 = q2 * q2 * q2;
                fr = b * (x6 - mk) * x6 * r2i + f * rinv;
              } else {
                rinv = rsqrt3(r2d);
                r2i = rinv * rinv;
                x6 = r2i * r2i * r2i;
                fr = __builtin_fma(__builtin_fma(a, x6, b) * x6, r2i, f * rinv);
              }
              fx = fma_t(fr, dx, fx);
              fy = fma_t(fr, dy, fy);
              fz = fma_t(fr, dz, fz);
              if constexpr (EN) {
                if constexpr (NS == 2 && MIXED) {
                  const float2 cv = s_ev[2 * ti + (int32_t)sp[u]];
                  pe += __builtin_fmaf(-12.0f, (r2 * rinv - cv.x) * f,
                                       __builtin_fmaf(b, (x6 - (mk + mk)) * x6, -cv.y));
                } else if constexpr (NS == 2) {
                  const double g =
                      __builtin_fma(12.0, f * (r2 * rinv), s_ev[2 * ti + (int32_t)sp[u]]);
                  pe += __builtin_fma(__builtin_fma(a, x6, b + b), x6, -g);
                } else {
                  const auto& W = s_en[0];
                  const T q2 = W.sig2[ab] * r2i, q6 = q2 * q2 * q2;
                  pe += W.c12[ab] * (q6 * q6) + W.c6[ab] * q6 - W.vc[ab] -
                        (r2 * rinv - W.rc[ab]) * W.fs[ab];
                }
                vw += fr * r2;
              }
            }
          }
        }
        wave_lds_sync();  // the next pass or group rewrites the words
      }
      fx += __shfl_xor(fx, 32, 64);
      fy += __shfl_xor(fy, 32, 64);
      fz += __shfl_xor(fz, 32, 64);
      if constexpr (EN) {
        sum_pe += (NS == 2 ? 1.0 / 24.0 : 0.5) * (double)pe;
        sum_w += 0.5 * (double)vw;
      }
      if (lane < gn) {
        if (!isfinite((double)(fx + fy + fz))) atomicOr(&st->err, kErrNonFinite);
        if constexpr (MODE != 2) {
          T* frc = (T*)frc_;
          frc[i] = fx;
          frc[stride + i] = fy;
          frc[2 * (size_t)stride + i] = fz;
        }
        const double m = s_mass[ti];
        double v0 = vel[i], v1 = vel[stride + i], v2 = vel[2 * (size_t)stride + i];
        if constexpr (MODE >= 1) {
          const double hm = 0.5 * dt / m;
          v0 += hm * (double)fx;
          v1 += hm * (double)fy;
          v2 += hm * (double)fz;
        }
        sum_ke += 0.5 * m * (v0 * v0 + v1 * v1 + v2 * v2);
        if constexpr (MODE == 2) {
          // the next step's first half kick and drift (as k_kick_drift)
          const double hk = 0.5 * dt * s_im[ti];
          v0 += hk * (double)fx;
          v1 += hk * (double)fy;
          v2 += hk * (double)fz;
          const double4 o = make_double4(px + dt * v0, py + dt * v1, pz + dt * v2, (double)ti);
          fo.pos_out[i] = o;
          const double e0 = o.x - fo.xref[i], e1 = o.y - fo.xref[stride + i],
                       e2 = o.z - fo.xref[2 * (size_t)stride + i];
          d2 = fmax(d2, e0 * e0 + e1 * e1 + e2 * e2);
        }
        if constexpr (MODE >= 1) {
          vel[i] = v0;
          vel[stride + i] = v1;
          vel[2 * (size_t)stride + i] = v2;
        }
      }
    }
  }
  // the tile's sums: each wave's lanes, then the waves in order
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    sum_pe += __shfl_xor(sum_pe, d, 64);
    sum_w += __shfl_xor(sum_w, d, 64);
    sum_ke += __shfl_xor(sum_ke, d, 64);
    d2 = fmax(d2, __shfl_xor(d2, d, 64));
  }
  if (lane == 0) {
    s_red[0][wv] = sum_pe;
    s_red[1][wv] = sum_w;
    s_red[2][wv] = sum_ke;
    s_red[3][wv] = d2;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int q = 1; q < nw; ++q) {
    sum_pe += s_red[0][q];
    sum_w += s_red[1][q];
    sum_ke += s_red[2][q];
    d2 = fmax(d2, s_red[3][q]);
  }
  double* o = part + 4 * (size_t)Tl.part;
  o[0] = sum_pe;
  o[1] = sum_w;
  o[2] = sum_ke;
  if constexpr (MODE == 2) o[3] = d2;
}

}  // namespace

int32_t search_waves() { return kWaves; }

void launch_force_search(hipStream_t s, int32_t mixed, int32_t mode, int32_t energy,
                         int32_t threads, int32_t four, const BrickArgs& A, const RepDesc* reps,
                         const PairTab* tab, const BrickPair* bp, const int32_t* cell_start,
                         const double4* pos, double* vel, void* frc, int32_t stride, double dt,
                         double* part, DevState* st, const FuseOut& fo) {
#define KF(M, MO, EN, NS)                                                                     \
  k_force_search<M, MO, EN, NS><<<A.ntiles, threads, 0, s>>>(A, reps, tab, bp, cell_start,    \
                                                             pos, vel, frc, stride, dt, part, \
                                                             st, fo)
  // mode 0 (a plain force evaluation) always forms the energies
#define KM(M, NS)                                                                 \
  if (mode == 0) { KF(M, 0, true, NS); }                                          \
  else if (mode == 1) { if (energy) KF(M, 1, true, NS); else KF(M, 1, false, NS); } \
  else { if (energy) KF(M, 2, true, NS); else KF(M, 2, false, NS); }
  if (mixed) {
    if (four) { KM(true, 4); } else { KM(true, 2); }
  } else {
    if (four) { KM(false, 4); } else { KM(false, 2); }
  }
#undef KM
#undef KF
}

}  // namespace mdk
