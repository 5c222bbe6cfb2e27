// force_brick.hip -- the pair-force hot spot on the brick path (brick.h):
// one block per tile copies the tile's neighbourhood into LDS (positions with
// their periodic shift applied, FP64) and its home particles walk 16-bit list
// entries against it.  The pair function is that of force.hip: Eq. (3) on
// Eq. (1)/(2), the displacement, r^2 and the cut-off test in FP64, the pair
// arithmetic in FP64 or, in the mixed form, FP32.
//
// Why LDS: a gather from memory costs one L1 tag access per lane and 16 bytes
// and runs at one per cycle and CU, which bounded the gather kernel (force.hip)
// at 261 us per launch for 1,048,576 particles (list radius 2.8, 92 entries);
// random 8- and 16-byte LDS reads of a whole wave take about 9 ns together
// (one ds_read_b128 for x and y, one ds_read_b64 for z; three b64: 14 ns),
// 60 us per launch.  What bounds this kernel is vector issue: of a SIMD's time
// an FP64 instruction of a wave and an FP32 one of three operands take 1.8 to
// 2.1 ns, a 32-bit one of two operands 1.0 to 1.3 ns, 1/sqrt 7 ns, and the
// vector units issue in 0.63 of the launch (mixed: 0.87; LDS is busy in 0.29 of
// it, 0.40), so the arithmetic below is kept short:
//  - the entry is the LDS byte offset, the species bit lands in the exponent
//    of a double (2.0 or 0.0) with one AND, and each species constant is one
//    FMA, p1 + d * 2, exact by choice of the base (BrickPair);
//  - 1/r by one third-order step from v_rsq_f64 (seed error 5e-8, result
//    within an ulp or two) instead of two Newton-Raphson steps;
//  - places past a row's end point at a slot infinitely far away, so there is
//    no bound test;
//  - r^2 is summed onto a number far below its last bit (BrickPair::tiny), so
//    that a pair at r = 0, which is skipped as on the other list paths, gives a
//    finite f(r) / r times a zero displacement (where FP32 or an energy would
//    overflow, it is tested).
// (BIG: contexts with wider cells take 3,072 slots, two blocks per CU.)
// Tiles of 2 x 2 x 2 cells (213 homes, 1,709 slots at rho = 1.2) put three
// blocks of eight waves on a CU (51 KB of LDS each).  Measured per launch of
// an NVE step (with the next step's kick and drift) at 1,048,576 particles,
// gather with its best variant -> here: after 400 steps FP64 261 -> 202 us,
// mixed 182 -> 146 us; in the first 25 launches of a process, before the card
// has raised its clocks, 270 -> 222 and 189 -> 166 us.
//
// Energies come from what the force has formed, with one constant more per
// species pair in FP64 and two in the mixed form (BrickPair), from registers;
// a table in LDS cost six reads per pair, and a force evaluation took longer
// than by gathers (FP64 / mixed, tables -> so: 131,072 particles 63 -> 54 /
// 51 -> 38 us, 1,048,576: 258 -> 223 / 218 -> 161 us).  With more than two
// species the table stays.
//
// TPP lanes take one particle: of each 8-entry chunk lane p takes the entries
// [8 p / TPP, 8 (p + 1) / TPP).  Sums are kept per pair of entries (0-1, 2-3,
// 4-5, 6-7 of every chunk) and combined in one fixed tree, and energies per 16
// home particles, so that results do not depend on TPP or the block size.
#include <type_traits>

#include "brick_device.h"

namespace mdk {
namespace {

constexpr int kTaskHomes = 16;  // homes per partial of the energies
constexpr int kAhead = 1;  // list chunks read ahead (2, 3 and 4 measured the same)
static_assert(kAhead <= kChunksAhead, "chunk_elems allocates what is read ahead");

// Registers: three blocks of eight waves fit a CU at 80 VGPRs, which the mixed
// form holds without spills.  The FP64 form with two lanes per particle spills
// there (203 us per NVE launch at 1,048,576 particles) and runs two blocks at
// 96 without (198 us in the same run; four lanes at 80 VGPRs: 11 % slower).
template <bool MIXED, int MODE, int TPP, bool EN, int NS, bool BIG>
__global__ __launch_bounds__(kBrickThreads)
__attribute__((amdgpu_waves_per_eu(BIG || (EN && NS > 2) || (!MIXED && (EN || TPP == 2)) ? 4 : 6))) void k_force_brick(
    BrickArgs A, const RepDesc* __restrict__ reps, const PairTab* __restrict__ tab,
    const BrickPair* __restrict__ bp, const double4* __restrict__ pos, double* __restrict__ vel,
    void* __restrict__ frc_, int32_t stride, double dt, double* __restrict__ part, DevState* st,
    FuseOut fo) {
  using T = typename std::conditional<MIXED, float, double>::type;
  constexpr int E = kChunkEntries / TPP;  // entries of a chunk per lane
  constexpr int NA = E / 2;               // sums per lane
  constexpr int kSlots = BIG ? kBrickSlotsBig : kBrickSlots, kPadSlot = kSlots - 1;
  constexpr int kTasks = kSlots / kTaskHomes;
  __shared__ double2 s_xy[kSlots];
  __shared__ double s_z[kSlots];
  __shared__ TileRow s_row[kTileRows];
  __shared__ HomeRow s_home[kTileHomeRows];
  __shared__ double s_ke[kTasks], s_pw[EN ? 2 * kTasks : 1], s_d2[kBrickThreads / 64];
  __shared__ typename std::conditional<EN && (NS > 2), EnergyTab<T>, char>::type s_en[1];
  __shared__ PairRow s_pair[NS > 2 ? 16 : 1];
  __shared__ double s_mass[4], s_im[4];
  const bool halt = halted(st);  // read beside the tile tables
  const int32_t lb = xcd_block(blockIdx.x, gridDim.x);
  const int32_t tb = lb / A.split, share = lb % A.split;
  const TileRow* trow = A.row + (size_t)tb * A.rows;
  const HomeRow* hrow = A.hrow + (size_t)tb * A.hrows;
  const int nthr = blockDim.x, nw = nthr / 64;
  const BrickTile Tl = A.tiles[tb];
  // this block's partials and homes of the tile
  const int32_t un0 = Tl.units * share / A.split, un1 = Tl.units * (share + 1) / A.split;
  const int32_t h0 = un0 * kUnitHomes;
  const int32_t nh = un1 == Tl.units ? A.head[tb].nh : min(A.head[tb].nh, un1 * kUnitHomes);
  const int32_t ry = Tl.ty + 2, nr = ry * (Tl.tz + 2), nhr = Tl.ty * Tl.tz;
  if ((int)threadIdx.x < nr) s_row[threadIdx.x] = trow[threadIdx.x];
  if ((int)threadIdx.x < nhr) s_home[threadIdx.x] = hrow[threadIdx.x];
  if (threadIdx.x < 4) {
    s_mass[threadIdx.x] = tab->mass[threadIdx.x];
    s_im[threadIdx.x] = tab->inv_mass[threadIdx.x];
  }
  if (threadIdx.x < 16) {
    const int k = threadIdx.x;
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
  __syncthreads();
  if (halt) {
    // a list build queued before this launch overflowed (see kHalt): the
    // step is not taken, and a fused launch hands the positions unchanged to
    // the buffer the host swaps in
    if (blockIdx.x == 0 && threadIdx.x == 0) st->any_rebuild = 0;
    if constexpr (MODE == 2) {
      for (int32_t h = h0 + threadIdx.x; h < nh; h += nthr) {
        const int32_t i = home_index(s_home, nhr, h, nh);
        fo.pos_out[i] = pos[i];
      }
    }
    return;
  }
  if constexpr (MODE == 2) {
    const uint32_t gz = blockIdx.x * (uint32_t)nthr + threadIdx.x;  // up to 2^32 (plan_bricks)
    if (gz < (uint32_t)fo.nzero) fo.counts[gz] = 0;
  }
  const RepDesc& R = reps[Tl.rep];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int lp = lane % TPP;
  constexpr int kHomes = 64 / TPP;  // homes per wave and round
  struct Home {
    int32_t i;
    int32_t nch;
    double4 p;
  };
  // the first round's home particle, in flight under the copy to LDS
  auto load_home = [&](int32_t h) {
    Home m{};
    m.i = home_index(s_home, nhr, h, nh);
    if (nh > 0) m.p = pos[m.i];
    m.nch = h < nh ? min(A.nchunk[m.i], A.capc) : 0;
    return m;
  };
  Home me = load_home(h0 + wv * kHomes + lane / TPP);
  copy_neighbourhood(Tl, R, s_row, pos, s_xy, s_z, kPadSlot, wv, nw, lane,
                     [](int32_t, const double4&) {});
  __syncthreads();

  const size_t base = list_base(s_home[0].g, A.capc) & ~(size_t)(kSlice - 1);
  const char* const list = reinterpret_cast<const char*>(A.list + base);
  double d2 = 0.0;
  const int32_t rounds = nh > h0 ? (nh - h0 + kHomes - 1) / kHomes : 0;
  for (int32_t task = wv; task < rounds; task += nw) {
    const int32_t h = h0 + task * kHomes + lane / TPP;
    if (task != wv) me = load_home(h);
    int32_t i = me.i;
    const double4 p = me.p;
    const int32_t ti = (int32_t)p.w;
    // list bytes from the tile's first particle on fit 32 bits (list_span_fits)
    uint32_t at_row = (uint32_t)((list_base(i, A.capc) - base) * sizeof(uint4)) + lp * 2 * E;
    constexpr uint32_t kStep = kSlice * sizeof(uint4);
    // constants of the home particle's species against either partner species
    double rc1 = 0, drc = 0;
    T a1 = 0, da = 0, b1 = 0, db = 0, f1 = 0, df = 0;
    const T mk = MIXED ? (T)bp->mk : (T)0;
    if constexpr (NS == 2) {
      rc1 = bp->rc2[ti][0];
      drc = bp->rc2[ti][1];
      if constexpr (MIXED) {
        a1 = bp->msig2[ti][0];
        da = bp->msig2[ti][1];
        b1 = bp->mf12[ti][0];
        db = bp->mf12[ti][1];
        f1 = bp->mfs[ti][0];
        df = bp->mfs[ti][1];
      } else {
        a1 = bp->a[ti][0];
        da = bp->a[ti][1];
        b1 = bp->b[ti][0];
        db = bp->b[ti][1];
        f1 = bp->fs[ti][0];
        df = bp->fs[ti][1];
      }
    }
    // and of the energies
    double v1 = 0, dv = 0;
    float mv0 = 0, mv1 = 0, mc0 = 0, mc1 = 0;
    if constexpr (EN && NS == 2 && !MIXED) {
      v1 = bp->v12[ti][0];
      dv = bp->v12[ti][1];
    }
    if constexpr (EN && NS == 2 && MIXED) {
      mv0 = bp->mv12[ti][0];
      mv1 = bp->mv12[ti][1];
      mc0 = bp->mrc[ti][0];
      mc1 = bp->mrc[ti][1];
    }
    const double tiny = bp->tiny;
    T fx[NA], fy[NA], fz[NA], pe[NA], vw[NA];
    // one pair: entry e, its LDS position, into sum u
    auto pair = [&](uint32_t e, double qx, double qy, double qz, int u) {
      const double ex = p.x - qx, ey = p.y - qy, ez = p.z - qz;
      const double r2d =
          __builtin_fma(ez, ez, __builtin_fma(ey, ey, __builtin_fma(ex, ex, tiny)));
      // 2.0 or 0.0 from bit 14
      const double sel = __hiloint2double((int)((e << 16) & 0x40000000u), 0);
      double rc2;
      int32_t ab = 0;
      if constexpr (NS == 2) {
        rc2 = __builtin_fma(drc, sel, rc1);
      } else {
        ab = ti * 4 + (int32_t)((e >> 14) & 3u);
        rc2 = s_pair[ab].rc2;
      }
      if (((!MIXED && !EN) | (r2d > tiny)) & (r2d < rc2)) {
        T a, b, f, fr, rinv, r2i, x6;  // x6: (s/r)^6 (mixed) or r^-6
        if constexpr (NS == 2) {
          const T sl = MIXED ? (T)__int_as_float((int)((e << 16) & 0x40000000u)) : (T)sel;
          a = fma_t(da, sl, a1);
          b = fma_t(db, sl, b1);
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
          const float s2 = a * r2i;
          x6 = s2 * s2 * s2;
          fr = b * (x6 - mk) * x6 * r2i + f * rinv;
        } else {
          rinv = rsqrt3(r2d);
          r2i = rinv * rinv;
          x6 = r2i * r2i * r2i;
          fr = __builtin_fma(__builtin_fma(a, x6, b) * x6, r2i, f * rinv);
        }
        fx[u] = fma_t(fr, dx, fx[u]);
        fy[u] = fma_t(fr, dy, fy[u]);
        fz[u] = fma_t(fr, dz, fz[u]);
        if constexpr (EN) {
          // twelve times the energy, from what the force has formed (NS = 2)
          if constexpr (NS == 2 && MIXED) {
            const bool set = (e & 0x4000u) != 0u;
            const float h = (r2 * rinv - (set ? mc1 : mc0)) * f;
            pe[u] += __builtin_fmaf(
                -12.0f, h, __builtin_fmaf(b, (x6 - (mk + mk)) * x6, -(set ? mv1 : mv0)));
          } else if constexpr (NS == 2) {
            const double g = __builtin_fma(12.0, f * (r2 * rinv), __builtin_fma(dv, sel, v1));
            pe[u] += __builtin_fma(__builtin_fma(a, x6, b + b), x6, -g);
          } else {
            const auto& W = s_en[0];
            const T s2 = W.sig2[ab] * r2i, s6 = s2 * s2 * s2;
            pe[u] += W.c12[ab] * (s6 * s6) + W.c6[ab] * s6 - W.vc[ab] -
                     (r2 * rinv - W.rc[ab]) * W.fs[ab];
          }
          vw[u] += fr * r2;
        }
      }
    };
    auto at = [&](uint32_t e, double& x, double& y, double& z) {
      // 16 and 8 bytes per slot from slot << 3 (BIG: << 2)
      const uint32_t o = e & (BIG ? 0x3ffcu : 0x3ff8u);
      const double2 v = *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(s_xy) +
                                                          (BIG ? 4 : 2) * o);
      x = v.x;
      y = v.y;
      z = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(s_z) +
                                           (BIG ? 2 : 1) * o);
    };
    auto clear = [&]() {
#pragma unroll
      for (int u = 0; u < NA; ++u) fx[u] = fy[u] = fz[u] = pe[u] = vw[u] = 0;
    };
    // the fixed tree over the sums of a particle: its lanes' own, then lanes
    auto combine = [&]() {
#pragma unroll
      for (int d = 1; d < NA; d <<= 1)
#pragma unroll
        for (int u = 0; u + d < NA; u += 2 * d) {
          fx[u] += fx[u + d];
          fy[u] += fy[u + d];
          fz[u] += fz[u + d];
          pe[u] += pe[u + d];
          vw[u] += vw[u + d];
        }
#pragma unroll
      for (int d = 1; d < TPP; d <<= 1) {
        fx[0] += __shfl_xor(fx[0], d, 64);
        fy[0] += __shfl_xor(fy[0], d, 64);
        fz[0] += __shfl_xor(fz[0], d, 64);
        if constexpr (EN) {
          pe[0] += __shfl_xor(pe[0], d, 64);
          vw[0] += __shfl_xor(vw[0], d, 64);
        }
      }
    };
    using Words = uint32_t[E / 2];
    auto load = [&](Words& w) {
      if constexpr (E == 4) {
        const uint2 v = *reinterpret_cast<const uint2*>(list + at_row);
        w[0] = v.x;
        w[1] = v.y;
      } else {
        w[0] = *reinterpret_cast<const uint32_t*>(list + at_row);
      }
      at_row += kStep;
    };
    clear();
    Words e[kAhead + 1];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) load(e[k]);
    for (int32_t c = 0; c < me.nch; ++c) {
      load(e[kAhead]);  // the chunks past a row's last one are allocated (chunk_elems)
      // two entries in flight: four held 24 registers and spilled at 80 in the
      // mixed form (166 us per launch, 145 so; FP64 201, 198)
#pragma unroll
      for (int k = 0; k < E / 2; ++k) {
        double qx[2], qy[2], qz[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) at(u ? e[0][k] >> 16 : e[0][k], qx[u], qy[u], qz[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u) pair(u ? e[0][k] >> 16 : e[0][k], qx[u], qy[u], qz[u], k);
      }
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
#pragma unroll
        for (int u = 0; u < E / 2; ++u) e[k][u] = e[k + 1][u];
    }
    combine();
    // the addresses below are formed here and not held in registers over the
    // walk (they cost a wave per SIMD)
    asm volatile("" : "+v"(i));
    double ke = 0.0;
    if (h < nh && lp == 0) {
      if (!isfinite((double)(fx[0] + fy[0] + fz[0]))) atomicOr(&st->err, kErrNonFinite);
      if constexpr (MODE != 2) {
        T* frc = (T*)frc_;
        frc[i] = fx[0];
        frc[stride + i] = fy[0];
        frc[2 * (size_t)stride + i] = fz[0];
      }
      const double m = s_mass[ti];
      double v0 = vel[i], v1 = vel[stride + i], v2 = vel[2 * (size_t)stride + i];
      if (MODE >= 1) {
        const double hm = 0.5 * dt / m;
        v0 += hm * (double)fx[0];
        v1 += hm * (double)fy[0];
        v2 += hm * (double)fz[0];
      }
      ke = 0.5 * m * (v0 * v0 + v1 * v1 + v2 * v2);
      if constexpr (MODE == 2) {
        // the next step's first half kick and drift (as k_kick_drift)
        const double hk = 0.5 * dt * s_im[ti];
        v0 += hk * (double)fx[0];
        v1 += hk * (double)fy[0];
        v2 += hk * (double)fz[0];
        const double4 o = make_double4(p.x + dt * v0, p.y + dt * v1, p.z + dt * v2, p.w);
        fo.pos_out[i] = o;
        const double e0 = o.x - fo.xref[i], e1 = o.y - fo.xref[stride + i],
                     e2 = o.z - fo.xref[2 * (size_t)stride + i];
        d2 = fmax(d2, e0 * e0 + e1 * e1 + e2 * e2);
      }
      if (MODE >= 1) {
        vel[i] = v0;
        vel[stride + i] = v1;
        vel[2 * (size_t)stride + i] = v2;
      }
    }
    // partials of 16 homes: lanes [16 TPP k, 16 TPP (k + 1)) of the wave
    double pi = 0.0, wi = 0.0;
    if constexpr (EN) {
      const bool on = h < nh && lp == 0;
      pi = on ? (NS == 2 ? 1.0 / 24.0 : 0.5) * (double)pe[0] : 0.0;
      wi = on ? 0.5 * (double)vw[0] : 0.0;
    }
#pragma unroll
    for (int d = kTaskHomes * TPP / 2; d >= TPP; d >>= 1) {
      ke += __shfl_xor(ke, d, 64);
      if constexpr (EN) {
        pi += __shfl_xor(pi, d, 64);
        wi += __shfl_xor(wi, d, 64);
      }
    }
    if (lane % (kTaskHomes * TPP) == 0) {
      const int32_t k =
          h0 / kTaskHomes + task * (kHomes / kTaskHomes) + lane / (kTaskHomes * TPP);
      if (k < kTasks) {
        s_ke[k] = ke;
        if constexpr (EN) {
          s_pw[k] = pi;
          s_pw[kTasks + k] = wi;
        }
      }
    }
  }
  if constexpr (MODE == 2) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) d2 = fmax(d2, __shfl_xor(d2, d, 64));
    if (lane == 0) s_d2[wv] = d2;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  // lane u: partial un0 + u, the tasks of its homes in order
  const int32_t u = un0 + lane;
  if (u >= un1) return;
  constexpr int kUnitTasks = kUnitHomes / kTaskHomes;
  const int32_t nt = (nh + kTaskHomes - 1) / kTaskHomes;
  const int32_t t1 = u + 1 == Tl.units ? nt : min(nt, (u + 1) * kUnitTasks);
  double k = 0.0, pe = 0.0, w = 0.0;
  for (int32_t t = u * kUnitTasks; t < t1; ++t) {
    k += s_ke[t];
    if constexpr (EN) {
      pe += s_pw[t];
      w += s_pw[kTasks + t];
    }
  }
  double* o = part + 4 * (size_t)(Tl.part + u);
  o[0] = pe;
  o[1] = w;
  o[2] = k;
  if constexpr (MODE == 2) {
    double m = 0.0;
    if (lane == 0)
      for (int q = 0; q < nw; ++q) m = fmax(m, s_d2[q]);
    o[3] = m;
  }
}

template <bool MIXED, int NS, bool BIG>
void launch_ns(hipStream_t s, int32_t mode, int32_t energy, int32_t tpp, int32_t threads,
               const BrickArgs& A, const RepDesc* reps, const PairTab* tab, const BrickPair* bp,
               const double4* pos, double* vel, void* frc, int32_t stride, double dt,
               double* part, DevState* st, const FuseOut& fo) {
#define KF(MO, TP, EN)                                                                      \
  k_force_brick<MIXED, MO, TP, EN, NS, BIG><<<A.ntiles * A.split, threads, 0, s>>>(A, reps, tab, bp, pos,  \
                                                                    vel, frc, stride, dt,   \
                                                                    part, st, fo)
#define KT(MO, EN) \
  if (tpp == 2) KF(MO, 2, EN); else KF(MO, 4, EN)
  // mode 0 (a plain force evaluation) always forms the energies
  if (mode == 0) { KT(0, true); }
  else if (mode == 1) { if (energy) { KT(1, true); } else { KT(1, false); } }
  else if constexpr (!MIXED) { if (energy) { KT(2, true); } else { KT(2, false); } }
  else { KT(2, false); }  // (mixed steps that form energies are not fused)
#undef KT
#undef KF
}

}  // namespace

void launch_force_brick(hipStream_t s, int32_t mixed, int32_t mode, int32_t energy, int32_t tpp,
                        int32_t threads, int32_t four, const BrickArgs& A, const RepDesc* reps,
                        const PairTab* tab, const BrickPair* bp, const double4* pos, double* vel,
                        void* frc, int32_t stride, double dt, double* part, DevState* st,
                        const FuseOut& fo) {
#define LB(M, NS, BIG)                                                                        \
  launch_ns<M, NS, BIG>(s, mode, energy, tpp, threads, A, reps, tab, bp, pos, vel, frc, stride, \
                        dt, part, st, fo)
#define LF(M, NS) \
  if (A.slots > kBrickSlots) LB(M, NS, true); else LB(M, NS, false)
  if (mixed) {
    if (four) { LF(true, 4); } else { LF(true, 2); }
  } else {
    if (four) { LF(false, 4); } else { LF(false, 2); }
  }
#undef LF
#undef LB
}

}  // namespace mdk
