// brick_device.h -- device functions that the kernels on tiles of cells share
// (force_brick.hip, force_search.hip, nlist_brick.hip).
#pragma once
#include "brick.h"

namespace mdk {

constexpr double kFarAway = 1.0e300;  // x of the far slot

__device__ inline double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ inline float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// 1/r from r^2: the seed of v_rsq_f64 and one third-order step
__device__ inline double rsqrt3(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double e = __builtin_fma(-r2 * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

// Species tables in LDS of the forms with more than two species, by
// (home species) * 4 + partner species; the first for launches with energies.
template <typename T>
struct EnergyTab {
  T sig2[16], c12[16], c6[16], vc[16], fs[16], rc[16];
};
struct PairRow {
  double rc2, a, b, fs;
  float sig2, f12, mfs, pad;
};
template <typename T>
__device__ inline void fill_energy(EnergyTab<T>& s, const PairTab* tab, int k) {
  s.sig2[k] = (T)tab->sig2[k];
  s.c12[k] = (T)tab->c12[k];
  s.c6[k] = (T)tab->c6[k];
  s.vc[k] = (T)tab->vc[k];
  s.fs[k] = (T)tab->fs[k];
  s.rc[k] = (T)tab->rc[k];
}
__device__ inline PairRow pair_row(const PairTab* tab, int k) {
  const double s2 = tab->sig2[k], s6 = s2 * s2 * s2;
  return PairRow{tab->rc2[k], tab->f12[k] * (s6 * s6), tab->f6[k] * s6, tab->fs[k],
                 (float)s2, (float)tab->f12[k], (float)tab->fs[k], 0.0f};
}

// Copies a tile's neighbourhood to LDS, positions with their periodic shift
// applied, and calls seen(slot, record) for each.  row: its rows, in LDS; the
// waves of the block share them.  Rows q and q + nw of a wave, 128 slots each,
// per round: four records in flight per lane.
template <typename Seen>
__device__ inline void copy_neighbourhood(const BrickTile& Tl, const RepDesc& R,
                                          const TileRow* row, const double4* __restrict__ pos,
                                          double2* xy, double* z_, int32_t pad_slot, int wv,
                                          int nw, int lane, Seen seen) {
  const double L = R.L;
  const int32_t nc = R.nc, ry = Tl.ty + 2, nr = ry * (Tl.tz + 2);
  auto fetch = [&](int q, int32_t v, bool& on, double4& c) {
    const TileRow w = row[q];
    on = v < min(w.l3, pad_slot);
    int32_t j = w.gm + (v - w.l1);
    if (v < w.l1) j = w.gl + (v - w.l0);
    if (v >= w.l2) j = w.gr + (v - w.l2);
    if (on) c = pos[j];
  };
  auto put = [&](int q, int32_t v, bool on, const double4& c) {
    const int32_t y = Tl.cy + q % ry - 1, z = Tl.cz + q / ry - 1;
    const double sy = y < 0 ? -L : (y >= nc ? L : 0.0), sz = z < 0 ? -L : (z >= nc ? L : 0.0);
    const TileRow w = row[q];
    const double sx = v < w.l1 ? -L : (v >= w.l2 ? L : 0.0);
    if (on) {
      xy[v] = make_double2(c.x + sx, c.y + sy);
      z_[v] = c.z + sz;
      seen(v, c);
    }
  };
  for (int q = wv; q < nr; q += 2 * nw) {
    const int q2 = q + nw < nr ? q + nw : q;  // (the last row alone: copied twice)
    const int32_t n = max(row[q].l3 - row[q].l0, row[q2].l3 - row[q2].l0);
    for (int32_t t = lane; t < n; t += 128) {
      bool on[4];
      double4 c[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int qk = k < 2 ? q : q2;
        fetch(qk, row[qk].l0 + t + 64 * (k & 1), on[k], c[k]);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int qk = k < 2 ? q : q2;
        put(qk, row[qk].l0 + t + 64 * (k & 1), on[k], c[k]);
      }
    }
  }
}

// Searches on the matrix cores: 32 home particles (columns of the product) at
// a time, a lane's 16 results of a 32 x 32 product.
constexpr int kGroup = 32;
constexpr float kNoHit = 1.0e4f;  // r^2 of the idle rows and columns, in squared cell sides
using f32x16 = __attribute__((ext_vector_type(16))) float;

// a = [a.lo, b.lo], b = [a.hi, b.hi] of the wave's halves: one value per
// candidate of a chunk in each of two registers becomes the two k-slices of
// the matrix operand for its first and its last 32 candidates.
__device__ inline void swap_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ inline void swap_halves(float& a, float& b) {
  uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
  swap_halves(x, y);
  a = __uint_as_float(x);
  b = __uint_as_float(y);
}

// Sign bits of a lane's 16 results: bit r = result r below zero.
__device__ inline uint32_t sign_bits(const f32x16& w) {
  uint32_t m = 0u;
#pragma unroll
  for (int r = 15; r >= 0; --r) m = __builtin_amdgcn_alignbit(m, __float_as_uint(w[r]), 31);
  return m;
}

__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace mdk
