// analysis.hip -- observables of the glass study: mean-squared displacement
// of the unwrapped positions, and the radial distribution function
//   g(r) = 2V/N^2 < sum_{i<j} delta(r - r_ij) >
// of the glass-transition section, as a histogram of all pair distances
// below rmax under the minimum image (exact FP64 distances; every unordered
// pair once).  Compiled without FMA contraction so the distances (and hence
// the bins) round exactly like a plain FP64 evaluation.
#include <algorithm>
#include <type_traits>

#include "md_internal.h"

#pragma clang fp contract(off)

namespace mdk {
namespace {

// Unwrapped positions u = x + img L of every particle into u0 (original id order).
__global__ __launch_bounds__(kTile) void k_msd_ref(const Tile* __restrict__ tiles,
                                                   const RepDesc* __restrict__ reps,
                                                   const double4* __restrict__ pos,
                                                   const int32_t* __restrict__ id,
                                                   const int32_t* __restrict__ img,
                                                   double* __restrict__ u0) {
  const Tile t = tiles[blockIdx.x];
  const int32_t i = t.start + threadIdx.x;
  if (i >= t.end) return;
  const double L = reps[t.rep].L;
  const double4 p = pos[i];
  const size_t o = 3 * (size_t)id[i];
  u0[o] = p.x + (double)img[o] * L;
  u0[o + 1] = p.y + (double)img[o + 1] * L;
  u0[o + 2] = p.z + (double)img[o + 2] * L;
}

// Per-tile sums of |u - u0|^2.
__global__ __launch_bounds__(kTile) void k_msd(const Tile* __restrict__ tiles,
                                               const RepDesc* __restrict__ reps,
                                               const double4* __restrict__ pos,
                                               const int32_t* __restrict__ id,
                                               const int32_t* __restrict__ img,
                                               const double* __restrict__ u0,
                                               double* __restrict__ part) {
  __shared__ double red[kTile / 64];
  const Tile t = tiles[blockIdx.x];
  const int32_t i = t.start + threadIdx.x;
  double s = 0.0;
  if (i < t.end) {
    const double L = reps[t.rep].L;
    const double4 p = pos[i];
    const size_t o = 3 * (size_t)id[i];
    const double dx = p.x + (double)img[o] * L - u0[o];
    const double dy = p.y + (double)img[o + 1] * L - u0[o + 1];
    const double dz = p.z + (double)img[o + 2] * L - u0[o + 2];
    s = (dx * dx + dy * dy) + dz * dz;
  }
  for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = red[0];
    for (int k = 1; k < kTile / 64; ++k) a += red[k];
    part[blockIdx.x] = a;
  }
}

// One block per replica: mean of the tile sums in a fixed order.
__global__ __launch_bounds__(256) void k_msd_reduce(const RepDesc* __restrict__ reps,
                                                    const double* __restrict__ part,
                                                    double* __restrict__ out) {
  __shared__ double red[256];
  const RepDesc R = reps[blockIdx.x];
  double s = 0.0;
  for (int32_t b = R.tile0 + threadIdx.x; b < R.tile1; b += 256) s += part[b];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0] / (double)R.n;
}

// Pair-distance histogram of particles [off, off + n): block b takes i in a
// tile of 256, loops over j tiles staged in LDS, counts j > i with r < rmax.
constexpr int kRdfTile = 256;
__global__ __launch_bounds__(kRdfTile) void k_rdf(const double4* __restrict__ pos, int32_t off,
                                                  int32_t n, double L, double rmax, double dr,
                                                  int32_t nbins,
                                                  unsigned long long* __restrict__ hist) {
  extern __shared__ unsigned int s_h[];
  __shared__ double jx[kRdfTile], jy[kRdfTile], jz[kRdfTile];
  for (int b = threadIdx.x; b < nbins; b += kRdfTile) s_h[b] = 0u;
  const int32_t i = blockIdx.x * kRdfTile + threadIdx.x;
  const bool act = i < n;
  const double4 pi = pos[off + (act ? i : 0)];
  for (int32_t j0 = blockIdx.x * kRdfTile; j0 < n; j0 += kRdfTile) {
    __syncthreads();
    const int32_t jl = j0 + threadIdx.x;
    if (jl < n) {
      const double4 q = pos[off + jl];
      jx[threadIdx.x] = q.x;
      jy[threadIdx.x] = q.y;
      jz[threadIdx.x] = q.z;
    }
    __syncthreads();
    const int32_t m = n - j0 < kRdfTile ? n - j0 : kRdfTile;
    if (act) {
      for (int32_t k = 0; k < m; ++k) {
        if (j0 + k <= i) continue;
        double dx = pi.x - jx[k], dy = pi.y - jy[k], dz = pi.z - jz[k];
        const double kx = rint(dx / L), ky = rint(dy / L), kz = rint(dz / L);
        const double tx = L * kx, ty = L * ky, tz = L * kz;
        dx = dx - tx;
        dy = dy - ty;
        dz = dz - tz;
        const double r = sqrt((dx * dx + dy * dy) + dz * dz);
        if (r < rmax) {
          int32_t b = (int32_t)(r / dr);
          b = b >= nbins ? nbins - 1 : b;
          atomicAdd(&s_h[b], 1u);
        }
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbins; b += kRdfTile)
    if (s_h[b]) atomicAdd(&hist[b], (unsigned long long)s_h[b]);
}

// Pair-distance histogram over the cells of replica [c0, c0 + nc^3) for any
// rmax: the cells within h of the home cell along each axis hold every
// partner closer than h cell sides minus the skin (while the skin rule
// holds), and 2 h + 1 <= nc makes them distinct.  Unordered pairs are met
// once by taking the home cell (partner index above the home's) and the
// half of the other offsets that follows it in (dz, dy, dx) order.
//
// A work item is one part of a home cell's particles and one wave: the lanes
// take packed candidates of the stencil's rows (each row of cells is one to
// two contiguous particle ranges), the wave walks the homes.  The image of a
// counted pair is the stencil's shift: with 2 h + 1 <= nc a pair whose
// minimum image is another one is at least h sides minus the skin apart in
// both, so d - L rint(d / L) is d - s L, the same subtraction of the same
// number without the division.
//
// Bound by vector issue: per (home, 64 candidates) about 14 instructions of
// FP64 distance, then for the lanes inside rmax (a tenth of them for h = 2)
// the bin from a single-precision estimate of r / dr, whose relative error
// stays below 4e-7; within 1e-6 nbins of a bin edge (or of rmax) the lane
// forms sqrt and the quotient in FP64 as k_rdf does, so every count is the
// one that arithmetic gives.  131,072 particles, rmax 4, 400 bins: all pairs
// (k_rdf) 31.5 ms, by cells 0.30 ms.  At most kRdfBlocks blocks walk the
// items, so that the bins are flushed to memory a fixed number of times.
constexpr int kRdfBlocks = 1024;
__global__ __launch_bounds__(256) void k_rdf_cells(int32_t c0, int32_t nc, int32_t h,
                                                   int32_t pshift, double reach,
                                                   const int32_t* __restrict__ cell_start,
                                                   const double4* __restrict__ pos, double L,
                                                   double rmax, double dr, int32_t nbins,
                                                   unsigned long long* __restrict__ hist) {
  extern __shared__ unsigned int s_h[];
  for (int b = threadIdx.x; b < nbins; b += 256) s_h[b] = 0u;
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t nitems = ((int64_t)nc * nc * nc) << pshift;
  const float inv_dr = (float)((double)nbins / rmax);
  const float eps = 1e-6f * (float)nbins + 1e-6f, top = (float)nbins - eps;
  const double reject = rmax * rmax * (1.0 + 4e-6);
  for (int64_t item = (int64_t)blockIdx.x * 4 + w; item < nitems;
       item += (int64_t)gridDim.x * 4) {
    const int32_t lc = (int32_t)(item >> pshift), part = (int32_t)item & ((1 << pshift) - 1);
    const int32_t qx = lc % nc, qy = (lc / nc) % nc, qz = lc / (nc * nc);
    const int32_t s0 = cell_start[c0 + lc], ns = cell_start[c0 + lc + 1] - s0;
    const int32_t i0 = s0 + (int32_t)(((int64_t)ns * part) >> pshift),
                  i1 = s0 + (int32_t)(((int64_t)ns * (part + 1)) >> pshift);
    if (i0 >= i1) continue;
    // candidates [k0, k1) of one piece with the shift s L of its image; HOME:
    // the piece starts with the home cell, whose pairs are taken for k > i
    auto piece = [&](auto home_tag, int32_t k0, int32_t k1, double sx, double sy, double sz) {
      constexpr bool HOME = decltype(home_tag)::value;
      for (int32_t base = k0; base < k1; base += 64) {
        const int32_t k = base + lane;
        const bool valid = k < k1;
        const double4 q = pos[valid ? k : k0];
        for (int32_t i = i0; i < i1; ++i) {
          const double4 pa = pos[i];  // wave-uniform
          const double dx = (pa.x - q.x) - sx, dy = (pa.y - q.y) - sy, dz = (pa.z - q.z) - sz;
          const double r2 = (dx * dx + dy * dy) + dz * dz;
          if (valid & (!HOME || k > i) & (r2 < reject)) {
            const float r2f = (float)r2;
            const float t = r2f * __builtin_amdgcn_rsqf(r2f) * inv_dr;
            const float fl = __builtin_floorf(t), f = t - fl;
            int32_t b = (int32_t)fl;
            bool count = true;
            if (!(t < top && f > eps && f < 1.0f - eps)) {
              const double r = sqrt(r2);
              count = r < rmax;
              b = (int32_t)(r / dr);
              b = b >= nbins ? nbins - 1 : b;
            }
            if (count) atomicAdd(&s_h[b], 1u);
          }
        }
      }
    };
    for (int32_t oz = 0; oz <= h; ++oz)
      for (int32_t oy = oz == 0 ? 0 : -h; oy <= h; ++oy) {
        int32_t y = qy + oy, z = qz + oz;
        const int32_t ky = y < 0 ? -1 : (y >= nc ? 1 : 0), kz = z >= nc ? 1 : 0;
        y -= ky * nc;
        z -= kz * nc;
        // rows beyond reach (rmax plus the skin, in cell sides) are skipped,
        // the others cut to the cells within it along x
        const double gy = (double)max(abs(oy) - 1, 0), gz = (double)max(oz - 1, 0);
        const double left2 = reach * reach - (gy * gy + gz * gz);
        if (left2 <= 0.0) continue;
        const int32_t hx = min(h, (int32_t)sqrt(left2) + 1);
        const int32_t* cs = cell_start + c0 + (z * nc + y) * nc;
        // d = x_i - (x_j + k L)
        const double sy = L * (double)ky, sz = L * (double)kz;
        const std::false_type other{};
        if (oz == 0 && oy == 0) {
          const int32_t x1 = qx + hx;
          piece(std::true_type{}, cs[qx], cs[x1 >= nc ? nc : x1 + 1], 0.0, 0.0, 0.0);
          if (x1 >= nc) piece(other, cs[0], cs[x1 - nc + 1], L, 0.0, 0.0);
        } else {
          const int32_t x0 = qx - hx, x1 = qx + hx;
          if (x0 < 0) piece(other, cs[nc + x0], cs[nc], -L, sy, sz);
          piece(other, cs[x0 < 0 ? 0 : x0], cs[x1 >= nc ? nc : x1 + 1], 0.0, sy, sz);
          if (x1 >= nc) piece(other, cs[0], cs[x1 - nc + 1], L, sy, sz);
        }
      }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbins; b += 256)
    if (s_h[b]) atomicAdd(&hist[b], (unsigned long long)s_h[b]);
}

__global__ void k_zero_u64(unsigned long long* __restrict__ a, int32_t n) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0ull;
}

}  // namespace

void launch_zero_u64(hipStream_t s, unsigned long long* a, int32_t n) {
  k_zero_u64<<<(n + 255) / 256, 256, 0, s>>>(a, n);
}

void launch_rdf_cells(hipStream_t s, int32_t c0, int32_t nc, int32_t h,
                      const int32_t* cell_start, const double4* pos, double L, double skin,
                      double rmax, int32_t nbins, unsigned long long* hist) {
  const double dr = rmax / nbins;
  const double reach = (rmax + skin) / (L / nc) * (1.0 + 1e-9);
  // small boxes: a cell's particles in up to 16 parts, so that the items fill
  // the chip (two waves per SIMD and more)
  const int64_t ncell = (int64_t)nc * nc * nc;
  int32_t pshift = 0;
  while (pshift < 4 && (ncell << pshift) < 4096) ++pshift;
  const int32_t grid = (int32_t)std::min<int64_t>(((ncell << pshift) + 3) / 4, kRdfBlocks);
  k_rdf_cells<<<grid, 256, sizeof(unsigned int) * nbins, s>>>(
      c0, nc, h, pshift, reach, cell_start, pos, L, rmax, dr, nbins, hist);
}

void launch_msd_ref(hipStream_t s, int32_t ntiles, const Tile* tiles, const RepDesc* reps,
                    const double4* pos, const int32_t* id, const int32_t* img, double* u0) {
  k_msd_ref<<<ntiles, kTile, 0, s>>>(tiles, reps, pos, id, img, u0);
}

void launch_msd(hipStream_t s, int32_t ntiles, int32_t nrep, const Tile* tiles,
                const RepDesc* reps, const double4* pos, const int32_t* id, const int32_t* img,
                const double* u0, double* part, double* out) {
  k_msd<<<ntiles, kTile, 0, s>>>(tiles, reps, pos, id, img, u0, part);
  k_msd_reduce<<<nrep, 256, 0, s>>>(reps, part, out);
}

void launch_rdf(hipStream_t s, const double4* pos, int32_t off, int32_t n, double L, double rmax,
                int32_t nbins, unsigned long long* hist) {
  const double dr = rmax / nbins;
  k_rdf<<<(n + kRdfTile - 1) / kRdfTile, kRdfTile, sizeof(unsigned int) * nbins, s>>>(
      pos, off, n, L, rmax, dr, nbins, hist);
}

}  // namespace mdk
