// Host-side checks of the tiles of cells (brick.h, plan_bricks), run by
// test_brick_plan.py on the CPU: no HIP call is made.
//   brick_plan_host empty N RHO FILL
//     a box whose particles fill the lower FILL of its height: home rows of
//     every tile from the cell counts, and the index that every load of a
//     home particle uses
//   brick_plan_host grid N RHO
//     the list-free path: threads of a force launch, which one launch holds
//     and its 32-bit index counts
//   brick_plan_host span N RHO CAP
//     the list path with a capacity of CAP entries (0: the default one): bytes
//     of list that the rows of a layer of tiles can take
#include "../paper_1105_5613_amd/csrc/md_api.cpp"

#include <cstdlib>
#include <random>

namespace {

// a context as md_init lays it out, one replica, without device buffers
void one_box(md_ctx c, int64_t n, double rho, int32_t path, const double* rc3, double skin) {
  md_params& p = c->p;
  p.ntypes = 2;
  p.skin = skin;
  p.dt = 0.005;
  p.path = path;
  const double eps[3] = {1.0, 1.5, 0.5}, sig[3] = {1.0, 0.8, 0.88};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) {
      p.eps[a * MD_MAXT + b] = eps[a + b];
      p.sig[a * MD_MAXT + b] = sig[a + b];
      p.rc[a * MD_MAXT + b] = rc3[a + b];
    }
  RepDesc d{};
  d.L = std::cbrt((double)n / rho);
  d.n = (int32_t)n;
  d.nc = (int32_t)std::floor(d.L / (max_rc(p) + skin));
  d.volume = d.L * d.L * d.L;
  d.cside = d.L / d.nc;
  d.tile1 = (int32_t)((n + kTile - 1) / kTile);
  c->nrep = 1;
  c->ntot = (int32_t)n;
  c->ntiles = d.tile1;
  c->ncells = d.nc * d.nc * d.nc;
  c->cells = path == MD_PATH_CELLS;
  c->reps_h.push_back(d);
}

int empty(int64_t n, double rho, double fill) {
  md_ctx_s c;
  const double rc[3] = {2.5, 2.0, 2.2};
  one_box(&c, n, rho, MD_PATH_AUTO, rc, 0.3);
  if (!plan_bricks(&c)) return std::puts("not on tiles of cells"), 2;
  const RepDesc& d = c.reps_h[0];
  const int32_t nc = d.nc;
  std::vector<int32_t> start((size_t)c.ncells + 1, 0);
  std::mt19937_64 gen(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int64_t k = 0; k < n; ++k) {
    auto cell = [&](double t) { return std::min(nc - 1, (int32_t)(t * nc)); };
    const int32_t x = cell(u(gen)), y = cell(u(gen)), z = cell(fill * u(gen));
    start[((int64_t)z * nc + y) * nc + x + 1] += 1;
  }
  for (int32_t k = 0; k < c.ncells; ++k) start[k + 1] += start[k];
  int32_t empty_tiles = 0, at_end = 0;
  for (const BrickTile& T : c.btiles_h) {
    HomeRow hr[kTileHomeRows];
    int32_t nh = 0;
    const int32_t nhr = T.ty * T.tz;
    for (int32_t r = 0; r < nhr; ++r) {
      const int32_t* s = &start[((T.cz + r / T.ty) * nc + T.cy + r % T.ty) * nc + T.cx];
      hr[r] = HomeRow{s[0], nh, 0, 0};
      nh += s[T.tx] - s[0];
    }
    empty_tiles += nh == 0;
    at_end += nh == 0 && hr[nhr - 1].g >= n;
    for (int32_t h = 0; h < std::max(nh, kBrickThreads); ++h) {
      const int32_t i = home_index(hr, nhr, h, nh);
      if (nh == 0 ? i != -1 : i < 0 || i >= n)
        return std::printf("tile at %d %d %d: home %d of %d reads particle %d of %lld\n", T.cx,
                           T.cy, T.cz, h, nh, i, (long long)n), 1;
    }
  }
  std::printf("%d tiles, %d empty, %d with rows that start at the end\n",
              (int)c.btiles_h.size(), empty_tiles, at_end);
  return empty_tiles && at_end ? 0 : 3;
}

int grid(int64_t n, double rho) {
  md_ctx_s c;
  const double rc[3] = {2.5, 2.0, 2.2};
  one_box(&c, n, rho, MD_PATH_CELLS, rc, 0.3);
  if (!plan_bricks(&c)) return std::puts("row tiles"), c.ba.ntiles != 0 || c.brick_parts != 0;
  const int64_t threads = (int64_t)c.ba.ntiles * c.search_threads;
  std::printf("%d tiles of %d threads: %.3f of 2^32\n", c.ba.ntiles, c.search_threads,
              (double)threads / 4294967296.0);
  // the clear of the cell counts reaches every cell
  return threads >= (1ll << 32) || threads < c.ncells;
}

int span(int64_t n, double rho, int32_t cap) {
  md_ctx_s c;
  const double rc[3] = {2.5, 2.0, 2.2};
  one_box(&c, n, rho, MD_PATH_AUTO, rc, 0.3);
  c.cap = cap ? cap : (int32_t)std::ceil(1.5 * rho * 4.0 / 3.0 * M_PI * 2.8 * 2.8 * 2.8) + 24;
  if (!plan_bricks(&c)) return std::puts("gather lists"), c.ba.ntiles != 0;
  const RepDesc& d = c.reps_h[0];
  c.ba.capc = chunk_capacity(&c, c.cap);
  int64_t layer = 0;  // particles at the mean density between a tile's first and last home
  for (const BrickTile& T : c.btiles_h)
    layer = std::max<int64_t>(
        layer, (int64_t)((double)n / c.ncells * (((T.tz - 1) * d.nc + T.ty - 1) * d.nc + T.tx)));
  std::printf("tiles of cells: %d chunks a row, %lld particles, at most %lld: %.3f of 4 GiB\n",
              c.ba.capc, (long long)layer, (long long)c.brick_layer,
              (double)(c.brick_layer / kSlice + 2) * c.ba.capc * kSlice * 16 / 4294967296.0);
  return layer > c.brick_layer || !list_span_fits(c.brick_layer, c.ba.capc);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "empty" && argc == 5)
    return empty(std::atoll(argv[2]), std::atof(argv[3]), std::atof(argv[4]));
  if (what == "grid" && argc == 4) return grid(std::atoll(argv[2]), std::atof(argv[3]));
  if (what == "span" && argc == 5)
    return span(std::atoll(argv[2]), std::atof(argv[3]), std::atoi(argv[4]));
  std::puts("unknown check");
  return 4;
}
