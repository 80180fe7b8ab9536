// Runs the register-block sweeps of ka_square.hip and ka_cube.hip on the CPU (hip/hip_runtime.h here).
// Between two barriers the threads of a workgroup run one after another, in ascending (order 0) or
// descending (order 1) index.
#include <ucontext.h>

#include <utility>
#include <vector>

#include "ka_internal.h"

namespace cpu {

dim3 thread, block, block_dim, grid_dim;
alignas(16) char dynamic_lds[160 << 10];

namespace {
constexpr size_t kStack = 256 << 10;
ucontext_t scheduler;
std::vector<ucontext_t> fiber;
std::vector<char> stacks;
std::vector<char> ended;
unsigned current = 0;
const std::function<void()> *body = nullptr;

void entry()
{
  (*body)();
  ended[current] = 1;
  swapcontext(&fiber[current], &scheduler);
}
}  // namespace

int order = 0;

void barrier()
{
  const unsigned me = current;
  swapcontext(&fiber[me], &scheduler);
}

void launch(dim3 grid, dim3 threads, const std::function<void()> &kernel)
{
  const unsigned n = threads.x;
  grid_dim = grid;
  block_dim = threads;
  body = &kernel;
  fiber.resize(n);
  stacks.resize(n * kStack);
  for (block.z = 0; block.z < grid.z; ++block.z)
    for (block.y = 0; block.y < grid.y; ++block.y)
      for (block.x = 0; block.x < grid.x; ++block.x) {
        ended.assign(n, 0);
        for (unsigned k = 0; k < n; ++k) {
          getcontext(&fiber[k]);
          fiber[k].uc_stack.ss_sp = stacks.data() + k * kStack;
          fiber[k].uc_stack.ss_size = kStack;
          fiber[k].uc_link = nullptr;
          makecontext(&fiber[k], entry, 0);
        }
        for (unsigned left = n; left > 0;)
          for (unsigned q = 0; q < n; ++q) {
            current = order ? n - 1 - q : q;
            if (ended[current]) continue;
            thread.x = current;
            swapcontext(&scheduler, &fiber[current]);
            left -= ended[current];
          }
      }
}

}  // namespace cpu

// State words [W][N] in canonical order, in place.  given: acceptance words drawn ahead; tile_sweeps:
// sweeps of a tile launch (0: one workgroup per word).
extern "C" int run_blocks(int d, int L, int W, int m, int noise, uint64_t seed, int t0, int sweeps, int given, int tile_sweeps,
                          int order, uint64_t *n, uint64_t *f)
{
  cpu::order = order;
  ka::SquareArgs a{};
  a.g.d = d;
  a.g.L = L;
  a.g.Q = L / 4;
  a.g.P = d == 2 ? a.g.Q * a.g.Q : a.g.Q * a.g.Q * a.g.Q;
  a.g.N = d == 2 ? L * L : L * L * L;
  a.g.qinv = ka::lattice_qinv(a.g.Q);
  a.W = W;
  a.wpt = W % 2 == 0 ? 2 : 1;
  a.noise = noise;
  a.key0 = (uint32_t)seed;
  a.key1 = (uint32_t)(seed >> 32);
  const size_t words = (size_t)a.g.N * W;
  std::vector<ka::u64> dn(words), df(words), next(words), acc;
  const auto place = [&](int w, int i) {
    int sub = 0, pos = 0, sm = 1, pm = 1, rest = i;
    for (int k = 0; k < d; ++k) {
      sub += (rest % L & 3) * sm;
      pos += (rest % L >> 2) * pm;
      rest /= L;
      sm *= 4;
      pm *= a.g.Q;
    }
    return ((size_t)(w / a.wpt) * a.g.N + (size_t)sub * a.g.P + pos) * a.wpt + (size_t)(w % a.wpt);
  };
  for (int w = 0; w < W; ++w)
    for (int i = 0; i < a.g.N; ++i) {
      dn[place(w, i)] = n[(size_t)w * a.g.N + i];
      df[place(w, i)] = f[(size_t)w * a.g.N + i];
    }
  a.n = dn.data();
  a.f = df.data();
  a.t0 = (uint32_t)t0;
  a.n_sweeps = sweeps;
  int rc = 0;
  if (given) {
    acc.resize((size_t)(d == 2 ? 32 : 192) * a.g.P * W * sweeps);
    a.acc = acc.data();
    rc |= d == 2 ? ka::launch_square_accept(a, nullptr) : ka::launch_cube_accept(a, nullptr);
  }
  if (tile_sweeps == 0) {
    rc |= d == 2 ? ka::launch_square_resident(a, m, nullptr) : ka::launch_cube_resident(a, m, nullptr);
  } else {
    for (int done = 0; done < sweeps;) {
      const int k = std::min(tile_sweeps, sweeps - done);
      a.n_out = next.data();
      a.sweep = done;
      if (!given) a.t0 = (uint32_t)(t0 + done);
      rc |= ka::launch_square_tile(a, k, m, nullptr);
      std::swap(dn, next);
      a.n = dn.data();
      done += k;
    }
  }
  for (int w = 0; w < W; ++w)
    for (int i = 0; i < a.g.N; ++i) {
      n[(size_t)w * a.g.N + i] = dn[place(w, i)];
      f[(size_t)w * a.g.N + i] = df[place(w, i)];
    }
  return rc;
}
