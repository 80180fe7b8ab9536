// ka_square.hip -- 2D lattices: sweeps on 4 x 4 blocks of sites held in registers (gfx950).
//
// Method: Boccagna, arXiv 1710.05155; the bit logic lives in ka_device.h.
//
// A thread owns the 16 words (n and moved-ever) of one 4 x 4 block, i.e. one position of the
// sublattice layout, for one 64-replica word.  The edge classes repeat with period 4 in both
// directions, so each class gives every thread four edges at places known at compile time: most
// words they read are the thread's own registers, and a workgroup keeps a copy of n in LDS only
// for what neighbouring blocks read (8 to 10 reads and 8 writes per class and thread, against 48
// LDS accesses for four edges of a kernel that keeps n and f there).  An edge that leaves the
// block is updated by the thread of its lower endpoint, in LDS; the other thread takes its new
// word, and the moved-ever bits from the change, after the class's barrier.
//
// k_square_resident: a whole lattice of at most 512 blocks (L <= 88) in one workgroup per word,
// for any number of sweeps.  k_square_tile: larger lattices, one workgroup per tile of 64 x 64
// sites and word, one to three sweeps per launch from one copy of n to another; sites within 9,
// 17 or 25 of the tile's edge are recomputed by the neighbouring tiles (a class along one
// direction reaches one site across it and, over its four classes, five along it: 5 + 4 sites in
// the first sweep, 8 in each one more).
//
// Measured per sweep, 64 replicas, against class passes over global memory (LDS-resident passes
// for L = 64): L = 64 3.4 us (7.2), L = 128 6.2 us (25), L = 256 8.2 us (28), L = 512 13.0 us (28),
// L = 1024 20 us (35), L = 4096 177 us (355); 256 replicas: L = 512 22 us (32), L = 4096 680 us
// (1600).  At 1024 threads (whole lattices up to L = 128, tiles of 128 x 128) the 128 registers a
// thread may have do not hold a block, and the spills cost more than the halos save (L = 128: 30
// us); tiles of 96 x 96 took longer at every size.
#include "ka_device.h"

namespace ka {
namespace {

using namespace dev;

// Acceptance words for one class of one sweep, drawn here or read.
struct SquareDraw {
  const u64 *acc;   // words drawn ahead for this sweep: [class * 4 + q][P], P = positions of the lattice
  int P;
  unsigned pos;     // this thread's position
  uint32_t t, key0, key1;
  uint32_t site;    // canonical id of the block's corner site
  uint32_t L;
  int word, noise;

  __device__ __forceinline__ void load(int c, u64 (&r)[4]) const
  {
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = (acc + (size_t)(c * 4 + q) * (size_t)P)[pos];
  }
};

template <int MU, int R, int Q>
__device__ __forceinline__ u64 square_draw(const SquareDraw &g)
{
  constexpr int a = (R + 2 * (Q & 1)) & 3;   // residue of the lower endpoint along MU, in row or column Q
  const uint32_t i = g.site + (MU == 0 ? (uint32_t)a + (uint32_t)Q * g.L : (uint32_t)Q + (uint32_t)a * g.L);
  u64 r[1];
  accept_words<1>(g.t, 4 * MU + R, 2 * i + MU, g.word, g.key0, g.key1, g.noise, r);
  return r[0];
}

// P: positions of the LDS copy, a constant so that the sublattice is part of an access's
// immediate offset (kept in registers, the addresses alone take more than the words).
template <int P>
struct Square {
  u64 *s;            // n of the tile in LDS: [16 sublattices][P]
  int off[3][3];     // position of the neighbouring block in direction (dy + 1, dx + 1)
  u64 n[4][4], f[4][4];   // [y][x]

  // the word of site (X, Y) relative to the block's corner, -1 <= X, Y <= 5
  template <int X, int Y>
  __device__ __forceinline__ u64 &lds() const
  {
    constexpr int bx = X < 0 ? 0 : X > 3 ? 2 : 1, by = Y < 0 ? 0 : Y > 3 ? 2 : 1;
    return s[((X & 3) + 4 * (Y & 3)) * P + off[by][bx]];
  }
  template <int X, int Y>
  __device__ __forceinline__ u64 at() const
  {
    if constexpr (X >= 0 && X < 4 && Y >= 0 && Y < 4) return n[Y][X];
    else return lds<X, Y>();
  }
  // site (a along MU, b across)
  template <int MU, int A, int B>
  __device__ __forceinline__ u64 along() const
  {
    if constexpr (MU == 0) return at<A, B>();
    else return at<B, A>();
  }

  // words read by edge Q of class (MU, R): the partner and the neighbours of both endpoints
  template <int MU, int R, int Q>
  __device__ __forceinline__ void gather(u64 (&x)[7]) const
  {
    constexpr int a = (R + 2 * (Q & 1)) & 3;
    x[0] = along<MU, a + 1, Q>();
    x[1] = along<MU, a - 1, Q>();
    x[2] = along<MU, a, Q + 1>();
    x[3] = along<MU, a, Q - 1>();
    x[4] = along<MU, a + 2, Q>();
    x[5] = along<MU, a + 1, Q + 1>();
    x[6] = along<MU, a + 1, Q - 1>();
  }

  template <int MU, int R, int Q>
  __device__ __forceinline__ void exchange(const u64 (&x)[7], u64 r, int m)
  {
    constexpr int a = (R + 2 * (Q & 1)) & 3;
    constexpr int iy = MU == 0 ? Q : a, ix = MU == 0 ? a : Q;
    const u64 xi[3] = {x[1], x[2], x[3]}, xj[3] = {x[4], x[5], x[6]};
    const u64 d = bit3<kTTAnd3>(bit3<kTTXorAnd>(n[iy][ix], x[0], activity<3>(xi, m)), activity<3>(xj, m), r);
    n[iy][ix] ^= d;
    f[iy][ix] |= d;
    lds<ix, iy>() = n[iy][ix];
    if constexpr (a < 3) {
      constexpr int jy = MU == 0 ? Q : a + 1, jx = MU == 0 ? a + 1 : Q;
      n[jy][jx] ^= d;
      f[jy][jx] |= d;
      lds<jx, jy>() = n[jy][jx];
    } else if constexpr (MU == 0) {
      lds<4, Q>() = x[0] ^ d;
    } else {
      lds<Q, 4>() = x[0] ^ d;
    }
  }

  // after the barrier of class (MU, R): the words that the block's lower neighbour changed
  template <int MU, int R, int Q>
  __device__ __forceinline__ void refresh()
  {
    if constexpr (((R + 2 * (Q & 1)) & 3) == 3) {
      constexpr int y = MU == 0 ? Q : 0, x = MU == 0 ? 0 : Q;
      const u64 v = lds<x, y>();
      f[y][x] |= n[y][x] ^ v;
      n[y][x] = v;
    }
  }

  // One class, number C = 4 MU + R of the sweep.  Words drawn ahead are in r[C % D]; once used,
  // those of D classes later take their place (`load`: there are such classes).
  template <int MU, int R, int D>
  __device__ __forceinline__ void step(u64 (&r)[D ? D : 1][4], const SquareDraw &g, int m, bool load)
  {
    constexpr int C = 4 * MU + R;
    constexpr bool GIVEN = D > 0;
    u64 (&rc)[4] = r[GIVEN ? C % (D ? D : 1) : 0];
    if constexpr (!GIVEN) {
      rc[0] = square_draw<MU, R, 0>(g);
      rc[1] = square_draw<MU, R, 1>(g);
      rc[2] = square_draw<MU, R, 2>(g);
      rc[3] = square_draw<MU, R, 3>(g);
      __builtin_amdgcn_sched_barrier(0);   // the draws end before the gathered words take registers
    }
    u64 x[4][7];
    gather<MU, R, 0>(x[0]);
    gather<MU, R, 1>(x[1]);
    gather<MU, R, 2>(x[2]);
    gather<MU, R, 3>(x[3]);
    exchange<MU, R, 0>(x[0], rc[0], m);
    exchange<MU, R, 1>(x[1], rc[1], m);
    exchange<MU, R, 2>(x[2], rc[2], m);
    exchange<MU, R, 3>(x[3], rc[3], m);
    if constexpr (GIVEN) {
      if (load) g.load(C + D, rc);   // entry 32 on: the next sweep
    }
    __syncthreads();
    refresh<MU, R, 0>();
    refresh<MU, R, 1>();
    refresh<MU, R, 2>();
    refresh<MU, R, 3>();
  }

  // One sweep.  D = 0: words drawn in the sweep; else r holds the words drawn ahead for classes
  // 0 .. D - 1 on entry, and on return those of the next sweep if there is one (`more`).
  template <int D>
  __device__ __forceinline__ void sweep(u64 (&r)[D ? D : 1][4], const SquareDraw &g, int m, bool more)
  {
    step<0, 0, D>(r, g, m, D < 8 || more);
    step<0, 1, D>(r, g, m, D < 7 || more);
    step<0, 2, D>(r, g, m, D < 6 || more);
    step<0, 3, D>(r, g, m, D < 5 || more);
    step<1, 0, D>(r, g, m, D < 4 || more);
    step<1, 1, D>(r, g, m, D < 3 || more);
    step<1, 2, D>(r, g, m, D < 2 || more);
    step<1, 3, D>(r, g, m, more);
  }
};

// Word `word` of the sites of a sublattice, in an array laid out in planes of wpt words: position
// pos is at [pos * wpt].  The same address on every lane.
template <typename T>
__device__ __forceinline__ T *sublattice_word(T *base, const SquareArgs &a, int word, int sub)
{
  return base + ((size_t)(word / a.wpt) * (size_t)a.g.N + (size_t)sub * (size_t)a.g.P) * (size_t)a.wpt + (size_t)(word % a.wpt);
}

// Acceptance words of sweeps t0 .. t0 + n_sweeps - 1: a.acc[((word * n_sweeps + s) * 32 + c * 4 + q) * P + pos].  A thread draws its position's
// four edges of a class, and one Philox call serves two words.
__global__ __launch_bounds__(256) void k_square_accept(SquareArgs a)
{
  const int pos = (int)blockIdx.x * (int)blockDim.x + (int)threadIdx.x;
  const int s = (int)blockIdx.y >> 3, c = (int)blockIdx.y & 7;
  const int pair = (int)blockIdx.z;
  if (pos >= a.g.P) return;
  const int p1 = div_q(a.g, pos), p0 = pos - p1 * a.g.Q;
  const int mu = c >> 2;
  u64 r[4][2];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e0 = ((c & 3) + 2 * (q & 1)) & 3;
    const int x = 4 * p0 + (mu == 0 ? e0 : q), y = 4 * p1 + (mu == 0 ? q : e0);
    accept_words<2>(a.t0 + (uint32_t)s, (uint32_t)c, (uint32_t)(x + a.g.L * y) * 2u + (uint32_t)mu, pair, a.key0, a.key1, a.noise,
                    r[q]);
  }
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const int word = 2 * pair + w;
    if (word >= a.W) continue;
    u64 *acc = a.acc + (((size_t)word * a.n_sweeps + s) * 32u + (size_t)c * 4u) * (size_t)a.g.P;
#pragma unroll
    for (int q = 0; q < 4; ++q) (acc + (size_t)q * (size_t)a.g.P)[pos] = r[q][w];
  }
}

// The thread's block from n at position `from` of the sublattice layout, into registers and LDS
// position `to`.
template <int P>
__device__ __forceinline__ void load_block(Square<P> &t, const SquareArgs &a, int word, int from, int to)
{
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x) t.n[y][x] = sublattice_word(a.n, a, word, x + 4 * y)[(unsigned)(from * a.wpt)];
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x) t.s[(x + 4 * y) * P + to] = t.n[y][x];
}

// Bound by issue and latency on one CU per word (0.44 us per class at 256 blocks).  The words of a
// pair, whose state interleaves, meet in one XCD's L2.  Two waves a SIMD, so that beyond 256 words a CU works
// on two: with draws among the gathers, and the products of every edge's id kept over the sweeps, a
// thread took 311 registers and a CU held one.  20 sweeps, before -> now: L = 64 x 24576 replicas 322 ->
// 212 us, L = 88 x 16384 265 -> 223; one sweep with its call L = 64 x 16384 41 -> 26.
template <int NT, bool GIVEN>
__global__ __launch_bounds__(NT, 2) void k_square_resident(SquareArgs a, int m)
{
  extern __shared__ u64 sq_lds[];
  const int word = xcd_remap((int)blockIdx.x, (int)gridDim.x);
  const int pos = (int)threadIdx.x;
  // threads that fill the last wave run a copy of block 0 with itself as neighbour, which is not stored
  const bool mine = pos < a.g.P;
  const int p = mine ? pos : 0;
  const int p1 = div_q(a.g, p), p0 = p - p1 * a.g.Q;
  Square<NT> t;
  t.s = sq_lds;
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      const int x = p0 + dx < 0 ? a.g.Q - 1 : p0 + dx == a.g.Q ? 0 : p0 + dx;
      const int y = p1 + dy < 0 ? a.g.Q - 1 : p1 + dy == a.g.Q ? 0 : p1 + dy;
      t.off[dy + 1][dx + 1] = mine ? x + a.g.Q * y : pos;
    }
  load_block(t, a, word, p, pos);
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x) t.f[y][x] = sublattice_word(a.f, a, word, x + 4 * y)[(unsigned)(p * a.wpt)];
  __syncthreads();
  SquareDraw g{};
  g.P = a.g.P;
  constexpr int D = GIVEN ? 4 : 0;   // classes of words in flight: they cover the words' latency
  u64 r[D ? D : 1][4];
  if constexpr (GIVEN) {
    g.acc = a.acc + (size_t)word * a.n_sweeps * 32u * (size_t)a.g.P;
    g.pos = (unsigned)p;
#pragma unroll
    for (int c = 0; c < D; ++c) g.load(c, r[c]);
  } else {
    g.t = a.t0;
    g.key0 = a.key0;
    g.key1 = a.key1;
    g.site = (uint32_t)(4 * p0) + (uint32_t)(4 * p1) * (uint32_t)a.g.L;
    g.L = (uint32_t)a.g.L;
    g.word = word;
    g.noise = a.noise;
  }
  const auto store = [&](u64 *n, u64 *f) {
    if (!mine) return;
    // not known to be the same from call to call, so that the addresses are not kept (spilled) over the sweeps
    int to = word;
    asm volatile("" : "+s"(to));
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        sublattice_word(n, a, to, x + 4 * y)[(unsigned)(pos * a.wpt)] = t.n[y][x];
        sublattice_word(f, a, to, x + 4 * y)[(unsigned)(pos * a.wpt)] = t.f[y][x];
      }
  };
  // observations: n and f as they are, for the observation kernel to count after this launch
  int row = 0;
  const size_t plane_words = (size_t)a.W * (size_t)a.g.N;
  const auto observe = [&](int64_t now) {
    for (; row < a.n_obs && (a.obs_times ? a.obs_times[row] == now : (int64_t)a.t0 + a.obs_at[row] == now); ++row) {
      u64 *dn = a.snap + (size_t)row * 2u * plane_words;
      store(dn, dn + plane_words);
    }
  };
  observe((int64_t)a.t0);
  for (int s = 0; s < a.n_sweeps; ++s) {
    if constexpr (!GIVEN) asm volatile("" : "+v"(g.site));   // else the products of all ids are kept (spilled) over the sweeps
    t.template sweep<D>(r, g, m, s + 1 < a.n_sweeps);
    g.acc += 32u * (size_t)a.g.P;
    g.t += 1;
    observe((int64_t)a.t0 + s + 1);
  }
  store(a.n, a.f);
}

// NS sweeps of a tile of TB x TB blocks, from a.n to a.n_out.  Sites [halo, halo + inner) of the
// tile are stored; the tile's first site is at inner * tile - 8 NS of the lattice, so blocks of
// the tile are blocks of the lattice and the stored windows cover it once.  Bound by issue and
// latency while a CU has one tile (about 6 us per launch and 4 us per sweep), by issue beyond.
constexpr int TB = 16;
constexpr int square_halo(int ns) { return 8 * ns + 1; }
constexpr int square_inner(int ns) { return (4 * TB - 2 * square_halo(ns)) & ~3; }
constexpr int square_tiles(int L, int ns) { return (L + square_inner(ns) - 1) / square_inner(ns); }   // per side

template <int NS, bool GIVEN>
__global__ __launch_bounds__(TB * TB) void k_square_tile(SquareArgs a, int m)
{
  constexpr int H = square_halo(NS), I = square_inner(NS);
  static_assert(I >= 4 && (H - 1) % 4 == 0, "block-aligned tiles");
  __shared__ u64 sq_lds[16 * TB * TB];
  const int lin = xcd_remap((int)blockIdx.x, (int)gridDim.x);
  const int side = square_tiles(a.g.L, NS);
  const int word = lin / (side * side);
  const int tile = lin - word * (side * side);
  const int ty = tile / side, tx = tile - ty * side;
  const int bx = (int)threadIdx.x % TB, by = (int)threadIdx.x / TB;
  int gx = tx * (I / 4) - (H - 1) / 4 + bx, gy = ty * (I / 4) - (H - 1) / 4 + by;
  gx = gx < 0 ? gx + a.g.Q : gx >= a.g.Q ? gx - a.g.Q : gx;
  gy = gy < 0 ? gy + a.g.Q : gy >= a.g.Q ? gy - a.g.Q : gy;
  const int pos = gx + a.g.Q * gy;
  Square<TB * TB> t;
  t.s = sq_lds;
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      // beyond the tile: any block will do, the sites it can reach are not stored
      const int x = min(max(bx + dx, 0), TB - 1), y = min(max(by + dy, 0), TB - 1);
      t.off[dy + 1][dx + 1] = x + TB * y;
    }
  load_block(t, a, word, pos, (int)threadIdx.x);
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x) t.f[y][x] = 0;
  SquareDraw g{};
  g.P = a.g.P;
  constexpr int D = GIVEN ? 8 : 0;   // a sweep's words at once
  u64 r[D ? D : 1][4];
  if constexpr (GIVEN) {
    g.acc = a.acc + ((size_t)word * a.n_sweeps + a.sweep) * 32u * (size_t)a.g.P;
    g.pos = (unsigned)pos;
#pragma unroll
    for (int c = 0; c < D; ++c) g.load(c, r[c]);
  } else {
    g.t = a.t0;
    g.key0 = a.key0;
    g.key1 = a.key1;
    g.site = (uint32_t)(4 * gx) + (uint32_t)(4 * gy) * (uint32_t)a.g.L;
    g.L = (uint32_t)a.g.L;
    g.word = word;
    g.noise = a.noise;
  }
  __syncthreads();
#pragma unroll 1
  for (int k = 0; k < NS; ++k) {
    t.template sweep<D>(r, g, m, k + 1 < NS);
    g.acc += 32u * (size_t)a.g.P;
    g.t += 1;
  }
  // n of the window is stored; a moved-ever word is read where its site moved and stored where it
  // gains a bit.  All of the reads are issued before any is used.
  const int nx = min(I, a.g.L - tx * I), ny = min(I, a.g.L - ty * I);
  const unsigned at = (unsigned)(pos * a.wpt);
  const auto stored = [&](int x, int y) {
    const int X = 4 * bx + x - H, Y = 4 * by + y - H;
    return X >= 0 && X < nx && Y >= 0 && Y < ny;
  };
  u64 had[4][4];
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x) had[y][x] = stored(x, y) && t.f[y][x] ? sublattice_word(a.f, a, word, x + 4 * y)[at] : ~0ull;
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x)
      if (stored(x, y)) sublattice_word(a.n_out, a, word, x + 4 * y)[at] = t.n[y][x];
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x)
      if (t.f[y][x] & ~had[y][x]) sublattice_word(a.f, a, word, x + 4 * y)[at] = had[y][x] | t.f[y][x];
}

template <int NS>
hipError_t launch_tile(const SquareArgs &a, int m, hipStream_t s)
{
  const int side = square_tiles(a.g.L, NS);
  const dim3 grid((unsigned)(side * side * a.W));
  if (a.acc) {
    hipLaunchKernelGGL((k_square_tile<NS, true>), grid, dim3(TB * TB), 0, s, a, m);
  } else {
    if constexpr (NS == 1) hipLaunchKernelGGL((k_square_tile<1, false>), grid, dim3(TB * TB), 0, s, a, m);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int NT, bool GIVEN>
hipError_t launch_resident(const SquareArgs &a, int m, hipStream_t s)
{
  const int threads = (a.g.P + 63) / 64 * 64;
  const size_t lds = (size_t)16 * NT * sizeof(u64);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_square_resident<NT, GIVEN>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_square_resident<NT, GIVEN>), dim3((unsigned)a.W), dim3((unsigned)threads), lds, s, a, m);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_square_accept(const SquareArgs &a, hipStream_t s)
{
  if (!a.acc || a.n_sweeps < 1 || a.n_sweeps > 8191) return hipErrorInvalidValue;   // grid y limit
  const int block = a.g.P > 64 ? 256 : 64;
  const dim3 grid((unsigned)((a.g.P + block - 1) / block), (unsigned)(8 * a.n_sweeps), (unsigned)((a.W + 1) / 2));
  hipLaunchKernelGGL(k_square_accept, grid, dim3((unsigned)block), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_square_resident(const SquareArgs &a, int m, hipStream_t s)
{
  if (a.g.d != 2 || a.g.P > kSquareResidentP || a.n_sweeps < 1) return hipErrorInvalidValue;
  if (a.acc)
    return a.g.P <= 64 ? launch_resident<64, true>(a, m, s) : a.g.P <= 256 ? launch_resident<256, true>(a, m, s)
                                                            : launch_resident<512, true>(a, m, s);
  return a.g.P <= 64 ? launch_resident<64, false>(a, m, s) : a.g.P <= 256 ? launch_resident<256, false>(a, m, s)
                                                           : launch_resident<512, false>(a, m, s);
}

// With one tile per CU a launch's fixed cost is shared by its sweeps, and the deeper halos cost
// nothing; with more tiles than CUs they do.  Per sweep with one / two / three sweeps a launch:
// L = 192 x 64 (25 / 49 / 256 tiles) 9.9 / 7.8 / 6.7 us, L = 256 x 64 (36 / 100 / 484) 10.1 / 8.1 / 8.5,
// L = 512 x 64 (144 / 361 / 1849) 12.7 / 12.3 / 24, L = 128 x 256 (36 / 100 / 484) 10.4 / 8.2 / 8.8.
int square_sweeps_per_launch(const SquareArgs &a)
{
  const auto tiles = [&](int ns) { return (int64_t)square_tiles(a.g.L, ns) * square_tiles(a.g.L, ns) * a.W; };
  if (!a.acc) return 1;
  return tiles(3) <= 256 ? 3 : tiles(2) <= 400 ? 2 : 1;
}

hipError_t launch_square_tile(const SquareArgs &a, int sweeps, int m, hipStream_t s)
{
  // a tile's blocks are distinct blocks of the lattice
  if (a.g.d != 2 || a.g.Q < TB || !a.n_out || (a.acc && a.sweep + sweeps > a.n_sweeps)) return hipErrorInvalidValue;
  switch (sweeps) {
    case 1: return launch_tile<1>(a, m, s);
    case 2: return launch_tile<2>(a, m, s);
    case 3: return launch_tile<3>(a, m, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ka
