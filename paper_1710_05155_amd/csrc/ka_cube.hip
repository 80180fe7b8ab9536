// ka_cube.hip -- small 3D lattices: the whole sweep loop of one word in one workgroup, on 4 x 4
// blocks of sites held in registers (gfx950).
//
// Method: Boccagna, arXiv 1710.05155; the bit logic lives in ka_device.h.
//
// The 3D form of the 2D register blocks: a thread owns the 16 words (n and moved-ever) of a 4 x 4
// block in x and y at one z, and LDS holds a copy of n for what other threads read.  Waves are
// ordered by z mod 4, so where a class's edges lie in a block is decided per wave.  Classes
// along x and y give every thread four edges; a class along z gives the blocks of two of the
// four residues eight edges each as lower endpoints, and the blocks above them take their new
// words (and the moved-ever bits from the change) from LDS after the barrier.  The waves of residues 0
// and 2, the active ones of every other such class, sit on different SIMDs.
//
// Bound by issue and latency on one CU per word.  Measured per sweep: L = 16 x 64 replicas 10.8 us
// (13.6 with n and f in LDS), L = 20 x 64 15.1 (24), L = 20 x 256 17.0 (51 as class passes over global
// memory).  Below L = 16 the four edges of a thread in turn take longer than one edge per
// thread (L = 12: 11.1 against 9.3 us, L = 8: 10.9 against 7.7), and the kernel of ka_lds.hip runs.
#include "ka_device.h"

namespace ka {
namespace {

using namespace dev;

// Where a thread's acceptance words come from: drawn ahead (acc: this sweep's, [class][16][P]) or drawn
// here from the canonical id of the block's corner site.
struct CubeDraw {
  const u64 *acc;
  int P, pos, az;
  uint32_t t, key0, key1, site, L;
  int word, noise;

  __device__ __forceinline__ u64 draw(int c, uint32_t x, uint32_t y, uint32_t mu) const
  {
    u64 r[1];
    accept_words<1>(t, (uint32_t)c, 3u * (site + x + L * y) + mu, word, key0, key1, noise, r);
    return r[0];
  }
  // the words of class c of the sweep at acc: four along x and y, eight along z for the two residues
  // of z with lower endpoints
  __device__ __forceinline__ void load(const u64 *from, int c, u64 (&r)[8]) const
  {
    const u64 *p = from + (size_t)(c * 16) * (size_t)P;
    if (c < 8) {
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] = (p + (size_t)(az * 4 + q) * (size_t)P)[pos];
    } else if (((az ^ c) & 1) == 0) {
      const int h = az == (c & 3) ? 0 : 8;
#pragma unroll
      for (int q = 0; q < 8; ++q) r[q] = (p + (size_t)(h + q) * (size_t)P)[pos];
    }
  }
};

// P: positions of the LDS copy, a constant so that the place in the block is part of an access's
// immediate offset.
template <int P>
struct Cube {
  u64 *s;                 // n in LDS: [64 sublattices][P]
  // element of (x = 0, y = 0) of blocks around this one, by direction: in this plane, one above, one
  // below, two above
  int here[3][3], above[3][3], below[3][3], above2;
  u64 n[4][4], f[4][4];   // [y][x]

  template <int X, int Y>
  __device__ __forceinline__ u64 &in(const int (&b)[3][3]) const
  {
    constexpr int bx = X < 0 ? 0 : X > 3 ? 2 : 1, by = Y < 0 ? 0 : Y > 3 ? 2 : 1;
    return s[((X & 3) + 4 * (Y & 3)) * P + b[by][bx]];
  }
  template <int X, int Y>
  __device__ __forceinline__ u64 at() const
  {
    if constexpr (X >= 0 && X < 4 && Y >= 0 && Y < 4) return n[Y][X];
    else return in<X, Y>(here);
  }

  // ---- classes along x (MU = 0) and y (MU = 1): edge Q is in row or column Q, from place
  // A = (R + 2 Q) mod 4 along MU, with R the class residue less twice the block's z
  template <int MU, int A, int B>
  __device__ __forceinline__ u64 along() const
  {
    if constexpr (MU == 0) return at<A, B>();
    else return at<B, A>();
  }
  template <int MU, int A, int B>
  __device__ __forceinline__ u64 along(const int (&b)[3][3]) const
  {
    if constexpr (MU == 0) return in<A, B>(b);
    else return in<B, A>(b);
  }
  template <int MU, int R, int Q>
  __device__ __forceinline__ void gather(u64 (&x)[11]) const
  {
    constexpr int a = (R + 2 * (Q & 1)) & 3;
    x[0] = along<MU, a + 1, Q>();
    x[1] = along<MU, a - 1, Q>();
    x[2] = along<MU, a, Q + 1>();
    x[3] = along<MU, a, Q - 1>();
    x[4] = along<MU, a, Q>(above);
    x[5] = along<MU, a, Q>(below);
    x[6] = along<MU, a + 2, Q>();
    x[7] = along<MU, a + 1, Q + 1>();
    x[8] = along<MU, a + 1, Q - 1>();
    x[9] = along<MU, a + 1, Q>(above);
    x[10] = along<MU, a + 1, Q>(below);
  }
  template <int MU, int R, int Q>
  __device__ __forceinline__ void exchange(const u64 (&x)[11], u64 r, int m)
  {
    constexpr int a = (R + 2 * (Q & 1)) & 3;
    constexpr int iy = MU == 0 ? Q : a, ix = MU == 0 ? a : Q;
    const u64 xi[5] = {x[1], x[2], x[3], x[4], x[5]}, xj[5] = {x[6], x[7], x[8], x[9], x[10]};
    const u64 d = bit3<kTTAnd3>(bit3<kTTXorAnd>(n[iy][ix], x[0], activity<5>(xi, m)), activity<5>(xj, m), r);
    n[iy][ix] ^= d;
    f[iy][ix] |= d;
    in<ix, iy>(here) = n[iy][ix];
    if constexpr (a < 3) {
      constexpr int jy = MU == 0 ? Q : a + 1, jx = MU == 0 ? a + 1 : Q;
      n[jy][jx] ^= d;
      f[jy][jx] |= d;
      in<jx, jy>(here) = n[jy][jx];
    } else if constexpr (MU == 0) {
      in<4, Q>(here) = x[0] ^ d;
    } else {
      in<Q, 4>(here) = x[0] ^ d;
    }
  }
  template <int X, int Y>
  __device__ __forceinline__ void take()   // the word another thread changed
  {
    const u64 v = in<X, Y>(here);
    f[Y][X] |= n[Y][X] ^ v;
    n[Y][X] = v;
  }
  template <int MU, int R, bool GIVEN>
  __device__ __forceinline__ void work_xy(u64 (&r)[8], const CubeDraw &g, int c, int m)
  {
    if constexpr (!GIVEN) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t a = (uint32_t)((R + 2 * (q & 1)) & 3);
        r[q] = g.draw(c, MU == 0 ? a : (uint32_t)q, MU == 0 ? (uint32_t)q : a, (uint32_t)MU);
      }
      __builtin_amdgcn_sched_barrier(0);   // the draws end before the gathered words take registers
    }
    u64 x[4][11];
    gather<MU, R, 0>(x[0]);
    gather<MU, R, 1>(x[1]);
    gather<MU, R, 2>(x[2]);
    gather<MU, R, 3>(x[3]);
    exchange<MU, R, 0>(x[0], r[0], m);
    exchange<MU, R, 1>(x[1], r[1], m);
    exchange<MU, R, 2>(x[2], r[2], m);
    exchange<MU, R, 3>(x[3], r[3], m);
  }
  template <int MU, int R>
  __device__ __forceinline__ void refresh_xy()
  {
    constexpr int q = (R & 1) ? (R == 3 ? 0 : 1) : -1;   // rows whose edge leaves the block: q and q + 2
    if constexpr (q >= 0) {
      if constexpr (MU == 0) {
        take<0, q>();
        take<0, q + 2>();
      } else {
        take<q, 0>();
        take<q + 2, 0>();
      }
    }
  }

  // ---- classes along z: the edges from the block's sites with x + y = E mod 2 to the plane above
  template <int X, int Y>
  __device__ __forceinline__ void gather_z(u64 (&x)[11]) const
  {
    x[0] = in<X, Y>(above);
    x[1] = at<X + 1, Y>();
    x[2] = at<X - 1, Y>();
    x[3] = at<X, Y + 1>();
    x[4] = at<X, Y - 1>();
    x[5] = in<X, Y>(below);
    x[6] = in<X + 1, Y>(above);
    x[7] = in<X - 1, Y>(above);
    x[8] = in<X, Y + 1>(above);
    x[9] = in<X, Y - 1>(above);
    x[10] = s[(X + 4 * Y) * P + above2];
  }
  template <int X, int Y>
  __device__ __forceinline__ void exchange_z(const u64 (&x)[11], u64 r, int m)
  {
    const u64 xi[5] = {x[1], x[2], x[3], x[4], x[5]}, xj[5] = {x[6], x[7], x[8], x[9], x[10]};
    const u64 d = bit3<kTTAnd3>(bit3<kTTXorAnd>(n[Y][X], x[0], activity<5>(xi, m)), activity<5>(xj, m), r);
    n[Y][X] ^= d;
    f[Y][X] |= d;
    in<X, Y>(here) = n[Y][X];
    in<X, Y>(above) = x[0] ^ d;
  }
  template <int E, int Y, bool GIVEN>   // rows Y and Y + 1, words r[2 Y] on
  __device__ __forceinline__ void rows_z(u64 (&r)[8], const CubeDraw &g, int c, int m)
  {
    constexpr int e0 = (Y + E) & 1, e1 = (Y + 1 + E) & 1;
    if constexpr (!GIVEN) {
      r[2 * Y] = g.draw(c, e0, Y, 2);
      r[2 * Y + 1] = g.draw(c, e0 + 2, Y, 2);
      r[2 * Y + 2] = g.draw(c, e1, Y + 1, 2);
      r[2 * Y + 3] = g.draw(c, e1 + 2, Y + 1, 2);
      __builtin_amdgcn_sched_barrier(0);
    }
    u64 x[4][11];
    gather_z<e0, Y>(x[0]);
    gather_z<e0 + 2, Y>(x[1]);
    gather_z<e1, Y + 1>(x[2]);
    gather_z<e1 + 2, Y + 1>(x[3]);
    exchange_z<e0, Y>(x[0], r[2 * Y], m);
    exchange_z<e0 + 2, Y>(x[1], r[2 * Y + 1], m);
    exchange_z<e1, Y + 1>(x[2], r[2 * Y + 2], m);
    exchange_z<e1 + 2, Y + 1>(x[3], r[2 * Y + 3], m);
  }
  template <int E, bool GIVEN>
  __device__ __forceinline__ void work_z(u64 (&r)[8], const CubeDraw &g, int c, int m)
  {
    rows_z<E, 0, GIVEN>(r, g, c, m);
    rows_z<E, 2, GIVEN>(r, g, c, m);
  }
  template <int E>
  __device__ __forceinline__ void refresh_z()
  {
    constexpr int e = E & 1, o = 1 - e;
    take<e, 0>();
    take<e + 2, 0>();
    take<o, 1>();
    take<o + 2, 1>();
    take<e, 2>();
    take<e + 2, 2>();
    take<o, 3>();
    take<o + 2, 3>();
  }
};

// Word `word` of the sites of a sublattice, in an array laid out in planes of wpt words: position
// pos is at [pos * wpt].  The same address on every lane.
template <typename T>
__device__ __forceinline__ T *sublattice_word(T *base, const SquareArgs &a, int word, int sub)
{
  return base + ((size_t)(word / a.wpt) * (size_t)a.g.N + (size_t)sub * (size_t)a.g.P) * (size_t)a.wpt + (size_t)(word % a.wpt);
}

// Acceptance words of sweeps t0 .. t0 + n_sweeps - 1: entry
// ((word * n_sweeps + s) * 12 + c) * 16 + group * 4 + q, times P, plus pos.  Along x and y
// the group is z mod 4 and q the row or column; along z group 2 h + k holds the sites of rows
// 2 k and 2 k + 1 with x + y = h mod 2.  A thread draws four edges; one Philox call serves two words.
__global__ __launch_bounds__(256) void k_cube_accept(SquareArgs a)
{
  const int k = (int)blockIdx.x * 256 + (int)threadIdx.x;   // group * P + pos
  if (k >= 4 * a.g.P) return;
  const int s = (int)blockIdx.y / 12, c = (int)blockIdx.y - 12 * s;
  const int pair = (int)blockIdx.z;
  const int group = k / a.g.P, pos = k - group * a.g.P;
  const Site b = decode(a.g, 3, 0, pos);
  const int mu = c >> 2;
  u64 r[4][2];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int x[3];
    if (mu < 2) {
      x[mu] = ((c & 3) + 2 * (q + group)) & 3;
      x[1 - mu] = q;
      x[2] = group;
    } else {
      const int h = group >> 1;
      x[1] = 2 * (group & 1) + (q >> 1);
      x[0] = 2 * (q & 1) + ((x[1] + h) & 1);
      x[2] = ((c & 3) + 2 * h) & 3;
    }
    const uint32_t i = (uint32_t)(4 * b.p[0] + x[0] + a.g.L * (4 * b.p[1] + x[1] + a.g.L * (4 * b.p[2] + x[2])));
    accept_words<2>(a.t0 + (uint32_t)s, (uint32_t)c, i * 3u + (uint32_t)mu, pair, a.key0, a.key1, a.noise, r[q]);
  }
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const int word = 2 * pair + w;
    if (word >= a.W) continue;
    u64 *acc = a.acc + (((size_t)word * a.n_sweeps + s) * 192u + (size_t)c * 16u + (size_t)group * 4u) * (size_t)a.g.P;
#pragma unroll
    for (int q = 0; q < 4; ++q) (acc + (size_t)q * (size_t)a.g.P)[pos] = r[q][w];
  }
}

// Every class has its own code, with both places that its edges can take: with loops over the
// classes, a quarter of the code, a sweep of L = 20 took 19.4 instead of 15.1 us.
template <int P, bool GIVEN>   // 64 or 128 positions of LDS: 256 or 512 threads
__global__ __launch_bounds__(4 * P, 2) void k_cube_resident(SquareArgs a, int m)
{
  __shared__ u64 lds[64 * P];
  const int word = xcd_remap((int)blockIdx.x, (int)gridDim.x);   // the words of a pair, whose state interleaves, in one XCD's L2
  const int slot = (int)threadIdx.x % P;
  // z mod 4 of this wave: residues 0, 2, 1, 3 in wave order
  const int g4 = __builtin_amdgcn_readfirstlane((int)threadIdx.x / P);
  const int az = ((g4 & 1) << 1) | (g4 >> 1);
  // threads that fill the last wave of a residue run a column of their own of zeros
  const bool mine = slot < a.g.P;
  const int pos = mine ? slot : 0;
  const Site b = decode(a.g, 3, 0, pos);
  Cube<P> t;
  t.s = lds;
  const auto block = [&](int dx, int dy, int dz) {   // element of (0, 0) of a block dx, dy away, dz planes up
    const int q[3] = {b.p[0] + dx, b.p[1] + dy, b.p[2] + ((az + dz) >> 2)};   // arithmetic shift: -1 for a plane below 0
    int w[3];
    for (int k = 0; k < 3; ++k) w[k] = q[k] < 0 ? q[k] + a.g.Q : q[k] >= a.g.Q ? q[k] - a.g.Q : q[k];
    const int p = mine ? w[0] + a.g.Q * (w[1] + a.g.Q * w[2]) : slot;
    return ((az + dz) & 3) * 16 * P + p;
  };
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      t.here[dy + 1][dx + 1] = block(dx, dy, 0);
      t.above[dy + 1][dx + 1] = block(dx, dy, 1);
      t.below[dy + 1][dx + 1] = block(dx, dy, -1);
    }
  t.above2 = block(0, 0, 2);
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int sub = x + 4 * y + 16 * az;
      t.n[y][x] = mine ? sublattice_word(a.n, a, word, sub)[(unsigned)(pos * a.wpt)] : 0;
      t.f[y][x] = mine ? sublattice_word(a.f, a, word, sub)[(unsigned)(pos * a.wpt)] : 0;
      lds[sub * P + slot] = t.n[y][x];
    }
  __syncthreads();

  const auto store = [&](u64 *n, u64 *f) {
    if (!mine) return;
    // not known to be the same from call to call, so that the addresses are not kept (spilled) over the sweeps
    int to = word;
    asm volatile("" : "+s"(to));
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        sublattice_word(n, a, to, x + 4 * y + 16 * az)[(unsigned)(pos * a.wpt)] = t.n[y][x];
        sublattice_word(f, a, to, x + 4 * y + 16 * az)[(unsigned)(pos * a.wpt)] = t.f[y][x];
      }
  };
  int row = 0;
  const size_t plane_words = (size_t)a.W * (size_t)a.g.N;
  const auto observe = [&](int64_t now) {
    for (; row < a.n_obs && (a.obs_times ? a.obs_times[row] == now : (int64_t)a.t0 + a.obs_at[row] == now); ++row) {
      u64 *dn = a.snap + (size_t)row * 2u * plane_words;
      store(dn, dn + plane_words);
    }
  };

  CubeDraw g{};
  g.P = a.g.P;
  g.pos = pos;
  g.az = az;
  const size_t sweep_words = 192u * (size_t)a.g.P;
  constexpr int D = 4;   // classes of words in flight: they cover the words' latency
  u64 r[D][8];
  if constexpr (GIVEN) {
    g.acc = a.acc + (size_t)word * a.n_sweeps * sweep_words;
#pragma unroll
    for (int c = 0; c < D; ++c) g.load(g.acc, c, r[c]);
  } else {
    g.t = a.t0;
    g.key0 = a.key0;
    g.key1 = a.key1;
    g.L = (uint32_t)a.g.L;
    g.site = (uint32_t)(4 * b.p[0]) + g.L * (uint32_t)(4 * b.p[1]) + g.L * g.L * (uint32_t)(4 * b.p[2] + az);
    g.word = word;
    g.noise = a.noise;
  }
  observe((int64_t)a.t0);
  const bool odd = az & 1;
  for (int s = 0; s < a.n_sweeps; ++s) {
    if constexpr (!GIVEN) asm volatile("" : "+v"(g.site));   // else the products of all ids are kept (spilled) over the sweeps
    // One class: the work at the places of this wave's z, the words of the class D later, the
    // barrier, and the words that other threads changed.  Those are read before the next barrier,
    // so the next class must not write them from another thread.  One pair of classes does: after
    // (1, 3) the blocks at z mod 4 = 3 take sites (1, 0) and (3, 0), which class (2, 0) writes from
    // the plane below; a barrier of its own orders the two.
#define KA_CUBE_XY(MU, R)                                                                          \
    if (odd) t.template work_xy<MU, (R ^ 2), GIVEN>(r[(4 * MU + R) % D], g, 4 * MU + R, m);        \
    else t.template work_xy<MU, R, GIVEN>(r[(4 * MU + R) % D], g, 4 * MU + R, m);                  \
    if constexpr (GIVEN) g.load(g.acc, 4 * MU + R + D, r[(4 * MU + R) % D]);                       \
    __syncthreads();                                                                               \
    if (odd) t.template refresh_xy<MU, (R ^ 2)>();                                                 \
    else t.template refresh_xy<MU, R>();
#define KA_CUBE_Z(R)                                                                               \
    if (az == R) t.template work_z<0, GIVEN>(r[R % D], g, 8 + R, m);                               \
    else if (az == (R ^ 2)) t.template work_z<1, GIVEN>(r[R % D], g, 8 + R, m);                    \
    if (GIVEN && s + 1 < a.n_sweeps) g.load(g.acc + sweep_words, 8 + R + D - 12, r[R % D]);        \
    __syncthreads();                                                                               \
    if (az == ((R + 1) & 3)) t.template refresh_z<0>();                                            \
    else if (az == ((R + 3) & 3)) t.template refresh_z<1>();
    KA_CUBE_XY(0, 0)
    KA_CUBE_XY(0, 1)
    KA_CUBE_XY(0, 2)
    KA_CUBE_XY(0, 3)
    KA_CUBE_XY(1, 0)
    KA_CUBE_XY(1, 1)
    KA_CUBE_XY(1, 2)
    KA_CUBE_XY(1, 3)
    __syncthreads();
    KA_CUBE_Z(0)
    KA_CUBE_Z(1)
    KA_CUBE_Z(2)
    KA_CUBE_Z(3)
#undef KA_CUBE_XY
#undef KA_CUBE_Z
    g.acc += sweep_words;
    g.t += 1;
    observe((int64_t)a.t0 + s + 1);
  }
  store(a.n, a.f);
}

}  // namespace

hipError_t launch_cube_accept(const SquareArgs &a, hipStream_t s)
{
  if (!a.acc || a.n_sweeps < 1 || a.n_sweeps > 5461) return hipErrorInvalidValue;   // grid y limit
  const dim3 grid((unsigned)((4 * a.g.P + 255) / 256), (unsigned)(12 * a.n_sweeps), (unsigned)((a.W + 1) / 2));
  hipLaunchKernelGGL(k_cube_accept, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_cube_resident(const SquareArgs &a, int m, hipStream_t s)
{
  if (a.g.d != 3 || a.g.P > kCubeResidentP || a.n_sweeps < 1) return hipErrorInvalidValue;
  const dim3 grid((unsigned)a.W);
#define KA_CUBE(P)                                                                          \
  do {                                                                                      \
    if (a.acc) hipLaunchKernelGGL((k_cube_resident<P, true>), grid, dim3(4 * P), 0, s, a, m); \
    else hipLaunchKernelGGL((k_cube_resident<P, false>), grid, dim3(4 * P), 0, s, a, m);      \
  } while (0)
  if (a.g.P <= 64) KA_CUBE(64);
  else KA_CUBE(128);
#undef KA_CUBE
  return hipGetLastError();
}

}  // namespace ka
