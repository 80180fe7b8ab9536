// ka_pairs.hip -- spatial four-point sums (gfx950).
//
// Method: Boccagna, arXiv 1710.05155, Sec. 2.2 (g4(r, t) and chi4 = sum_r g4) and Sec. 3.3
// (Phi(r, t) as the popcount of the AND of the words n_i(t), n_i(0), n_j(t), n_j(0)).  With
// Q_i = n_i(t) & n_i(0) per word (one bit per replica), for every minimum-image displacement
// delta with |delta|^2 = r2 <= r2_max:
//     S2[r2]  += popcount(Q_i & Q_{i+delta})            summed over sites i and words,
//     S11[r2] += popcount(Q_i) * popcount(Q_{i+delta})  with popcounts over all words,
// i.e. the replica sums of q_i q_j and the products of the replica sums, over ordered pairs.
// Both sums are the same for delta and -delta, so only one of the two is computed and counts twice.
//
// k_pairs_tile: a workgroup takes some rows of one plane, with the Q words and replica sums of the
// plane dz above (their halo included) in LDS; for every displacement with that dz a thread ANDs
// its sites' Q, held in registers, with the words at one offset from them.  k_pairs, one thread
// per site gathering from global memory, covers radii whose halo does not fit in LDS, and those
// where loading the tiles would take longer than the gathers (pairs_tiles).
#include <algorithm>

#include "ka_device.h"

namespace ka {
namespace {

using namespace dev;

constexpr int kPairBlock = 256;
constexpr int kPairChunk = 32;     // most displacements of a workgroup
constexpr int kMaxWords = 16;      // up to 1024 replicas
constexpr int kTileBlock = 512, kTileSites = 2;   // threads of k_pairs_tile, sites per thread
constexpr size_t kTileLds = 80 << 10;   // two workgroups to a CU

__device__ __forceinline__ unsigned wave_sum(unsigned v)
{
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += (unsigned)__shfl_xor((int)v, off);
  return v;
}

// element index of canonical coordinates in the sublattice layout
__device__ __forceinline__ int element_of(const LatticeGeom &g, const int (&x)[3])
{
  int sub = 0, pos = 0, sm = 1, pm = 1;
  for (int k = 0; k < g.d; ++k) {
    sub += (x[k] & 3) * sm;
    pos += (x[k] >> 2) * pm;
    sm *= 4;
    pm *= g.Q;
  }
  return sub * g.P + pos;
}

template <int WPT>
__global__ __launch_bounds__(kPairBlock) void k_pairs(PairArgs a, int chunk)
{
  __shared__ unsigned long long acc2[kMaxPairShells];
  __shared__ unsigned long long acc11[kMaxPairShells];
  const int tid = (int)threadIdx.x;
  for (int q = tid; q <= a.r2_max; q += kPairBlock) {
    acc2[q] = 0;
    acc11[q] = 0;
  }
  __syncthreads();
  const int idx = (int)blockIdx.x * kPairBlock + tid;
  const bool valid = idx < a.g.N;
  const int e = valid ? idx : 0;
  const int sub = e / a.g.P, pos = e - (e / a.g.P) * a.g.P;
  const Site s = decode(a.g, a.g.d, sub, pos);
  int x[3];
  for (int k = 0; k < 3; ++k) x[k] = 4 * s.p[k] + s.a[k];
  const size_t plane_words = (size_t)a.g.N * WPT;
  u64 qi[kMaxWords];
  unsigned pci = 0;
#pragma unroll
  for (int q = 0; q < kMaxWords; ++q) {
    qi[q] = 0;
    const int p = q / WPT, w = q % WPT;
    if (p < a.planes) {
      const size_t off = (size_t)p * plane_words + (size_t)e * WPT + w;
      qi[q] = a.n[off] & a.n0[off];
      pci += (unsigned)__popcll(qi[q]);
    }
  }
  const int d0 = (int)blockIdx.y * chunk;
  const int d1 = min(a.n_disp, d0 + chunk);
  for (int dq = d0; dq < d1; ++dq) {
    const int4 dv = a.disp[dq];   // components, shell * 2 + whether it counts twice
    const int r2 = dv.w >> 1;
    const u64 times = 1u + (unsigned)(dv.w & 1);
    int y[3] = {x[0] + dv.x, x[1] + dv.y, x[2] + dv.z};
    for (int k = 0; k < a.g.d; ++k) {
      if (y[k] < 0) y[k] += a.g.L;
      else if (y[k] >= a.g.L) y[k] -= a.g.L;
    }
    const int j = element_of(a.g, y);
    unsigned c2 = 0, pcj = 0;
#pragma unroll
    for (int q = 0; q < kMaxWords; ++q) {
      const int p = q / WPT, w = q % WPT;
      if (p < a.planes) {
        const size_t off = (size_t)p * plane_words + (size_t)j * WPT + w;
        const u64 qj = a.n[off] & a.n0[off];
        c2 += (unsigned)__popcll(qi[q] & qj);
        pcj += (unsigned)__popcll(qj);
      }
    }
    unsigned c11 = pci * pcj;
    if (!valid) c2 = c11 = 0;
    c2 = wave_sum(c2);
    c11 = wave_sum(c11);
    if (__lane_id() == 0) {
      atomicAdd(&acc2[r2], (u64)c2 * times);
      atomicAdd(&acc11[r2], (u64)c11 * times);
    }
  }
  __syncthreads();
  for (int q = tid; q <= a.r2_max; q += kPairBlock) {
    if (acc2[q]) atomicAdd(&a.S2[q], acc2[q]);
    if (acc11[q]) atomicAdd(&a.S11[q], acc11[q]);
  }
}

// Sum over the wave, on lane 63: adds of lanes 1, 2, 4 and 8 below within rows of 16, then of the
// last lane of the row and of the two rows before.
__device__ __forceinline__ unsigned wave_sum_last(unsigned v)
{
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr:2
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr:4
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr:8
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Word w of q at element e.
__device__ __forceinline__ u64 site_word(const PairArgs &a, int wpt, int e, int w)
{
  const size_t at = ((size_t)(w / wpt) * (size_t)a.g.N + (size_t)e) * (size_t)wpt + (size_t)(w % wpt);
  return a.n[at] & a.n0[at];
}

// Bound by VALU and LDS: per site, displacement and word two ANDs, two population counts and an 8
// byte LDS read.  WC words at a time (S11 comes with the first of them).
// 3D L = 64 x 256 replicas, squared radius to 36: 177 us, of which the LDS reads alone take 50; 190
// with 32-bit products (a quarter of the rate of 24-bit ones) and each displacement's record
// fetched where it is used.
template <int WC>
__global__ __launch_bounds__(kTileBlock) void k_pairs_tile(PairArgs a, int wpt)
{
  extern __shared__ u64 pair_lds[];
  const int tid = (int)threadIdx.x;
  const int L = a.g.L, h = a.halo, T = a.tiles.rows;
  const int width = L + 2 * h, area = (T + 2 * h) * width;
  // word pairs in one 16-byte read (WC = 1: single words)
  constexpr int V = WC > 1 ? 2 : 1, G = WC / V;
  u64 *q = pair_lds;                                                  // [G][area][V]
  u64 *acc2 = q + (size_t)WC * area, *acc11 = acc2 + a.r2_max + 1;
  unsigned short *sum = reinterpret_cast<unsigned short *>(acc11 + a.r2_max + 1);   // [area]
  const int y0 = (int)blockIdx.x * T, z = (int)blockIdx.y, dz = (int)blockIdx.z / a.tiles.parts;
  const int part = (int)blockIdx.z - dz * a.tiles.parts;
  const int zb = z + dz < L ? z + dz : z + dz - L;
  const int first = a.start[dz], listed = a.start[dz + 1] - first;   // at most 2^13 displacements in a plane
  const int d0 = first + listed * part / a.tiles.parts, d1 = first + listed * (part + 1) / a.tiles.parts;
  if (d0 == d1) return;
  for (int k = tid; k <= a.r2_max; k += kTileBlock) acc2[k] = acc11[k] = 0;
  // this thread's sites: tile positions tid + k * kTileBlock (rows beyond the lattice hold none)
  const int W = a.planes * wpt;
  int at[kTileSites], elem[kTileSites];
  unsigned p[kTileSites];
#pragma unroll
  for (int k = 0; k < kTileSites; ++k) {
    const int s = tid + k * kTileBlock, y = s / L, x = s - y * L;
    const bool valid = y < T && y0 + y < L;
    const int xyz[3] = {x, valid ? y0 + y : 0, z};
    elem[k] = valid ? element_of(a.g, xyz) : -1;
    at[k] = valid ? (y + h) * width + x + h : h * width + h;
    p[k] = 0;
  }
  const float inv = 1.0f / (float)width;
  constexpr int U = 4;   // tile sites a thread loads at a time
  for (int w0 = 0; w0 < W; w0 += WC) {
    __syncthreads();   // the previous words' reads are done
    for (int k0 = tid; k0 < area; k0 += U * kTileBlock) {
      u64 v[U][WC];
      int e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(k0 + u * kTileBlock, area - 1);
        int y = (int)((float)k * inv);   // k below 2^14: exact after one correction
        y -= y * width > k;
        y += (y + 1) * width <= k;
        int x = k - y * width - h;
        y += y0 - h;
        x = x < 0 ? x + L : x >= L ? x - L : x;
        y = y < 0 ? y + L : y >= 2 * L ? y - 2 * L : y >= L ? y - L : y;
        const int xyz[3] = {x, y, zb};
        e[u] = element_of(a.g, xyz);
#pragma unroll
        for (int w = 0; w < WC; ++w) v[u][w] = w0 + w < W ? site_word(a, wpt, e[u], w0 + w) : 0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(k0 + u * kTileBlock, area - 1);   // (the last site more than once, with the same words)
        unsigned sites = 0;
#pragma unroll
        for (int w = 0; w < WC; ++w) {
          q[((w / V) * area + k) * V + w % V] = v[u][w];
          sites += (unsigned)__popcll(v[u][w]);
        }
        if (w0 == 0) {   // replica sum: the words that are here, and the others
          for (int w = WC; w < W; ++w) sites += (unsigned)__popcll(site_word(a, wpt, e[u], w));
          sum[k] = (unsigned short)sites;
        }
      }
    }
    u64 qi[kTileSites][WC];
#pragma unroll
    for (int k = 0; k < kTileSites; ++k) {
#pragma unroll
      for (int w = 0; w < WC; ++w) {
        qi[k][w] = elem[k] >= 0 && w0 + w < W ? site_word(a, wpt, elem[k], w0 + w) : 0;
        if (w0 == 0) p[k] += (unsigned)__popcll(qi[k][w]);
      }
      if (w0 == 0 && elem[k] >= 0)
        for (int w = WC; w < W; ++w) p[k] += (unsigned)__popcll(site_word(a, wpt, elem[k], w));
    }
    __syncthreads();
    // Displacements of one shell follow each other, and are summed over the wave together (at
    // most 16 of them: a product of replica sums takes 2^27 over a wave).
    unsigned c2 = 0, c11 = 0;
    int4 next = a.disp[d0];
    for (int d = d0, run = 1; d < d1; ++d, ++run) {
      const int4 dv = next;   // offset in the tile, shell, how often it counts, whether the next one differs in these
      next = a.disp[min(d + 1, d1 - 1)];
#pragma unroll
      for (int k = 0; k < kTileSites; ++k) {
        const int j = at[k] + dv.x;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const Elem<V> x = ld<V>(q + (size_t)g * area * V, j);
#pragma unroll
          for (int w = 0; w < V; ++w) c2 += (unsigned)__popcll(qi[k][g * V + w] & x.w[w]);
        }
        if (w0 == 0) c11 += __umul24(p[k], (unsigned)sum[j]);   // both at most 1024
      }
      if (!dv.w && run < 16 && d + 1 < d1) continue;
      c2 = wave_sum_last(c2);
      if (w0 == 0) c11 = wave_sum_last(c11);
      if (__lane_id() == 63) {
        if (c2) atomicAdd(&acc2[dv.y], (u64)c2 * (u64)dv.z);
        if (w0 == 0 && c11) atomicAdd(&acc11[dv.y], (u64)c11 * (u64)dv.z);
      }
      c2 = c11 = 0;
      run = 0;
    }
  }
  __syncthreads();
  for (int k = tid; k <= a.r2_max; k += kTileBlock) {
    if (acc2[k]) atomicAdd(&a.S2[k], acc2[k]);
    if (acc11[k]) atomicAdd(&a.S11[k], acc11[k]);
  }
}

size_t tile_lds(int L, int halo, int rows, int r2_max, int wc)
{
  const size_t area = (size_t)(rows + 2 * halo) * (size_t)(L + 2 * halo);
  return area * (size_t)(8 * wc + 2) + (size_t)(r2_max + 1) * 16u + 16u;
}

// Graphs without a geometry (Sec. 3.3: distance 0 for i = j, 1 otherwise): only the per-site
// replica sums Q_i = sum_b q_i^b are needed, through sum_i Q_i and sum_i Q_i^2 (out[0], out[1]).
template <int WPT>
__global__ __launch_bounds__(kPairBlock) void k_pairs_graph(PairGraphArgs a)
{
  const int i = (int)blockIdx.x * kPairBlock + (int)threadIdx.x;
  unsigned q = 0;
  if (i < a.N) {
    const size_t plane_words = (size_t)a.N * WPT;
    for (int p = 0; p < a.planes; ++p)
#pragma unroll
      for (int w = 0; w < WPT; ++w) {
        const size_t off = (size_t)p * plane_words + (size_t)i * WPT + w;
        q += (unsigned)__popcll(a.n[off] & a.n0[off]);
      }
  }
  // per wave: sum Q <= 64 * 1024 and sum Q^2 <= 64 * 2^20, both within 32 bits
  const unsigned s1 = wave_sum(q);
  const unsigned s2 = wave_sum(q * q);
  if (__lane_id() == 0 && s1) {
    atomicAdd(&a.out[0], (unsigned long long)s1);
    atomicAdd(&a.out[1], (unsigned long long)s2);
  }
}

}  // namespace

hipError_t launch_pairs_graph(const PairGraphArgs &a, int wpt, hipStream_t s)
{
  const dim3 grid((unsigned)((a.N + kPairBlock - 1) / kPairBlock));
  if (wpt == 2)
    hipLaunchKernelGGL((k_pairs_graph<2>), grid, dim3(kPairBlock), 0, s, a);
  else
    hipLaunchKernelGGL((k_pairs_graph<1>), grid, dim3(kPairBlock), 0, s, a);
  return hipGetLastError();
}

// Displacements of a gather workgroup: fewer while that leaves CUs idle.
static int gather_chunk(const LatticeGeom &g, int n_disp)
{
  int chunk = kPairChunk;
  while (chunk > 8 && (int64_t)((g.N + kPairBlock - 1) / kPairBlock) * ((n_disp + chunk - 1) / chunk) < 256) chunk /= 2;
  return chunk;
}

// Microseconds of either kernel beyond what they share (the tiles' estimate, the rougher one, has to be below
// the other by a margin), fitted to L = 8 to 512 in 2D and 4 to 64 in 3D,
// 1 to 16 words, squared radii 0 to 2048 (within 10% for the gathers and 25% for the tiles).  A workgroup of
// the gathers takes up to 32 displacements of 256 sites; one of the tiles loads its tile and then takes its
// part of the displacements, so that more parts fill the device and cost more loads.
// A call, tiles in one part -> as chosen here: 2D L = 64 x 1024 replicas to r2 = 400 2423 -> 149 us (gathers),
// L = 64 x 64 236 -> 57 us (tiles in 64 parts; gathers 83); 3D L = 64 x 256 to r2 = 36, where one part fills the
// device, 208 us (two parts 255, gathers 868).
static double gather_us(const LatticeGeom &g, int W, int n_disp)
{
  const int chunk = gather_chunk(g, n_disp);
  const double blocks = (double)((g.N + kPairBlock - 1) / kPairBlock) * ((n_disp + chunk - 1) / chunk);
  const double each = std::min(n_disp, chunk);
  return each * (0.10 * W + 0.78) + 0.03 * W + blocks / 906.0 * each * (1.0 + 0.138 * W);
}

static double tile_us(const LatticeGeom &g, int W, int halo, int n_disp, int r2_max, const PairTiles &t)
{
  const int planes = g.d == 3 ? halo + 1 : 1;
  const double area = (double)(t.rows + 2 * halo) * (g.L + 2 * halo) / 1024.0;
  const double passes = (W + t.words - 1) / t.words;
  const double listed = ((n_disp + planes - 1) / planes + t.parts - 1) / t.parts;
  const double blocks = (double)((g.L + t.rows - 1) / t.rows) * (g.d == 3 ? g.L : 1) * planes * t.parts;
  const double at_once = 256.0 * std::min<size_t>(2, (160 << 10) / tile_lds(g.L, halo, t.rows, r2_max, t.words));
  return ((1.45 * passes + 0.80 * W) * area + 0.16 * listed * W + 2.1 * passes) * (1.0 + 1.54 * std::max(0.0, blocks / at_once - 1.0));
}

PairTiles pairs_tiles(const LatticeGeom &g, int W, int halo, int n_disp, int r2_max)
{
  PairTiles best{0, 0, 0};
  if (g.L > kTileSites * kTileBlock) return best;
  PairTiles t{std::min(g.L, kTileSites * kTileBlock / g.L), 4, 1};
  while (t.words >= 1 && tile_lds(g.L, halo, t.rows, r2_max, t.words) > kTileLds) t.words /= 2;
  if (t.words < 1) return best;
  double least = 0.85 * gather_us(g, W, n_disp);
  const int listed = n_disp / (g.d == 3 ? halo + 1 : 1);
  for (; t.parts <= 64 && (t.parts == 1 || 2 * t.parts <= listed); t.parts *= 2) {
    const double us = tile_us(g, W, halo, n_disp, r2_max, t);
    if (us >= least) continue;
    least = us;
    best = t;
  }
  return best;
}

hipError_t launch_pairs_tile(const PairArgs &a, int wpt, hipStream_t s)
{
  const int rows = a.tiles.rows, words = a.tiles.words;
  const size_t lds = tile_lds(a.g.L, a.halo, rows, a.r2_max, words);
  if (rows < 1 || a.tiles.parts < 1 || rows * a.g.L > kTileSites * kTileBlock || 2 * a.halo > a.g.L || lds > kTileLds)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)((a.g.L + rows - 1) / rows), (unsigned)(a.g.d == 3 ? a.g.L : 1),
                  (unsigned)((a.g.d == 3 ? a.halo + 1 : 1) * a.tiles.parts));
#define KA_PT(WC)                                                                                        \
  do {                                                                                                   \
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_pairs_tile<WC>),           \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTileLds); \
    if (e != hipSuccess) return e;                                                                       \
    hipLaunchKernelGGL((k_pairs_tile<WC>), grid, dim3(kTileBlock), lds, s, a, wpt);                      \
  } while (0)
  if (words == 4) KA_PT(4);
  else if (words == 2) KA_PT(2);
  else KA_PT(1);
#undef KA_PT
  return hipGetLastError();
}

hipError_t launch_pairs(const PairArgs &a, int wpt, hipStream_t s)
{
  const int chunk = gather_chunk(a.g, a.n_disp);
  const dim3 grid((unsigned)((a.g.N + kPairBlock - 1) / kPairBlock), (unsigned)((a.n_disp + chunk - 1) / chunk));
  if (wpt == 2)
    hipLaunchKernelGGL((k_pairs<2>), grid, dim3(kPairBlock), 0, s, a, chunk);
  else
    hipLaunchKernelGGL((k_pairs<1>), grid, dim3(kPairBlock), 0, s, a, chunk);
  return hipGetLastError();
}

}  // namespace ka
