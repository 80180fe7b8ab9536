// ka_pass.hip -- global-memory class passes and observables (gfx950).
//
// Method: Boccagna, arXiv 1710.05155; the per-edge bit logic lives in ka_device.h.
#include <algorithm>
#include <mutex>

#include "ka_device.h"

// Fixed device scratch of the observation entry point that allocates nothing (see
// observe_scratch_setup below): one copy per device, held until the process ends.
static __device__ __align__(256) unsigned long long scratch[ka::kObserveScratchWords];

namespace ka {
namespace {

using namespace dev;

constexpr int kPassBlock = 256;
constexpr int kObsBlock = 512;
// Workgroups of one observation launch: at most two for each CU over all planes and states, at
// most one for each CU of one plane, and about a third of the CUs before lanes take four sites
constexpr int kObsBlocks = 512, kObsPlaneBlocks = 256, kObsSpread = 80;
// Graph classes are uneven (greedy colouring): a class with fewer edges than this (over all
// planes) runs in 64-thread workgroups, which spread it over more CUs; larger ones in
// kPassBlock-thread workgroups.
constexpr int kGraphSmallBlock = 64;
constexpr long long kGraphSmallEdges = 65536;

// Lattice passes of at most this many edge-words (edges of a class x words of the launch) load
// the moved-ever words together with the state words.  Up to there a pass is bound by its chain
// of dependent loads, and the words come from the caches; above, by bytes, and at low mobility
// most edges exchange nothing and need neither word.  Microseconds per class, loaded late -> with
// the state, 64 replicas: L = 48 3.49 -> 3.32 at density 0.8, L = 64 3.57 -> 3.41, L = 128 (2^19
// edge-words) 7.62 -> 7.52 and 6.57 -> 6.32 at density 0.9; 256 replicas, L = 64 (2^18) 4.48 ->
// 4.36, but L = 128 (2^21) 22.4 -> 22.3 and, at density 0.9, 15.1 -> 17.1.
constexpr long long kEarlyEdges = 1 << 19;

// ------------------------------------------------------------------------------------
// Global-memory class pass kernels: one launch per (class, sweep) over a range of planes.
// ------------------------------------------------------------------------------------
// Thread order: a wave covers 64 consecutive positions of one lower-endpoint sublattice
// (coalesced 64 x 16 B loads); consecutive waves cover the class's other lower-endpoint
// sublattices at the same positions, so the neighbour sublattices they share are fetched
// once and then served from L2 (together with the XCD-contiguous block order).
template <int D, int MU, int WPT, bool EARLY>
__global__ __launch_bounds__(kPassBlock) void k_pass_lattice(PassLattice a, int m)
{
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int pl = lin / a.blocks_per_plane;
  const int blk = lin - pl * a.blocks_per_plane;
  const int plane = a.plane0 + pl;
  const int gid = blk * kPassBlock + (int)threadIdx.x;
  constexpr int nsub = D == 2 ? 4 : 16;   // lower-endpoint sublattices per class
  const int span = nsub * 64;              // threads per 64-position chunk
  const int chunk = gid / span;
  const int rem = gid - chunk * span;
  // Waves are 64-thread aligned and span is a multiple of 64, so q is the same on every lane
  // of the wave: take it (and the sublattice) in scalar registers.
  const int q = __builtin_amdgcn_readfirstlane(rem >> 6);
  int chk = chunk;
  if (D == 3 && a.row_tile_log2 > 0) {
    // Rows (p1, p2) of whole chunks visited in tiles of T = 2^row_tile_log2 rows along p1,
    // p2 next: the +-e_2 neighbour rows are then T rows apart instead of Q (inside one L2),
    // at the cost of the +-e_1 neighbours at tile edges.  A permutation of the chunks.
    const int lt = a.row_tile_log2, lq = a.q_log2, lr = lq - 6;
    const int row = chk >> lr, xc = chk & ((1 << lr) - 1);
    const int tb = row >> (lt + lq);
    const int in = row & ((1 << (lt + lq)) - 1);
    const int p2 = in >> lt, p1 = (tb << lt) | (in & ((1 << lt) - 1));
    chk = ((p1 | (p2 << lq)) << lr) | xc;
  }
  const int pos = chk * 64 + (rem & 63);
  if (pos >= a.g.P) return;
  const int sub = class_sublattice(D, MU, (int)(a.c & 3u), q);
  const size_t off = (size_t)plane * (size_t)a.g.N * WPT;
  lattice_edge<D, MU, WPT, EARLY>(a.n + off, a.f + off, a.g, sub, pos, plane, m, a.t, a.c,
                                  a.key0, a.key1, a.noise);
}

template <int Z, int WPT, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_pass_graph(PassGraph a, int m)
{
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int pl = lin / a.blocks_per_plane;
  const int blk = lin - pl * a.blocks_per_plane;
  const int plane = a.plane0 + pl;
  const int k = blk * BLOCK + (int)threadIdx.x;
  if (k >= a.count) return;
  const size_t off = (size_t)plane * (size_t)a.N * WPT;
  if (a.fsat)
    graph_edge<Z, WPT>(a.n + off, a.f + off, a.edges, a.nbr, a.stride, a.first + k, plane, m, a.t,
                       a.c, a.key0, a.key1, a.noise, FSat{a.fsat, plane * a.N});
  else
    graph_edge<Z, WPT>(a.n + off, a.f + off, a.edges, a.nbr, a.stride, a.first + k, plane, m, a.t,
                       a.c, a.key0, a.key1, a.noise);
}

// One launch counts a.rows states (blockIdx.z): the sim's own state, or snapshots taken by the
// LDS-resident sweep loop.
// Bound by reading n, n0 and f once (24 B per site-word).  The wave counts are added in LDS and
// a workgroup makes one global add per count: with one per wave, the adds of all waves to the
// same few lines took longer than the reads.
template <int WPT>
__global__ __launch_bounds__(kObsBlock) void k_observe(ObserveArgs a)
{
  __shared__ unsigned cnt[3 * 64 * WPT];
  const int plane = blockIdx.y;
  const int row = blockIdx.z;
  const int tid = (int)threadIdx.x;
  const int lane = (int)__lane_id();
  for (int q = tid; q < 3 * 64 * WPT; q += kObsBlock) cnt[q] = 0;
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane((int)blockIdx.x * (kObsBlock / 64) + tid / 64);
  const int nwaves = (int)(gridDim.x * (kObsBlock / 64));
  const size_t off = (size_t)plane * (size_t)a.N * WPT;
  const size_t soff = off + (size_t)row * a.row_stride;
  unsigned acc[3][WPT];
#pragma unroll
  for (int o = 0; o < 3; ++o)
#pragma unroll
    for (int w = 0; w < WPT; ++w) acc[o][w] = 0;
  observe_sites<WPT>(a.n + soff, a.n0 + off, a.f + soff, a.N, wave * 64, nwaves * 64, acc);
#pragma unroll
  for (int o = 0; o < 3; ++o)
#pragma unroll
    for (int w = 0; w < WPT; ++w)
      if (acc[o][w]) atomicAdd(&cnt[(o * WPT + w) * 64 + lane], acc[o][w]);
  __syncthreads();
  unsigned long long *out = a.out + (size_t)row * 3u * (size_t)a.R;
  for (int q = tid; q < 3 * 64 * WPT; q += kObsBlock) {
    const int o = q / (64 * WPT), b = q - o * (64 * WPT);
    if (cnt[q]) atomicAdd(&out[(size_t)o * a.R + (size_t)plane * (64 * WPT) + b], (unsigned long long)cnt[q]);
  }
}

}  // namespace

// ------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------
hipError_t launch_pass_lattice(const PassLattice &a, int m, int wpt, hipStream_t s)
{
  const dim3 grid((unsigned)(a.blocks_per_plane * a.planes));
  const dim3 block(kPassBlock);
  const bool early = (long long)a.g.N / 4 * a.planes * wpt <= kEarlyEdges;
#define KA_LAT(D, MU, W)                                                                   \
  do {                                                                                     \
    if (early)                                                                             \
      hipLaunchKernelGGL((k_pass_lattice<D, MU, W, true>), grid, block, 0, s, a, m);       \
    else                                                                                   \
      hipLaunchKernelGGL((k_pass_lattice<D, MU, W, false>), grid, block, 0, s, a, m);      \
  } while (0)
  if (a.g.d == 2) {
    if (wpt == 2) {
      if (a.mu == 0) KA_LAT(2, 0, 2); else KA_LAT(2, 1, 2);
    } else {
      if (a.mu == 0) KA_LAT(2, 0, 1); else KA_LAT(2, 1, 1);
    }
  } else {
    if (wpt == 2) {
      if (a.mu == 0) KA_LAT(3, 0, 2); else if (a.mu == 1) KA_LAT(3, 1, 2); else KA_LAT(3, 2, 2);
    } else {
      if (a.mu == 0) KA_LAT(3, 0, 1); else if (a.mu == 1) KA_LAT(3, 1, 1); else KA_LAT(3, 2, 1);
    }
  }
#undef KA_LAT
  return hipGetLastError();
}

hipError_t launch_pass_graph(const PassGraph &args, int z, int m, int wpt, hipStream_t s)
{
  PassGraph a = args;
  const bool small = (long long)a.count * a.planes < kGraphSmallEdges;
  const int bs = small ? kGraphSmallBlock : kPassBlock;
  a.blocks_per_plane = (a.count + bs - 1) / bs;
  const dim3 grid((unsigned)(a.blocks_per_plane * a.planes));
  const dim3 block((unsigned)bs);
#define KA_GR(Z, W)                                                                        \
  do {                                                                                     \
    if (small)                                                                             \
      hipLaunchKernelGGL((k_pass_graph<Z, W, kGraphSmallBlock>), grid, block, 0, s, a, m); \
    else                                                                                   \
      hipLaunchKernelGGL((k_pass_graph<Z, W, kPassBlock>), grid, block, 0, s, a, m);       \
  } while (0)
  switch (z * 4 + wpt) {
    case 3 * 4 + 1: KA_GR(3, 1); break;
    case 3 * 4 + 2: KA_GR(3, 2); break;
    case 4 * 4 + 1: KA_GR(4, 1); break;
    case 4 * 4 + 2: KA_GR(4, 2); break;
    case 5 * 4 + 1: KA_GR(5, 1); break;
    case 5 * 4 + 2: KA_GR(5, 2); break;
    case 6 * 4 + 1: KA_GR(6, 1); break;
    case 6 * 4 + 2: KA_GR(6, 2); break;
    default: return hipErrorInvalidValue;
  }
#undef KA_GR
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Fixed scratch for the observation entry point that allocates nothing (ka_observe_noalloc):
// the per-replica counts accumulate here instead of in a sim's own buffer.  One copy per
// device, held until the process ends; every call on a device shares it.
// ------------------------------------------------------------------------------------
namespace {

__global__ void k_fill_u64(unsigned long long *p, int n, unsigned long long v)
{
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < n) p[i] = v;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned long long *g_scratch_ptr[kMaxDevices] = {};

}  // namespace

hipError_t observe_scratch_setup(int device)
{
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  // the array's name is only a host-side stand-in: the device address comes from the runtime,
  // taken with this device current
  void *ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(::scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = static_cast<unsigned long long *>(ptr);
  return hipSuccess;
}

unsigned long long *observe_scratch(int device)
{
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

hipError_t launch_fill_u64(unsigned long long *p, int n, unsigned long long v, hipStream_t s)
{
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_observe(const ObserveArgs &a, int wpt, hipStream_t s)
{
  if (a.rows < 1 || a.rows > 65535) return hipErrorInvalidValue;
  // Four sites per lane (one counter step), fewer only while that leaves most CUs idle, and at
  // most kObsPlaneBlocks workgroups for one plane of one state: all of them add into the same
  // 192 counts per word.  One state of 2^18 sites takes 7.2 us in 128 workgroups and 15.5 us in
  // 512; 10 states of 4096 sites take 6.9 us in 2 workgroups each and 6.1 us in 8 each.
  const int chunks = (a.N + kObsBlock - 1) / kObsBlock;
  const int sets = (int)std::min<int64_t>((int64_t)a.planes * a.rows, kObsBlocks);   // planes x states
  const int spread = std::max((chunks + 3) / 4, std::min(chunks, kObsSpread / sets));
  const int bx = std::max(1, std::min(spread, std::min(kObsPlaneBlocks, kObsBlocks / sets)));
  // a grid holds fewer than 2^16 workgroups in y: more planes than that are counted in parts
  constexpr int kGridY = 1 << 15;
  for (int first = 0; first < a.planes; first += kGridY) {
    ObserveArgs p = a;
    const size_t words = (size_t)first * (size_t)wpt;
    p.n += words * (size_t)a.N;
    p.n0 += words * (size_t)a.N;
    p.f += words * (size_t)a.N;
    p.out += words * 64u;
    p.planes = std::min(kGridY, a.planes - first);
    const dim3 grid((unsigned)bx, (unsigned)p.planes, (unsigned)a.rows);
    if (wpt == 2) hipLaunchKernelGGL((k_observe<2>), grid, dim3(kObsBlock), 0, s, p);
    else hipLaunchKernelGGL((k_observe<1>), grid, dim3(kObsBlock), 0, s, p);
  }
  return hipGetLastError();
}

}  // namespace ka
