// ka_init.hip -- initial state: a uniform K-subset of the sites per replica (gfx950).
//
// Method: Boccagna, arXiv 1710.05155, Sec. 3.1 (a configuration of fixed density drawn at
// random).  Replica b occupies the K sites with the smallest keys (u_i, i), u_i = half (b & 1) of
// Philox4x32-10(0, 0xFFFFFFFF, i, b >> 1).
//
// Large instances draw every key once.  The K-th smallest of N uniform keys lies within a few
// standard deviations sqrt(p (1 - p) / N), p = K/N, of p, so k_init_keys compares the keys with a
// window around p: below it a site is occupied, above it empty, and the few sites inside are
// listed per replica.  k_init_pick then finds the threshold among a replica's listed sites and
// sets the bits of those at or below it.  A replica whose threshold falls outside the window (about one in 10^5)
// is selected by radix over all its keys instead, and its bits set site by site.
#include <algorithm>
#include <cmath>

#include "ka_device.h"

namespace ka {
namespace {

using namespace dev;

constexpr int kSelBlock = 1024;
constexpr int kDig = 12;
constexpr int kBins = 1 << kDig;
constexpr int kCap = 2048;
// Below this many sites every key is ranked against every other; above, one histogram first
// (1024 sites: 83 us without it).
constexpr int kRankAll = 128;
constexpr int kBinsPerThread = kBins / kSelBlock;
constexpr int kKeysBlock = 256;
constexpr int kKeysEntries = 4096;   // candidates a workgroup of k_init_keys lists in LDS

// Element index -> canonical site id.
__device__ __forceinline__ int element_site(const InitArgs &a, int idx)
{
  if (!a.is_lattice) return a.site_of[idx];
  const int sub = idx / a.g.P;
  const int pos = idx - sub * a.g.P;
  const Site s = decode(a.g, a.g.d, sub, pos);
  return canonical(a.g, a.g.d, s);
}

// The draw of replica pair hp at a site: Philox4x32-10(0, 0xFFFFFFFF, site, hp).  Its first round
// leaves hp in one word by itself, so with a wave-uniform hp the next round's product with it is
// a scalar one, and the products with the site's words do not change from pair to pair.
__device__ __forceinline__ uint4 key_draw(const InitArgs &a, uint32_t site, uint32_t hp)
{
  const u64 p1 = (u64)0xCD9E8D57u * (u64)site;
  const uint4 c = make_uint4((uint32_t)(p1 >> 32) ^ 0xFFFFFFFFu ^ a.key0, (uint32_t)p1, hp ^ a.key1, 0u);
  return philox_rounds<1>(c, a.key0 + 0x9E3779B9u, a.key1 + 0xBB67AE85u);
}

__device__ __forceinline__ u64 site_key(const InitArgs &a, int site, int b)
{
  const uint4 o = key_draw(a, (uint32_t)site, (uint32_t)(b >> 1));
  return (b & 1) ? hi_half(o) : lo_half(o);
}

// Exclusive prefix sum of v over the kSelBlock threads of the block (every thread calls it;
// tmp holds one value per wave).  Counts stay below 2^32: at most N <= 2^31 keys.
__device__ __forceinline__ unsigned block_exclusive_scan(unsigned v, unsigned *tmp)
{
  const int lane = (int)__lane_id();
  const int wave = (int)threadIdx.x / 64;
  unsigned x = v;   // inclusive scan within the wave
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) tmp[wave] = x;
  __syncthreads();
  unsigned off = 0;
  for (int w = 0; w < wave; ++w) off += tmp[w];
  return off + x - v;
}

// Workgroup scratch of the selection of one replica.
struct Select {
  unsigned hist[kBins];
  u64 cand_u[kCap];
  int cand_i[kCap];     // canonical site
  int cand_at[kCap];    // element index
  unsigned scan[kSelBlock / 64];
  int bin;              // bin that holds the wanted key, -1 if none does
  unsigned before;      // keys in lower bins
  unsigned in_bin;
  int ncand;
  u64 thr_u;            // wanted key
  int thr_i;
};

// The bin of s.hist that holds the need-th smallest key (need >= 1), into s.bin, s.before and
// s.in_bin; thread t scans bins kBinsPerThread * t ...  Starts and ends with a barrier.
__device__ __forceinline__ void find_bin(Select &s, int64_t need)
{
  const int tid = (int)threadIdx.x;
  __syncthreads();   // the histogram is complete
  if (tid == 0) {
    s.bin = -1;
    s.before = s.in_bin = 0;
  }
  unsigned c[kBinsPerThread];
  unsigned sum = 0;
#pragma unroll
  for (int q = 0; q < kBinsPerThread; ++q) {
    c[q] = s.hist[kBinsPerThread * tid + q];
    sum += c[q];
  }
  unsigned e = block_exclusive_scan(sum, s.scan);   // its barrier orders the initial values first
#pragma unroll
  for (int q = 0; q < kBinsPerThread; ++q) {
    if ((int64_t)e < need && need <= (int64_t)e + (int64_t)c[q]) {
      s.bin = kBinsPerThread * tid + q;
      s.before = e;
      s.in_bin = c[q];
    }
    e += c[q];
  }
  __syncthreads();
}

// Key number `need` (1-based) in (u, i) order among the s.ncand <= kCap collected ones, into
// s.thr_u and s.thr_i.  Starts and ends with a barrier.
__device__ __forceinline__ void rank_candidates(Select &s, int64_t need)
{
  __syncthreads();
  const int nc = s.ncand;
  for (int k = (int)threadIdx.x; k < nc; k += (int)blockDim.x) {
    const u64 us = s.cand_u[k];
    const int is = s.cand_i[k];
    int rank = 0;
    for (int q = 0; q < nc; ++q) rank += (s.cand_u[q] < us) || (s.cand_u[q] == us && s.cand_i[q] < is);
    if (rank == need - 1) {
      s.thr_u = us;
      s.thr_i = is;
    }
  }
  __syncthreads();
}

// Threshold (s.thr_u, s.thr_i) of replica b over all N keys, 1 <= K <= N: 12-bit digits of u, most
// significant first, histogrammed among the keys that match the digits fixed so far, until the
// bin that holds the K-th key has at most kCap keys; those are collected and ranked exactly.
// Called by the whole workgroup.
__device__ void select_full(const InitArgs &a, int b, Select &s)
{
  const int tid = (int)threadIdx.x;
  u64 prefix = 0;
  int pbits = 0;
  int64_t need = a.K;
  bool small = a.N <= kRankAll;   // all of this is the same on every thread
  while (!small && pbits < 64) {
    const int dig = 64 - pbits < kDig ? 64 - pbits : kDig;
    __syncthreads();
    for (int q = tid; q < kBins; q += kSelBlock) s.hist[q] = 0;
    __syncthreads();
    for (int64_t i = tid; i < a.N; i += kSelBlock) {
      const u64 u = site_key(a, (int)i, b);
      if (pbits != 0 && (u >> (64 - pbits)) != prefix) continue;
      atomicAdd(&s.hist[(unsigned)((u >> (64 - pbits - dig)) & ((1ull << dig) - 1ull))], 1u);
    }
    find_bin(s, need);
    int bin = s.bin;
    if (bin < 0) {   // unreachable: need <= keys under the prefix
      bin = (1 << dig) - 1;
      if (tid == 0) atomicOr(a.err, 2);
    }
    need -= s.before;
    prefix = (prefix << dig) | (u64)bin;
    pbits += dig;
    small = s.in_bin <= (unsigned)kCap;
  }
  __syncthreads();
  if (tid == 0) s.ncand = 0;
  __syncthreads();
  for (int64_t i = tid; i < a.N; i += (int)blockDim.x) {
    const u64 u = site_key(a, (int)i, b);
    if (pbits != 0 && (u >> (64 - pbits)) != prefix) continue;
    const int slot = atomicAdd(&s.ncand, 1);
    if (slot < kCap) {
      s.cand_u[slot] = u;
      s.cand_i[slot] = (int)i;
    }
  }
  __syncthreads();
  if (tid == 0 && s.ncand > kCap) {   // more than kCap equal 64-bit keys
    atomicOr(a.err, 1);
    s.ncand = kCap;
  }
  rank_candidates(s, need);
}

// Small instances: the threshold of replica a.first + blockIdx.x.  A thread keeps the keys it drew (at most
// kKeep) from the histogram to the collection, so that every key is drawn once.  Bound by those draws with many
// replicas: 2D L = 88 x 16384 replicas, init and free 765 us when the keys were drawn again, 579 now.
constexpr int kKeep = 16;   // N < kSelBlock * kKeep
__global__ __launch_bounds__(kSelBlock) void k_init_select(InitArgs a)
{
  __shared__ Select s;
  const int b = a.first + (int)blockIdx.x;
  const int tid = (int)threadIdx.x;
  if (a.K > 0 && a.N > kRankAll) {
    u64 key[kKeep];
    for (int q = tid; q < kBins; q += kSelBlock) s.hist[q] = 0;
    if (tid == 0) s.ncand = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kKeep; ++k) {
      const int i = tid + k * kSelBlock;
      if (i >= a.N) break;
      key[k] = site_key(a, i, b);
      atomicAdd(&s.hist[(unsigned)(key[k] >> (64 - kDig))], 1u);
    }
    find_bin(s, a.K);
    const int bin = s.bin;
    if (bin >= 0 && s.in_bin <= (unsigned)kCap) {   // the same on every thread
      const int64_t need = a.K - (int64_t)s.before;
#pragma unroll
      for (int k = 0; k < kKeep; ++k) {
        const int i = tid + k * kSelBlock;
        if (i >= a.N) break;
        if ((int)(key[k] >> (64 - kDig)) != bin) continue;
        const int slot = atomicAdd(&s.ncand, 1);   // at most in_bin <= kCap of them
        s.cand_u[slot] = key[k];
        s.cand_i[slot] = i;
      }
      rank_candidates(s, need);
    } else {
      select_full(a, b, s);
    }
  } else if (a.K > 0) {
    select_full(a, b, s);
  }
  if (tid == 0) {
    a.thr_u[b] = a.K > 0 ? s.thr_u : 0;
    a.thr_i[b] = a.K > 0 ? s.thr_i : -1;
  }
}

// Small instances: a workgroup sets one word of 64 sites, wave q the replicas 8q .. 8q + 7, so
// that a site's 32 draws are not one thread's serial chain (a lattice of a few thousand sites
// has far fewer threads than the device).
constexpr int kFillBlock = 512;

template <int WPT>
__global__ __launch_bounds__(kFillBlock) void k_init_fill(InitArgs a)
{
  __shared__ u64 bits[64];
  const int word = a.first + (int)blockIdx.y;
  const int lane = (int)__lane_id();
  const int q = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int idx = (int)blockIdx.x * 64 + lane;
  unsigned mine = 0;
  if (idx < a.N) {
    const int i = element_site(a, idx);
#pragma unroll
    for (int l = 0; l < 8; l += 2) {
      const int b = word * 64 + q * 8 + l;
      const uint4 o = key_draw(a, (uint32_t)i, (uint32_t)(b >> 1));
      const u64 u0 = lo_half(o), u1 = hi_half(o);
      const u64 t0 = a.thr_u[b], t1 = a.thr_u[b + 1];
      const long long i0 = a.thr_i[b], i1 = a.thr_i[b + 1];
      mine |= (unsigned)((u0 < t0) || (u0 == t0 && (long long)i <= i0)) << l;
      mine |= (unsigned)((u1 < t1) || (u1 == t1 && (long long)i <= i1)) << (l + 1);
    }
  }
  reinterpret_cast<unsigned char *>(bits)[lane * 8 + q] = (unsigned char)mine;
  __syncthreads();
  if (q == 0 && idx < a.N) {
    const size_t at = ((size_t)(word / WPT) * (size_t)a.N + (size_t)idx) * WPT + (size_t)(word % WPT);
    a.n[at] = bits[lane];
    a.n0[at] = bits[lane];
    a.f[at] = 0;
  }
}

// Candidate list of replica b: N/16 element indices in the rows of n0 (replicas 0..31 of a word)
// or f (32..63) of its word, which hold nothing else until k_init_copy.
__device__ __forceinline__ uint32_t *candidate_list(const InitArgs &a, int b)
{
  u64 *row = ((b & 32) ? a.f : a.n0) + (size_t)(b >> 6) * (size_t)a.N;
  return reinterpret_cast<uint32_t *>(row) + (size_t)(b & 31) * (size_t)(a.N >> 4);
}

// Candidates listed and sites below the window of replica b (global counters).
__device__ __forceinline__ unsigned *listed_count(const InitArgs &a, int b) { return reinterpret_cast<unsigned *>(a.thr_u) + 2 * b; }
__device__ __forceinline__ unsigned *below_count(const InitArgs &a, int b) { return listed_count(a, b) + 1; }

// Occupation bits of the sites below the window, the candidates and the counts.  Bound by the
// Philox calls, one per site and replica pair (268 M for 3D L=128 x 256 replicas).  A thread holds
// the WPT words of one site; candidates (a few in 1000 keys) are noted in a mask and listed
// after the draws, in LDS first, so that the draws have no branches and a workgroup makes one
// global add per replica.
template <int WPT>
__global__ __launch_bounds__(kKeysBlock) void k_init_keys(InitArgs a)
{
  constexpr int RB = 64 * WPT;   // replicas of a plane
  __shared__ unsigned cnt[RB], first[RB], below[RB];
  __shared__ uint2 ent[kKeysEntries];   // element, replica of the plane | slot << 8
  __shared__ unsigned total;
  const int plane = a.first + (int)blockIdx.y;
  const int tid = (int)threadIdx.x;
  const int lane = (int)__lane_id();
  for (int q = tid; q < RB; q += kKeysBlock) cnt[q] = below[q] = 0;
  if (tid == 0) total = 0;
  __syncthreads();
  u64 *n = a.n + (size_t)plane * (size_t)a.N * WPT;
  LaneCounter lc[WPT];
  unsigned acc[WPT];
#pragma unroll
  for (int w = 0; w < WPT; ++w) {
    lc[w].clear();
    acc[w] = 0;
  }
  int words = 0;
  const int step = (int)gridDim.x * kKeysBlock;
  int64_t base = (int64_t)blockIdx.x * kKeysBlock + __builtin_amdgcn_readfirstlane(tid & ~63);
  for (; base < a.N; base += step) {
    const int64_t idx = base + lane;
    Elem<WPT> x;
#pragma unroll
    for (int w = 0; w < WPT; ++w) x.w[w] = 0;
    if (idx < a.N) {
      const int i = element_site(a, (int)idx);
#pragma unroll
      for (int w = 0; w < WPT; ++w) {
        u64 in = 0, near = 0;
        for (int q = 0; q < 64; q += 8) {
          unsigned inq = 0, nearq = 0;
#pragma unroll
          for (int l = 0; l < 8; l += 2) {
            const uint4 o = key_draw(a, (uint32_t)i, (uint32_t)(((plane * WPT + w) * 64 + q + l) >> 1));
            inq |= (unsigned)(o.y < a.lo) << l | (unsigned)(o.w < a.lo) << (l + 1);
            nearq |= (unsigned)(o.y - a.lo < a.width) << l | (unsigned)(o.w - a.lo < a.width) << (l + 1);
          }
          in |= (u64)inq << q;
          near |= (u64)nearq << q;
        }
        x.w[w] = in;
        while (near) {
          const int l = __ffsll((unsigned long long)near) - 1;
          near &= near - 1;
          const unsigned e = atomicAdd(&total, 1u);
          if (e < (unsigned)kKeysEntries) {
            ent[e] = make_uint2((unsigned)idx, (unsigned)(w * 64 + l) | atomicAdd(&cnt[w * 64 + l], 1u) << 8);
          } else {   // LDS list full: straight into the replica's list
            const int b = (plane * WPT + w) * 64 + l;
            const unsigned slot = atomicAdd(listed_count(a, b), 1u);
            if (slot < (unsigned)a.cap) candidate_list(a, b)[slot] = (uint32_t)idx;
          }
        }
      }
      st<WPT>(n, (int)idx, x);
    }
#pragma unroll
    for (int w = 0; w < WPT; ++w) lc[w].add4(x.w[w], 0, 0, 0);
    if (++words == LaneCounter::kMaxWords) {
#pragma unroll
      for (int w = 0; w < WPT; ++w) {
        count_planes(lc[w], words, acc[w]);
        lc[w].clear();
      }
      words = 0;
    }
  }
#pragma unroll
  for (int w = 0; w < WPT; ++w) {
    count_planes(lc[w], words, acc[w]);
    if (acc[w]) atomicAdd(&below[w * 64 + lane], acc[w]);
  }
  __syncthreads();
  for (int q = tid; q < RB; q += kKeysBlock) {
    if (cnt[q]) first[q] = atomicAdd(listed_count(a, plane * RB + q), cnt[q]);
    if (below[q]) atomicAdd(below_count(a, plane * RB + q), below[q]);
  }
  __syncthreads();
  const int m = (int)min(total, (unsigned)kKeysEntries);
  for (int e = tid; e < m; e += kKeysBlock) {
    const unsigned q = ent[e].y & 255u, slot = first[q] + (ent[e].y >> 8);
    if (slot < (unsigned)a.cap) candidate_list(a, plane * RB + (int)q)[slot] = ent[e].x;
  }
}

// The threshold of replica a.first + blockIdx.x among its candidates, and the bits of those at or below it.
template <int WPT>
__global__ __launch_bounds__(kSelBlock) void k_init_pick(InitArgs a)
{
  __shared__ Select s;
  const int b = a.first + (int)blockIdx.x;
  const int tid = (int)threadIdx.x;
  const int word = b >> 6;
  u64 *n = a.n + (size_t)(word / WPT) * (size_t)a.N * WPT + (size_t)(word % WPT);   // + idx * WPT
  const u64 bit = 1ull << (b & 63);
  const int64_t listed = *listed_count(a, b);
  const int64_t need = a.K - (int64_t)*below_count(a, b);   // candidates to occupy
  if (need == 0) return;   // the window holds no occupied site
  bool found = need > 0 && need <= listed && listed <= a.cap;
  const uint32_t *list = candidate_list(a, b);
  if (found) {   // the same on every thread
    // histogram of the keys' high words over the window, monotonic in the key
    for (int q = tid; q < kBins; q += kSelBlock) s.hist[q] = 0;
    if (tid == 0) s.ncand = 0;
    __syncthreads();
    for (int64_t k = tid; k < listed; k += kSelBlock) {
      const u64 u = site_key(a, element_site(a, (int)list[k]), b);
      atomicAdd(&s.hist[((u64)((uint32_t)(u >> 32) - a.lo) * a.bin_mul) >> 32], 1u);
    }
    find_bin(s, need);
    const int bin = s.bin;
    found = bin >= 0 && s.in_bin <= (unsigned)kCap;
    if (found) {
      for (int64_t k = tid; k < listed; k += kSelBlock) {
        const int idx = (int)list[k];
        const int i = element_site(a, idx);
        const u64 u = site_key(a, i, b);
        const int at = (int)(((u64)((uint32_t)(u >> 32) - a.lo) * a.bin_mul) >> 32);
        if (at < bin) {
          atomicOr(n + (size_t)idx * WPT, bit);
        } else if (at == bin) {
          const int slot = atomicAdd(&s.ncand, 1);   // at most in_bin <= kCap of them
          s.cand_u[slot] = u;
          s.cand_i[slot] = i;
          s.cand_at[slot] = idx;
        }
      }
      rank_candidates(s, need - (int64_t)s.before);
      for (int k = tid; k < s.ncand; k += kSelBlock)
        if (s.cand_u[k] < s.thr_u || (s.cand_u[k] == s.thr_u && s.cand_i[k] <= s.thr_i))
          atomicOr(n + (size_t)s.cand_at[k] * WPT, bit);
      return;
    }
  }
  // the threshold is not among the candidates: select over all keys and set every site's bit
  if (a.K > 0) select_full(a, b, s);
  for (int64_t idx = tid; idx < a.N; idx += kSelBlock) {
    const int i = element_site(a, (int)idx);
    const u64 u = site_key(a, i, b);
    const bool in = a.K > 0 && (u < s.thr_u || (u == s.thr_u && i <= s.thr_i));
    if (in) atomicOr(n + (size_t)idx * WPT, bit);
    else atomicAnd(n + (size_t)idx * WPT, ~bit);
  }
}

// n0 = n, f = 0.
__global__ __launch_bounds__(256) void k_init_copy(const u64 *n, u64 *n0, u64 *f, size_t words)
{
  for (size_t q = (size_t)blockIdx.x * 256 + threadIdx.x; q < words; q += (size_t)gridDim.x * 256) {
    n0[q] = n[q];
    f[q] = 0;
  }
}

__global__ void k_init_clear(unsigned *counters, int n, int *err)
{
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < n) counters[i] = 0;
  if (i == 0) *err = 0;
}

// Smallest N of the window selection: its lists (N/16 sites per replica) hold the widest window.
constexpr int kWindowMinN = 1 << 14;
static_assert(kWindowMinN <= kSelBlock * kKeep, "k_init_select keeps every key");

// A grid holds fewer than 2^32 threads in x and 2^16 workgroups in y, and a launch beyond that runs
// with the number of them cut off, without an error; so larger ones are made in parts.
template <typename Launch>
void in_parts(InitArgs a, int total, int part, Launch launch)
{
  for (a.first = 0; a.first < total; a.first += part) launch(a, (unsigned)std::min(part, total - a.first));
}
constexpr int kGridX = 1 << 21, kGridY = 1 << 15;   // at most 1024 threads a workgroup

}  // namespace

hipError_t launch_init(const InitArgs &args, int R, int wpt, hipStream_t s)
{
  InitArgs a = args;
  const int words = R / 64;
  hipLaunchKernelGGL(k_init_clear, dim3((unsigned)((2 * (size_t)R + 255) / 256)), dim3(256), 0, s, reinterpret_cast<unsigned *>(a.thr_u),
                     2 * R, a.err);
  if (a.N < kWindowMinN) {
    // (ranking needs a thread per site: 2D L = 4 x 262144 replicas 2740 us with 1024 of them, 980 with 128)
    const int threads = a.N <= kRankAll ? kRankAll : kSelBlock;
    in_parts(a, R, kGridX, [&](const InitArgs &p, unsigned n) { hipLaunchKernelGGL(k_init_select, dim3(n), dim3((unsigned)threads), 0, s, p); });
    in_parts(a, words, kGridY, [&](const InitArgs &p, unsigned n) {
      const dim3 grid((unsigned)((a.N + 63) / 64), n);
      if (wpt == 2) hipLaunchKernelGGL((k_init_fill<2>), grid, dim3(kFillBlock), 0, s, p);
      else hipLaunchKernelGGL((k_init_fill<1>), grid, dim3(kFillBlock), 0, s, p);
    });
    return hipGetLastError();
  }
  // Window of 4.5 standard deviations of the K-th key and 12 sites to either side (the second
  // term covers densities where the count is not normal): the threshold of about one replica
  // in 10^5 lies outside it.
  const double N = (double)a.N, p = (double)a.K / N;
  const double half = (4.5 * std::sqrt(p * (1.0 - p) / N) + 12.0 / N) * 4294967296.0;
  const double lo = std::min(std::max(p * 4294967296.0 - half, 0.0), 4294967295.0);
  const double hi = std::min(std::max(p * 4294967296.0 + half, lo + 1.0), 4294967296.0);
  a.lo = (uint32_t)lo;
  a.width = (uint32_t)(std::ceil(hi) - (double)a.lo);
  a.bin_mul = ((u64)kBins << 32) / a.width;
  a.cap = a.N >> 4;
  // 2048 workgroups fill the device (8 waves a SIMD)
  const unsigned bx = (unsigned)std::min((a.N + kKeysBlock - 1) / kKeysBlock, std::max(1, 2048 / a.planes));
  in_parts(a, a.planes, kGridY, [&](const InitArgs &p, unsigned n) {
    if (wpt == 2) hipLaunchKernelGGL((k_init_keys<2>), dim3(bx, n), dim3(kKeysBlock), 0, s, p);
    else hipLaunchKernelGGL((k_init_keys<1>), dim3(bx, n), dim3(kKeysBlock), 0, s, p);
  });
  in_parts(a, R, kGridX, [&](const InitArgs &p, unsigned n) {
    if (wpt == 2) hipLaunchKernelGGL((k_init_pick<2>), dim3(n), dim3(kSelBlock), 0, s, p);
    else hipLaunchKernelGGL((k_init_pick<1>), dim3(n), dim3(kSelBlock), 0, s, p);
  });
  const size_t total = (size_t)a.N * (size_t)words;
  hipLaunchKernelGGL(k_init_copy, dim3((unsigned)std::min<size_t>((total + 255) / 256, 4096)), dim3(256), 0, s, a.n, a.n0, a.f, total);
  return hipGetLastError();
}

}  // namespace ka
