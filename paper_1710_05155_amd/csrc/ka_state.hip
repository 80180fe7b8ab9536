// ka_state.hip -- state words between the device layout and the canonical one (gfx950).
//
// The canonical layout is [W][N] words, word w of canonical site i at w N + i; the device layout is
// described in ka_internal.h.  Both kernels move the canonical words [t0, t1) of one array to or from
// a staging buffer, from which they are copied whole: the reordering took the host 5 to 10 ns a
// word, and here it streams at memory speed under the copy over the bus.
#include <algorithm>

#include "ka_device.h"

namespace ka {
namespace {

using namespace dev;

// Place in the device array and canonical index of this thread's word: lattices by canonical index,
// general graphs by device index (their table goes that way).
struct Place {
  size_t at;
  int64_t t;
};

__device__ __forceinline__ Place state_place(const StateArgs &a, int64_t k)
{
  const int w = (int)(k / a.N), j = (int)(k - (int64_t)w * a.N);
  int el, i;
  if (a.site_of) {
    el = j;
    i = a.site_of[j];
  } else {
    i = j;
    int rest = i, sub = 0, pos = 0, sm = 1, pm = 1;
    for (int d = 0; d < a.g.d; ++d) {
      const int up = rest / a.g.L, x = rest - up * a.g.L;
      rest = up;
      sub += (x & 3) * sm;
      pos += (x >> 2) * pm;
      sm *= 4;
      pm *= a.g.Q;
    }
    el = sub * a.g.P + pos;
  }
  return {((size_t)(w / a.wpt) * (size_t)a.N + (size_t)el) * (size_t)a.wpt + (size_t)(w % a.wpt), (int64_t)w * a.N + i};
}

template <bool OUT>
__global__ __launch_bounds__(256) void k_state(StateArgs a)
{
  // general graphs: every word of the sites' rows that the range touches, to find those inside it
  const int64_t first = a.site_of ? a.t0 / a.N * a.N : a.t0;
  const int64_t last = a.site_of ? (a.t1 + a.N - 1) / a.N * a.N : a.t1;
  for (int64_t k = first + (int64_t)blockIdx.x * 256 + threadIdx.x; k < last; k += (int64_t)gridDim.x * 256) {
    const Place p = state_place(a, k);
    if (p.t < a.t0 || p.t >= a.t1) continue;
    if (OUT) a.staging[p.t - a.t0] = a.state[p.at];
    else a.state[p.at] = a.staging[p.t - a.t0];
  }
}

}  // namespace

hipError_t launch_state(const StateArgs &a, bool out, hipStream_t s)
{
  if (a.t0 < 0 || a.t1 <= a.t0 || a.N < 1) return hipErrorInvalidValue;
  const int64_t words = (a.t1 - a.t0) + (a.site_of ? 2 * (int64_t)a.N : 0);
  const dim3 grid((unsigned)std::min<int64_t>((words + 255) / 256, 8192));
  if (out) hipLaunchKernelGGL((k_state<true>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_state<false>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace ka
