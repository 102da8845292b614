// Global operators (Table 2): operators that read every pixel of an image
// and produce a few values.  Each kernel streams the image once in 16-byte
// chunks (the chunks of all rows dealt out over all threads, several loaded
// together per thread so that every lane has independent loads in flight: eight
// in the histogram, four in the others) and reduces inside the wave with lane
// exchanges.  Work-groups combine with one global atomic per group (per bin for
// the histogram) into a result that a small kernel in the same stream has
// initialised; the counts of the extremes go to a key per group, which a last
// kernel merges.  Kernels only, so the sequence can be captured into a HIP graph.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "dev_reduce.hpp"
#include "gen_abi.h"
#include "global.h"
#include "hvx_desc.h"

namespace hvx {

constexpr int kGThreads = 256;

// Launch shapes.  The histogram's groups each add up to 256 counts to the
// result, so there are few of them and each lane loads eight chunks at a time
// (3840x2160: 253 groups 9.9 us, 506 of four chunks 13.8, 2025 of one 41); on
// large images two groups a CU feed the LDS (four where the bins are
// computed).  Min/max and the sums combine through two words each:
// same-address atomics serialise, so those kernels reduce a whole 1024-thread
// group in LDS first and launch one group per CU.
constexpr int kRThreads = 1024;
constexpr int kRGroups = 256;
static_assert(kRGroups <= kMMSubKeys && kMMSubKeys <= kRThreads, "one counting key per group, and a thread for each");

// Work-groups of NT threads for an image read in steps of K chunks a thread.
static int global_grid(const GlobalImg& im, int per, int nt, int k, int cap) {
  const long long chunks = (long long)((im.w + per - 1) / per) * im.h, step = (long long)nt * k;
  const long long g = (chunks + step - 1) / step;
  return (int)(g < cap ? g : cap);
}

// Calls f(chunks, valid elements) for the 16-byte chunks of the image (PER
// elements each) that this thread of an NT-thread group reads, K of them
// loaded together; chunks past the image's end have no valid elements.  The
// rows' chunks are taken as one sequence, so images of any width keep every
// lane busy (dealt out by rows, 330x15000 pixels took 21.7 us for min / max,
// 8.5 so), and f is called by whole waves.  Only the last step tests its
// loads, and images of whole chunks have no element counts: min / max of
// 268 MB 44 -> 41 us (6.5 TB/s); with the tests in every step it took 52.
template <int PER, int NT, int K, class F>
__device__ __forceinline__ void stream_image(const GlobalImg& im, F&& f) {
  const uint32_t h = (uint32_t)im.h, chunks = (uint32_t)(im.w + PER - 1) / PER, total = chunks * h;
  const uint32_t stride = gridDim.x * NT;  // chunks from one load of a thread to its next
  const uint32_t dy = stride / chunks, dc = stride - dy * chunks;
  const uint32_t first = blockIdx.x * NT + threadIdx.x;
  uint32_t c = first % chunks;
  // the chunk's address, and what a step adds to it
  const uint8_t* p = im.base + (int64_t)(first / chunks) * im.pitch + 16 * (int64_t)c;
  const int64_t dp = (int64_t)dy * im.pitch + 16 * (int64_t)dc, wrap = im.pitch - 16 * (int64_t)chunks;
  auto advance = [&]() {
    c += dc;
    const bool over = c >= chunks;
    p += dp + (over ? wrap : 0);
    c -= over ? chunks : 0;
  };
  uint32_t i = blockIdx.x * NT;
  uint4 q[K];
  int n[K];
  // steps in which every load of the group lies inside the image
  if (im.w % PER == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) n[k] = PER;
    for (; i + (K - 1) * stride + NT <= total; i += K * stride) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        q[k] = *(const uint4*)p;
        advance();
      }
      f(q, n);
    }
  } else {
    for (; i + (K - 1) * stride + NT <= total; i += K * stride) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        n[k] = min(PER, im.w - (int)(PER * c));
        q[k] = *(const uint4*)p;
        advance();
      }
      f(q, n);
    }
  }
  if (i < total) {  // the last step
#pragma unroll
    for (int k = 0; k < K; ++k) {
      // past the end: the first chunk again, with no valid element
      const bool in = i + k * stride + threadIdx.x < total;
      n[k] = in ? min(PER, im.w - (int)(PER * c)) : 0;
      q[k] = *(const uint4*)(in ? p : im.base);
      advance();
    }
    f(q, n);
  }
}

// the same, f(chunk, valid elements) for each chunk that holds any
template <int PER, int NT, int K, class F>
__device__ __forceinline__ void stream_each(const GlobalImg& im, F&& f) {
  stream_image<PER, NT, K>(im, [&](const uint4 (&q)[K], const int (&n)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (n[k] > 0) f(q[k], n[k]);
  });
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, int n, uint32_t a, uint32_t b) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = i == 0 ? a : b;
}

// ---- histogram of a U8 image ------------------------------------------------
// Bin of value v: (v - offset) * num_bins / range for offset <= v < offset +
// range, none otherwise.  With y = (v - offset) * num_bins * 256 (mod 2^32),
// formed as one 24-bit multiply-add v * B + D, the bin is the high word of
// y * m for m = ceil(2^24 / range) (0 for range 1): y and m fit 24 bits, so
// both products run on the full-rate 24-bit multiplier, and the quotient is
// exact because (v - offset) * num_bins * (m * range - 2^24) < 2^16 * 2^8.
// v lies in the interval exactly when y < R = range * num_bins * 256 (below
// the offset y wraps past 2^32 - 2^24).  The 256-bin histogram over [0, 256)
// takes the byte itself.
//
// A group counts into one LDS histogram held as 16 interleaved copies (copy c
// of bin b at word b * 16 + c, lane l adding to copy l mod 16): at most four
// lanes of a wave share a counter, whatever the data, and the lanes of a
// quarter of a wave add to different banks.  Pixels outside the interval, and
// the bytes past a row's end, add zero.
// What bounds it: LDS additions, one a pixel.  268 MB, a smooth image 51 us
// (5.3 TB/s), uniform noise 47 us; with a histogram per wave in four copies,
// where up to sixteen lanes that drew one bin waited for each other, 101 and
// 63 us.  (A byte counter per lane and bin, conflict-free but summed every
// 192 pixels and 64 KB a group, took 84 and 80 us.)
struct HistBins {
  uint32_t B, D, R, m;
};

constexpr int kHistCopies = 16, kHistLoads = 8;

template <bool kIdentity>
__global__ __launch_bounds__(kGThreads) void k_histogram(GlobalImg im, int num_bins, HistBins hb,
                                                         uint32_t* __restrict__ counts) {
  constexpr int K = kHistLoads;
  __shared__ __attribute__((aligned(16))) uint32_t sub[256 * kHistCopies];
  const int t = threadIdx.x;
  for (int k = t; k < 256 * kHistCopies / 4; k += kGThreads) ((uint4*)sub)[k] = uint4{0, 0, 0, 0};
  __syncthreads();
  uint32_t* mine = sub + (t & (kHistCopies - 1));
  const uint32_t B = hb.B & 0xFFFFFFu, m = hb.m & 0xFFFFFFu;
  stream_image<16, kGThreads, K>(im, [&](const uint4 (&q)[K], const int (&n)[K]) {
#pragma unroll
    for (int r = 0; r < K; ++r) {
      const uint32_t wd[4] = {q[r].x, q[r].y, q[r].z, q[r].w};
      auto add = [&](int k, bool in) {
        const uint32_t v = (wd[k >> 2] >> (8 * (k & 3))) & 0xFFu;
        uint32_t b = v;
        if constexpr (!kIdentity) {
          const uint32_t y = v * B + hb.D;
          b = (uint32_t)(((uint64_t)(y & 0xFFFFFFu) * m) >> 32) & 0xFFu;
          in = in && y < hb.R;
        }
        atomicAdd(&mine[b * kHistCopies], in ? 1u : 0u);
      };
      if (__all(n[r] == 16)) {
#pragma unroll
        for (int k = 0; k < 16; ++k) add(k, true);
      } else if (n[r] > 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) add(k, k < n[r]);
      }
    }
  });
  __syncthreads();
  for (int b = t; b < num_bins; b += kGThreads) {
    const uint4* p = (const uint4*)(sub + b * kHistCopies);
    uint32_t s = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies / 4; ++c) {
      const uint4 q = p[(c + b) & (kHistCopies / 4 - 1)];
      s += q.x + q.y + q.z + q.w;
    }
    if (s) atomicAdd(&counts[b], s);
  }
}

hipError_t launch_histogram(const GlobalImg& im, int num_bins, int offset, int range, uint32_t* counts,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3((num_bins + 255) / 256), dim3(256), 0, s, counts, num_bins, 0u, 0u);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || im.w <= 0 || im.h <= 0) return e;
  HistBins hb;
  hb.B = (uint32_t)num_bins << 8;
  hb.D = 0u - (uint32_t)offset * hb.B;
  hb.R = (uint32_t)range * hb.B;
  hb.m = range == 1 ? 0u : (uint32_t)(((1u << 24) + (uint32_t)range - 1) / (uint32_t)range);
  const bool identity = offset == 0 && range == 256 && num_bins == 256;
  // full steps, but at least 32 groups while a thread has a chunk (10 bins of
  // 440x559 8.8 -> 7.0 us)
  const int few = global_grid(im, 16, kGThreads, 1, 32);
  const dim3 grid(std::max(few, global_grid(im, 16, kGThreads, kHistLoads, identity ? 512 : 1024)));
  if (identity)
    hipLaunchKernelGGL(k_histogram<true>, grid, dim3(kGThreads), 0, s, im, num_bins, hb, counts);
  else
    hipLaunchKernelGGL(k_histogram<false>, grid, dim3(kGThreads), 0, s, im, num_bins, hb, counts);
  return hipGetLastError();
}

// ---- histogram equalisation of a U8 image ----------------------------------------
// From the 256-bin histogram: cdf(v) by a scan of the group, cdf_min the cdf at the
// first nonzero bin, and lut[v] = round((cdf(v) - cdf_min) * 255 / (N -
// cdf_min)) clamped to 0..255, or v itself for an image of one value.
// (256 threads; returns the entry of value threadIdx.x)
__device__ __forceinline__ uint8_t eq_entry(const uint32_t* __restrict__ hist, long long n, uint32_t (&sums)[2][4]) {
  // the counts before and at t (fewer than 2^31 pixels): a scan by lane
  // exchange in each of the four waves, then the waves' sums; the first
  // nonzero count is the smallest nonzero cumulative one
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t h = hist[t];
  uint32_t cdf = h;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t add = __shfl_up(cdf, d);
    cdf += lane >= d ? add : 0u;
  }
  const unsigned long long any = __ballot(h != 0);
  const uint32_t first = __shfl(h, any ? __builtin_ctzll(any) : 0);
  if (lane == 63) {
    sums[0][wave] = cdf;
    sums[1][wave] = first;
  }
  __syncthreads();
  uint32_t lowest = 0;
#pragma unroll
  for (int w = 3; w >= 0; --w) {
    cdf += w < wave ? sums[0][w] : 0u;
    lowest = sums[1][w] ? sums[1][w] : lowest;
  }
  const long long cmin = (long long)lowest;
  const long long den = n - cmin;
  int v = t;
  if (den > 0) {
    const long long num = ((long long)cdf - cmin) * 255;
    long long r = num >= 0 ? (2 * num + den) / (2 * den) : 0;
    v = (int)(r > 255 ? 255 : r);
  }
  return (uint8_t)v;
}

__global__ __launch_bounds__(256) void k_eq_lut(const uint32_t* __restrict__ hist, uint8_t* __restrict__ lut,
                                                 long long n) {
  __shared__ uint32_t sums[2][4];
  lut[threadIdx.x] = eq_entry(hist, n, sums);
}

// out = the mapping of in, 16 bytes per lane per step; rows strided over the
// grid.  A thread reads and writes the same chunk, so in place is allowed.
// Every group forms the mapping from the histogram itself (about a
// microsecond, behind the other groups' streaming; as a kernel of its own it
// held the stream for 5 us); the first also writes it to `lut`.  With the scan
// by lane exchange and one barrier instead of sixteen, 440x559 takes 3.4 us
// (6.2) and 1500x1100 4.1 (7.7); an equalize call of 3840x2160 19.4 -> 14.7.
__global__ __launch_bounds__(kGThreads) void k_apply_lut(GlobalImg im, const uint32_t* __restrict__ hist, uint8_t* lut,
                                                         uint8_t* out, int64_t out_pitch) {
  __shared__ uint8_t tab[256];
  __shared__ uint32_t sums[2][4];
  const uint8_t entry = eq_entry(hist, (long long)im.w * im.h, sums);
  tab[threadIdx.x] = entry;
  if (blockIdx.x == 0) lut[threadIdx.x] = entry;
  __syncthreads();
  const int chunks = (im.w + 15) >> 4;
  for (int y = blockIdx.x; y < im.h; y += gridDim.x) {
    const uint8_t* row = im.base + (size_t)y * im.pitch;
    uint8_t* orow = out + (size_t)y * out_pitch;
    for (int c = threadIdx.x; c < chunks; c += kGThreads) {
      const uint4 q = *(const uint4*)(row + 16 * c);
      const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
      uint32_t o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        o[j] = (uint32_t)tab[wd[j] & 0xFF] | (uint32_t)tab[(wd[j] >> 8) & 0xFF] << 8 |
               (uint32_t)tab[(wd[j] >> 16) & 0xFF] << 16 | (uint32_t)tab[wd[j] >> 24] << 24;
      }
      // streamed past the caches: nothing here reads the output again
      typedef unsigned int u4v __attribute__((ext_vector_type(4)));
      __builtin_nontemporal_store(u4v{o[0], o[1], o[2], o[3]}, (u4v*)(orow + 16 * c));
    }
  }
}

hipError_t launch_equalize_mapping(const GlobalImg& im, void* workspace, hipStream_t s) {
  static_assert(kEqHistBytes <= (int)kEqualizeScratchBytes, "the fixed workspace holds the counts and the mapping");
  uint32_t* hist = (uint32_t*)workspace;
  uint8_t* lut = (uint8_t*)workspace + 256 * 4;
  hipError_t e = launch_histogram(im, 256, 0, 256, hist, s);
  if (e != hipSuccess || im.w <= 0 || im.h <= 0) return e;
  hipLaunchKernelGGL(k_eq_lut, dim3(1), dim3(256), 0, s, (const uint32_t*)hist, lut, (long long)im.w * im.h);
  return hipGetLastError();
}

hipError_t launch_equalize_hist(const GlobalImg& im, uint8_t* out, int64_t out_pitch, void* workspace,
                                hipStream_t s) {
  uint32_t* hist = (uint32_t*)workspace;
  uint8_t* lut = (uint8_t*)workspace + 256 * 4;
  hipError_t e = launch_histogram(im, 256, 0, 256, hist, s);
  if (e != hipSuccess || im.w <= 0 || im.h <= 0) return e;
  hipLaunchKernelGGL(k_apply_lut, dim3(im.h < 2048 ? im.h : 2048), dim3(kGThreads), 0, s, im, (const uint32_t*)hist, lut,
                     out, out_pitch);
  return hipGetLastError();
}

// ---- EqualizeHist without a caller workspace ------------------------------------
// For callers that cannot allocate: the histogram and the mapping live in a
// fixed device array, `scratch`, one copy per GPU, held until the process
// ends.  In host code the array's name is only a host-side stand-in, so it
// is never passed to a kernel: its device address is resolved once per
// device (with that device current) and kept.  Every call on a GPU shares
// that GPU's copy; the histogram part is cleared by a kernel at the start
// of each call, and calls that overlap on one GPU race.
static __device__ __align__(256) uint8_t scratch[kEqualizeScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];
}  // namespace

hipError_t equalize_scratch(int device, void** ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> l(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = p;
  }
  *ptr = g_scratch_ptr[device];
  return hipSuccess;
}

// ---- smallest and largest element of a U8 or S16 image ------------------------
template <bool S16>
__global__ __launch_bounds__(kRThreads) void k_min_max(GlobalImg im, int32_t* __restrict__ out) {
  constexpr int kPer = S16 ? 8 : 16;  // elements per 16-byte chunk
  __shared__ int part[2][kRThreads / 64];
  int mn = INT_MAX, mx = INT_MIN;
  const int t = threadIdx.x;
  stream_each<kPer, kRThreads, 4>(im, [&](const uint4& q, int n) {
    const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int v = S16 ? (int)(int16_t)(wd[k >> 1] >> (16 * (k & 1))) : (int)((wd[k >> 2] >> (8 * (k & 3))) & 0xFF);
      if (k < n) {
        mn = min(mn, v);
        mx = max(mx, v);
      }
    }
  });
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mn = min(mn, __shfl_xor(mn, off));
    mx = max(mx, __shfl_xor(mx, off));
  }
  if ((t & 63) == 0) {
    part[0][t >> 6] = mn;
    part[1][t >> 6] = mx;
  }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < kRThreads / 64; ++w) {
      mn = min(mn, part[0][w]);
      mx = max(mx, part[1][w]);
    }
    // the result only moves one way: a group that cannot improve it skips
    // the atomic (a stale read only costs an unneeded atomic)
    if (mn < __atomic_load_n(&out[0], __ATOMIC_RELAXED)) atomicMin(&out[0], mn);
    if (mx > __atomic_load_n(&out[1], __ATOMIC_RELAXED)) atomicMax(&out[1], mx);
  }
}

// Number of elements of the 32-bit word w equal to the element value whose
// copies fill `splat` (SWAR: an element of x = w ^ splat is zero exactly
// where w matches; adding 0x7F.. to its low bits sets its top bit unless the
// element is zero, and no carry crosses an element), added to acc.
template <bool S16>
__device__ __forceinline__ uint32_t count_eq(uint32_t w, uint32_t splat, uint32_t acc) {
  const uint32_t lo = S16 ? 0x7FFF7FFFu : 0x7F7F7F7Fu, hi = S16 ? 0x80008000u : 0x80808080u;
  const uint32_t x = w ^ splat;
  const uint32_t y = ((x & lo) + lo) | x;
  return acc + (uint32_t)__popc(~y & hi);
}

// One pass for the smallest and the largest value and how many pixels take
// each.  Every lane keeps a running (value, count) pair per extreme: for each
// 16-byte chunk it takes the chunk's extremes, restarts a count when the
// value improves, and adds the chunk's matches counted word-wise.  The pairs
// are merged across the wave and the group, and stored as the group's own
// 64-bit key of each extreme (at most kMMSubKeys groups run; the keys no group
// owns are set neutral, so nothing is initialised before).
template <bool S16>
__global__ __launch_bounds__(kRThreads) void k_min_max_count(GlobalImg im, unsigned long long* __restrict__ keys) {
  constexpr int kPer = S16 ? 8 : 16;
  __shared__ int part[4][kRThreads / 64];
  int mn = S16 ? 32767 : 255, mx = S16 ? -32768 : 0;
  uint32_t cmn = 0, cmx = 0;
  const int t = threadIdx.x;
  stream_each<kPer, kRThreads, 4>(im, [&](const uint4& q, int n) {
    const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
    if (n == kPer) {
      int a = S16 ? 32767 : 255, b = S16 ? -32768 : 0;
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int v = S16 ? (int)(int16_t)(wd[k >> 1] >> (16 * (k & 1))) : (int)((wd[k >> 2] >> (8 * (k & 3))) & 0xFF);
        a = min(a, v);
        b = max(b, v);
      }
      cmn = a < mn ? 0u : cmn;
      cmx = b > mx ? 0u : cmx;
      mn = min(mn, a);
      mx = max(mx, b);
      const uint32_t sl = S16 ? ((uint32_t)mn & 0xFFFFu) * 0x10001u : (uint32_t)mn * 0x01010101u;
      const uint32_t sh = S16 ? ((uint32_t)mx & 0xFFFFu) * 0x10001u : (uint32_t)mx * 0x01010101u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        cmn = count_eq<S16>(wd[j], sl, cmn);
        cmx = count_eq<S16>(wd[j], sh, cmx);
      }
    } else {  // the last chunk of a row: element by element
      for (int k = 0; k < n; ++k) {
        const int v = S16 ? (int)(int16_t)(wd[k >> 1] >> (16 * (k & 1))) : (int)((wd[k >> 2] >> (8 * (k & 3))) & 0xFF);
        cmn = v < mn ? 1u : cmn + (v == mn ? 1u : 0u);
        cmx = v > mx ? 1u : cmx + (v == mx ? 1u : 0u);
        mn = min(mn, v);
        mx = max(mx, v);
      }
    }
  });
  wave_merge_extremes(mn, cmn, mx, cmx);
  if ((t & 63) == 0) {
    part[0][t >> 6] = mn;
    part[1][t >> 6] = (int)cmn;
    part[2][t >> 6] = mx;
    part[3][t >> 6] = (int)cmx;
  }
  __syncthreads();
  if (t == 0) {
    unsigned long long kmin = kMinKeyInit, kmax = kMaxKeyInit;
    for (int w = 0; w < kRThreads / 64; ++w) {
      kmin = mm_merge(kmin, mm_key(part[0][w], (uint32_t)part[1][w]), true);
      kmax = mm_merge(kmax, mm_key(part[2][w], (uint32_t)part[3][w]), false);
    }
    keys[blockIdx.x] = kmin;
    keys[kMMSubKeys + blockIdx.x] = kmax;
  }
  // the keys that no group owns, by a thread each (by thread 0 alone they
  // made a call of 64x64 take 17.0 us on the device instead of 6.7)
  if (blockIdx.x == 0 && t < kMMSubKeys && t >= (int)gridDim.x) {
    keys[t] = kMinKeyInit;
    keys[kMMSubKeys + t] = kMaxKeyInit;
  }
}

// The sub-keys merged into {min, max, count of min, count of max} at the
// front of the result.
// (One wave: each lane merges every 64th key, then the lanes merge by
// exchange.)
__global__ __launch_bounds__(64) void k_unpack_keys(int32_t* __restrict__ mm) {
  const unsigned long long* k = (const unsigned long long*)((uint8_t*)mm + kMMKeyOffset);
  const int lane = threadIdx.x;
  unsigned long long kmin = kMinKeyInit, kmax = kMaxKeyInit;
  for (int i = lane; i < kMMSubKeys; i += 64) {
    kmin = mm_merge(kmin, k[i], true);
    kmax = mm_merge(kmax, k[kMMSubKeys + i], false);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    kmin = mm_merge(kmin, __shfl_xor(kmin, off), true);
    kmax = mm_merge(kmax, __shfl_xor(kmax, off), false);
  }
  if (lane == 0) {
    mm[0] = mm_value(kmin);
    mm[1] = mm_value(kmax);
    mm[2] = (int32_t)(uint32_t)kmin;
    mm[3] = (int32_t)(uint32_t)kmax;
  }
}

__global__ __launch_bounds__(256) void k_init_keys(int32_t* __restrict__ mm) {
  unsigned long long* k = (unsigned long long*)((uint8_t*)mm + kMMKeyOffset);
  for (int i = threadIdx.x; i < 2 * kMMSubKeys; i += blockDim.x) k[i] = i < kMMSubKeys ? kMinKeyInit : kMaxKeyInit;
}

hipError_t launch_min_max_count(const GlobalImg& im, int32_t* result, hipStream_t s) {
  unsigned long long* keys = (unsigned long long*)((uint8_t*)result + kMMKeyOffset);
  hipError_t e = hipSuccess;
  if (im.w <= 0 || im.h <= 0) {
    hipLaunchKernelGGL(k_init_keys, dim3(1), dim3(256), 0, s, result);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else {
    // every group has a key of its own, so a small image takes as many as it has
    // chunks for: a call of 440x559 10.8 us in 16 groups of one chunk a thread,
    // 17.9 in 4 of four (min / max and the sums, whose groups meet in atomics,
    // are faster in few: 3840x2160 8.5 against 9.9 and 10.0 against 13.2)
    const dim3 grid(global_grid(im, im.bpp == 2 ? 8 : 16, kRThreads, 1, kRGroups));
    if (im.bpp == 2) hipLaunchKernelGGL(k_min_max_count<true>, grid, dim3(kRThreads), 0, s, im, keys);
    else hipLaunchKernelGGL(k_min_max_count<false>, grid, dim3(kRThreads), 0, s, im, keys);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_unpack_keys, dim3(1), dim3(64), 0, s, result);
  return hipGetLastError();
}

// MinMaxLoc: the (x, y) of pixels equal to mm[0] (into lmin) and to mm[1]
// (into lmax), two words per location, at most `cap` of each list, in no
// particular order; mm[4], mm[5] count the reserved slots (the exact counts
// come from k_min_max_count).  One 1024-thread group per CU streams K rows a
// grid apart per step, one 16-byte chunk per lane and row.  Each lane marks
// its matches, the counts are scanned across the wave and summed over the
// group in LDS, and one thread reserves the group's slots of each list with
// a single atomic; then every lane writes its entries.  Once both lists are
// full the groups stop (thread 0 reads the counters and the decision goes
// through LDS, so the whole group leaves together).
template <bool S16>
__global__ __launch_bounds__(kRThreads) void k_extreme_locs(GlobalImg im, int32_t* __restrict__ mm,
                                                            uint32_t* __restrict__ lmin, uint32_t* __restrict__ lmax,
                                                            uint32_t cap) {
  constexpr int kPer = S16 ? 8 : 16, K = 4, NW = kRThreads / 64;
  __shared__ uint32_t wtot[2][NW];  // wave totals, then their exclusive prefix
  __shared__ uint32_t gbase[2];     // the group's first slot of each list (cap: none)
  __shared__ int stop;
  const int lo = mm[0], hi = mm[1];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int chunks = (im.w + kPer - 1) / kPer;
  const int G = gridDim.x;
  for (int y = blockIdx.x; y < im.h; y += K * G) {
    if (t == 0)
      stop = (uint32_t)__atomic_load_n(&mm[4], __ATOMIC_RELAXED) >= cap &&
             (uint32_t)__atomic_load_n(&mm[5], __ATOMIC_RELAXED) >= cap;
    __syncthreads();
    if (stop) return;
    for (int cb = 0; cb < chunks; cb += kRThreads) {
      const int c = cb + t;
      uint32_t m[2][K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        m[0][k] = m[1][k] = 0;
        const int yy = y + k * G;
        if (c < chunks && yy < im.h) {
          const uint4 q = *(const uint4*)(im.base + (size_t)yy * im.pitch + 16 * c);
          const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
          const int n = min(kPer, im.w - kPer * c);
#pragma unroll
          for (int e = 0; e < kPer; ++e) {
            const int v = S16 ? (int)(int16_t)(wd[e >> 1] >> (16 * (e & 1))) : (int)((wd[e >> 2] >> (8 * (e & 3))) & 0xFF);
            m[0][k] |= (e < n && v == lo) ? 1u << e : 0u;
            m[1][k] |= (e < n && v == hi) ? 1u << e : 0u;
          }
        }
      }
      uint32_t cnt[2], inc[2];
#pragma unroll
      for (int l = 0; l < 2; ++l) {
        cnt[l] = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) cnt[l] += (uint32_t)__popc(m[l][k]);
        inc[l] = cnt[l];  // inclusive scan across the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t u = (uint32_t)__shfl_up((int)inc[l], off);
          if (lane >= off) inc[l] += u;
        }
        if (lane == 63) wtot[l][wv] = inc[l];
      }
      __syncthreads();
      if (t < 2) {  // exclusive prefix over the waves, one reservation per list
        uint32_t run = 0;
        for (int w = 0; w < NW; ++w) {
          const uint32_t x = wtot[t][w];
          wtot[t][w] = run;
          run += x;
        }
        uint32_t base = cap;
        if (run && (uint32_t)__atomic_load_n(&mm[4 + t], __ATOMIC_RELAXED) < cap)
          base = (uint32_t)atomicAdd(&mm[4 + t], (int)run);
        gbase[t] = base;
      }
      __syncthreads();
#pragma unroll
      for (int l = 0; l < 2; ++l) {
        uint32_t i = gbase[l] + wtot[l][wv] + inc[l] - cnt[l];
        if (gbase[l] >= cap || i >= cap) continue;
        uint32_t* out = l ? lmax : lmin;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          uint32_t mk = m[l][k];
          while (mk && i < cap) {
            const int e = __ffs(mk) - 1;
            mk &= mk - 1;
            out[2 * i] = (uint32_t)(kPer * c + e);
            out[2 * i + 1] = (uint32_t)(y + k * G);
            ++i;
          }
        }
      }
      __syncthreads();  // wtot and gbase are rewritten by the next step
    }
  }
}

hipError_t launch_extreme_locs(const GlobalImg& im, int32_t* result, uint32_t* lmin, uint32_t* lmax, uint32_t cap,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, (uint32_t*)result + 4, 2, 0u, 0u);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || im.w <= 0 || im.h <= 0 || cap == 0) return e;
  const int steps = (im.h + 3) / 4;  // four rows a step
  const dim3 grid(steps < kRGroups ? steps : kRGroups);
  if (im.bpp == 2) hipLaunchKernelGGL(k_extreme_locs<true>, grid, dim3(kRThreads), 0, s, im, result, lmin, lmax, cap);
  else hipLaunchKernelGGL(k_extreme_locs<false>, grid, dim3(kRThreads), 0, s, im, result, lmin, lmax, cap);
  return hipGetLastError();
}

hipError_t launch_min_max_loc(const GlobalImg& im, int32_t* result, uint32_t* lmin, uint32_t* lmax, uint32_t cap,
                              hipStream_t s) {
  hipError_t e = launch_min_max_count(im, result, s);
  if (e != hipSuccess) return e;
  return launch_extreme_locs(im, result, lmin, lmax, cap, s);
}

// Slot counters of the location lists clamped to the capacity: the number of
// locations each list holds.
__global__ void k_clamp_slots(int32_t* __restrict__ mm, uint32_t cap) {
  if (threadIdx.x < 2) {
    const uint32_t v = (uint32_t)mm[4 + threadIdx.x];
    mm[4 + threadIdx.x] = (int32_t)(v < cap ? v : cap);
  }
}

hipError_t launch_clamp_slots(int32_t* result, uint32_t cap, hipStream_t s) {
  hipLaunchKernelGGL(k_clamp_slots, dim3(1), dim3(64), 0, s, result, cap);
  return hipGetLastError();
}

hipError_t launch_min_max(const GlobalImg& im, int32_t* min_max, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, (uint32_t*)min_max, 2, (uint32_t)INT_MAX,
                     (uint32_t)INT_MIN);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || im.w <= 0 || im.h <= 0) return e;
  const dim3 grid(global_grid(im, im.bpp == 2 ? 8 : 16, kRThreads, 4, kRGroups));
  if (im.bpp == 2) hipLaunchKernelGGL(k_min_max<true>, grid, dim3(kRThreads), 0, s, im, min_max);
  else hipLaunchKernelGGL(k_min_max<false>, grid, dim3(kRThreads), 0, s, im, min_max);
  return hipGetLastError();
}

// ---- mean and standard deviation of a U8 image ----------------------------------
// Exact sums S1 = sum v and S2 = sum v^2 (64-bit), then one thread forms
// mean = S1 / N and stddev = sqrt(S2 / N - mean^2) in double precision.
// result: u64 S1, u64 S2, f32 mean, f32 stddev.
__global__ __launch_bounds__(kRThreads) void k_sums(GlobalImg im, unsigned long long* __restrict__ sums) {
  __shared__ unsigned long long part[2][kRThreads / 64];
  unsigned long long s1 = 0, s2 = 0;
  const int t = threadIdx.x;
  stream_each<16, kRThreads, 4>(im, [&](const uint4& q, int n) {
    const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
    uint32_t a = 0, b = 0;  // at most 16 * 255^2 < 2^21
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const uint32_t v = k < n ? (wd[k >> 2] >> (8 * (k & 3))) & 0xFF : 0u;
      a += v;
      b += v * v;
    }
    s1 += a;
    s2 += b;
  });
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s1 += __shfl_xor(s1, off);
    s2 += __shfl_xor(s2, off);
  }
  if ((t & 63) == 0) {
    part[0][t >> 6] = s1;
    part[1][t >> 6] = s2;
  }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < kRThreads / 64; ++w) {
      s1 += part[0][w];
      s2 += part[1][w];
    }
    atomicAdd(&sums[0], s1);
    atomicAdd(&sums[1], s2);
  }
}

__device__ __forceinline__ void mean_std(unsigned long long* sums, double n) {
  const double mean = (double)sums[0] / n;
  const double var = (double)sums[1] / n - mean * mean;
  float* f = (float*)(sums + 2);
  f[0] = (float)mean;
  f[1] = (float)sqrt(var > 0.0 ? var : 0.0);
}

__global__ void k_mean_std_final(unsigned long long* __restrict__ sums, double n) {
  if (threadIdx.x == 0) mean_std(sums, n);
}

hipError_t launch_mean_std_dev(const GlobalImg& im, void* result, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, (uint32_t*)result, 6, 0u, 0u);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || im.w <= 0 || im.h <= 0) return e;
  hipLaunchKernelGGL(k_sums, dim3(global_grid(im, im.bpp == 2 ? 8 : 16, kRThreads, 4, kRGroups)), dim3(kRThreads), 0, s, im,
                     (unsigned long long*)result);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mean_std_final, dim3(1), dim3(64), 0, s, (unsigned long long*)result,
                     (double)im.w * (double)im.h);
  return hipGetLastError();
}

// ---- results of the generated reducing kernels ---------------------------------
// Every work-group of such a kernel wrote its partial results to its own slot
// (red_slot_words); here they become the operators' results, with plain
// stores: nothing is initialised before and no atomic is needed.  A block of
// 1024 threads sums 16 bins of a histogram (64 slots at a time, up to eight
// loads in flight), or merges one operator's words over all slots and forms
// the final values.  After 3840x2160 Gaussian3x3 -> Histogram + MeanStdDev it
// takes 4.7 us, where merging 2025 slots by atomics, two initialising kernels
// and a final one took 17.
constexpr int kFinishThreads = 1024, kFinishBins = 16;

__global__ __launch_bounds__(kFinishThreads) void k_finish_partials(const GProg* __restrict__ P, const IOTable io,
                                                                    const uint32_t* __restrict__ ws, int nslots,
                                                                    int slot_words, double npix) {
  constexpr int NW = kFinishThreads / 64, GROUPS = kFinishThreads / kFinishBins;
  __shared__ uint32_t bins[NW][kFinishBins];
  __shared__ unsigned long long part[2][NW];
  const int t = threadIdx.x, wv = t >> 6, lane = t & 63;
  int blk = blockIdx.x, off = 0;
  for (int oi = 0; oi < P->nops; ++oi) {
    const GOp& o = P->ops[oi];
    if (!is_reduce_op(o.kind)) continue;
    const bool hist = o.kind == OP_HISTOGRAM || o.kind == OP_EQHIST;
    const int blocks = hist ? (o.p0 + kFinishBins - 1) / kFinishBins : 1;
    if (blk >= blocks) {
      blk -= blocks;
      off += red_block_words(o.kind, o.p0);
      continue;
    }
    void* out = io.ptr[P->vals[o.out].io];
    if (hist) {
      const int b = blk * kFinishBins + (t & (kFinishBins - 1));
      uint32_t c = 0;
      if (b < o.p0) {
        const uint32_t* p = ws + off + b;
#pragma unroll 8
        for (int sl = t / kFinishBins; sl < nslots; sl += GROUPS) c += p[(size_t)sl * slot_words];
      }
#pragma unroll
      for (int sh = kFinishBins; sh < 64; sh <<= 1) c += (uint32_t)__shfl_xor((int)c, sh);
      if (lane < kFinishBins) bins[wv][lane] = c;
      __syncthreads();
      if (t < kFinishBins && b < o.p0) {
        uint32_t sum = 0;
        for (int w = 0; w < NW; ++w) sum += bins[w][t];
        ((uint32_t*)out)[b] = sum;
      }
      return;
    }
    unsigned long long x = 0, y = 0;
    if (o.kind == OP_MINMAX) {
      x = (unsigned)INT_MAX;
      y = (unsigned)INT_MIN;
    } else if (o.kind == OP_MMCOUNT) {
      x = kMinKeyInit;
      y = kMaxKeyInit;
    }
    for (int sl = t; sl < nslots; sl += kFinishThreads) {
      const uint32_t* w = ws + (size_t)sl * slot_words + off;
      if (o.kind == OP_MINMAX) red_merge(OP_MINMAX, x, y, w[0], w[1]);
      else red_merge(o.kind, x, y, w[0] | (unsigned long long)w[1] << 32, w[2] | (unsigned long long)w[3] << 32);
    }
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) red_merge(o.kind, x, y, __shfl_xor(x, sh), __shfl_xor(y, sh));
    if (lane == 0) {
      part[0][wv] = x;
      part[1][wv] = y;
    }
    __syncthreads();
    if (t != 0) return;
    for (int w = 1; w < NW; ++w) red_merge(o.kind, x, y, part[0][w], part[1][w]);
    if (o.kind == OP_MINMAX) {
      ((int32_t*)out)[0] = (int)(unsigned)x;
      ((int32_t*)out)[1] = (int)(unsigned)y;
    } else if (o.kind == OP_MMCOUNT) {
      int32_t* mm = (int32_t*)out;
      mm[0] = mm_value(x);
      mm[1] = mm_value(y);
      mm[2] = (int32_t)(uint32_t)x;
      mm[3] = (int32_t)(uint32_t)y;
      mm[4] = mm[5] = 0;  // no locations stored (yet)
    } else {
      unsigned long long* sums = (unsigned long long*)out;
      sums[0] = x;
      sums[1] = y;
      mean_std(sums, npix);
    }
    return;
  }
}

hipError_t launch_finish_partials(const GProg& P, const GProg* dev_prog, const IOTable& io, const uint32_t* ws,
                                  int nslots, hipStream_t s) {
  int blocks = 0;
  for (int i = 0; i < P.nops; ++i) {
    const GOp& o = P.ops[i];
    if (o.kind == OP_HISTOGRAM || o.kind == OP_EQHIST) blocks += (o.p0 + kFinishBins - 1) / kFinishBins;
    else if (is_reduce_op(o.kind)) ++blocks;
  }
  if (blocks == 0 || nslots <= 0) return hipSuccess;
  const double npix = (double)P.w * (double)P.h;
  hipLaunchKernelGGL(k_finish_partials, dim3(blocks), dim3(kFinishThreads), 0, s, dev_prog, io, ws, nslots,
                     red_slot_words(P), npix);
  hipError_t e = hipGetLastError();
  for (int i = 0; i < P.nops && e == hipSuccess; ++i)
    if (P.ops[i].kind == OP_EQHIST)
      e = launch_reduce_finish(OP_EQHIST, io.ptr[P.vals[P.ops[i].out].io], (long long)P.w * P.h, s);
  return e;
}

// ---- first and last steps of global operators reduced by the interpreter -----------
// It merges its groups' results into the operator's result buffer with atomics;
// these kernels set the starting value before and form the final values
// after, in the same stream.

hipError_t launch_reduce_init(int kind, void* result, int num_bins, hipStream_t s) {
  switch (kind) {
    case OP_HISTOGRAM:
    case OP_EQHIST: {
      const int n = kind == OP_EQHIST ? 256 : num_bins;
      hipLaunchKernelGGL(k_fill_u32, dim3((n + 255) / 256), dim3(256), 0, s, (uint32_t*)result, n, 0u, 0u);
      break;
    }
    case OP_MINMAX:
      hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, (uint32_t*)result, 2, (uint32_t)INT_MAX,
                         (uint32_t)INT_MIN);
      break;
    case OP_MMCOUNT: hipLaunchKernelGGL(k_init_keys, dim3(1), dim3(256), 0, s, (int32_t*)result); break;
    case OP_SUMS: hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, (uint32_t*)result, 6, 0u, 0u); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_zero_words(void* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3((n + 255) / 256), dim3(256), 0, s, (uint32_t*)p, n, 0u, 0u);
  return hipGetLastError();
}

hipError_t launch_reduce_finish(int kind, void* result, long long npix, hipStream_t s) {
  switch (kind) {
    case OP_EQHIST:
      hipLaunchKernelGGL(k_eq_lut, dim3(1), dim3(256), 0, s, (const uint32_t*)result, (uint8_t*)result + 256 * 4,
                         npix);
      break;
    case OP_MMCOUNT: hipLaunchKernelGGL(k_unpack_keys, dim3(1), dim3(64), 0, s, (int32_t*)result); break;
    case OP_SUMS:
      hipLaunchKernelGGL(k_mean_std_final, dim3(1), dim3(64), 0, s, (unsigned long long*)result, (double)npix);
      break;
    default: return hipSuccess;
  }
  return hipGetLastError();
}

}  // namespace hvx
