// Cross section and unweighted events from weighted events f_i = w_i |M|^2_i
// (the two outputs of a matrix-element generator, Sec. II: a fiducial cross
// section and a sample of unweighted events obtained from a larger set of
// weighted ones by Monte Carlo).
//
// xsec_partial_kernel + xsec_final_kernel: FP64 sums of f and f^2, the
// maximum and the number of finite f in two passes of fixed shape (blocks
// over contiguous event ranges, then one block over their partials), so the
// result does not depend on timing.  Non-finite f are left out.
//
// Hit-or-miss unweighting: event i is kept iff u_i fmax < f_i with u_i the
// Philox uniform of (seed, event evt_offset + i) at block UNW_BLOCK (a
// counter block no sampler uses, so the same seed may serve both).  The
// kept indices are written in increasing order (stream compaction):
//   unw_count_kernel   per block of R groups of 256 events: number kept -> ws
//   unw_scan_kernel    one block: exclusive prefix sum in place, total
//   unw_write_kernel   per block: wave ballots + LDS offsets -> idx_out
#include <mutex>

#include "mg5mi.h"
#include "common.h"
#include "internal.h"
#include "philox.h"

namespace mg {

constexpr uint32_t UNW_BLOCK = 0x80000000u;

__device__ __forceinline__ double unweight_uniform(uint64_t seed, uint64_t ievt) {
  uint32_t c0 = (uint32_t)ievt, c1 = (uint32_t)(ievt >> 32), c2 = UNW_BLOCK, c3 = 0u;
  philox10(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
  return bits_to_u(c0, c1);
}

// Deterministic two-pass reduction of (sum f, sum f^2, max f, finite count).
// Pass 1: block b reduces the contiguous event range [b*chunk, (b+1)*chunk)
// (coalesced: thread t reads events b*chunk + t + 256 k), then a fixed tree
// over its 256 threads -> ws[4b .. 4b+3].  Pass 2: one block of 1024 threads
// reduces the nb partials (thread t: partials t, t + 1024, ...) by a fixed
// tree.  The block count and ranges depend on n only, so the result does not
// depend on timing.
constexpr int XS_THREADS = 256;
constexpr int64_t XS_MAX_BLOCKS = 2048;
constexpr int64_t XS_MIN_CHUNK = 4096;

int64_t xsec_blocks(int64_t n) {
  int64_t nb = (n + XS_MIN_CHUNK - 1) / XS_MIN_CHUNK;
  return nb < 1 ? 1 : (nb > XS_MAX_BLOCKS ? XS_MAX_BLOCKS : nb);
}

template <int NT>
__device__ __forceinline__ void reduce4(double (&s)[4][NT], int t) {
  for (int st = NT / 2; st > 0; st >>= 1) {
    if (t < st) {
      s[0][t] += s[0][t + st];
      s[1][t] += s[1][t + st];
      s[2][t] = s[2][t + st] > s[2][t] ? s[2][t + st] : s[2][t];
      s[3][t] += s[3][t + st];
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(XS_THREADS) xsec_partial_kernel(const double* __restrict__ f,
                                                                  int64_t n, int64_t chunk,
                                                                  double* __restrict__ ws) {
  __shared__ double s[4][XS_THREADS];
  const int t = threadIdx.x;
  const int64_t b = (int64_t)blockIdx.x * chunk;
  const int64_t e = b + chunk < n ? b + chunk : n;
  double sum = 0.0, sq = 0.0, mx = 0.0, cnt = 0.0;
  for (int64_t i = b + t; i < e; i += XS_THREADS) {
    const double v = f[i];
    if (isfinite(v)) {
      sum += v;
      sq += v * v;
      mx = v > mx ? v : mx;
      cnt += 1.0;
    }
  }
  s[0][t] = sum;
  s[1][t] = sq;
  s[2][t] = mx;
  s[3][t] = cnt;
  __syncthreads();
  reduce4<XS_THREADS>(s, t);
  if (t < 4) ws[4 * blockIdx.x + t] = s[t][0];
}

__global__ void __launch_bounds__(1024) xsec_final_kernel(const double* __restrict__ ws,
                                                          int64_t nb, double* __restrict__ out) {
  __shared__ double s[4][1024];
  const int t = threadIdx.x;
  double sum = 0.0, sq = 0.0, mx = 0.0, cnt = 0.0;
  for (int64_t k = t; k < nb; k += 1024) {
    sum += ws[4 * k];
    sq += ws[4 * k + 1];
    mx = ws[4 * k + 2] > mx ? ws[4 * k + 2] : mx;
    cnt += ws[4 * k + 3];
  }
  s[0][t] = sum;
  s[1][t] = sq;
  s[2][t] = mx;
  s[3][t] = cnt;
  __syncthreads();
  reduce4<1024>(s, t);
  if (t < 4) out[t] = s[t][0];
}

// f of event i, NaN (never kept) past the end
__device__ __forceinline__ double weight_at(const double* f, int64_t i, int64_t n) {
  return i < n ? f[i] : __builtin_nan("");
}
__device__ __forceinline__ bool keep(double v, int64_t i, double fmax, uint64_t seed, int64_t off) {
  return unweight_uniform(seed, (uint64_t)(off + i)) * fmax < v;  // false for NaN
}

// Block b of 256 threads takes the R groups of 256 events from 256 R b on, in
// chunks of 64 (one ballot each): chunk 4 q + w of group q to wave w.  Its kept
// events go to ws[R b], and which of its 4 R chunks keep any, one bit each, to
// ws[R b + 1] where the workspace (a word per group) has that word.
template <int R>
__global__ void __launch_bounds__(256) unw_count_kernel(const double* __restrict__ f, int64_t n,
                                                        double fmax, uint64_t seed, int64_t off,
                                                        int64_t slots, int64_t* __restrict__ ws) {
  __shared__ int cnt[4];
  __shared__ uint64_t any[4];
  const int t = threadIdx.x, w = t >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * (256 * R) + t;
  int c = 0;
  uint64_t bits = 0;
  double v[R];  // all loads in flight at once
#pragma unroll
  for (int q = 0; q < R; ++q) v[q] = weight_at(f, i0 + 256 * q, n);
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const uint64_t m = __ballot(keep(v[q], i0 + 256 * q, fmax, seed, off));
    c += __popcll(m);
    bits |= (uint64_t)(m != 0) << (4 * q + w);
  }
  if ((t & 63) == 0) {
    cnt[w] = c;
    any[w] = bits;
  }
  __syncthreads();
  const int64_t k = (int64_t)blockIdx.x * R;
  if (t == 0) ws[k] = cnt[0] + cnt[1] + cnt[2] + cnt[3];
  if (R > 1 && t == 1 && k + 1 < slots) ws[k + 1] = (int64_t)(any[0] | any[1] | any[2] | any[3]);
}

// inclusive sum over the lanes of a wave up to this one
__device__ __forceinline__ int64_t wave_prefix(int64_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t o = __shfl_up(v, d);
    v += lane >= d ? o : 0;
  }
  return v;
}

// exclusive scan of the nb counts ws[0], ws[stride], ... in place; total -> *count
__global__ void __launch_bounds__(1024) unw_scan_kernel(int64_t* __restrict__ ws, int64_t nb,
                                                        int64_t stride,
                                                        int64_t* __restrict__ count) {
  __shared__ int64_t part[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t chunk = (nb + 1023) / 1024;
  const int64_t b = (int64_t)t * chunk, e = b + chunk < nb ? b + chunk : nb;
  int64_t s = 0;
  for (int64_t k = b; k < e; ++k) s += ws[k * stride];
  const int64_t incl = wave_prefix(s, lane);
  if (lane == 63) part[w] = incl;
  __syncthreads();
  int64_t run = incl - s;
  for (int v = 0; v < w; ++v) run += part[v];
  for (int64_t k = b; k < e; ++k) {
    const int64_t c = ws[k * stride];
    ws[k * stride] = run;
    run += c;
  }
  if (t == 1023) *count = run;
}

template <int R>
__global__ void __launch_bounds__(256) unw_write_kernel(const double* __restrict__ f, int64_t n,
                                                        double fmax, uint64_t seed, int64_t off,
                                                        int64_t slots,
                                                        const int64_t* __restrict__ ws,
                                                        int64_t* __restrict__ idx) {
  constexpr int C = 4 * R;
  __shared__ uint64_t kept[C];
  __shared__ int before[C];
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  const int64_t k = (int64_t)blockIdx.x * R;
  const int64_t i0 = (int64_t)blockIdx.x * (256 * R) + t;
  const uint64_t any = R > 1 && k + 1 < slots ? (uint64_t)ws[k + 1] : ~0ull;
  if (any == 0) return;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int c = 4 * q + w;
    uint64_t m = 0;
    if ((any >> c) & 1) {
      const int64_t i = i0 + 256 * q;
      m = __ballot(keep(weight_at(f, i, n), i, fmax, seed, off));
    }
    if (l == 0) kept[c] = m;
  }
  __syncthreads();
  if (w == 0) {
    const int64_t p = l < C ? __popcll(kept[l]) : 0;
    const int64_t incl = wave_prefix(p, l);
    if (l < C) before[l] = (int)(incl - p);
  }
  __syncthreads();
  const int64_t base = ws[k];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int c = 4 * q + w;
    const uint64_t m = kept[c];
    if ((m >> l) & 1) idx[base + before[c] + __popcll(m & ((1ull << l) - 1ull))] = i0 + 256 * q;
  }
}

// Fixed device scratch of the allocation-free unweighting entry point: one
// int64 per 256-event block, for at most MG_UNWEIGHT_NOALLOC_MAX_EVENTS
// events.  Every GPU the library runs on holds its own copy until the
// process ends.  In host code `scratch` names a host-side stand-in: its
// device address comes from hipGetSymbolAddress, once per device.
constexpr int64_t SCRATCH_BLOCKS = (MG_UNWEIGHT_NOALLOC_MAX_EVENTS + 255) / 256;
static __device__ __align__(256) int64_t scratch[SCRATCH_BLOCKS];

constexpr int MAX_DEVICES = 64;
static std::mutex scratch_mutex;
static int64_t* scratch_ptr[MAX_DEVICES];

// Device address of `scratch` on the current device (nullptr on error).
int64_t* unweight_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    scratch_ptr[dev] = (int64_t*)ptr;
  }
  return scratch_ptr[dev];
}

int launch_xsec_stats(const double* f, int64_t n, double* out, double* ws, hipStream_t s) {
  const int64_t nb = xsec_blocks(n);
  const int64_t chunk = n > 0 ? (n + nb - 1) / nb : 0;
  xsec_partial_kernel<<<(unsigned)nb, XS_THREADS, 0, s>>>(f, n, chunk, ws);
  xsec_final_kernel<<<1, 1024, 0, s>>>(ws, nb, out);
  return 0;
}

int64_t unweight_blocks(int64_t n) { return (n + 255) / 256; }

template <int R>
static void unweight_kernels(const double* f, int64_t n, double fmax, uint64_t seed, int64_t off,
                             int64_t* idx, int64_t* count, int64_t* ws, int64_t slots,
                             hipStream_t s) {
  const int64_t nb = (slots + R - 1) / R;
  if (nb > 0)
    unw_count_kernel<R><<<(unsigned)nb, 256, 0, s>>>(f, n, fmax, seed, off, slots, ws);
  unw_scan_kernel<<<1, 1024, 0, s>>>(ws, nb, R, count);  // nb = 0: writes count = 0
  if (nb > 0)
    unw_write_kernel<R><<<(unsigned)nb, 256, 0, s>>>(f, n, fmax, seed, off, slots, ws, idx);
}

// Groups of 256 events per block: as many as leave about a thousand blocks (four
// per CU), so that the one block of the scan has few counts to go through (5e6
// events: 19532 counts in 34.6 us with one group per block, 1221 in 5.0 us
// with 16) and the second pass draws random numbers for the chunks with kept
// events only.
int launch_unweight(const double* f, int64_t n, double fmax, uint64_t seed, int64_t off,
                    int64_t* idx, int64_t* count, int64_t* ws, hipStream_t s) {
  const int64_t slots = unweight_blocks(n);
  if (slots > 0x7FFFFFFF) return -1;
  if (n > (1 << 22)) unweight_kernels<16>(f, n, fmax, seed, off, idx, count, ws, slots, s);
  else if (n > (1 << 20)) unweight_kernels<4>(f, n, fmax, seed, off, idx, count, ws, slots, s);
  else unweight_kernels<1>(f, n, fmax, seed, off, idx, count, ws, slots, s);
  return 0;
}

}  // namespace mg
