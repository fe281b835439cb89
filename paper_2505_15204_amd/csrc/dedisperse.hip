// dedisperse.hip — incoherent de-dispersion: out[k][t] = mean over channels c of
// in[t + d(k, c)][c], FP64 sums in channel order, divided by C and rounded to float once.
#include <hip/hip_runtime.h>

#include "launch.hpp"

namespace blink {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 16;                       // waves of a tiled workgroup
constexpr int kDms = 2;                          // trials of one wave
constexpr int kPx = 64;                          // pixels of a workgroup, one per lane
constexpr int kStage = 4;                        // channels per LDS stage
constexpr int kMaxRows = 60;                     // time steps of one channel in a stage
constexpr int kMaxChannels = 4096;               // row ranges kept in the LDS
constexpr int kMinReads2 = 5;                    // twice the reads per copied step that the tiled form needs
constexpr int kMinGroups = 96;                   // workgroups below which the tiled form is not taken

// One output value per thread and pixel quad, every input read where it is used: for the shapes
// that the tiled kernel does not take.
__global__ __launch_bounds__(256) void k_dedisperse(const float4* __restrict__ in, int C, long nn4,
                                                    const int* __restrict__ delays, int t_out,
                                                    float4* __restrict__ out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nn4) return;
  const int t = blockIdx.y, k = blockIdx.z;
  const int* dk = delays + (size_t)k * C;
  double sx = 0.0, sy = 0.0, sz = 0.0, sw = 0.0;
  for (int c = 0; c < C; ++c) {
    const float4 v = in[((size_t)(t + dk[c]) * C + c) * nn4 + i];
    sx += v.x;
    sy += v.y;
    sz += v.z;
    sw += v.w;
  }
  const double cd = (double)C;
  out[((size_t)k * t_out + t) * nn4 + i] = make_float4((float)(sx / cd), (float)(sy / cd), (float)(sz / cd),
                                                       (float)(sw / cd));
}

// Tiled form. A workgroup takes 64 pixels and up to 16 units, one per wave; a unit is 2 trials x TB
// output steps, whose 2 TB sums a lane keeps in registers over all channels. Per stage of 4
// channels the workgroup copies to LDS the time steps that any of its units reads (so each input
// is read from memory once per workgroup instead of once per output), and the next stage's loads
// are in flight during the sums. A lane reads its TB steps of each trial from LDS at compile-time
// offsets. (Letting two trials of nearly equal delay share reads and conversions needs a branch per
// delay difference; keeping the values over it spills: 15.8 ms. Eight waves of four trials: 11.3 ms.)
//
// Bounds: 512^2 pixels x 768 channels x 40 steps and 16 trials read 26.5 GB (4.3 ms at the rate of
// a copy) and convert and add 84 G values in FP64 (4.3 ms of VALU issue): 9.2 ms; 54 ms when every
// output read its 768 inputs (335 GB through the caches).
template <int TB>
__global__ __launch_bounds__(64 * kWaves) void k_dedisperse_tile(const float* __restrict__ in, int C, int log_nn,
                                                                    const int* __restrict__ delays, int n_dm, int t_out,
                                                                    int tiles, int units, int groups, int rows_max,
                                                                    float* __restrict__ out) {
  extern __shared__ __align__(16) float lds[];   // two stages of kStage x rows_max x 64 (and the reads past them), row ranges
  const int rows4 = (rows_max + 3) & ~3;
  const int slot = rows4 * kPx;                  // floats of one channel
  int2* range = reinterpret_cast<int2*>(lds + 2 * kStage * slot + TB * kPx);   // per channel {first step, steps}
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  // the workgroups of one pixel block (their inputs are largely the same) share one XCD's L2
  const unsigned span = 8u * groups;
  const int u0 = (int)(blockIdx.x % span / 8) * kWaves;
  const long px0 = (long)(blockIdx.x / span * 8 + blockIdx.x % 8) * kPx;
  const long nn = 1L << log_nn;
  if (px0 >= nn) return;
  // this wave's unit: trials k0 and k0 + 1 (a last one alone repeats itself), steps t0 .. t0 + TB - 1
  const int u = u0 + wave < units ? u0 + wave : units - 1;
  const int k0 = u / tiles * kDms, t0 = u % tiles * TB;
  {
    // steps that the workgroup's units read of each channel: the units' trials and tiles
    const int u1 = u0 + kWaves < units ? u0 + kWaves : units;
    for (int c = tid; c < C; c += 64 * kWaves) {
      int lo = 0x7fffffff, hi = 0;
      for (int q = u0; q < u1; ++q) {
        const int ka = q / tiles * kDms, ta = q % tiles * TB, tb = ta + TB < t_out ? ta + TB : t_out;
        for (int k = ka; k < ka + kDms && k < n_dm; ++k) {
          const int d = delays[(size_t)k * C + c];
          lo = ta + d < lo ? ta + d : lo;
          hi = tb + d > hi ? tb + d : hi;
        }
      }
      range[c] = make_int2(lo, hi - lo);
    }
  }
  __syncthreads();
  // A stage's copy: 16 threads read one step's 64 pixels (16 bytes each); thread group tid / 16
  // takes the steps tid / 16, + STEPS, ... of the stage's kStage x rows4 slots. Every load is
  // unconditional (slots past a channel's steps repeat its last one).
  constexpr int STEPS = 64 * kWaves / 16;        // steps copied at a time
  constexpr int COPY = (kStage * kMaxRows + STEPS - 1) / STEPS;
  f32x4 held[COPY];
  int where[COPY];                               // channel of the stage | step of its slot << 8
#pragma unroll
  for (int i = 0; i < COPY; ++i) {
    const int s = tid / 16 + STEPS * i, ch = s / rows4 < kStage ? s / rows4 : kStage - 1;
    where[i] = ch | (s - ch * rows4) << 8;
  }
  const float* src = in + px0 + (tid & 15) * 4;
  auto fetch = [&](int c0) {
#pragma unroll
    for (int i = 0; i < COPY; ++i) {
      if (STEPS * i >= kStage * rows4) continue;    // uniform
      const int c = c0 + (where[i] & 0xff), cc = c < C ? c : C - 1, r = where[i] >> 8;
      const int2 g = range[cc];
      const unsigned step = (unsigned)(g.x + (r < g.y ? r : g.y - 1));
      held[i] = *reinterpret_cast<const f32x4*>(src + ((size_t)(step * (unsigned)C + (unsigned)cc) << log_nn));
    }
  };
  auto stash = [&](float* stage) {
#pragma unroll
    for (int i = 0; i < COPY; ++i) {
      const int s = tid / 16 + STEPS * i;
      if (s < kStage * rows4) *reinterpret_cast<f32x4*>(stage + s * kPx + (tid & 15) * 4) = held[i];
    }
  };
  double acc[kDms][TB];
#pragma unroll
  for (int k = 0; k < kDms; ++k)
#pragma unroll
    for (int t = 0; t < TB; ++t) acc[k][t] = 0.0;
  int kk[kDms];
#pragma unroll
  for (int k = 0; k < kDms; ++k) kk[k] = k0 + k < n_dm ? k0 + k : n_dm - 1;
  // a channel's delays (uniform over the wave) and first step, requested one channel ahead
  auto rows_of = [&](int c) {
    const int cc = c < C ? c : C - 1;
    return make_int3(delays[(size_t)kk[0] * C + cc], delays[(size_t)kk[1] * C + cc], range[cc].x);
  };
  fetch(0);
  stash(lds);
  __syncthreads();
  int3 next = rows_of(0);
  for (int c0 = 0, b = 0; c0 < C; c0 += kStage, b ^= 1) {
    if (c0 + kStage < C) fetch(c0 + kStage);
    const float* stage = lds + b * kStage * slot + lane;
#pragma unroll 1
    for (int ch = 0; ch < kStage && c0 + ch < C; ++ch) {
      const int3 now = next;
      next = rows_of(c0 + ch + 1);
      const int base = ch * rows4 + t0 - __builtin_amdgcn_readfirstlane(now.z);
      // steps past t_out (the last tile) are read from what follows in the LDS and never stored
      const float* p = stage + (base + now.x) * kPx;
      const float* q = stage + (base + now.y) * kPx;
      float x[2 * TB];                           // every read is issued before the first sum
#pragma unroll
      for (int t = 0; t < TB; ++t) x[t] = p[t * kPx];
#pragma unroll
      for (int t = 0; t < TB; ++t) x[TB + t] = q[t * kPx];
#pragma unroll
      for (int t = 0; t < TB; ++t) acc[0][t] += (double)x[t];
#pragma unroll
      for (int t = 0; t < TB; ++t) acc[1][t] += (double)x[TB + t];
    }
    if (c0 + kStage < C) stash(lds + (b ^ 1) * kStage * slot);
    __syncthreads();
  }
  const int last = t_out - t0 < TB ? t_out - t0 - 1 : TB - 1;   // last step of this wave's tile
  if (u0 + wave >= units) return;
  const double cd = (double)C;
#pragma unroll
  for (int k = 0; k < kDms; ++k)
#pragma unroll
    for (int t = 0; t < TB; ++t)
      if (k0 + k < n_dm && t <= last) out[((size_t)(k0 + k) * t_out + t0 + t) * nn + px0 + lane] = (float)(acc[k][t] / cd);
}

struct Tiling {
  int tb, tiles, units, groups, rows;
};

template <int TB>
hipError_t launch_tile(int tb, const float* in, int C, int log_nn, const int* delays, int n_dm, int t_out, const Tiling& g,
                       float* out, hipStream_t s) {
  if (tb == TB) {
    const int rows4 = (g.rows + 3) & ~3;
    const size_t lds = ((size_t)2 * kStage * rows4 + TB) * kPx * sizeof(float) + (size_t)C * sizeof(int2);
    const void* fn = reinterpret_cast<const void*>(k_dedisperse_tile<TB>);
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    const unsigned blocks = (unsigned)((1L << log_nn) / kPx + 7) / 8 * 8 * (unsigned)g.groups;
    k_dedisperse_tile<TB><<<blocks, 64 * kWaves, lds, s>>>(in, C, log_nn, delays, n_dm, t_out, g.tiles, g.units, g.groups,
                                                           g.rows, out);
    return hipGetLastError();
  }
  if constexpr (TB > 1) return launch_tile<TB - 1>(tb, in, C, log_nn, delays, n_dm, t_out, g, out, s);
  else return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_dedisperse(const float* in, int C, int logn, const int* delays, const int32_t* host_delays, int n_dm,
                             int t_out, float* out, hipStream_t s) {
  if (n_dm <= 0 || t_out <= 0) return hipSuccess;
  const long nn = 1L << (2 * logn);
  // Tiles of at most 13 steps (2 x 13 FP64 sums and 26 values: 78 registers), as even as they go; the steps that
  // one workgroup's units read of a channel have to fit the stage.
  Tiling g{};
  constexpr int kMaxTb = 13;
  g.tiles = (t_out + kMaxTb - 1) / kMaxTb;
  g.tb = (t_out + g.tiles - 1) / g.tiles;
  g.units = (n_dm + kDms - 1) / kDms * g.tiles;
  g.groups = (g.units + kWaves - 1) / kWaves;
  // One workgroup takes as long as any, so few of them (small images) leave the chip idle: 128^2
  // pixels x 768 channels x 16 trials (256 workgroups) take 0.73 ms tiled and 2.6 ms untiled, 64^2
  // (64 workgroups) 0.57 and 0.43 ms.
  const int nk = (n_dm + kDms - 1) / kDms;
  // The steps copied to LDS have to be read often enough, by enough of the workgroup's waves: 3 trials
  // to a large DM (100 channels of 256^2, 30 steps) read each copied step 1.4 times and take 292 us tiled
  // and 140 untiled; 2 trials to a small one 1.9 times, 201 and 218 us; 8 trials of 60 channels of 128^2 63
  // and 117.
  long copied = 0;
  bool fits = C <= kMaxChannels && g.groups <= 4096 && nn / kPx * g.groups >= kMinGroups && g.units >= kWaves / 2;
  for (int c = 0; fits && c < C; ++c) {
    for (int q = 0; q < g.groups; ++q) {
      const int u0 = q * kWaves, u1 = u0 + kWaves < g.units ? u0 + kWaves : g.units;
      int lo = 0x7fffffff, hi = 0;
      for (int a = u0 / g.tiles; a <= (u1 - 1) / g.tiles && a < nk; ++a) {
        const int ua = a * g.tiles > u0 ? 0 : u0 - a * g.tiles, ub = (a + 1) * g.tiles < u1 ? g.tiles : u1 - a * g.tiles;
        const int tb = ub * g.tb < t_out ? ub * g.tb : t_out;
        for (int k = a * kDms; k < a * kDms + kDms && k < n_dm; ++k) {
          const int d = host_delays[(size_t)k * C + c];
          lo = ua * g.tb + d < lo ? ua * g.tb + d : lo;
          hi = tb + d > hi ? tb + d : hi;
        }
      }
      g.rows = hi - lo > g.rows ? hi - lo : g.rows;
      copied += hi - lo;
    }
    fits = g.rows <= kMaxRows;
  }
  fits = fits && 2 * (long)n_dm * t_out * C >= kMinReads2 * copied;
  if (fits) return launch_tile<kMaxTb>(g.tb, in, C, 2 * logn, delays, n_dm, t_out, g, out, s);
  const long nn4 = nn / 4;
  dim3 grid((unsigned)((nn4 + 255) / 256), (unsigned)t_out, (unsigned)n_dm);
  k_dedisperse<<<grid, 256, 0, s>>>((const float4*)in, C, nn4, delays, t_out, (float4*)out);
  return hipGetLastError();
}

}  // namespace blink
