// kernels.hip — gfx950 kernels of the batched dirty-imaging path.
//
//   k_twiddles       FP64 sincospi -> FP32 stage-ordered twiddle table
//   k_bin            cell indices (FP64 product + rint), flags, out-of-grid drop, counting sort
//                    of the placements into column strips, or tiles of the full grid (Section
//                    6.2.4 gridding, one workgroup per (time, channel), shared by the polarisations)
//   k_grid_full      LDS-private tiles -> complex grid in HBM, counts
//   k_grid_colfft    LDS-private strip grid -> inverse FFT along v -> half-spectrum H
//   k_dense_colfft   Hermitian part of a dense grid -> inverse FFT along v -> H
//   k_row_c2r        two H rows -> Hermitian-extended inverse FFT along u -> two image rows,
//                    scaled by 1/W of the image (computed from the kept count or occupancy)
//   k_bin_conv, k_grid_colfft_conv, k_conv_correction
//                    the convolutional-gridding variant (conv_device.hpp)
//
// The dirty image is I = Re(IDFT2(G)) / W (Section 4, Eq. 5). The shift of Section 6.2.4 is
// folded into the input as the modulation (-1)^(ku + kv), which for even N moves the phase
// centre to pixel (N/2, N/2). Because the grid is Hermitian only the columns ku < N/2 are
// transformed along v; the row pass rebuilds the other half by symmetry, and H's column 0 packs
// the two real-valued columns ku = 0 (real part) and ku = N/2 (imaginary part).
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace blink {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- twiddles
// The stage-ordered table of one size N (fft_device.hpp): FP64 sincospi of an exact dyadic
// argument, rounded to FP32. Unused rows of A (m >= R1) hold zero.
__global__ void k_twiddles(float2* tw, int logn) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= tw_total(logn)) return;
  const int n = 1 << logn;
  const int r1 = logn <= 4 ? 1 : (logn >= 8 ? 16 : n / 16);
  long num = 0, den = 1;
  bool used = true;
  if (j < 256) {                      // A: row m, column k
    const int m = j / 16, k = j % 16;
    used = m < r1;
    num = (long)k * m;
    den = 16L * r1;
  } else if (j < kTwA) {              // D: 16-point DFT entries
    num = j - 256;
    den = 16;
  } else if (j >= tw_size(logn)) {    // linear table
    num = j - tw_size(logn);
    den = n;
  } else {                            // B: row m, column k
    const int m = (j - kTwA) / 256, k = (j - kTwA) % 256;
    num = (long)k * m;
    den = n;
  }
  double s = 0.0, c = 0.0;
  sincospi(2.0 * (double)(num % den) / (double)den, &s, &c);
  tw[j] = used ? make_float2((float)c, (float)s) : make_float2(0.f, 0.f);
}

int twiddle_table_size(int logn) { return tw_total(logn); }

// ---------------------------------------------------------------- split-form DFT operands
__global__ void k_dft_operands(const float2* __restrict__ tw, uint4* ops) {
  const int lane = threadIdx.x & 63;
  if (threadIdx.x < 64) make_dft_operands<kPrecSplitF16>(tw, ops, lane);
  else if (threadIdx.x < 128) make_dft_operands<kPrecSplitBf16>(tw, ops, lane);
}

hipError_t launch_dft_operands(const float2* tw, uint4* ops, hipStream_t s) {
  k_dft_operands<<<1, 128, 0, s>>>(tw, ops);
  return hipGetLastError();
}

hipError_t launch_twiddles(float2* tw, int logn, hipStream_t s) {
  const int n = tw_total(logn);
  k_twiddles<<<(n + 255) / 256, 256, 0, s>>>(tw, logn);
  return hipGetLastError();
}

// ---------------------------------------------------------------- binning
template <bool TILES>
__global__ __launch_bounds__(kBinThreads) void k_bin(BinArgs a) {
  __shared__ BinShared sh;
  const int tcl = blockIdx.x;
  const long tc = (long)a.tc0 + tcl;
  const int t = (int)(tc / a.C), c = (int)(tc % a.C);
  const int N = 1 << a.logn;
  const int nstrips = a.ku_limit >> a.log_strip;
  const double k = (a.freq[c] / kSpeedOfLight) * ((double)N * a.pixel_scale);
  bin_visibilities<TILES>(a.uvw + (size_t)t * a.B * 3, a.flags ? a.flags + (size_t)tc * a.B : nullptr, a.B, k, a.logn,
                   a.log_strip, a.ku_limit, a.plc + (size_t)tcl * 2 * a.B, a.strip_off + (size_t)tcl * (nstrips + 1),
                   a.n_kept + tcl, a.n_out ? a.n_out + tc : nullptr, a.cell_idx ? a.cell_idx + (size_t)tc * a.B : nullptr,
                   sh, a.ext ? a.ext + tcl : nullptr);
  if (threadIdx.x < a.P) a.occ[(size_t)tcl * a.P + threadIdx.x] = 0;
}

hipError_t launch_bin(const BinArgs& a, hipStream_t s) {
  if (a.Q <= 0) return hipSuccess;
  if (a.tiles) k_bin<true><<<a.Q, kBinThreads, 0, s>>>(a);
  else k_bin<false><<<a.Q, kBinThreads, 0, s>>>(a);
  return hipGetLastError();
}

// ---------------------------------------------------------------- convolutional binning
__global__ __launch_bounds__(kBinThreads) void k_bin_conv(BinArgs a, ConvSpec cs, int rec_stride) {
  __shared__ BinShared sh;
  const int tcl = blockIdx.x;
  const long tc = (long)a.tc0 + tcl;
  const int t = (int)(tc / a.C), c = (int)(tc % a.C);
  const int N = 1 << a.logn;
  const int nstrips = (N / 2) >> a.log_strip;
  const double k = (a.freq[c] / kSpeedOfLight) * ((double)N * a.pixel_scale);
  const int log_band = conv_log_band(a.logn), nb = N >> log_band;
  bin_visibilities_conv(a.uvw + (size_t)t * a.B * 3, a.flags ? a.flags + (size_t)tc * a.B : nullptr, a.B, k, a.logn,
                        a.log_strip, log_band, cs, reinterpret_cast<ConvRec*>(a.plc) + (size_t)tcl * rec_stride,
                        a.strip_off + (size_t)tcl * (nstrips * nb + 1), a.n_kept + tcl,
                        a.n_out ? a.n_out + tc : nullptr, sh, a.ext ? a.ext + tcl : nullptr);
}

// A placement's W < N/2 tap columns reach at most ceil(W / S) + 1 strips and its W <= 16 tap rows
// at most two 16-row bands; with bands every bin holds at most three padding records.
int conv_records_per_pair(int B, int width, int min_strip, int logn) {
  const bool banded = conv_log_band(logn) < logn;
  return 2 * B * ((width + min_strip - 1) / min_strip + 2) * (banded ? 2 : 1) +
         (banded ? 3 * conv_bins_per_pair(logn, min_strip) : 0);
}

int conv_bins_per_pair(int logn, int strip) { return ((1 << logn) / 2 / strip) * ((1 << logn) >> conv_log_band(logn)); }

hipError_t launch_bin_conv(const BinArgs& a, ConvParams cp, int rec_stride, hipStream_t s) {
  if (a.Q <= 0) return hipSuccess;
  k_bin_conv<<<a.Q, kBinThreads, 0, s>>>(a, ConvSpec{cp.width, (float)cp.beta}, rec_stride);
  return hipGetLastError();
}

__global__ __launch_bounds__(kCorrThreads) void k_conv_correction(float* corr, int n, int width, double beta, int shift) {
  __shared__ double s_part[kCorrNodes];
  conv_correction_entry(corr, n, blockIdx.x, width, beta, shift, s_part);
}

hipError_t launch_conv_correction(float* corr, int logn, ConvParams cp, int shift, hipStream_t s) {
  const int n = 1 << logn;
  k_conv_correction<<<n, kCorrThreads, 0, s>>>(corr, n, cp.width, cp.beta, shift);
  return hipGetLastError();
}

template <int LOGN>
struct ConvStrip {
  static hipError_t run(int* out) {
    *out = ColSmax<LOGN, false>::value;
    return hipSuccess;
  }
};

int conv_strip_width(int logn) {
  int s = 0;
  return by_logn<ConvStrip>(logn, &s) == hipSuccess ? s : 0;
}

hipError_t launch_grid_colfft_conv(const ColArgs& a, int n_img, ConvParams cp, int prec, const float2* tw,
                                   hipStream_t s) {
  const float beta = (float)cp.beta;
  switch (prec) {
    case BLINK_PREC_FP32: return PrecLaunch<BLINK_PREC_FP32>::grid_colfft_conv(a, n_img, cp.width, beta, tw, s);
    case BLINK_PREC_SPLIT_F16:
      return PrecLaunch<BLINK_PREC_SPLIT_F16>::grid_colfft_conv(a, n_img, cp.width, beta, tw, s);
    case BLINK_PREC_SPLIT_BF16:
      return PrecLaunch<BLINK_PREC_SPLIT_BF16>::grid_colfft_conv(a, n_img, cp.width, beta, tw, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------- visibility corrections
// Antenna pair (i, j), i > j, of baseline b = i (i - 1) / 2 + j: the lower-triangular order in
// which the correlation step stores visibilities (Section 6.2.2).
__device__ __forceinline__ void antenna_pair(long long b, int& i, int& j) {
  long long r = (long long)((1.0 + sqrt(1.0 + 8.0 * (double)b)) * 0.5);
  while (r * (r - 1) / 2 > b) --r;
  while ((r + 1) * r / 2 <= b) ++r;
  i = (int)r;
  j = (int)(b - r * (r - 1) / 2);
}

// One thread per (pair, baseline); the phase of the new phase centre is shared by the pols.
// Workgroup w covers baselines (w % nbx) * 256 .. of pair w / nbx.
__global__ __launch_bounds__(256) void k_correct_vis(CorrArgs a, int nbx) {
  const int q = (int)(blockIdx.x / (unsigned)nbx);
  const int b = (int)(blockIdx.x % (unsigned)nbx) * 256 + (int)threadIdx.x;
  if (b >= a.B) return;
  const long tc = (long)a.tc0 + q;
  const long t = tc / a.C, c = tc % a.C;
  const double* x = a.uvw + 3 * ((size_t)t * a.B + b);
  // geometric delay in turns (FP64), reduced exactly to [-1/2, 1/2]; the sine and cosine of the
  // reduced angle are taken in FP32 (|angle| <= pi, so their error is a few 1e-8)
  const double turns = (a.freq[c] / kSpeedOfLight) * (x[0] * a.l0 + x[1] * a.m0 + x[2] * a.n0m1);
  float snf, csf;
  sincospif((float)(2.0 * (turns - rint(turns))), &snf, &csf);
  const double sn = snf, cs = csf;
  int i = 0, j = 0;
  if (a.gains) antenna_pair(b, i, j);
  for (int p = 0; p < a.P; ++p) {
    const size_t at = ((size_t)q * a.P + p) * a.B + b;
    const float2 v = a.vis[at];
    double re = v.x, im = v.y;
    if (a.gains) {
      const float2 gi = a.gains[((size_t)c * a.P + p) * a.n_ant + i];
      const float2 gj = a.gains[((size_t)c * a.P + p) * a.n_ant + j];
      const double r1 = (double)gi.x * re - (double)gi.y * im, i1 = (double)gi.x * im + (double)gi.y * re;
      re = r1 * gj.x + i1 * gj.y;          // (r1 + i i1) conj(gj)
      im = i1 * gj.x - r1 * gj.y;
    }
    a.out[at] = make_float2((float)(re * cs - im * sn), (float)(re * sn + im * cs));
  }
}

hipError_t launch_correct_vis(const CorrArgs& a, hipStream_t s) {
  if (a.Q <= 0 || a.B <= 0) return hipSuccess;
  const long nbx = ((long)a.B + 255) / 256;
  if (nbx * a.Q > 0x7fffffffL) return hipErrorInvalidValue;
  k_correct_vis<<<(unsigned)(nbx * a.Q), 256, 0, s>>>(a, (int)nbx);
  return hipGetLastError();
}

// ---------------------------------------------------------------- image averages
// Averages of images [T][C][P][N][N] over the axes in `axes` (1 time, 2 channel, 4 polarisation;
// Sections 7.2 and 7.3 average over time and over the band, the polarisation average of XX and YY
// is Stokes I). Four consecutive pixels of one output per lane, FP64 sums. The inputs of an output
// are runs of n1 images at a stride of s1, n2 runs at a stride of s2; groups of WIDTH waves take equal
// parts of the inputs of the same 256 WIDTH pixels and their sums meet in LDS, which keeps enough
// loads in flight for small images too (8 per lane). Bound by reading the inputs: 1536 of 1024^2 in 1.02 ms,
// 6.3 TB/s (a copy, which also writes as much, moves 6.2).
struct AvgRuns {
  int n1, n2;
  long s1, s2;                                  // in images
};

template <int SLICES, int WIDTH>
__global__ __launch_bounds__(64 * SLICES * WIDTH) void k_image_average(const f32x4* __restrict__ in, int C, int P, long nn4,
                                                                int axes, int Co, int Po, AvgRuns r,
                                                                f32x4* __restrict__ out) {
  __shared__ double part[SLICES > 1 ? SLICES - 1 : 1][4][64 * WIDTH];
  const int lane = threadIdx.x % (64 * WIDTH), slice = __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * WIDTH));
  const long blocks = (nn4 + 64 * WIDTH - 1) / (64 * WIDTH), img = blockIdx.x / blocks;
  const long px = (blockIdx.x - img * blocks) * (64 * WIDTH) + lane;
  const int po = (int)(img % Po), co = (int)((img / Po) % Co), to = (int)(img / ((long)Po * Co));
  const long first = ((long)((axes & 1) ? 0 : to) * C + ((axes & 2) ? 0 : co)) * P + ((axes & 4) ? 0 : po);
  const long n = (long)r.n1 * r.n2;
  const f32x4* src = in + first * nn4 + (px < nn4 ? px : 0);
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  long k = n * slice / SLICES;
  const long k1 = n * (slice + 1) / SLICES;
  while (k < k1) {                              // uniform over the wave
    const long run = k / r.n1, at = k - run * r.n1;
    const int m = (int)(r.n1 - at < k1 - k ? r.n1 - at : k1 - k);
    const f32x4* p = src + (run * r.s2 + at * r.s1) * nn4;
    const long step = r.s1 * nn4;
    int i = 0;
    for (; i + 8 <= m; i += 8, p += 8 * step) {
      f32x4 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(p + j * step);
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] += (double)v[j][q];
    }
    for (; i < m; ++i, p += step) {
      const f32x4 v = __builtin_nontemporal_load(p);
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] += (double)v[q];
    }
    k += m;
  }
  if constexpr (SLICES > 1) {
    if (slice > 0)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[slice - 1][q][lane] = a[q];
    __syncthreads();
    if (slice > 0) return;
    for (int s = 0; s < SLICES - 1; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] += part[s][q][lane];
  }
  const double inv = 1.0 / (double)n;
  if (px < nn4) out[img * nn4 + px] = f32x4{(float)(a[0] * inv), (float)(a[1] * inv), (float)(a[2] * inv), (float)(a[3] * inv)};
}

// One thread per pixel quad and output, every input through the caches: for short sums. Small images leave a
// thread little but its index to work out, which takes 32-bit divisions (80000 outputs of two inputs of
// 8^2: 26.7 us with 64-bit ones and a product per input).
__global__ __launch_bounds__(256) void k_image_average_few(const f32x4* __restrict__ in, int C, int P, int log_nn4,
                                                           int axes, unsigned Co, unsigned Po, long n_quads, AvgRuns r,
                                                           f32x4* __restrict__ out) {
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  if (gid >= n_quads) return;
  const unsigned img = (unsigned)(gid >> log_nn4), tc = img / Po, po = img - tc * Po, to = tc / Co, co = tc - to * Co;
  const long first = ((long)((axes & 1) ? 0u : to) * C + ((axes & 2) ? 0u : co)) * P + ((axes & 4) ? 0u : po);
  const f32x4* src = in + (first << log_nn4) + (gid & ((1L << log_nn4) - 1));
  const long step1 = r.s1 << log_nn4, step2 = r.s2 << log_nn4;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int i = 0; i < r.n2; ++i, src += step2) {
    const f32x4* p = src;
    for (int j = 0; j < r.n1; ++j, p += step1) {
      const f32x4 v = *p;
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] += (double)v[q];
    }
  }
  const double inv = 1.0 / ((double)r.n1 * r.n2);
  out[gid] = f32x4{(float)(a[0] * inv), (float)(a[1] * inv), (float)(a[2] * inv), (float)(a[3] * inv)};
}

hipError_t launch_image_average(const float* in, int T, int C, int P, int logn, int axes, float* out, hipStream_t s) {
  const long nn4 = (1L << (2 * logn)) / 4;
  const int To = (axes & 1) ? 1 : T, Co = (axes & 2) ? 1 : C, Po = (axes & 4) ? 1 : P;
  const long n_img = (long)To * Co * Po;
  if (n_img * nn4 <= 0) return hipSuccess;
  // the averaged axes as runs: polarisation and channel merge into one when both are averaged (or
  // there is one polarisation), channel and time likewise
  struct { long n, s; } d[3] = {{(axes & 4) ? P : 1, 1}, {(axes & 2) ? C : 1, P}, {(axes & 1) ? T : 1, (long)C * P}}, m[3];
  int nd = 0;
  for (auto& x : d) {
    if (x.n == 1) continue;
    if (nd > 0 && m[nd - 1].n * m[nd - 1].s == x.s) m[nd - 1].n *= x.n;
    else m[nd++] = {x.n, x.s};
  }
  AvgRuns r{1, 1, 1, 1};
  if (nd > 0) r.n1 = (int)m[0].n, r.s1 = m[0].s;
  if (nd > 1) r.n2 = (int)m[1].n, r.s2 = m[1].s;   // (three separate axes always merge)
  const long n = (long)r.n1 * r.n2;
  const f32x4* src = (const f32x4*)in;
  f32x4* dst = (f32x4*)out;
  auto blocks = [&](int width) { return (unsigned)((nn4 + 64 * width - 1) / (64 * width) * n_img); };
  if ((nn4 + 63) / 64 * n_img > 0x7fffffffL) return hipErrorInvalidValue;
  // Below 16 inputs the sum is short, and it is below 64 where the pixels alone fill the chip: there
  // plain loads with a thread per pixel quad (40 inputs of 2048^2: 119 us, 126 with 8 slices; 3 inputs: 11.6
  // and 13.4), unless there are many outputs and more data than the last-level cache keeps, which the 64-thread
  // blocks' loads pass by (80 of 2 inputs of 1024^2: 155 us against 167 plain; but 80 of 2 of 256^2, 63
  // MB: 14.9 against 11.9) and which need whole waves of an image's pixels (80000 of 2 inputs of 8^2: 37.3
  // against 11.7). 84 inputs of 2048^2 take 235 us with 8 slices, 250 plain. Below 2048 blocks of 256 pixels
  // (256^2 and smaller, one output; from 512 on short sums stay plain: 100 outputs of 20 inputs of 64^2 15.8
  // us with 16 slices, 8.7 plain) more waves per output are needed than the 8 slices of the wider form give:
  // 8400 images of 256^2 take 337 us with 16 slices, 3886 us with one; 1536 of 1024^2 1055 us with 8 slices of
  // 512 pixels, 1078 with 4 of 256, 1228 with 4 of 1024, 1211 with one (one thread per pixel quad).
  const bool streams = (n + 1) * n_img * nn4 * 16 > 300000000L && nn4 >= 256;
  if (n < 16 ? n_img == 1 || !streams : n < 64 && blocks(1) >= (n < 32 ? 512u : 2048u))
    k_image_average_few<<<(unsigned)((nn4 * n_img + 255) / 256), 256, 0, s>>>(src, C, P, 2 * logn - 2, axes, Co, Po,
                                                                                nn4 * n_img, r, dst);
  else if (n < 16) k_image_average<1, 1><<<blocks(1), 64, 0, s>>>(src, C, P, nn4, axes, Co, Po, r, dst);
  else if (blocks(1) >= 2048) k_image_average<8, 2><<<blocks(2), 1024, 0, s>>>(src, C, P, nn4, axes, Co, Po, r, dst);
  else k_image_average<16, 1><<<blocks(1), 1024, 0, s>>>(src, C, P, nn4, axes, Co, Po, r, dst);
  return hipGetLastError();
}

// ---------------------------------------------------------------- full grid (blink_grid)
// A workgroup writes H x W cells of an image (64 x 64): it clears them in LDS, adds the placements of its
// tile that lie in them, and stores them as whole 512-byte runs. Bound by the writes; parts of 4096 cells so
// that several workgroups share a compute unit and their chains (offsets, records, visibilities, LDS
// atomics, stores) overlap. Tiles have both sides short, and their two parts divide them crosswise, so that a
// coverage along either axis (an east-west array, v = 0) spreads over many. The same tile of all pairs comes before the next one, the tiles with the
// dense centre first, so that these spread over the XCDs and no long one comes last; the parts and polarisations
// of a tile are placed 8 workgroups apart: they share one XCD's L2, which then reads its records once.
// 96 grids of 512^2 with counts of 48 pairs (252 MB): 67 us (strips of rows, 8192 cells each: 84; strips of 16
// columns, one workgroup per compute unit, 164); 128 grids of 256^2 with v = 0 throughout: 62 us a call
// (strips of rows: 377, of columns: 90).
template <int LOGN, bool UNIFORM, bool COUNT>
__global__ __launch_bounds__(kGridThreads) void k_grid_full(GridArgs a) {
  using Cfg = GridCfg<LOGN>;
  constexpr int N = 1 << LOGN, H = Cfg::H, W = Cfg::W, PART = H * W, PARTS = Cfg::PARTS;
  constexpr int TR = N / H, TC = N / Cfg::TW, STRIPS = TR * TC;
  static_assert(STRIPS == N / Cfg::S && PART % 4 == 0, "a tile has as many cells as a strip");
  constexpr bool COUNTS = UNIFORM || COUNT;
  __shared__ __align__(16) float2 sbuf[PART];
  __shared__ __align__(16) unsigned scnt[COUNTS ? PART : 4];
  __shared__ int s_tmp;
  const unsigned share = PARTS * a.P, sub = blockIdx.x / 8 % share, item = blockIdx.x / (8 * share) * 8 + blockIdx.x % 8;
  if (item >= (unsigned)a.Q * STRIPS) return;      // uniform over the workgroup
  const int tile = item / a.Q, tcl = item - tile * a.Q, p = sub / PARTS, img = tcl * a.P + p;
  const int jr = tile / TC, tr = jr & 1 ? TR - 1 - jr / 2 : jr / 2, tc = tile % TC, strip = tr * TC + tc;
  const int row0 = tr * H, col0 = tc * Cfg::TW;
  // of two parts, one takes the left columns of the tile's upper rows and the right ones of its lower rows
  static_assert(PARTS == 1 || PARTS == 2, "parts of a tile");
  const int part = (sub + item / 8) % PARTS;       // (in turn, so that busy parts don't meet on every other compute unit)
  auto left = [&](int row) { return PARTS == 1 ? 0 : W * (part ^ (row / (H / 2))); };
  const int* so = a.strip_off + (size_t)tcl * (STRIPS + 1);
  const int o0 = so[strip], o1 = so[strip + 1];
  const int2* plc = a.plc + (size_t)tcl * 2 * a.B;
  const float2* V = a.vis + (size_t)img * a.B;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int i = threadIdx.x; i < PART / 2; i += kGridThreads) reinterpret_cast<float4*>(sbuf)[i] = zero;
  if constexpr (COUNTS)
    for (int i = threadIdx.x; i < PART / 4; i += kGridThreads) reinterpret_cast<float4*>(scnt)[i] = zero;
  if (threadIdx.x == 0) s_tmp = 0;
  __syncthreads();
  // The strips at the centre hold thousands of records: four of a thread's loads are in flight
  // together, unconditional (their index clamped), and then the visibilities that fall in the part.
  for (int i = o0 + (int)threadIdx.x; i < o1; i += kGridBatch * kGridThreads) {
    int2 r[kGridBatch];
    float2 v[kGridBatch];
#pragma unroll
    for (int j = 0; j < kGridBatch; ++j) r[j] = plc[i + j * kGridThreads < o1 ? i + j * kGridThreads : o0];
#pragma unroll
    for (int j = 0; j < kGridBatch; ++j) {
      const int row = (r[j].x >> LOGN) - row0, col = (r[j].x & (N - 1)) - col0 - left(row);
      const bool in = i + j * kGridThreads < o1 && (unsigned)col < (unsigned)W;
      r[j].x = in ? row * W + col : -1;
      v[j] = V[in ? r[j].y & 0x7fffffff : 0];
    }
#pragma unroll
    for (int j = 0; j < kGridBatch; ++j)
      if (r[j].x >= 0) {
        atomicAdd(&sbuf[r[j].x].x, v[j].x);
        atomicAdd(&sbuf[r[j].x].y, r[j].y < 0 ? -v[j].y : v[j].y);
        if constexpr (COUNTS) atomicAdd(&scnt[r[j].x], 1u);
      }
  }
  __syncthreads();
  if constexpr (UNIFORM) {
    int occ = 0;
    for (int i = threadIdx.x; i < PART; i += kGridThreads) {
      const unsigned n = scnt[i];
      if (n) {
        const float inv = 1.0f / (float)n;
        sbuf[i].x *= inv;
        sbuf[i].y *= inv;
        ++occ;
      }
    }
    block_add_to_global(occ, &s_tmp, a.occ + img);
    __syncthreads();
  }
  // where cell i of the part (its row i / W, column i % W) lies from the tile's first
  auto at = [&](int i) { return (size_t)(i / W) * N + left(i / W) + i % W; };
  const size_t cell0 = (size_t)row0 * N + col0;
  float2* G = a.grids + (size_t)img * N * N + cell0;
  if (((uintptr_t)a.grids & 15) == 0) {
    for (int i = 2 * threadIdx.x; i < PART; i += 2 * kGridThreads)
      *reinterpret_cast<float4*>(G + at(i)) = *reinterpret_cast<const float4*>(sbuf + i);
  } else {                                         // the caller's array may start at any complex value
    for (int i = threadIdx.x; i < PART; i += kGridThreads) G[at(i)] = sbuf[i];
  }
  if constexpr (COUNT) {
    if (p == 0) {
      int32_t* cnt = a.counts + (size_t)tcl * N * N + cell0;
      if (((uintptr_t)a.counts & 15) == 0) {
        for (int i = 4 * threadIdx.x; i < PART; i += 4 * kGridThreads)
          *reinterpret_cast<int4*>(cnt + at(i)) = *reinterpret_cast<const int4*>(scnt + i);
      } else {
        for (int i = threadIdx.x; i < PART; i += kGridThreads) cnt[at(i)] = (int32_t)scnt[i];
      }
    }
  }
}

// ---------------------------------------------------------------- weights
// Images img0 .. img0+n_img-1 of a chunk: W from the pair's kept count (natural) or the image's
// occupancy (uniform); inv_w and weight_sum are indexed by the chunk image index.
__global__ void k_image_weights(const int* n_kept, const int* occ, int uniform, int P, int img0, int n_img,
                                float* inv_w, double* weight_sum) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_img) return;
  const int i = img0 + j;
  const int W = uniform ? occ[i] : 2 * n_kept[i / P];
  if (inv_w) inv_w[i] = W > 0 ? (float)(1.0 / (double)W) : 0.f;
  if (weight_sum) weight_sum[i] = (double)W;
}

hipError_t launch_image_weights(const int* n_kept, const int* occ, int uniform, int P, int img0, int n_img,
                                float* inv_w, double* weight_sum, hipStream_t s) {
  if (n_img <= 0) return hipSuccess;
  k_image_weights<<<(n_img + 255) / 256, 256, 0, s>>>(n_kept, occ, uniform, P, img0, n_img, inv_w, weight_sum);
  return hipGetLastError();
}

// Strip-width and row-block options compiled for each size (largest first).
template <int LOGN>
struct Options {
  static hipError_t run(bool uniform, int* col, int* ncol, int* row, int* nrow, int* grid) {
    const int sm = uniform ? ColSmax<LOGN, true>::value : ColSmax<LOGN, false>::value;
    *ncol = 0;
    for (int k = 0; k < (LOGN >= kTunedLogn ? 3 : 1); ++k)
      if ((sm >> k) >= 1) col[(*ncol)++] = sm >> k;
    *nrow = 0;
    if (LOGN >= kTunedLogn) {
      if (RowFits<LOGN, 8>::value) row[(*nrow)++] = 8;
      if (RowFits<LOGN, 4>::value) row[(*nrow)++] = 4;
      if (RowFits<LOGN, 2>::value) row[(*nrow)++] = 2;
      if (RowFits<LOGN, 1>::value) row[(*nrow)++] = 1;
    } else {
      row[(*nrow)++] = RowDefault<LOGN>::value;
    }
    *grid = GridCfg<LOGN>::S;
    return hipSuccess;
  }
};

int col_strip_options(int logn, bool uniform, int* out) {
  int col[4], row[4], nc = 0, nr = 0, g = 0;
  if (by_logn<Options>(logn, uniform, col, &nc, row, &nr, &g) != hipSuccess) return 0;
  for (int i = 0; i < nc; ++i) out[i] = col[i];
  return nc;
}

int row_block_options(int logn, int* out) {
  int col[4], row[4], nc = 0, nr = 0, g = 0;
  if (by_logn<Options>(logn, false, col, &nc, row, &nr, &g) != hipSuccess) return 0;
  for (int i = 0; i < nr; ++i) out[i] = row[i];
  return nr;
}

int grid_strip_width(int logn) {
  int col[4], row[4], nc = 0, nr = 0, g = 0;
  (void)by_logn<Options>(logn, false, col, &nc, row, &nr, &g);
  return g;
}

template <int LOGN>
struct GridFullL {
  static hipError_t run(const GridArgs* a, hipStream_t s) {
    using Cfg = GridCfg<LOGN>;
    const long items = (long)a->Q * (Cfg::N / Cfg::S), blocks = (items + 7) / 8 * 8 * Cfg::PARTS * a->P;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)blocks;
    if (a->uniform && a->counts) k_grid_full<LOGN, true, true><<<grid, kGridThreads, 0, s>>>(*a);
    else if (a->uniform) k_grid_full<LOGN, true, false><<<grid, kGridThreads, 0, s>>>(*a);
    else if (a->counts) k_grid_full<LOGN, false, true><<<grid, kGridThreads, 0, s>>>(*a);
    else k_grid_full<LOGN, false, false><<<grid, kGridThreads, 0, s>>>(*a);
    return hipGetLastError();
  }
};

hipError_t launch_grid_full(const GridArgs& a, hipStream_t s) {
  if (a.Q <= 0) return hipSuccess;
  return by_logn<GridFullL>(a.logn, &a, s);
}

// ---------------------------------------------------------------- FFT launchers
template struct PrecLaunch<BLINK_PREC_FP32>;

hipError_t launch_grid_colfft(const ColArgs& a, int n_img, int strip, int prec, const float2* tw, hipStream_t s) {
  switch (prec) {
    case BLINK_PREC_FP32: return PrecLaunch<BLINK_PREC_FP32>::grid_colfft(a, n_img, strip, tw, s);
    case BLINK_PREC_SPLIT_F16: return PrecLaunch<BLINK_PREC_SPLIT_F16>::grid_colfft(a, n_img, strip, tw, s);
    case BLINK_PREC_SPLIT_BF16: return PrecLaunch<BLINK_PREC_SPLIT_BF16>::grid_colfft(a, n_img, strip, tw, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_dense_colfft(const float2* grids, int n_img, int logn, int shift, int prec, float2* H,
                               const float2* tw, const uint4* ops, hipStream_t s) {
  switch (prec) {
    case BLINK_PREC_FP32: return PrecLaunch<BLINK_PREC_FP32>::dense_colfft(grids, n_img, logn, shift, H, tw, ops, s);
    case BLINK_PREC_SPLIT_F16:
      return PrecLaunch<BLINK_PREC_SPLIT_F16>::dense_colfft(grids, n_img, logn, shift, H, tw, ops, s);
    case BLINK_PREC_SPLIT_BF16:
      return PrecLaunch<BLINK_PREC_SPLIT_BF16>::dense_colfft(grids, n_img, logn, shift, H, tw, ops, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_chunk_colfft(const DescArgs& a, int chunk, int logn, int strip, int col_loop, int slots, int prec,
                               hipStream_t s) {
  switch (prec) {
    case BLINK_PREC_FP32: return StagedLaunch<BLINK_PREC_FP32>::colfft(a, chunk, logn, strip, col_loop, slots, s);
    case BLINK_PREC_SPLIT_F16:
      return StagedLaunch<BLINK_PREC_SPLIT_F16>::colfft(a, chunk, logn, strip, col_loop, slots, s);
    case BLINK_PREC_SPLIT_BF16:
      return StagedLaunch<BLINK_PREC_SPLIT_BF16>::colfft(a, chunk, logn, strip, col_loop, slots, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_chunk_row(const DescArgs& a, int chunk, int logn, int tpb, int slots, int prec, hipStream_t s) {
  switch (prec) {
    case BLINK_PREC_FP32: return StagedLaunch<BLINK_PREC_FP32>::row(a, chunk, logn, tpb, slots, s);
    case BLINK_PREC_SPLIT_F16: return StagedLaunch<BLINK_PREC_SPLIT_F16>::row(a, chunk, logn, tpb, slots, s);
    case BLINK_PREC_SPLIT_BF16: return StagedLaunch<BLINK_PREC_SPLIT_BF16>::row(a, chunk, logn, tpb, slots, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_row_c2r(const RowArgs& a, int n_img, int tpb, int prec, const float2* tw, hipStream_t s) {
  switch (prec) {
    case BLINK_PREC_FP32: return PrecLaunch<BLINK_PREC_FP32>::row_c2r(a, n_img, tpb, tw, s);
    case BLINK_PREC_SPLIT_F16: return PrecLaunch<BLINK_PREC_SPLIT_F16>::row_c2r(a, n_img, tpb, tw, s);
    case BLINK_PREC_SPLIT_BF16: return PrecLaunch<BLINK_PREC_SPLIT_BF16>::row_c2r(a, n_img, tpb, tw, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace blink
