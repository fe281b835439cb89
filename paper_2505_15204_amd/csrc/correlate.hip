// correlate.hip — the correlator (Section 4, Eq. 3; Section 6.2.2) on the matrix cores.
//
// For one integration interval and one output channel the visibilities of all input pairs form
// R = X X^H, X the complex int8 voltages of the 2A inputs (antenna, polarisation) over the
// K = n_int n_favg (sample, fine channel) terms. Each input's terms are kept as interleaved
// (re, im) byte pairs, so one int8 dot product over 2K bytes gives, for rows r and c,
//   (re, im)_r . (re, im)_c = sum Xr[r] Xr[c] + Xi[r] Xi[c]       = Re R[r][c]
//   (im, ~re)_r . (re, im)_c = sum Xi[r] Xr[c] + (~Xr[r]) Xi[c]  = Im R[r][c] - sum Xi[c]
// with ~x = -x - 1 the bitwise complement (exact in int8, unlike -x for x = -128); the per-input
// sum of Xi over K is added back at the end. Both byte layouts are staged in LDS (planes P and
// Q), so the products read their operands directly. Each 32 x 32 output tile therefore needs two
// int32 accumulators and two v_mfma_i32_32x32x32_i8 per 16 terms, all exact
// (|R| <= 2 K 128^2 < 2^31 for K <= 65535). Only the tiles on or below the diagonal are
// formed. A workgroup of 12 waves owns up to 36 tiles (three per wave, along tile rows so that a
// row's operands are read once per step) of one (interval, channel), all of them up to 128
// antennas, so every input is staged once, and keeps their accumulators in registers over all of
// K; K is staged through LDS in chunks of 64 terms (each input's 128 bytes contiguous), and the
// global loads of the next chunk are issued before the current chunk's matrix products.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch.hpp"

namespace blink {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kTile = 32;                 // MFMA tile (inputs)
constexpr int kKc = 64;                   // terms per LDS chunk
constexpr int kRow = 2 * kKc + 16;        // LDS row stride in bytes (spreads rows over the banks)
constexpr int kTilesPerWave = 3;
constexpr int kWaves = 12;
constexpr int kTilesPerGroup = kTilesPerWave * kWaves;
constexpr int kThreads = 64 * kWaves;
constexpr int kOctets = kKc / 8;               // 8-term octets per chunk
constexpr int kItemsPerSlab = 4 * kOctets;     // (8-input group, 8-term octet) pairs per 32-input slab

// Tile tau of the lower triangle in row order: (a, b), b <= a, tau = a (a + 1) / 2 + b (at most
// 16 tile rows).
__device__ __forceinline__ void tile_of(int tau, int& a, int& b) {
  int r = 0;
  while ((r + 1) * (r + 2) / 2 <= tau) ++r;
  a = r;
  b = tau - r * (r + 1) / 2;
}

// (float)((double)x / K) for an integer |x| < 2^31 and K <= 65535, without a division: with inv the
// correctly rounded 1 / K, q = x inv is within an ulp of x / K, the fma forms its remainder exactly,
// and q + r inv rounds to the correctly rounded quotient (Markstein 1990).
__device__ __forceinline__ float mean_rn(int x, double K, double inv) {
  const double d = (double)x, q = d * inv;
  return (float)fma(fma(-K, q, d), inv, q);
}

// One staging item: 16 bytes (8 inputs, re and im) for each of 8 consecutive terms.
struct Staged {
  uint4 w[8];
};

// A workgroup of 12 waves owns 36 tiles: every tile of one (interval, channel) up to 128 antennas
// (8 slabs), so each input is staged once per chunk; larger arrays take several workgroups. Each
// thread stages at most one item (n_slabs * kItemsPerSlab <= 512 items up to 256 antennas).
// With DB (two plane buffers, up to 8 slabs) the staging waves store chunk i + 1 into one buffer
// while every wave forms chunk i's products from the other: one barrier per chunk, and the other
// waves' matrix products cover the staging's byte permutes on each SIMD.
template <bool DB>
__global__ __launch_bounds__(kThreads, 1) void k_correlate(CorrelateArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int IP = a.n_slabs * kTile;               // padded input count
  const size_t plane = (size_t)IP * kRow;
  unsigned char* x0 = lds;                        // plane P [IP][kRow]: (re, im) pairs, terms contiguous
  unsigned char* xq0 = lds + plane;               // plane Q [IP][kRow]: (im, ~re) pairs
  unsigned char* x1 = DB ? lds + 2 * plane : x0;  // second buffer (DB)
  unsigned char* xq1 = DB ? lds + 3 * plane : xq0;
  int* colsum = reinterpret_cast<int*>(lds + (DB ? 4 : 2) * plane);   // [IP]: sum of Xi over K
  __shared__ unsigned s_need;                     // bit s: slab s is used by this workgroup

  // Workgroups are dispatched to the 8 XCDs in turn (workgroup w to XCD w % 8): the n_groups
  // workgroups of one (interval, channel) pair are w, w + 8, ..., so they share one XCD's L2 and
  // the voltages they all stage are read from HBM once.
  const long w = blockIdx.x, span = 8L * a.n_groups;
  const int group = (int)((w % span) / 8);
  const long pair = (w / span) * 8 + w % 8;
  if (pair >= (long)a.T * a.C) return;             // padding workgroups of the last span
  const int t = (int)(pair / a.C), c = (int)(pair % a.C);
  const int ntiles = a.n_slabs * (a.n_slabs + 1) / 2;
  const int tau0 = group * kTilesPerGroup;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = (int)threadIdx.x % 64;
  const int n = lane % 32, g = lane / 32;
  int ta[kTilesPerWave], tb[kTilesPerWave], tv[kTilesPerWave];
#pragma unroll
  for (int u = 0; u < kTilesPerWave; ++u) {
    const int tau = tau0 + wave * kTilesPerWave + u;
    tv[u] = tau < ntiles;
    if (tv[u]) tile_of(tau, ta[u], tb[u]);
    else ta[u] = tb[u] = 0;
  }
  for (int i = threadIdx.x; i < IP; i += kThreads) colsum[i] = 0;
  if (threadIdx.x == 0) {
    unsigned need = 0;
    for (int k = 0; k < kTilesPerGroup && tau0 + k < ntiles; ++k) {
      int y, z;
      tile_of(tau0 + k, y, z);
      need |= (1u << y) | (1u << z);
    }
    s_need = need;
  }

  v16i re[kTilesPerWave], im[kTilesPerWave];
#pragma unroll
  for (int u = 0; u < kTilesPerWave; ++u) re[u] = im[u] = v16i{};

  const int K = a.n_int * a.n_favg;
  const int in2 = 2 * a.A;                          // inputs (antenna, polarisation)
  const size_t rec = (size_t)in2 * 2;               // bytes per (sample, fine channel)
  const int n_items = a.n_slabs * kItemsPerSlab;
  __syncthreads();
  const unsigned need = s_need;

  // item -> (8-input group rg, term octet o): consecutive items are the 8 octets of one input
  // group, so a global load of a wave reads 128-byte runs (8 groups) of 8 records, and the LDS
  // rows are stored without a swizzle: with the 144-byte row stride (9 16-byte slots) the 16
  // lanes of one LDS cycle write rows r and r + 8 of their groups at octets 0..7, slots 9 row + o,
  // all distinct modulo 16, and the operand reads (16 consecutive rows, one octet) are distinct too
  const int item = (int)threadIdx.x;
  const int o = item % kOctets, rg = item / kOctets, row0 = rg * 8, slab = rg / 4;
  const bool staged = item < n_items && ((need >> slab) & 1u);   // this thread writes rows of P, Q
  const bool on = staged && row0 < in2;                           // ... and loads voltages for them
  // global loads of one chunk's item of this thread (unused slabs, inputs past 2A and terms past K
  // are not loaded and stage zeros). Term k is (sample k / n_favg, fine channel k % n_favg) of the
  // block; one division per chunk.
  auto load = [&](int k0, Staged& st) {
    const int kb = k0 + 8 * o;
    int sl = kb / a.n_favg, fl = kb - sl * a.n_favg;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      st.w[e] = make_uint4(0, 0, 0, 0);
      if (on && kb + e < K) {
        const size_t at = ((size_t)(t * a.n_int + sl) * a.F + (size_t)(c * a.n_favg + fl)) * rec + (size_t)row0 * 2;
        st.w[e] = *reinterpret_cast<const uint4*>(a.volt + at);
      }
      if (++fl == a.n_favg) {
        fl = 0;
        ++sl;
      }
    }
  };
  // transpose: row row0 + r gets the (re, im) pairs of its 8 terms as one 16-byte vector in P and
  // the (im, ~re) pairs in Q (byte permutes of two loaded words each). The chunk's imaginary parts
  // of each row are added to colsum: the eight lanes of an input group hold the group's rows' sums
  // over their octets, and exchange them so that lane o adds the total of row o, one LDS atomic to
  // distinct words in place of eight with eight lanes on each (768 products of 128 antennas and 800
  // terms: 243 -> 216 us).
  auto store = [&](const Staged& st, unsigned char* x, unsigned char* xq) {
    if (staged) {
      int part[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        // v_perm_b32 byte selectors (0-3: bytes of the second source, 4-7: of the first): row r's
        // (re, im) pair is bytes j, j + 1 of its word, j = 2 (r % 2)
        const unsigned j = 2u * (r % 2);
        const unsigned sel_p = j | (j + 1) << 8 | (j + 4) << 16 | (j + 5) << 24;
        const unsigned sel_q = (j + 1) | j << 8 | (j + 5) << 16 | (j + 4) << 24;
        unsigned d[4], e[4];
        int isum = 0;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const uint4& w0 = st.w[2 * h];
          const uint4& w1 = st.w[2 * h + 1];
          const unsigned a0 = r < 2 ? w0.x : r < 4 ? w0.y : r < 6 ? w0.z : w0.w;
          const unsigned a1 = r < 2 ? w1.x : r < 4 ? w1.y : r < 6 ? w1.z : w1.w;
          d[h] = __builtin_amdgcn_perm(a1, a0, sel_p);                 // (re, im) of terms 2h, 2h + 1
          e[h] = __builtin_amdgcn_perm(a1, a0, sel_q) ^ 0xff00ff00u;   // (im, ~re)
          isum = __builtin_amdgcn_sdot4((int)d[h], 0x01000100, isum, false);   // the two im bytes
        }
        const size_t at = (size_t)(row0 + r) * kRow + 16 * o;
        *reinterpret_cast<uint4*>(x + at) = make_uint4(d[0], d[1], d[2], d[3]);
        *reinterpret_cast<uint4*>(xq + at) = make_uint4(e[0], e[1], e[2], e[3]);
        part[r] = isum;
      }
      // keep the half of the rows that this lane ends with, hand its partner the other half
      const bool h4 = o & 4, h2 = o & 2, h1 = o & 1;
      int q4[4], q2[2];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        q4[r] = (h4 ? part[r + 4] : part[r]) +
                __builtin_amdgcn_update_dpp(0, h4 ? part[r] : part[r + 4], 0x141, 0xf, 0xf, true);   // lane 7 - o
#pragma unroll
      for (int r = 0; r < 2; ++r)
        q2[r] = (h2 ? q4[r + 2] : q4[r]) +
                __builtin_amdgcn_update_dpp(0, h2 ? q4[r] : q4[r + 2], 0x4e, 0xf, 0xf, true);        // lane o ^ 2
      const int sum = (h1 ? q2[1] : q2[0]) + __builtin_amdgcn_update_dpp(0, h1 ? q2[0] : q2[1], 0xb1, 0xf, 0xf, true);
      atomicAdd(&colsum[row0 + o], sum);
    }
  };

  // the products of one staged chunk: the wave's tiles run along tile rows (row order), so the
  // row operands A and As are read once per tile row and step and reused by the following tiles
  // of that row
  auto products = [&](const unsigned char* x, const unsigned char* xq) {
#pragma unroll
    for (int kk = 0; kk < 2 * kKc; kk += 32) {
      const int q = kk / 16 + g;                    // this lane's term octet of the step
      v4i A = {}, As = {};
      int cur = -1;
#pragma unroll
      for (int u = 0; u < kTilesPerWave; ++u) {
        if (!tv[u]) continue;
        if (ta[u] != cur) {
          cur = ta[u];
          const int rowa = cur * kTile + n;
          const size_t oa = (size_t)rowa * kRow + 16 * q;
          A = *reinterpret_cast<const v4i*>(x + oa);
          As = *reinterpret_cast<const v4i*>(xq + oa);
        }
        const int rowb = tb[u] * kTile + n;
        const v4i B = *reinterpret_cast<const v4i*>(x + (size_t)rowb * kRow + 16 * q);
        re[u] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, B, re[u], 0, 0, 0);
        im[u] = __builtin_amdgcn_mfma_i32_32x32x32_i8(As, B, im[u], 0, 0, 0);
      }
    }
  };
  Staged st;
  load(0, st);
  if constexpr (DB) {
    // chunk i + 1 (loaded during chunk i - 1) is stored into the free buffer and chunk i + 2
    // requested before chunk i's products; the barrier closes both the products' reads of one
    // buffer and the stores into the other
    store(st, x0, xq0);
    if (kKc < K) load(kKc, st);
    __syncthreads();
    int i = 0;
    for (int k0 = 0; k0 < K; k0 += kKc, ++i) {
      if (k0 + kKc < K) {
        store(st, (i & 1) ? x0 : x1, (i & 1) ? xq0 : xq1);
        if (k0 + 2 * kKc < K) load(k0 + 2 * kKc, st);
      }
      products((i & 1) ? x1 : x0, (i & 1) ? xq1 : xq0);
      __syncthreads();
    }
  } else {
    // one buffer: stage the registers into LDS, request the next chunk (answered during this
    // chunk's products), then the products
    for (int k0 = 0; k0 < K; k0 += kKc) {
      store(st, x0, xq0);
      __syncthreads();
      if (k0 + kKc < K) load(k0 + kKc, st);
      products(x0, xq0);
      __syncthreads();   // the chunk's operands are read before the next chunk overwrites them
    }
  }

  // Output: element v of the lane is R[32 a + 8 (v / 4) + 4 g + v % 4][32 b + n].
  const double Kd = (double)K, inv = 1.0 / Kd;
  const int B = (int)((long)a.A * (a.A - 1) / 2);
  float2* vis = a.vis + ((size_t)t * a.C + c) * a.pol_mode * B;
#pragma unroll
  for (int u = 0; u < kTilesPerWave; ++u) {
    if (!tv[u]) continue;
    const int ci = tb[u] * kTile + n;
    const int csum = ci < in2 ? colsum[ci] : 0;
    const int j = ci / 2, q = ci % 2;
    // Im R = im + csum fits in int32 (|R| <= 2 K 128^2 < 2^31); the sum is formed modulo 2^32
    auto value = [&](int v) {
      return make_float2(mean_rn(re[u][v], Kd, inv), mean_rn((int)((unsigned)im[u][v] + (unsigned)csum), Kd, inv));
    };
    if (ta[u] > tb[u] && (ta[u] + 1) * kTile <= in2 && a.pol_mode == 4) {
      // whole tile below the diagonal: every element is a baseline's (uniform over the wave); without
      // the tests per element and with 32-bit offsets 216 -> 199 us for the same products
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const int i = ta[u] * (kTile / 2) + 4 * (v / 4) + 2 * g + v % 4 / 2, b = i * (i - 1) / 2 + j + q * B;
        vis[b] = value(v);
        vis[b + 2 * B] = value(v + 1);
      }
      continue;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int ri = ta[u] * kTile + 8 * (v / 4) + 4 * g + v % 4;
      if (ri >= in2 || ci >= in2) continue;
      const int i = ri / 2, p = ri % 2;
      if (i < j) continue;
      const float2 r = value(v);
      if (i == j) {
        if (a.autos) a.autos[(((size_t)t * a.C + c) * a.A + i) * 4 + 2 * p + q] = r;
        continue;
      }
      int pp;
      if (a.pol_mode == 4) pp = 2 * p + q;
      else if (p == q) pp = p;
      else continue;
      vis[(size_t)pp * B + (i * (i - 1) / 2 + j)] = r;
    }
  }
}

}  // namespace

// Two plane buffers when they fit the 160 KB of LDS (up to 8 slabs, 128 antennas), else one.
static bool correlate_db(int slabs) { return (size_t)slabs * kTile * (4 * kRow + sizeof(int)) <= 160 * 1024; }

size_t correlate_lds_bytes(int A) {
  const int slabs = (2 * A + kTile - 1) / kTile;
  return (size_t)slabs * kTile * ((correlate_db(slabs) ? 4 : 2) * kRow + sizeof(int));
}

hipError_t launch_correlate(const CorrelateArgs& a, hipStream_t s) {
  const int T = a.S / a.n_int, C = a.F / a.n_favg;
  if (T == 0 || C == 0) return hipSuccess;
  const int ntiles = a.n_slabs * (a.n_slabs + 1) / 2;
  const int n_groups = (ntiles + kTilesPerGroup - 1) / kTilesPerGroup;
  const long n_wg = 8L * n_groups * (((long)T * C + 7) / 8);
  if (n_wg > 0x7fffffffL) return hipErrorInvalidValue;
  CorrelateArgs b = a;
  b.C = C;
  b.T = T;
  b.n_groups = n_groups;
  const unsigned grid = (unsigned)n_wg;
  const size_t lds_bytes = correlate_lds_bytes(a.A);
  if (a.n_slabs * kItemsPerSlab > kThreads) return hipErrorInvalidValue;   // one item per thread
  const bool db = correlate_db(a.n_slabs);
  const void* fn = db ? reinterpret_cast<const void*>(k_correlate<true>)
                      : reinterpret_cast<const void*>(k_correlate<false>);
  if (lds_bytes > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
  }
  if (db) k_correlate<true><<<grid, kThreads, lds_bytes, s>>>(b);
  else k_correlate<false><<<grid, kThreads, lds_bytes, s>>>(b);
  return hipGetLastError();
}

}  // namespace blink
