// fold_bin.hip — binning for the folded imaging path (fold_device.hpp): cell indices, the
// segments of folded cells, and every image's placement values in the segments' order.
#include "fold_device.hpp"

namespace blink {
namespace {

constexpr int kFoldThreads = 1024;
constexpr int kFoldWaves = kFoldThreads / 64;
constexpr int kFoldLoad = 4;                     // baselines per thread whose loads are in flight together
constexpr int kFields = kFoldDiag / 2 + 1;       // packed counters: two segment lengths per word, placements beyond
constexpr int kFoldLong = 4 * 64;                // placements of a segment above which the workgroup counts them
static_assert(kFoldDiag == 16 && kFoldCells <= 8 * kFoldThreads, "lengths are counted in the 16 bytes of two words");

// STAGE: bytes of the area in which placement records and values are put in order before they are
// written, so that global memory sees contiguous stores only.
template <int STAGE>
struct FoldShared {
  union {
    unsigned cell[kFoldCells];                   // placements of each folded cell, then segment | beyond << 14
    uint32_t rec[STAGE / 4];
    float2 val[STAGE / 8];
  };
  unsigned part[kFields][kFoldWaves];            // per-wave totals, then their exclusive sums
  unsigned total[kFields];
  int joff[kFoldDiag + 1], cum[kFoldDiag];
  int kept, outside, ext, occ;
  uint16_t deep[2 * kFoldMaxB / kFoldDiag];  // segments that fill the diagonals: their first placement beyond
  unsigned hist[kFoldThreads];                   // placements of one segment by factor index (at most 1024)
  uint16_t longest[2 * kFoldMaxB / kFoldLong];   // segments longer than kFoldLong
  int n_long;
};

// Field i (16 bits) of packed words.
__device__ __forceinline__ int field(const unsigned (&f)[kFields], int i) {
  unsigned v = f[0];
#pragma unroll
  for (int k = 1; k < kFoldDiag / 2; ++k) v = (i >> 1) == k ? f[k] : v;
  return (int)((v >> (16 * (i & 1))) & 0xffffu);
}

// Uniform weighting: the weight of every placement, one over the placements of its grid cell (equal records in
// its segment), to wts; returns how many cells of the image the first placements of this thread's cells occupy.
// All records are in the LDS.
//
// Segments within the diagonals: a thread each (the longest first, so the lanes of a wave have nearly equal
// work), whose records it holds in registers. Longer ones (a dense core, a compact array, a small field): a wave
// each, whose lanes find their equals by ballots; the longest are counted by their factor index. One
// image of 1024^2 with 8128 placements in one cell took 8.4 ms where every placement compared itself with
// its whole segment, 48 us now (natural weighting: 45).
template <int STAGE>
__device__ __forceinline__ int fold_weights(FoldShared<STAGE>& sh, int over0, int n_over, int logn, int logm,
                                            float* __restrict__ wts) {
  const int N = 1 << logn, logr = logn - logm;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int full = __builtin_amdgcn_readfirstlane(sh.cum[kFoldDiag - 1]);
  int occ = 0;
  // of a placement and its mirror: column 0, the first of each half of a row pair, holds both by itself
  const unsigned inv = 0xffffffffu / (unsigned)padded_len(N) + 1u;   // exact for 15 bits by 4353 at most
  auto cells_of = [&](uint32_t r) {
    const unsigned key = r >> 17, in_pair = key - __umulhi(key, inv) * (unsigned)padded_len(N);
    return in_pair == 0u || in_pair == (unsigned)pad_index(N / 2) ? 1 : 2;
  };
  auto beyond = [&](int s) { return s < full ? (s + 1 < full ? (int)sh.deep[s + 1] : n_over) - (int)sh.deep[s] : 0; };
  auto segment = [&](int s, auto depth) {
    constexpr int D = decltype(depth)::value;
    uint32_t r[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int cum = __builtin_amdgcn_readfirstlane(sh.cum[j]), off = __builtin_amdgcn_readfirstlane(sh.joff[j]);
      r[j] = s < cum ? sh.rec[off + s] : ~(uint32_t)j;
    }
#pragma unroll 1
    for (int i = 0; i < D && s < sh.cum[i]; ++i) {
      const int pos = sh.joff[i] + s;
      const uint32_t own = sh.rec[pos];
      int n = 0, first = D;
#pragma unroll
      for (int j = D - 1; j >= 0; --j) {
        n += r[j] == own;
        first = r[j] == own ? j : first;
      }
      if (first == i) occ += cells_of(own);
      wts[pos] = 1.0f / (float)n;
    }
  };
#pragma unroll 1
  for (int s = tid; s < sh.cum[0]; s += kFoldThreads) {
    asm volatile("" ::: "memory");               // the offsets are read again, not kept in registers
    const int s0 = __builtin_amdgcn_readfirstlane(s - lane);   // the longest of the wave's segments
    if (beyond(s) > 0) continue;
    if (s0 >= sh.cum[1]) segment(s, std::integral_constant<int, 1>{});
    else if (s0 >= sh.cum[2]) segment(s, std::integral_constant<int, 2>{});
    else if (s0 >= sh.cum[4]) segment(s, std::integral_constant<int, 4>{});
    else if (s0 >= sh.cum[8]) segment(s, std::integral_constant<int, 8>{});
    else segment(s, std::integral_constant<int, kFoldDiag>{});
  }
#pragma unroll 1
  for (int s = wave; s < full; s += kFoldWaves) {
    const int n = __builtin_amdgcn_readfirstlane(kFoldDiag + beyond(s)), x = over0 + sh.deep[s] - kFoldDiag;
    if (n == kFoldDiag) continue;
    auto pos_of = [&](int i) { return i < kFoldDiag ? sh.joff[i] + s : x + i; };
    if (n > kFoldLong) {
      if (lane == 0) sh.longest[atomicAdd(&sh.n_long, 1)] = (uint16_t)s;
      continue;
    }
    // every 64 against every 64, through ballots over the bits of the factor index
#pragma unroll 1
    for (int a = 0; a < n; a += 64) {
      const bool in = a + lane < n;
      const int pos = pos_of(in ? a + lane : 0);
      const uint32_t r = sh.rec[pos];
      int equal = 0;
      bool first = true;
#pragma unroll 1
      for (int b = 0; b < n; b += 64) {
        const bool in_b = b + lane < n;
        const uint32_t rb = b == a ? r : sh.rec[pos_of(in_b ? b + lane : 0)];
        unsigned long long same = __ballot(in_b);    // the lanes whose index this lane's placement has
        for (int k = 3; k < 3 + logr; ++k) {
          const unsigned long long m = __ballot((rb >> k) & 1u);
          const int bit = __builtin_amdgcn_sbfe((int)r, k, 1);        // 0 or -1
          same &= ~(m ^ (unsigned long long)(long long)bit);
        }
        equal += __popcll(same);
        if (b < a) first = first && same == 0;
        else if (b == a) first = first && __ffsll(same) - 1 == lane;
      }
      if (in) {
        if (first) occ += cells_of(r);
        wts[pos] = 1.0f / (float)equal;
      }
    }
  }
  // the longest: counted by their factor index, all waves on one segment
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < sh.n_long; ++i) {
    const int s = sh.longest[i], n = kFoldDiag + beyond(s), x = over0 + sh.deep[s] - kFoldDiag;
    auto each = [&](auto f) {
#pragma unroll 1
      for (int j = tid; j < n; j += kFoldThreads) {
        const int pos = j < kFoldDiag ? sh.joff[j] + s : x + j;
        const uint32_t r = sh.rec[pos];
        f(pos, r, &sh.hist[(r & 0x1ff8u) >> 3]);
      }
      __syncthreads();
    };
    sh.hist[tid] = 0u;
    __syncthreads();
    each([&](int, uint32_t r, unsigned* w) {
      const unsigned long long all = __ballot(true);
      unsigned count = 1u;
      if (__ballot(r == (uint32_t)__builtin_amdgcn_readfirstlane((int)r)) == all) {   // a pile: one atomic for the wave
        if (lane != __ffsll(all) - 1) return;
        count = (unsigned)__popcll(all);
      }
      if (atomicAdd(w, count) == 0u) occ += cells_of(r);
    });
    each([&](int pos, uint32_t, unsigned* w) { wts[pos] = 1.0f / (float)*w; });
  }
  return occ;
}

// One workgroup bins one visibility set of at most NB * 1024 baselines, which every thread reads
// once and keeps in registers; the rank of a placement in its folded cell is what the counting
// pass's LDS atomic returns, so there is no second counting pass. A baseline on the u = 0 column
// has a second placement there, the mirror of the first.
template <int NB, bool UNIFORM, int STAGE>
__device__ __forceinline__ void fold_bin(const double* __restrict__ uvw, const uint8_t* __restrict__ fl, int B, double k,
                                         int logn, int logm, int shift, const float2* __restrict__ vis, int P,
                                         size_t vis_stride, FoldHeader* hdr, uint32_t* __restrict__ rows,
                                         uint32_t* __restrict__ rec, float2* __restrict__ val, size_t val_stride,
                                         int* nout_out, FoldShared<STAGE>& sh, uint32_t* __restrict__ place = nullptr,
                                         float2* __restrict__ coef = nullptr) {
  const int N = 1 << logn, mask = N - 1, HALF = N / 2, M = 1 << logm, cells = M * HALF;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double half = (double)HALF;
  for (int i = tid; i < cells; i += kFoldThreads) sh.cell[i] = 0u;
  if (tid == 0) sh.kept = sh.outside = sh.ext = sh.occ = sh.n_long = 0;
  __syncthreads();
  int code[NB];                                  // folded cell | h << 13 | conj << 24, or -1
  unsigned at[NB];                               // ranks of the placement and its mirror (16 bits each), later positions
  int kept = 0, outside = 0, ext = 0;
#pragma unroll
  for (int c = 0; c < NB; c += kFoldLoad) {
    double u[kFoldLoad], v[kFoldLoad];
    bool off[kFoldLoad];
#pragma unroll
    for (int i = 0; i < kFoldLoad; ++i) {
      const int b = (c + i) * kFoldThreads + tid, bs = b < B ? b : 0;
      u[i] = uvw[3 * (size_t)bs];
      v[i] = uvw[3 * (size_t)bs + 1];
      off[i] = fl ? fl[bs] != 0 : false;
      if (b >= B) off[i] = true;
    }
#pragma unroll
    for (int i = 0; i < kFoldLoad; ++i) {
      int iu, iv;
      code[c + i] = -1;
      at[c + i] = 0;
      if (off[i]) continue;
      if (nearest_cell(u[i], v[i], k, half, iu, iv)) {
        ++kept;
        const bool conj = iu < 0;
        const int ku = conj ? -iu : iu, kv = (conj ? -iv : iv) & mask;
        ext = ku + 1 > ext ? ku + 1 : ext;
        const int cell = (kv & (M - 1)) * HALF + ku;
        at[c + i] = atomicAdd(&sh.cell[cell], 1u);
        if (ku == 0) at[c + i] |= atomicAdd(&sh.cell[((-kv) & (M - 1)) * HALF], 1u) << 16;
        code[c + i] = cell | (kv >> logm) << 13 | (conj ? 1 << 24 : 0);
      } else {
        ++outside;
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    kept += __shfl_xor(kept, o, 64);
    outside += __shfl_xor(outside, o, 64);
    const int e = __shfl_xor(ext, o, 64);
    ext = e > ext ? e : ext;
  }
  if (lane == 0) {
    atomicAdd(&sh.kept, kept);
    atomicAdd(&sh.outside, outside);
    atomicMax(&sh.ext, ext);
  }
  __syncthreads();
  // Segments by length: exclusive scan over the threads of how many segments of each length (and
  // placements beyond the diagonals) their cells hold. A thread has at most 8 cells, so it counts
  // in the bytes of two 64-bit words; the scan runs on 16-bit fields (totals <= 8192).
  unsigned long long own8[2] = {};
  int own_over = 0;
  for (int i = tid; i < cells; i += kFoldThreads) {
    const int n = (int)sh.cell[i], cls = (n < kFoldDiag ? n : kFoldDiag) - 1;
    const unsigned long long one = 1ull << (8 * (cls & 7));
    if (n > 0) {
      own8[0] += cls < 8 ? one : 0ull;
      own8[1] += cls < 8 ? 0ull : one;
    }
    own_over += n > kFoldDiag ? n - kFoldDiag : 0;
  }
  unsigned run[kFields];
#pragma unroll
  for (int f = 0; f < kFields; ++f) {
    const unsigned b2 = f < kFoldDiag / 2 ? (unsigned)(own8[(f >> 2) & 1] >> (16 * (f & 3))) & 0xffffu : 0u;
    const unsigned own = f < kFoldDiag / 2 ? (b2 & 0xffu) | (b2 >> 8) << 16 : (unsigned)own_over;
    unsigned x = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    run[f] = x - own;
    if (lane == 63) sh.part[f][wave] = x;
  }
  __syncthreads();
  if (tid < kFields * kFoldWaves) {              // exclusive sums over the waves: 16 lanes per field
    const int f = tid / kFoldWaves, w = tid % kFoldWaves;
    const unsigned own = sh.part[f][w];
    unsigned x = own;
#pragma unroll
    for (int o = 1; o < kFoldWaves; o <<= 1) {
      const unsigned y = __shfl_up(x, o, kFoldWaves);
      if (w >= o) x += y;
    }
    sh.part[f][w] = x - own;
    if (w == kFoldWaves - 1) sh.total[f] = x;
  }
  __syncthreads();
  unsigned total[kFields];
#pragma unroll
  for (int f = 0; f < kFields; ++f) {
    run[f] += sh.part[f][wave];
    total[f] = sh.total[f];
  }
  int start = 0;
#pragma unroll
  for (int n = kFoldDiag - 1; n >= 0; --n) {     // segments of length n + 1 start behind the longer ones
    run[n >> 1] += (unsigned)start << (16 * (n & 1));
    start += (int)((total[n >> 1] >> (16 * (n & 1))) & 0xffffu);
    if (tid == 0) sh.cum[n] = start;
  }
  unsigned long long used[2] = {};               // this thread's segments of each length so far
  unsigned x0 = run[kFields - 1];
  for (int i = tid; i < cells; i += kFoldThreads) {
    const int n = (int)sh.cell[i];
    if (n == 0) continue;
    const int cls = (n < kFoldDiag ? n : kFoldDiag) - 1;
    const unsigned long long one = 1ull << (8 * (cls & 7)), have = cls < 8 ? used[0] : used[1];
    const int s = field(run, cls) + (int)((have >> (8 * (cls & 7))) & 0xffu);
    used[0] += cls < 8 ? one : 0ull;
    used[1] += cls < 8 ? 0ull : one;
    sh.cell[i] = (unsigned)s | x0 << 14;
    if (UNIFORM && n >= kFoldDiag) sh.deep[s] = (uint16_t)x0;   // (in the order of s)
    x0 += n > kFoldDiag ? (unsigned)(n - kFoldDiag) : 0u;
  }
  if (tid == 0) {
    int o = 0;
    for (int j = 0; j < kFoldDiag; ++j) {
      sh.joff[j] = o;
      o += (sh.cum[j] + 63) & ~63;               // whole rows
    }
    sh.joff[kFoldDiag] = o;
    hdr->first_over = o;
    hdr->n_over = (int)total[kFields - 1];
    hdr->ext = sh.ext;
    hdr->kept = sh.kept;
    if (nout_out) *nout_out = sh.outside;
  }
  __syncthreads();
  // Row table: the rows (diagonal j of 64 segments) of each wave of the imaging workgroup. Chunk
  // c of 64 segments goes to the waves in turn, forth and back, so that the long ones spread.
  {
    const int nw = (M << logn) >= 4096 ? (M << logn) / 2048 : 1, chunks = (sh.cum[0] + 63) / 64;
    auto depth = [&](int c) {                    // diagonals of chunk c
      int d = 0;
      for (int j = 0; j < kFoldDiag; ++j) d += sh.cum[j] > 64 * c;
      return d;
    };
    auto chunk_of = [&](int w, int t) { return t * nw + ((t & 1) ? nw - 1 - w : w); };
    if (tid < chunks) {
      const int t = tid / nw, w = (t & 1) ? nw - 1 - tid % nw : tid % nw, d = depth(tid);
      int o = 0;
      for (int p = 0; p < t; ++p) o += depth(chunk_of(w, p));
      for (int j = 0; j < d; ++j)
        rows[w * kFoldRowsPerWave + o + j] = (uint32_t)(sh.joff[j] + 64 * tid) | (j == 0 ? kFoldRowFirst : 0u) | (j == d - 1 ? kFoldRowLast : 0u);
    }
    if (tid < nw) {
      int o = 0;
      for (int p = 0; p * nw < chunks; ++p) o += depth(chunk_of(tid, p));
      hdr->rows[tid] = o;
      for (; o < 2 * kFoldRowBatch || o % kFoldRowBatch; ++o) rows[tid * kFoldRowsPerWave + o] = 0u;
    }
  }
  // positions of the placements
  const int over0 = sh.joff[kFoldDiag], n_ent = over0 + (int)total[kFields - 1];
  auto mirror = [&](int cell, int h) { return (-((h << logm) + (cell >> (logn - 1)))) & mask; };
  auto slot_of = [&](int cell, unsigned r) {
    const unsigned c = sh.cell[cell];
    return (unsigned)(r < kFoldDiag ? sh.joff[r] + (int)(c & 0x3fffu) : over0 + (int)(c >> 14) + (int)(r - kFoldDiag));
  };
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (code[i] < 0) continue;
    const int cell = code[i] & 0x1fff, h = (code[i] >> 13) & 0x7ff;
    unsigned p = slot_of(cell, at[i] & 0xffffu) | 0xffff0000u;
    if ((cell & (HALF - 1)) == 0) p = (p & 0xffffu) | slot_of((mirror(cell, h) & (M - 1)) * HALF, at[i] >> 16) << 16;
    at[i] = p;
  }
  __syncthreads();                               // the cells are no longer needed: the area stages records now
  // records: the factor's index h and the cell's LDS index in the imaging kernel
  auto record = [&](int cell, int h) {
    const int kk = cell >> (logn - 1), c = cell & (HALF - 1);
    const int idx = (kk >> 1) * padded_len(N) + pad_index((kk & 1) * HALF + c);
    return (uint32_t)(8 * h) | (uint32_t)idx << 17;
  };
  const uint32_t pad_rec = (uint32_t)((M / 2) * padded_len(N)) << 17;
  int pad_at = n_ent;                            // this thread's padding placement of the diagonals
  {
    const int j = tid / 64, p = sh.joff[j] + sh.cum[j] + lane;
    if (p < sh.joff[j + 1]) pad_at = p;
  }
  constexpr int RW = STAGE / 4, VW = STAGE / 8;
  for (int w0 = 0; w0 < n_ent; w0 += RW) {       // one window unless most baselines lie on the u = 0 column
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (code[i] < 0) continue;
      const int cell = code[i] & 0x1fff, h = (code[i] >> 13) & 0x7ff;
      const unsigned p = (at[i] & 0xffffu) - (unsigned)w0, q = (at[i] >> 16) - (unsigned)w0;
      if (p < (unsigned)RW) sh.rec[p] = record(cell, h);
      if (at[i] < 0xffff0000u && q < (unsigned)RW) {
        const int kv = mirror(cell, h);
        sh.rec[q] = record((kv & (M - 1)) * HALF, kv >> logm);
      }
    }
    if (pad_at < n_ent && (unsigned)(pad_at - w0) < (unsigned)RW) sh.rec[pad_at - w0] = pad_rec;
    __syncthreads();
    for (int j = tid; j < RW && w0 + j < n_ent; j += kFoldThreads) rec[w0 + j] = sh.rec[j];
    if (w0 + RW < n_ent) __syncthreads();
  }
  float wt[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) wt[i] = 1.f;
  if constexpr (UNIFORM) {
    // the weights pass through the value array
    static_assert(RW >= fold_entries(NB * kFoldThreads), "uniform weighting compares the records in the LDS");
    float* wts = reinterpret_cast<float*>(val);
    const int occ = fold_weights<STAGE>(sh, over0, (int)total[kFields - 1], logn, logm, wts);
    if (occ) atomicAdd(&sh.occ, occ);
    __syncthreads();                             // the weights are visible to the workgroup
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (code[i] >= 0) wt[i] = wts[at[i] & 0xffffu];
  }
  __syncthreads();
  if (UNIFORM && tid == 0) hdr->occ = sh.occ;
  const float scale = inverse_weight(UNIFORM ? (double)sh.occ : 2.0 * (double)sh.kept);
  // factors of a visibility's parts: its weight over the image's, with (-1)^(ku + kv) when the image is
  // shifted, and conjugated where the placement is the mirror's
  auto factors = [&](int cd, float w) {
    const int cell = cd & 0x1fff;
    const bool neg = shift && ((((cd >> 13) & 0x7ff) << logm) + (cell >> (logn - 1)) + cell) & 1;
    const float ws = w * scale, re = neg ? -ws : ws;
    return make_float2(re, (cd >> 24) & 1 ? -re : re);
  };
  if (place) {                                   // uniform over the workgroup: k_fold_values writes the values
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int b = i * kFoldThreads + tid;
      if (b >= B) continue;
      place[b] = code[i] < 0 ? ~0u : at[i];
      coef[b] = code[i] < 0 ? make_float2(0.f, 0.f) : factors(code[i], wt[i]);
    }
    return;
  }
  for (int p = 0; p < P; ++p) {
    for (int w0 = 0; w0 < n_ent; w0 += VW) {
      // Addresses and signs are formed again for every polarisation and window: kept over these loops
      // (they do not change) they took up to 288 spilled registers a thread.
      int t = tid;
      asm volatile("" : "+v"(t));
#pragma unroll
      for (int c = 0; c < NB; c += kFoldLoad) {
        float2 v[kFoldLoad];
#pragma unroll
        for (int i = 0; i < kFoldLoad; ++i) {
          const int b = (c + i) * kFoldThreads + t;
          v[i] = vis[p * vis_stride + (b < B ? b : 0)];
        }
#pragma unroll
        for (int i = 0; i < kFoldLoad; ++i) {
          int cd = code[c + i];                  // (see t)
          asm volatile("" : "+v"(cd));
          if (cd < 0) continue;
          const float2 f = factors(cd, wt[c + i]);
          const unsigned a0 = (at[c + i] & 0xffffu) - (unsigned)w0, a1 = (at[c + i] >> 16) - (unsigned)w0;
          if (a0 < (unsigned)VW) sh.val[a0] = make_float2(v[i].x * f.x, v[i].y * f.y);
          if (at[c + i] < 0xffff0000u && a1 < (unsigned)VW) sh.val[a1] = make_float2(v[i].x * f.x, -(v[i].y * f.y));
        }
      }
      if (pad_at < n_ent && (unsigned)(pad_at - w0) < (unsigned)VW) sh.val[pad_at - w0] = make_float2(0.f, 0.f);
      __syncthreads();
      for (int j = tid; j < VW && w0 + j < n_ent; j += kFoldThreads) val[p * val_stride + w0 + j] = sh.val[j];
      __syncthreads();
    }
  }
}

template <int NB, bool UNIFORM, int STAGE, bool VALUES>
__global__ __launch_bounds__(kFoldThreads, NB > 8 ? 4 : 8) void k_fold_bin(FoldBinArgs a) {
  __shared__ FoldShared<STAGE> sh;
  const int q = blockIdx.x;
  const long tc = (long)a.tc0 + q;
  const int t = (int)(tc / a.C), c = (int)(tc % a.C);
  const double k = (a.freq[c] / kSpeedOfLight) * ((double)(1 << a.logn) * a.pixel_scale);
  fold_bin<NB, UNIFORM, STAGE>(a.uvw + (size_t)t * a.B * 3, a.flags ? a.flags + (size_t)tc * a.B : nullptr, a.B, k, a.logn,
                               a.logm, a.shift, a.vis + (size_t)q * a.P * a.B, a.P, (size_t)a.B, a.hdr + q,
                               a.rows + (size_t)q * kFoldRows, a.rec + (size_t)q * a.ent_stride,
                               a.val + (size_t)q * a.P * a.ent_stride, (size_t)a.ent_stride,
                               a.n_out ? a.n_out + tc : nullptr, sh, VALUES ? nullptr : a.place + (size_t)q * a.B,
                               VALUES ? nullptr : a.coef + (size_t)q * a.B);
}

// The values of one image (workgroup), where the binning's workgroups, one a pair, would write too many of
// them one after the other: one pair of 8128 baselines takes 3 us for each polarisation. (16 polarisations of one pair,
// 512^2: 84 us a call with the values in the binning, 47 so, 51 in the two-pass form.)
__global__ __launch_bounds__(kFoldThreads) void k_fold_values(FoldBinArgs a) {
  constexpr int VW = 8192;                         // positions put in order at a time
  __shared__ float2 out[VW];
  const int tid = threadIdx.x, q = blockIdx.x / a.P;
  const int n_ent = a.hdr[q].first_over + a.hdr[q].n_over;
  const uint32_t* place = a.place + (size_t)q * a.B;
  const float2* coef = a.coef + (size_t)q * a.B;
  const float2* vis = a.vis + (size_t)blockIdx.x * a.B;
  float2* val = a.val + (size_t)blockIdx.x * a.ent_stride;
  for (int w0 = 0; w0 < n_ent; w0 += VW) {
    for (int j = tid; j < VW; j += kFoldThreads) out[j] = make_float2(0.f, 0.f);   // also the diagonals' padding
    __syncthreads();
    for (int b0 = tid; b0 < a.B; b0 += kFoldLoad * kFoldThreads) {
      uint32_t at[kFoldLoad];
      float2 f[kFoldLoad], v[kFoldLoad];
#pragma unroll
      for (int i = 0; i < kFoldLoad; ++i) {
        const int b = b0 + i * kFoldThreads < a.B ? b0 + i * kFoldThreads : b0;
        at[i] = place[b];
        f[i] = coef[b];
        v[i] = vis[b];
      }
#pragma unroll
      for (int i = 0; i < kFoldLoad; ++i) {
        const unsigned a0 = (at[i] & 0xffffu) - (unsigned)w0, a1 = (at[i] >> 16) - (unsigned)w0;
        if ((at[i] & 0xffffu) != 0xffffu && a0 < (unsigned)VW) out[a0] = make_float2(v[i].x * f[i].x, v[i].y * f[i].y);
        if (at[i] < 0xffff0000u && a1 < (unsigned)VW) out[a1] = make_float2(v[i].x * f[i].x, -(v[i].y * f[i].y));
      }
    }
    __syncthreads();
    for (int j = tid; j < VW && w0 + j < n_ent; j += kFoldThreads) val[w0 + j] = out[j];
    __syncthreads();
  }
}

// Uneven batches: workgroup w bins the image at position pos0 + w of the descriptor pass's order.
template <int NB, bool UNIFORM, int STAGE>
__global__ __launch_bounds__(kFoldThreads, NB > 8 ? 4 : 8) void k_fold_bin_desc(DescArgs a) {
  __shared__ FoldShared<STAGE> sh;
  const int at = blockIdx.x, img = a.order[a.pos0 + at];
  if (!a.valid[img]) return;                       // uniform over the workgroup
  const blink_image_desc d = a.desc[img];
  const int logn = 31 - __clz(d.grid_n), logm = 31 - __clz(fold_rows(logn));
  const double k = (d.freq_hz / kSpeedOfLight) * ((double)d.grid_n * d.pixel_scale);
  // The loads of an image without baselines, whose values are not used, go to its own header.
  const bool some = d.n_baselines > 0;
  const double* uvw = some ? a.uvw + 3 * d.uvw_offset : reinterpret_cast<const double*>(a.hdr + at);
  const float2* vis = some ? a.vis + d.vis_offset : reinterpret_cast<const float2*>(a.hdr + at);
  fold_bin<NB, UNIFORM, STAGE>(uvw, some && a.flags ? a.flags + d.flag_offset : nullptr, d.n_baselines, k, logn, logm,
                               a.shift, vis, 1, 0, a.hdr + at,
                               a.rows + (size_t)at * kFoldRows, a.rec + (size_t)at * a.ent_stride,
                               a.val + (size_t)at * a.ent_stride, 0, a.n_out ? a.n_out + img : nullptr, sh);
}

}  // namespace

hipError_t launch_fold_bin_desc(const DescArgs& a, hipStream_t s) {
  if (a.n_pos <= 0) return hipSuccess;
  if (a.max_b > kFoldMaxB) return hipErrorInvalidValue;
  if (a.max_b <= 8 * kFoldThreads) {
    if (a.weighting) k_fold_bin_desc<8, true, 68 * 1024><<<a.n_pos, kFoldThreads, 0, s>>>(a);
    else k_fold_bin_desc<8, false, 68 * 1024><<<a.n_pos, kFoldThreads, 0, s>>>(a);
  } else {
    if (a.weighting) k_fold_bin_desc<16, true, 132 * 1024><<<a.n_pos, kFoldThreads, 0, s>>>(a);
    else k_fold_bin_desc<16, false, 132 * 1024><<<a.n_pos, kFoldThreads, 0, s>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_fold_desc(const DescArgs& a, int prec, unsigned items, hipStream_t s) {
  switch (prec) {
    case BLINK_PREC_FP32: return FoldLaunch<BLINK_PREC_FP32>::desc(a, items, s);
    case BLINK_PREC_SPLIT_F16: return FoldLaunch<BLINK_PREC_SPLIT_F16>::desc(a, items, s);
    case BLINK_PREC_SPLIT_BF16: return FoldLaunch<BLINK_PREC_SPLIT_BF16>::desc(a, items, s);
    default: return hipErrorInvalidValue;
  }
}

template <bool VALUES>
static void bin_pairs(const FoldBinArgs& a, hipStream_t s) {
  // uniform weighting keeps every record in the LDS at once (two per baseline at most)
  if (a.B <= 8 * kFoldThreads) {
    if (a.uniform) k_fold_bin<8, true, 68 * 1024, VALUES><<<a.Q, kFoldThreads, 0, s>>>(a);
    else k_fold_bin<8, false, 68 * 1024, VALUES><<<a.Q, kFoldThreads, 0, s>>>(a);
  } else {
    if (a.uniform) k_fold_bin<16, true, 132 * 1024, VALUES><<<a.Q, kFoldThreads, 0, s>>>(a);
    else k_fold_bin<16, false, 132 * 1024, VALUES><<<a.Q, kFoldThreads, 0, s>>>(a);
  }
}

hipError_t launch_fold_bin(const FoldBinArgs& a, hipStream_t s) {
  if (a.Q <= 0) return hipSuccess;
  if (a.B <= 0 || a.B > kFoldMaxB) return hipErrorInvalidValue;
  if (!a.place) {
    bin_pairs<true>(a, s);
    return hipGetLastError();
  }
  if ((long)a.Q * a.P >= 1L << 22) return hipErrorInvalidValue;   // threads of a launch stay below 2^32
  bin_pairs<false>(a, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_fold_values<<<(unsigned)(a.Q * a.P), kFoldThreads, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_fold_image(const FoldArgs& a, int prec, const float2* tw, hipStream_t s) {
  switch (prec) {
    case BLINK_PREC_FP32: return FoldLaunch<BLINK_PREC_FP32>::image(a, tw, s);
    case BLINK_PREC_SPLIT_F16: return FoldLaunch<BLINK_PREC_SPLIT_F16>::image(a, tw, s);
    case BLINK_PREC_SPLIT_BF16: return FoldLaunch<BLINK_PREC_SPLIT_BF16>::image(a, tw, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace blink
