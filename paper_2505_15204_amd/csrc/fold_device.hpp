// fold_device.hpp — the folded form of the fused imaging path: no half spectrum in memory.
//
// The uv plane of one image is sparse (a few thousand placements on N^2 / 2 cells). With the rows
// of the image taken in R = N / M residue classes y = r + R s (s < M), the column transform
//   X[y] = sum_kv x[kv] w_N^(y kv),   kv = k + M h (k < M),  w_n = exp(2 pi i / n)
// of one class needs only the M folded values
//   z[k] = w_N^(r k) sum_h x[k + M h] w_R^(r h),   X[r + R s] = sum_k z[k] w_M^(s k),
// because w_N^(R M s h) = 1. The inner sum runs over the placements themselves, so the first
// stages of the dense column transform disappear; the M x N/2 folded cells of a class fit the LDS
// of one compute unit twice over (M N = 16384), and the M rows that come out of the M-point transforms are
// complete half rows: the same workgroup transforms them along u and stores the pixels. Every
// class reads the image's placements once more (from L2: 8 B per placement), which costs far less
// than the half spectrum's trip to memory and back (16 B per column and row of the grid).
//
// What bounds it: 1536 images of 1024^2 write 6.44 GB, 0.94 ms at the rate of a fill (6.87 TB/s); the kernel
// takes 2.18 ms with two workgroups per compute unit, whose phases overlap: VALU issue 64% of the time, waves
// waiting 35% of theirs (16% for the LDS). A call on 256 images takes 400 us with 8128 baselines, of which 87 are the
// fold: 313 with 45. One workgroup of M N = 32768 per compute unit halves the fold's work but runs its phases one
// after the other (2.82 ms against 2.23 when both were built); M N = 16384 measured faster at 256^2 .. 1024^2 and
// equal above. The two-pass form (column pass, half spectrum, row pass) took 3.9 ms.
//
// Placement layout of one (time, channel) pair (k_fold_bin): the placements of one folded cell
// (k, ku) form a segment; segments are numbered by length, longest first, and stored as jagged
// diagonals: placement j of segment s lies at joff[j] + s, so 64 neighbouring segments are read
// with contiguous loads and the lanes of a wave have nearly equal work. Placements beyond the first
// kFoldDiag of a segment (the shortest baselines of a dense core) lie behind the diagonals and are
// added with LDS atomics, runs of one cell summed up first.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "imaging_device.hpp"
#include "launch.hpp"

namespace blink {

// 32-point inverse DFT: 32 = 4 x 8, inner DFT4 over n1 of x[8 n1 + n2], twiddle w32^(n2 k1), outer
// DFT8 over n2; output k1 + 4 k2.
__device__ __forceinline__ void dft32(float2* v) {
  constexpr float c[22] = {1.f, 0.98078528040323044913f, 0.92387953251128675613f, 0.83146961230254523708f,
                           0.70710678118654752440f, 0.55557023301960222474f, 0.38268343236508977173f,
                           0.19509032201612826785f, 0.f, -0.19509032201612826785f, -0.38268343236508977173f,
                           -0.55557023301960222474f, -0.70710678118654752440f, -0.83146961230254523708f,
                           -0.92387953251128675613f, -0.98078528040323044913f, -1.f, -0.98078528040323044913f,
                           -0.92387953251128675613f, -0.83146961230254523708f, -0.70710678118654752440f,
                           -0.55557023301960222474f};   // cos(pi t / 16); sin(pi t / 16) = cos(pi (t - 8) / 16)
  float2 a[8][4];
#pragma unroll
  for (int n2 = 0; n2 < 8; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < 4; ++n1) a[n2][n1] = v[8 * n1 + n2];
    dft4(a[n2]);
#pragma unroll
    for (int k1 = 1; k1 < 4; ++k1) {
      const int t = n2 * k1;
      if (t == 8) a[n2][k1] = mul_i(a[n2][k1]);
      else if (t > 0) a[n2][k1] = cmul(a[n2][k1], make_float2(c[t], t < 8 ? c[8 - t] : c[t - 8]));
    }
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    float2 b[8];
#pragma unroll
    for (int n2 = 0; n2 < 8; ++n2) b[n2] = a[n2][k1];
    dft8(b);
#pragma unroll
    for (int k2 = 0; k2 < 8; ++k2) v[k1 + 4 * k2] = b[k2];
  }
}

template <int M>
__device__ __forceinline__ void fold_dft(float2* v) {
  if constexpr (M == 32) dft32(v);
  else dft<M>(v);
}

// The M-point column transforms run as one radix pass up to M = 32 and as two above (M = A x B,
// index k = n2 + B n1): pass 1 transforms the A values n1 of one n2 and multiplies value k1 by
// w_M^(n2 k1), pass 2 transforms the B values n2 of one k1. Both passes are in place, so slot
// k2 + B k1 ends up with row s = k1 + A k2 of the class; the row pass accounts for that order.
template <int M>
struct FoldRadix {
  static constexpr int A = M <= 32 ? M : 8, B = M / A;
  static_assert(A * B == M && B <= 16, "one or two radix passes");
  // row of the class held by slot p
  __host__ __device__ static constexpr int row_of(int p) { return B == 1 ? p : p / B + A * (p % B); }
};

// Raw buffer over `bytes` bytes at p (uniform over the wave); a load at or past the end returns
// zero without touching memory, so loads that some lanes do not need stay unconditional.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t fold_rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, kBufferRsrcWord3);
}

// Residue class r of one image: see the head of this file. sbuf holds
// M / 2 row pairs (slot p of the class at (p / 2) NP + pad((p % 2) N/2 + column)), later each pair's
// transform buffer, and one word behind them for the padding placements. The workgroup has BLOCK >=
// M N / 32 threads; the others only join the barriers and the loops over columns.
template <int LOGN, int M, int PREC, int BLOCK>
__device__ __forceinline__ void fold_class(const FoldImage& im, int r, int tid, float2* sbuf, float2* s_w,
                                           const float2* __restrict__ tw, const float2* __restrict__ lin, SplitCtx sp) {
  using P = FftPlan<LOGN>;
  using FR = FoldRadix<M>;
  constexpr int N = P::N, T = P::T, NP = P::NP, HALF = N / 2, R = N / M, NT = (M / 2) * T, NW = NT >= 64 ? NT / 64 : 1;
  constexpr int A = FR::A, B = FR::B;
  constexpr bool SPLIT = PREC != kPrecFp32 && LOGN >= 4;
  static_assert(BLOCK % 64 == 0 && BLOCK >= NT, "whole waves");
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int ext = im.hdr->ext, first_over = im.hdr->first_over, n_over = im.hdr->n_over, n_ent = first_over + n_over;
  const bool folds = BLOCK / 64 == NW || wave < NW;   // uniform over the wave
  const int nrows = folds ? im.hdr->rows[wave] : 0;
  const uint32_t* rows = im.rows + wave * kFoldRowsPerWave;
  // (whole vectors of the list beyond the diagonals, which may reach into what is unused of the arrays)
  const int n_buf = (n_ent + kFoldOver - 1) / kFoldOver * kFoldOver;
  const __amdgpu_buffer_rsrc_t rv = fold_rsrc(im.val, n_buf * 8), rr = fold_rsrc(im.rec, n_buf * 4);
  auto load_val = [&](int at, int base) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rv, at * 8, base * 8, 0));
  };
  auto load_rec = [&](int at, int base) { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rr, at * 4, base * 4, 0); };
  auto w_of = [&](uint32_t rec) {
    return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(s_w) + (rec & 0x1ff8u));
  };
  // Rows of this wave, eight per batch. All lanes of a row hold a placement: the diagonals are
  // padded to whole rows with zero values, whose segments' sums go to the word behind the pairs.
  struct Rows {
    float2 v[kFoldRowBatch];
    uint32_t rec[kFoldRowBatch], row[kFoldRowBatch];
  };
  auto load_rows = [&](Rows& q, int i0) {
#pragma unroll
    for (int i = 0; i < kFoldRowBatch; ++i) {
      q.row[i] = rows[i0 + i];
      q.v[i] = load_val(lane, (int)(q.row[i] & 0xffffu));
      q.rec[i] = load_rec(lane, (int)(q.row[i] & 0xffffu));
    }
  };
  float2 acc = make_float2(0.f, 0.f);            // of this lane's segment
  uint32_t cell = 0;                             // its LDS index, from its first placement
  auto add_rows = [&](const Rows& q) {
    float2 w[kFoldRowBatch];
#pragma unroll
    for (int i = 0; i < kFoldRowBatch; ++i) w[i] = w_of(q.rec[i]);
#pragma unroll
    for (int i = 0; i < kFoldRowBatch; ++i) {
      if (q.row[i] & kFoldRowFirst) {            // uniform over the wave
        acc = make_float2(0.f, 0.f);
        cell = q.rec[i] >> 17;
      }
      acc.x = fmaf(q.v[i].x, w[i].x, acc.x);
      acc.y = fmaf(q.v[i].x, w[i].y, acc.y);
      acc.x = fmaf(-q.v[i].y, w[i].y, acc.x);
      acc.y = fmaf(q.v[i].y, w[i].x, acc.y);
      if (q.row[i] & kFoldRowLast) sbuf[cell] = acc;
    }
  };
  // this thread's first placement beyond the diagonals
  const float2 xv = __builtin_bit_cast(
      float2, __builtin_amdgcn_raw_buffer_load_b64(fold_rsrc(im.val + first_over, n_over * 8), tid * 8, 0, 0));
  const uint32_t xr =
      (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(fold_rsrc(im.rec + first_over, n_over * 4), tid * 4, 0, 0);
  auto slot = [&](int p, int pc) { return (p >> 1) * NP + (p & 1) * pad_offset(HALF) + pc; };
  // padded LDS index of a + b T (a <= T): one base plus compile-time steps when T is a multiple of 16
  auto pad_at = [](int a, int b) { return T % 16 == 0 ? pad_index(a) + pad_offset(b * T) : pad_index(a + b * T); };
  // row pairs: pair j holds the rows of slots 2 j and 2 j + 1
  const bool active = BLOCK == NT || tid < NT;
  const int jt = active ? tid / T : 0, j = T % 64 == 0 ? __builtin_amdgcn_readfirstlane(jt) : jt, lt = tid % T;
  float2* buf = sbuf + j * NP;
  // The first two batches are requested whatever their number (the table holds that many rows for
  // every wave, empty ones reading placement 0), so that the header and the table cost one wait.
  Rows qa, qb;
  if (folds) {
    load_rows(qa, 0);
    load_rows(qb, kFoldRowBatch);
  }
  if (active) {
#pragma unroll
    for (int i = 0; i < P::R; ++i) buf[lt + i * T] = make_float2(0.f, 0.f);
    for (int i = N + lt; i < NP; i += T) buf[i] = make_float2(0.f, 0.f);
  }
  for (int i = tid; i < R; i += BLOCK) s_w[i] = lin[(r * i * M) & (N - 1)];   // w_R^(r h)
  if constexpr (SPLIT) {
    if (tid == 0) *sp.s_max = 0u;
  }
  __syncthreads();
  if (nrows > 0) add_rows(qa);
  if (nrows > kFoldRowBatch) add_rows(qb);
  for (int i = 2 * kFoldRowBatch; i < nrows; i += kFoldRowBatch) {   // uniform over the wave
    load_rows(qa, i);
    add_rows(qa);
  }
  __syncthreads();
  if (n_over > 0) {                            // uniform over the workgroup
    // They lie segment by segment, so where segments run on for many of them (a compact array, a
    // small field) the lanes of a wave would add to a few words: the 16 lanes of a DPP row sum up each
    // run of theirs first, and its first lane alone adds the sum. 256 images of 1024^2 with their 8128
    // placements in one cell: 1971 us with an atomic per placement, 409 now (spread over the grid: 400).
    auto add_to = [&](float2 v, int key) {
      atomicAdd(&sbuf[key].x, v.x);
      atomicAdd(&sbuf[key].y, v.y);
    };
    auto add_row = [&](float2 v, int key, bool on) {
      if (!on) key = -1;
      if (__any(on && key == __builtin_amdgcn_update_dpp(-1, key, 0x104, 0xf, 0xf, false))) {   // lane + 4
        auto step = [&](auto o) {              // lane + o
          constexpr int kCtrl = 0x100 + decltype(o)::value;
          const bool same = key == __builtin_amdgcn_update_dpp(-2, key, kCtrl, 0xf, 0xf, false);
          const float x = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v.x), kCtrl, 0xf, 0xf, false));
          const float y = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v.y), kCtrl, 0xf, 0xf, false));
          if (same) v = make_float2(v.x + x, v.y + y);
        };
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 4>{});
        step(std::integral_constant<int, 8>{});
        on = on && key != __builtin_amdgcn_update_dpp(-2, key, 0x111, 0xf, 0xf, false);          // lane - 1
      }
      if (on) add_to(v, key);
    };
    if (n_over <= BLOCK) {
      if (wave * 64 < n_over) add_row(cmul(xv, w_of(xr)), (int)(xr >> 17), tid < n_over);
    } else {
      // long lists: a lane sums up runs in several neighbours first
      for (int x = tid * kFoldOver; x - lane * kFoldOver < n_over; x += BLOCK * kFoldOver) {   // uniform over the wave
        float2 v[kFoldOver];
        uint32_t rec[kFoldOver];
#pragma unroll
        for (int i = 0; i < kFoldOver; i += 2) {
          const auto two = __builtin_amdgcn_raw_buffer_load_b128(rv, (x + i) * 8, first_over * 8, 0);
          v[i] = make_float2(__uint_as_float(two[0]), __uint_as_float(two[1]));
          v[i + 1] = make_float2(__uint_as_float(two[2]), __uint_as_float(two[3]));
        }
#pragma unroll
        for (int i = 0; i < kFoldOver; i += 4) {
          const auto four = __builtin_amdgcn_raw_buffer_load_b128(rr, (x + i) * 4, first_over * 4, 0);
#pragma unroll
          for (int j = 0; j < 4; ++j) rec[i + j] = four[j];
        }
#pragma unroll
        for (int i = 0; i < kFoldOver; ++i) {
          if (x + i >= n_over) {
            v[i] = make_float2(0.f, 0.f);
            rec[i] = i > 0 ? rec[i - 1] : 0u;
          }
        }
        float2 sum = cmul(v[0], w_of(rec[0]));
        int key = (int)(rec[0] >> 17);
#pragma unroll
        for (int i = 1; i < kFoldOver; ++i) {
          const float2 t = cmul(v[i], w_of(rec[i]));
          const int k = (int)(rec[i] >> 17);
          if (k == key) {
            sum = cadd(sum, t);
          } else {
            add_to(sum, key);
            sum = t;
            key = k;
          }
        }
        add_row(sum, key, x < n_over);
      }
    }
    __syncthreads();
  }
  // M-point transforms of the columns below the extent, in place, with the factors w_N^(r k)
  for (int i = tid; i < B * HALF; i += BLOCK) {
    const int c = i % HALF, n2 = HALF % 64 == 0 ? __builtin_amdgcn_readfirstlane(i / HALF) : i / HALF;
    const int pc = pad_index(c);
    if (c >= ext) continue;
    float2 v[A];
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) {
      const int k = n2 + B * n1;
      v[n1] = cmul(sbuf[slot(k, pc)], lin[(r * k) & (N - 1)]);
    }
    fold_dft<A>(v);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      if constexpr (B > 1) {
        if (k1 > 0) v[k1] = cmul(v[k1], lin[(n2 * k1) * R]);
      }
      sbuf[slot(n2 + B * k1, pc)] = v[k1];
    }
  }
  __syncthreads();
  if constexpr (B > 1) {
    for (int i = tid; i < A * HALF; i += BLOCK) {
      const int c = i % HALF, k1 = i / HALF, pc = pad_index(c);
      if (c >= ext) continue;
      float2 v[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) v[n2] = sbuf[slot(n2 + B * k1, pc)];
      dft<B>(v);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) sbuf[slot(k2 + B * k1, pc)] = v[k2];
    }
    __syncthreads();
  }
  float2 v[P::R];
#pragma unroll
  for (int m = 0; m < P::R / 2; ++m) {
    const float2 a = buf[pad_at(lt, m)], b = buf[pad_at(lt, m + P::R / 2)];
    v[m] = make_float2(a.x - b.y, a.y + b.x);
    if (m == 0 && lt == 0) v[m] = make_float2(a.x, b.x);
  }
#pragma unroll
  for (int m = P::R / 2; m < P::R; ++m) {
    // column N - e in (0, N/2]; the Nyquist column is empty
    const float2 a = buf[pad_at(T - lt, P::R - 1 - m)], b = buf[pad_at(T - lt, P::R - 1 - m + P::R / 2)];
    v[m] = make_float2(a.x + b.y, b.x - a.y);
    if (m == P::R / 2 && lt == 0) v[m] = make_float2(0.f, 0.f);
  }
  float* o = im.out + (size_t)r * N;
  auto row_at = [&](int p) { return o + (size_t)(FR::row_of(p) * R) * N; };
  if constexpr (SPLIT) {
    stage_sync<T>();                           // every load of the row pair is done
    if (active) {
#pragma unroll
      for (int m = 0; m < P::R; ++m) buf[pad_at(lt, m)] = v[m];
    }
    __syncthreads();
    fft_inverse_split<LOGN, PREC, false, true>(sbuf, M / 2, tw, [](int, int) { return make_float2(0.f, 0.f); },
                                               [&](int c, int e, float2 z) {
                                                 __builtin_nontemporal_store(z.x, row_at(2 * c) + e);
                                                 __builtin_nontemporal_store(z.y, row_at(2 * c + 1) + e);
                                               }, sp, tid);
  } else {
    float* o1 = row_at(2 * j);
    float* o2 = row_at(2 * j + 1);
    fft_inverse<LOGN, false>(v, buf, tw, lt, [&](int e, float2 z) {
      __builtin_nontemporal_store(z.x, &o1[e]);
      __builtin_nontemporal_store(z.y, &o2[e]);
    }, active);
  }
}

}  // namespace blink
