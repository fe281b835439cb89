// fold.hip — the folded imaging kernel (fold_device.hpp) of one precision form; built once per
// form. The binning of the folded form is in fold_bin.hip.
#include "fold_device.hpp"

#ifndef BLINK_FOLD_PREC
#error "BLINK_FOLD_PREC: 0 (FP32), 1 (split FP16) or 2 (split BF16)"
#endif

namespace blink {

// Workgroup id -> (image, class). Consecutive workgroups go to the 8 XCDs in turn, so the classes
// of one image are placed 8 apart: they share one XCD's L2, which then reads the image's
// placements from memory once. The last n_img % 8 images keep their classes together instead, so
// that a small batch still spreads over the whole chip.
template <int R>
__device__ __forceinline__ void fold_item(unsigned w, unsigned n_img, int& img, int& r) {
  const unsigned full = n_img & ~7u;
  if (w < full * R) {
    img = (int)(w / (8 * R) * 8 + w % 8);
    r = (int)(w / 8 % R);
  } else {
    img = (int)(w / R);
    r = (int)(w % R);
  }
}

template <int LOGN, int M, int PREC>
__global__ __launch_bounds__((M << LOGN) >> 5, 4) void k_fold_image(FoldArgs a, const float2* __restrict__ tw,
                                                                    const float2* __restrict__ lin) {
  using P = FftPlan<LOGN>;
  constexpr int N = P::N, R = N / M;
  __shared__ __align__(16) float2 sbuf[(M / 2) * P::NP + 1];   // row pairs and the padding's word
  __shared__ float2 s_w[R];
  __shared__ unsigned s_max;
  int img, r;
  fold_item<R>(blockIdx.x, a.n_img, img, r);
  const int pair = img / a.P;
  const FoldHeader* h = a.hdr + pair;
  if (a.weight_sum && r == 0 && threadIdx.x == 0)
    a.weight_sum[img] = a.uniform ? (double)h->occ : 2.0 * (double)h->kept;
  FoldImage im;
  im.hdr = h;
  im.rows = a.rows + (size_t)pair * kFoldRows;
  im.rec = a.rec + (size_t)pair * a.ent_stride;
  im.val = a.val + (size_t)img * a.ent_stride;
  im.out = a.images + (size_t)img * N * N;
  fold_class<LOGN, M, PREC, ((M << LOGN) >> 5)>(im, r, threadIdx.x, sbuf, s_w, tw, lin, SplitCtx{&s_max, a.dft_ops});
}

// ---------------------------------------------------------------- uneven batches
// One launch images every grid size of an uneven batch. Its items are the classes of the images at
// positions [pos0, pos0 + n_pos) of the order, the largest size first, each size's count rounded up
// to a multiple of 8; every size takes 512 threads and 68 to 76 KB of LDS, so that the kernel's
// resources fit all of them. The host knows only that images which do not overlap have at most
// images_len / 16384 + n_pos items and launches that many workgroups; should descriptors share
// pixels there can be more, which a second launch (LOOP) takes in turn.
// 400 images of 512^2 to 2048^2 (3.6 GB of pixels): 2721 us with the half spectra in memory (chunks
// of one size, a column and a row launch each), 1500 us folded.
constexpr int kDescBlock = 512;
template <int LOGN>
constexpr int fold_lds() {
  return (fold_rows(LOGN) / 2) * FftPlan<LOGN>::NP + 1 + (1 << LOGN) / fold_rows(LOGN);   // float2
}

template <int LOGN, int PREC>
__device__ __forceinline__ void fold_desc_item(const DescArgs& a, int first, int count, unsigned w, int tid, float2* lds,
                                               unsigned* s_max) {
  constexpr int M = fold_rows(LOGN), R = (1 << LOGN) / M;
  int k, r;
  fold_item<R>(w, count, k, r);
  if (k >= count) return;                          // padding of the size's items
  const int q = first + k, at = q - a.pos0, img = a.order[q];
  const FoldHeader* h = a.hdr + at;
  if (a.weight_sum && r == 0 && tid == 0) a.weight_sum[img] = a.weighting ? (double)h->occ : 2.0 * (double)h->kept;
  FoldImage im;
  im.hdr = h;
  im.rows = a.rows + (size_t)at * kFoldRows;
  im.rec = a.rec + (size_t)at * a.ent_stride;
  im.val = a.val + (size_t)at * a.ent_stride;
  im.out = a.images + a.desc[img].image_offset;
  fold_class<LOGN, M, PREC, kDescBlock>(im, r, tid, lds, lds + (M / 2) * FftPlan<LOGN>::NP + 1, a.tw[LOGN],
                                        a.tw[LOGN] + tw_size(LOGN), SplitCtx{s_max, a.dft_ops});
}

template <int PREC, bool LOOP>
__global__ __launch_bounds__(kDescBlock, 4) void k_fold_desc(DescArgs a, unsigned first_item) {
  __shared__ __align__(16) float2 lds[fold_lds<12>()];
  __shared__ unsigned s_max;
  static_assert(fold_lds<12>() >= fold_lds<11>() && fold_lds<12>() >= fold_lds<7>() && fold_lds<12>() >= fold_lds<3>(),
                "the largest grid needs the most LDS");
  for (unsigned item = first_item + blockIdx.x;; item += gridDim.x) {
    // the size, and the item within it (uniform over the workgroup)
    unsigned w = item;
    int tid = threadIdx.x;
    if (LOOP) {
      // what follows from the thread's index is formed again for every item: kept over the loop it took
      // 1120 (FP32) to 1608 bytes of scratch memory a lane, outside the caller's workspace
      asm volatile("" : "+v"(tid));
      __builtin_assume(tid >= 0 && tid < kDescBlock);
    }
    int l = a.max_logn, lo = 0, count = 0;
    for (; l >= 3; --l) {
      const int4 z = a.sizes[l];
      lo = z.x > a.pos0 ? z.x : a.pos0;
      count = (z.x + z.y < a.pos0 + a.n_pos ? z.x + z.y : a.pos0 + a.n_pos) - lo;
      if (count <= 0) continue;
      const unsigned n = ((unsigned)count * (unsigned)((1 << l) / fold_rows(l)) + 7u) & ~7u;
      if (w < n) break;
      w -= n;
    }
    switch (l) {
      case 3: fold_desc_item<3, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 4: fold_desc_item<4, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 5: fold_desc_item<5, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 6: fold_desc_item<6, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 7: fold_desc_item<7, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 8: fold_desc_item<8, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 9: fold_desc_item<9, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 10: fold_desc_item<10, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 11: fold_desc_item<11, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      case 12: fold_desc_item<12, PREC>(a, lo, count, w, tid, lds, &s_max); break;
      default: return;                             // past the last item
    }
    if (!LOOP) return;
    __syncthreads();                               // the item is done with the LDS
  }
}

template <int PREC>
struct FoldFor {
  template <int LOGN>
  static hipError_t size(const FoldArgs& a, const float2* tw, hipStream_t s) {
    constexpr int M = fold_rows(LOGN);
    const long n = (long)a.n_img * ((1 << LOGN) / M);
    if (n > 0x7fffffffL) return hipErrorInvalidValue;
    k_fold_image<LOGN, M, PREC><<<(unsigned)n, (M << LOGN) >> 5, 0, s>>>(a, tw, tw + tw_size(LOGN));
    return hipGetLastError();
  }
};

template <int PREC>
hipError_t FoldLaunch<PREC>::image(const FoldArgs& a, const float2* tw, hipStream_t s) {
  if (a.n_img <= 0) return hipSuccess;
  using F = FoldFor<PREC>;
  switch (a.logn) {
    case 8: return F::template size<8>(a, tw, s);
    case 9: return F::template size<9>(a, tw, s);
    case 10: return F::template size<10>(a, tw, s);
    case 11: return F::template size<11>(a, tw, s);
    case 12: return F::template size<12>(a, tw, s);
    default: return hipErrorInvalidValue;
  }
}

template <int PREC>
hipError_t FoldLaunch<PREC>::desc(const DescArgs& a, unsigned items, hipStream_t s) {
  if (a.n_pos <= 0 || items == 0) return hipSuccess;
  k_fold_desc<PREC, false><<<items, kDescBlock, 0, s>>>(a, 0u);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_fold_desc<PREC, true><<<512, kDescBlock, 0, s>>>(a, items);
  return hipGetLastError();
}

template struct FoldLaunch<BLINK_FOLD_PREC>;

}  // namespace blink
