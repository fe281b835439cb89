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
  fold_class<LOGN, M, PREC>(im, r, sbuf, s_w, tw, lin, SplitCtx{&s_max, a.dft_ops});
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
    case 6: return F::template size<6>(a, tw, s);
    case 7: return F::template size<7>(a, tw, s);
    case 8: return F::template size<8>(a, tw, s);
    case 9: return F::template size<9>(a, tw, s);
    case 10: return F::template size<10>(a, tw, s);
    case 11: return F::template size<11>(a, tw, s);
    case 12: return F::template size<12>(a, tw, s);
    default: return hipErrorInvalidValue;
  }
}

template struct FoldLaunch<BLINK_FOLD_PREC>;

}  // namespace blink
