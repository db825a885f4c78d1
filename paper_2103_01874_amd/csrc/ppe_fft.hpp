// ppe_fft.hpp -- launches of the kernels that depend on a transform length.
//
// The row and z transforms are compiled per length, in five groups of lengths
// and for both spectrum precisions, each pair a translation unit of its own
// (ppe_fft.hip with PPE_FFT_GROUP and PPE_FFT_TS), so that they build side by
// side.  Group 0 holds the run-time plans.
#pragma once

#include "ppe_kernels.hpp"

namespace ppe {

#define PPE_FFT_GROUP_1(X) X(16) X(32) X(64) X(128) X(256) X(512) X(1024) X(2048)
#define PPE_FFT_GROUP_2(X) X(24) X(48) X(72) X(96) X(144) X(192) X(288) X(384) X(432) X(768)
#define PPE_FFT_GROUP_3(X) X(18) X(27) X(36) X(54) X(81) X(108) X(162) X(216) X(243) X(324) X(486)
#define PPE_FFT_GROUP_4(X) X(576) X(648) X(729) X(864) X(972) X(1152) X(1296) X(1458) X(1536) X(1728) X(1944)

// Group of a length's compile-time plan; 0: none, the run-time plan (lengths
// below 16: a stage or two).
inline int fft_group(int n) {
#define PPE_FFT_CASE(NN) case NN:
  switch (n) {
    PPE_FFT_GROUP_1(PPE_FFT_CASE) return 1;
    PPE_FFT_GROUP_2(PPE_FFT_CASE) return 2;
    PPE_FFT_GROUP_3(PPE_FFT_CASE) return 3;
    PPE_FFT_GROUP_4(PPE_FFT_CASE) return 4;
    default: return 0;
  }
#undef PPE_FFT_CASE
}

struct FftLaunch {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
};

// Each enqueues its kernel for the plan f (n = f.n); false: no such kernel.
template <int GROUP, typename TS>
struct FftGroup {
  // src: FP64 values, or the residual in the spectrum's precision (src_ts)
  static bool r2c(const FftLaunch& l, const FftDev& f, const PtrTable& tab, const Geom& g, const Work<TS>& W,
                  const void* src, bool src_ts, int rp, int check, const FinishArgs& fin);
  static bool c2r(const FftLaunch& l, const FftDev& f, const PtrTable& tab, const Geom& g, const Work<TS>& W, int rp,
                  int mode, int check);
  static bool fft_z(const FftLaunch& l, const FftDev& f, const Geom& g, const Work<TS>& W, int tx, int dir, int check,
                    int kx0, int pair);
  // dynamic LDS above 64 KiB, for the z kernels of plan `only` (nullptr: of the group)
  static bool allow_lds(int bytes, const FftDev* only);
};

// Elements and threads per transform of a length's compile-time plan.
inline void fft_ct_shape(int n, int& e, int& tc) {
#define PPE_FFT_CASE(NN) \
  case NN:               \
    e = CFft<NN>::e;     \
    tc = CFft<NN>::tc;   \
    return;
  switch (n) {
    PPE_FFT_GROUP_1(PPE_FFT_CASE)
    PPE_FFT_GROUP_2(PPE_FFT_CASE)
    PPE_FFT_GROUP_3(PPE_FFT_CASE)
    PPE_FFT_GROUP_4(PPE_FFT_CASE)
    default: return;
  }
#undef PPE_FFT_CASE
}

}  // namespace ppe
