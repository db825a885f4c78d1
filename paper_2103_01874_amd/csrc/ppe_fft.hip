// ppe_fft.hip -- one group of transform lengths in one spectrum precision
// (PPE_FFT_GROUP, PPE_FFT_TS: see ppe_fft.hpp).
#include <hip/hip_runtime.h>

#include "ppe_fft.hpp"
#include "ppe_kernels.hip.inc"

namespace ppe {
namespace {

// CALL with F the kernels' plan and E its elements per thread.
#define PPE_FFT_CT(NN)              \
  case NN: {                        \
    constexpr int E = CFft<NN>::e;  \
    const CFft<NN> F{f.tw};         \
    return call(std::integral_constant<int, E>{}, F); \
  }
#define PPE_FFT_RT(EE) \
  case EE: return call(std::integral_constant<int, EE>{}, f);

template <typename Call>
bool with_plan(const FftDev& f, Call call) {
#if PPE_FFT_GROUP == 0
  switch (f.e) {
    PPE_FFT_RT(1) PPE_FFT_RT(2) PPE_FFT_RT(3) PPE_FFT_RT(4) PPE_FFT_RT(6) PPE_FFT_RT(8) PPE_FFT_RT(12)
    default: return false;
  }
#else
  switch (f.n) {
#if PPE_FFT_GROUP == 1
    PPE_FFT_GROUP_1(PPE_FFT_CT)
#elif PPE_FFT_GROUP == 2
    PPE_FFT_GROUP_2(PPE_FFT_CT)
#elif PPE_FFT_GROUP == 3
    PPE_FFT_GROUP_3(PPE_FFT_CT)
#else
    PPE_FFT_GROUP_4(PPE_FFT_CT)
#endif
    default: return false;
  }
#endif
}

}  // namespace

template <int GROUP, typename TS>
bool FftGroup<GROUP, TS>::r2c(const FftLaunch& l, const FftDev& f, const PtrTable& tab, const Geom& g,
                              const Work<TS>& W, const void* src, bool src_ts, int rp, int check,
                              const FinishArgs& fin) {
  return with_plan(f, [&](auto e, const auto& F) {
    constexpr int E = decltype(e)::value;
    if (src_ts)
      k_r2c<TS, E><<<l.grid, l.block, l.lds, l.stream>>>(tab, g, F, W, static_cast<const TS*>(src), rp, check, fin);
    else
      k_r2c<TS, E><<<l.grid, l.block, l.lds, l.stream>>>(tab, g, F, W, static_cast<const double*>(src), rp, check, fin);
    return true;
  });
}

template <int GROUP, typename TS>
bool FftGroup<GROUP, TS>::c2r(const FftLaunch& l, const FftDev& f, const PtrTable& tab, const Geom& g,
                              const Work<TS>& W, int rp, int mode, int check) {
  return with_plan(f, [&](auto e, const auto& F) {
    k_c2r<TS, decltype(e)::value><<<l.grid, l.block, l.lds, l.stream>>>(tab, g, F, W, rp, mode, check);
    return true;
  });
}

template <int GROUP, typename TS>
bool FftGroup<GROUP, TS>::fft_z(const FftLaunch& l, const FftDev& f, const Geom& g, const Work<TS>& W, int tx, int dir,
                                int check, int kx0, int pair) {
  return with_plan(f, [&](auto e, const auto& F) {
    constexpr int E = decltype(e)::value;
    if (dir < 0) k_fft_z<TS, E, -1><<<l.grid, l.block, l.lds, l.stream>>>(g, F, W, tx, check, kx0, pair);
    else k_fft_z<TS, E, +1><<<l.grid, l.block, l.lds, l.stream>>>(g, F, W, tx, check, kx0, pair);
    return true;
  });
}

template <int GROUP, typename TS>
bool FftGroup<GROUP, TS>::allow_lds(int bytes, const FftDev* only) {
  const auto allow = [&](auto e, const auto& F) {
    using P = std::decay_t<decltype(F)>;
    constexpr int E = decltype(e)::value;
    const void* fns[] = {reinterpret_cast<const void*>(&k_fft_z<TS, E, -1, P>),
                         reinterpret_cast<const void*>(&k_fft_z<TS, E, +1, P>)};
    for (const void* f : fns)
      if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return false;
    return true;
  };
  if (only) return with_plan(*only, allow);
  FftDev f{};
  bool ok = true;
#if PPE_FFT_GROUP == 0
  for (int e : {1, 2, 3, 4, 6, 8, 12}) {
    f.e = e;
    ok = ok && with_plan(f, allow);
  }
#else
#define PPE_FFT_ALLOW(NN) \
  f.n = NN;               \
  ok = ok && with_plan(f, allow);
#if PPE_FFT_GROUP == 1
  PPE_FFT_GROUP_1(PPE_FFT_ALLOW)
#elif PPE_FFT_GROUP == 2
  PPE_FFT_GROUP_2(PPE_FFT_ALLOW)
#elif PPE_FFT_GROUP == 3
  PPE_FFT_GROUP_3(PPE_FFT_ALLOW)
#else
  PPE_FFT_GROUP_4(PPE_FFT_ALLOW)
#endif
#endif
  return ok;
}

template struct FftGroup<PPE_FFT_GROUP, PPE_FFT_TS>;

}  // namespace ppe
