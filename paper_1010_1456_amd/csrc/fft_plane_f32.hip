// Passes over kz-outer grids for float2: the run-time length selects the compiled
// kernel set.
#include "fft_plane.h"

namespace aim {
void fft_plane_pass(const float2 *in, float2 *out, const fftk::PlaneOut &om, const FftPlan &pl, int Nx,
                    int Ny, int F, int Pz, int Hy, const float2 *ghat, const float2 *tw,
                    const int32_t *yrange, hipStream_t s) {
  if (F <= 0) return;
  switch (pl.P) {
#define AIM_X(P, a, b, c)                                                                      \
  case P:                                                                                      \
    fftk::launch_plane<float, fftk::PlanC<a, b, c>>(in, out, om, Nx, Ny, F, Pz, Hy, ghat, tw,  \
                                                    yrange, s);                                \
    return;
    AIM_FOR_EACH_FFT_PLAN(AIM_X)
#undef AIM_X
    default:
      break;
  }
  fftk::bad_length(pl.P);
}

void fft_zplane_pass(const float2 *in, float2 *out, const FftPlan &pl, int n_in, int n_out, int F,
                     int64_t nl, const int32_t *sel, const int32_t *range, int64_t A1,
                     bool inverse, const float2 *tw, hipStream_t s) {
  if (F <= 0 || nl <= 0) return;
  switch (pl.P) {
#define AIM_X(P, a, b, c)                                                                      \
  case P:                                                                                      \
    fftk::launch_zplane<float, fftk::PlanC<a, b, c>>(in, out, n_in, n_out, F, nl, sel, range,  \
                                                     A1, inverse, tw, s);                      \
    return;
    AIM_FOR_EACH_FFT_PLAN(AIM_X)
#undef AIM_X
    default:
      break;
  }
  fftk::bad_length(pl.P);
}

PlaneRange fft_plane_range(const float2 *, const FftPlan &pl) {
  switch (pl.P) {
#define AIM_X(P, a, b, c) \
  case P:                 \
    return fftk::plane_range<float, fftk::PlanC<a, b, c>>();
    AIM_FOR_EACH_FFT_PLAN(AIM_X)
#undef AIM_X
    default:
      return PlaneRange{};
  }
}
bool fft_zplane_available(const float2 *, const FftPlan &pl) {
  switch (pl.P) {
#define AIM_X(P, a, b, c) \
  case P:                 \
    return fftk::zplane_ok<fftk::PlanC<a, b, c>>();
    AIM_FOR_EACH_FFT_PLAN(AIM_X)
#undef AIM_X
    default:
      return false;
  }
}
}  // namespace aim
