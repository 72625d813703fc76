// K-a: launches of the decorrelation factors and records (k_decorr_bin.hpp),
// and the kernels of one wave per bin and of Method 1.
#include "k_decorr_bin.hpp"

namespace psf {

// Few long bins: one wave per bin.  When an observation has too few bins
// to fill the GPU with one lane each but many samples per bin (the host's
// choice, use_wave_bins), every wave takes one bin: lane l sums the bin's
// samples l, l + 64, ... in (time, channel) order, then the wave's partial
// sums are combined by a fixed butterfly of lane exchanges (deterministic,
// rounded in another order than the one-lane loop).  The per-sample phase
// is formed exactly as there (no fused multiply-add, so that identical rows
// still cancel exactly).  Four waves per block; source y of the launch in
// grid row y, as for k_decorr.
template <bool kGrad>
__global__ __launch_bounds__(256) void k_decorr_wave(ObsView o, double l0, double m0, double dl, double dm,
                                                     const double* __restrict__ dirs, int64_t dir_stride,
                                                     int64_t rec_stride, float2* __restrict__ D_out,
                                                     BinRec* __restrict__ rec_out, float2* __restrict__ c_out,
                                                     float2* __restrict__ coef_out) {
#pragma clang fp contract(off)
  const int64_t k = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (k >= o.K) return;  // the whole wave
  const int lane = threadIdx.x & 63;
  if (dirs != nullptr) {
    l0 = dirs[blockIdx.y * dir_stride];
    m0 = dirs[blockIdx.y * dir_stride + 1];
    dl = dirs[blockIdx.y * dir_stride + 4];
    dm = dirs[blockIdx.y * dir_stride + 5];
  }
  if (rec_out != nullptr) rec_out += blockIdx.y * rec_stride;
  if (c_out != nullptr) c_out += blockIdx.y * rec_stride;
  const BinRef r = locate_bin(o.koff, o.tboff, o.bl_bin, o.n_bl, o.n_t, o.n_ch, k);
  const double n0 = sqrt(1.0 - l0 * l0 - m0 * m0);
  const double Lw = n0 - 1.0;
  const double nu_k = bin_freq(o.freq, r.c0, r.c1);
  const double uc = o.uvw_c[3 * r.tb + 0], vc = o.uvw_c[3 * r.tb + 1], wc = o.uvw_c[3 * r.tb + 2];
  const double A_k = uc * l0 + vc * m0 + wc * Lw;
  const double A_knu = A_k * nu_k;
  const double l0_n0 = l0 / n0, m0_n0 = m0 / n0;
  const bool win = o.win_t != nullptr || o.win_c != nullptr;
  const int nc = r.c1 - r.c0, n = (r.t1 - r.t0) * nc;
  const double* rows = o.uvw + 3 * (static_cast<int64_t>(r.b) * o.n_t);
  float v[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // S re, im; G_l re, im; G_m re, im; window sum
  for (int idx = lane; idx < n; idx += 64) {
    const int t = r.t0 + idx / nc, c = r.c0 + idx % nc;
    const double u = rows[3 * t], vv = rows[3 * t + 1], w = rows[3 * t + 2];
    const double nu_c = o.freq[c];
    const double A_t = u * l0 + vv * m0 + w * Lw;
    const double phi = (A_t * nu_c - A_knu) * kInvCLight;
    const cf32 e = expi_turns_hw(-phi);
    float x = 1.f;
    if (win) {
      x = (o.win_t != nullptr ? o.win_t[static_cast<int64_t>(r.b) * o.n_t + t] : 1.f) *
          (o.win_c != nullptr ? o.win_c[static_cast<int64_t>(r.b) * o.n_ch + c] : 1.f);
      v[6] += x;
    }
    v[0] += x * e.re;
    v[1] += x * e.im;
    if constexpr (kGrad) {
      const double du = (u * nu_c - uc * nu_k) * kInvCLight;
      const double dv = (vv * nu_c - vc * nu_k) * kInvCLight;
      const double dw = (w * nu_c - wc * nu_k) * kInvCLight;
      const float gl = x * static_cast<float>(du - dw * l0_n0);
      const float gm = x * static_cast<float>(dv - dw * m0_n0);
      v[2] += gl * e.im;
      v[3] -= gl * e.re;
      v[4] += gm * e.im;
      v[5] -= gm * e.re;
    }
  }
#pragma unroll
  for (int q = 0; q < 7; ++q)
    for (int off = 32; off > 0; off >>= 1) v[q] += __shfl_xor(v[q], off);
  if (lane != 0) return;
  const float inv = win ? (v[6] != 0.f ? 1.0f / v[6] : 0.f) : 1.0f / static_cast<float>(n);
  const float sc = 6.283185307179586f * inv;
  finish_bin<kGrad>(o, k, l0, m0, n0, dl, dm, nu_k, uc, vc, wc, v[0] * inv, v[1] * inv, v[2] * sc, v[3] * sc,
                    v[4] * sc, v[5] * sc, true, D_out, rec_out, c_out, coef_out);
}

// One wave per bin pays off when one lane per bin leaves the GPU mostly
// idle: fewer bins than 512 waves' worth and at least 64 samples per bin
// on average.
bool use_wave_bins(const ObsView& o) {
  const double samples = static_cast<double>(o.n_bl) * o.n_t * o.n_ch;
  return o.K > 0 && o.K < 512 * 64 && samples >= 64.0 * static_cast<double>(o.K);
}

// The kernel without derivatives: wide where there are channels enough, with
// windows only from 128 samples per bin on average (the bins' own sizes are on
// the device), since that form takes 126 registers to the other's 66.
static decltype(&k_decorr<false, kNotWide>) decorr_kernel(const ObsView& o) {
  if (o.n_ch < kEvenBin) return k_decorr<false, kNotWide>;
  if (o.win_t == nullptr && o.win_c == nullptr) return k_decorr<false, kWideBoxcar>;
  const bool many = static_cast<double>(o.n_bl) * o.n_t * o.n_ch >= 128.0 * static_cast<double>(o.K);
  return many ? k_decorr<false, kWideWindow> : k_decorr<false, kNotWide>;
}

// Without derivatives also for observations of few bins: one wave per bin
// where all of them run at once and a bin has samples for a quarter of the
// lanes (420 bins of 30 samples: 8.5 us with one lane each, whose loads follow
// one another, 5.6 with a wave each).
static bool few_bins(const ObsView& o) {
  const double samples = static_cast<double>(o.n_bl) * o.n_t * o.n_ch;
  return use_wave_bins(o) || (o.K > 0 && o.K <= 8192 && samples >= 16.0 * static_cast<double>(o.K));
}

hipError_t launch_decorr(const ObsView& o, double l0, double m0, double dl, double dm, const float2* D_in,
                         float2* D_out, BinRec* rec_out, float2* c_out, float2* coef_out, hipStream_t stream,
                         const double* dir) {
  const int threads = 256;
  const int64_t blocks = (o.K + threads - 1) / threads;
  if (D_in == nullptr && (coef_out != nullptr ? use_wave_bins(o) : few_bins(o))) {
    const dim3 g(static_cast<unsigned>((o.K + 3) / 4));
    if (coef_out != nullptr)
      hipLaunchKernelGGL(k_decorr_wave<true>, g, dim3(256), 0, stream, o, l0, m0, dl, dm, dir, int64_t(0),
                         int64_t(0), D_out, rec_out, c_out, coef_out);
    else
      hipLaunchKernelGGL(k_decorr_wave<false>, g, dim3(256), 0, stream, o, l0, m0, dl, dm, dir, int64_t(0),
                         int64_t(0), D_out, rec_out, c_out, nullptr);
    return hipGetLastError();
  }
  if (coef_out != nullptr && D_in == nullptr)
    hipLaunchKernelGGL((k_decorr<true, kNotWide>), dim3(static_cast<unsigned>(blocks)), dim3(threads), 0, stream, o, l0, m0,
                       dl, dm, dir, int64_t(0), int64_t(0), D_in, D_out, rec_out, c_out, coef_out);
  else
    hipLaunchKernelGGL(decorr_kernel(o),
                       dim3(static_cast<unsigned>(blocks)), dim3(threads), 0, stream, o, l0, m0, dl, dm, dir, int64_t(0), int64_t(0), D_in, D_out, rec_out, c_out, nullptr);
  return hipGetLastError();
}

hipError_t launch_decorr_sources(const ObsView& o, const double* dirs, int64_t dir_stride, int n_src,
                                 BinRec* rec_out, float2* c_out, int64_t rec_stride, hipStream_t stream) {
  const int threads = 256;
  const int64_t blocks = (o.K + threads - 1) / threads;
  if (few_bins(o)) {
    hipLaunchKernelGGL(k_decorr_wave<false>, dim3(static_cast<unsigned>((o.K + 3) / 4), static_cast<unsigned>(n_src)),
                       dim3(256), 0, stream, o, 0.0, 0.0, 0.0, 0.0, dirs, dir_stride, rec_stride, nullptr, rec_out,
                       c_out, nullptr);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(decorr_kernel(o),
                     dim3(static_cast<unsigned>(blocks), static_cast<unsigned>(n_src)), dim3(threads), 0, stream, o, 0.0, 0.0, 0.0, 0.0, dirs, dir_stride, rec_stride, nullptr, nullptr, rec_out, c_out,
                     nullptr);
  return hipGetLastError();
}

}  // namespace psf

namespace psf {

// Method 1, the uv-plane approximation [section 3.1]: D_k replaced by
// sinc(dPsi/2) sinc(dPhi/2), dPsi = 2 pi du.(l0, m0) across the bin's time
// interval at its centre frequency, dPhi the same across its frequency
// interval at its centre time (2-D: w is dropped), sinc(x) = sin(x)/x.  A
// bin of n samples spaced by s covers n s: the change across it is n times
// the per-sample step, taken from the bin's first and last samples (from a
// neighbour for a one-sample bin; zero if the axis has one sample).  Only
// the bin's end rows are read, not its samples.  FP64; written as (D, 0).
__device__ __forceinline__ double sinc_of(double x) { return x == 0.0 ? 1.0 : sin(x) / x; }

__global__ __launch_bounds__(256) void k_decorr_sinc(ObsView o, double l0, double m0, float2* __restrict__ D_out) {
  const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= o.K) return;
  const BinRef r = locate_bin(o.koff, o.tboff, o.bl_bin, o.n_bl, o.n_t, o.n_ch, k);
  const double nu_k = bin_freq(o.freq, r.c0, r.c1);
  const double* row = o.uvw + 3 * (static_cast<int64_t>(r.b) * o.n_t);
  // per-sample step in time (metres)
  const int nt = r.t1 - r.t0;
  int ta, tb2;
  double div;
  if (nt > 1) {
    ta = r.t0;
    tb2 = r.t1 - 1;
    div = nt - 1;
  } else if (o.n_t > 1) {
    ta = r.t0 + 1 < o.n_t ? r.t0 : r.t0 - 1;
    tb2 = ta + 1;
    div = 1.0;
  } else {
    ta = tb2 = r.t0;
    div = 1.0;
  }
  const double su = (row[3 * tb2] - row[3 * ta]) / div, sv = (row[3 * tb2 + 1] - row[3 * ta + 1]) / div;
  // per-channel frequency step (Hz)
  const int nc = r.c1 - r.c0;
  double sf;
  if (nc > 1)
    sf = (o.freq[r.c1 - 1] - o.freq[r.c0]) / (nc - 1);
  else if (o.n_ch > 1)
    sf = r.c0 + 1 < o.n_ch ? o.freq[r.c0 + 1] - o.freq[r.c0] : o.freq[r.c0] - o.freq[r.c0 - 1];
  else
    sf = 0.0;
  const double pi = 3.141592653589793;
  const double x_t = pi * (nt * (su * l0 + sv * m0) * (nu_k * kInvCLight));
  const double uc = o.uvw_c[3 * r.tb], vc = o.uvw_c[3 * r.tb + 1];
  const double x_f = pi * ((uc * l0 + vc * m0) * (nc * sf * kInvCLight));
  D_out[k] = make_float2(static_cast<float>(sinc_of(x_t) * sinc_of(x_f)), 0.0f);
}

hipError_t launch_decorr_sinc(const ObsView& o, double l0, double m0, float2* D_out, hipStream_t stream) {
  const int threads = 256;
  const int64_t blocks = (o.K + threads - 1) / threads;
  hipLaunchKernelGGL(k_decorr_sinc, dim3(static_cast<unsigned>(blocks)), dim3(threads), 0, stream, o, l0, m0, D_out);
  return hipGetLastError();
}

}  // namespace psf
