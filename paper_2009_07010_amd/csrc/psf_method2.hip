// Method 2, the image-plane approximation [section 3.2]: every baseline is
// given the same decorrelation, pixelised over the uv plane from a
// fringe-rate model [Algorithm 1], and applied to the effective PSF (the
// PSF at the phase centre, section 2.2) as a product in the Fourier domain:
//   P^_d(l0, .) = F^-1 { F{P_eff} D^(l0) } .
// The effective PSF is computed once (psf_method2_spectrum: the patch
// contraction at l0 = m0 = 0, where every D_k is exactly 1, then a 2-D FFT);
// each source then costs one pointwise product and one inverse 2-D FFT
// (psf_method2_patch, up to kChunk sources per launch).
//
// Grid: N x N (N a power of two), pixel i at offset (i - N/2) cell; uv cell
// a at frequency a' du, du = 1/(N cell), with a' = a for a < N/2 and a - N
// otherwise (the DFT's own order, in which the spectrum is kept).
// Fringe-rate model: a circular track of radius |u0| turning at omega_E, so
//   dPsi = 2 pi omega_E (-v0 l0 + u0 m0) dt,  dPhi = 2 pi (dnu/nu) |l0| |u0|,
//   D^ = sinc(dPsi/2) sinc(dPhi/2).
//
// FFTs: Stockham (self-sorting) of radix 4, with a last pass of radix 2 where
// N is an odd power, FP32, twiddles exp(+-2 pi i k/N) from sincospif of an
// exactly representable argument, once per workgroup.  A workgroup holds
// several lines in LDS, so that column passes read and write whole 64- or
// 128-byte pieces of rows.  The patch is the real part of the transform, which
// depends on the Hermitian part of F{P_eff} D^ only: rows a <= N/2 of that
// are formed (with the model, in the kernel that transforms them), and two of
// the real columns share one complex transform of the second pass, which
// writes the patch.  16 sources at N = 512: 34 us in two launches, against 176
// us in four with one radix-2 line per workgroup (50 MB of traffic instead of
// 250; bound now by latency, of loads from other dies' caches and of passes
// through LDS, with vector issue at 42% of the cycles of the first kernel, most
// of it the model in FP64, and 24% of the second's).
#include <algorithm>
#include <cmath>

#include "psf_host.hpp"

namespace psf {

namespace {

constexpr double kOmegaEarth = 7.2921150e-5;  // rad / s, sidereal
constexpr int kChunk = 16;                    // sources per launch
constexpr int kFftThreads = 256;
constexpr int kPad = 4;  // per line: 8 lines x 4 elements fall on different LDS banks

// patches and workspace may begin at any element
typedef float m2_f32x2 __attribute__((ext_vector_type(2), aligned(4)));
typedef float m2_f32x4 __attribute__((ext_vector_type(4), aligned(8)));

// Complex elements per workgroup: kFly radix-4 butterflies per thread.
template <int kFly>
constexpr int kElems = 4 * kFftThreads * kFly;

// tw[k] = exp(sign 2 pi i k / N), k < 3 N / 4
__device__ __forceinline__ void twiddles(float2* tw, int N, float sign) {
  for (int k = threadIdx.x; k < 3 * N / 4; k += kFftThreads) {
    float sn, cs;
    sincospif(sign * 2.0f * static_cast<float>(k) / static_cast<float>(N), &sn, &cs);
    tw[k] = make_float2(cs, sn);
  }
}

__device__ __forceinline__ float2 times(float2 a, float2 w) {
  return make_float2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}

// DFTs of the kElems / N lines in v (pitch N + kPad), sign as the twiddles'.
// Enters and leaves with all of v written and visible.
template <int kFly>
__device__ __forceinline__ void fft_block(float2* v, const float2* tw, int N, int logN, float sign) {
  const int quarter = N >> 2, lq = logN - 2;
  int ls = 0;  // log2 of the stride
  for (; ls + 2 <= logN; ls += 2) {
    float2 x[kFly][4];
#pragma unroll
    for (int f = 0; f < kFly; ++f) {
      const int g = threadIdx.x + f * kFftThreads;
      const float2* in = v + (g >> lq) * (N + kPad) + (g & (quarter - 1));
#pragma unroll
      for (int k = 0; k < 4; ++k) x[f][k] = in[k * quarter];
    }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < kFly; ++f) {
      const int g = threadIdx.x + f * kFftThreads;
      const int t = g & (quarter - 1), p = t >> ls, q = t - (p << ls);
      const float2 a = x[f][0], b = x[f][1], c = x[f][2], d = x[f][3];
      const float2 s0 = make_float2(a.x + c.x, a.y + c.y), s1 = make_float2(a.x - c.x, a.y - c.y);
      const float2 s2 = make_float2(b.x + d.x, b.y + d.y);
      const float2 s3 = make_float2(-sign * (b.y - d.y), sign * (b.x - d.x));  // sign i (b - d)
      float2* out = v + (g >> lq) * (N + kPad) + q + (p << (ls + 2));
      out[0] = make_float2(s0.x + s2.x, s0.y + s2.y);
      out[1 << ls] = times(make_float2(s1.x + s3.x, s1.y + s3.y), tw[p << ls]);
      out[2 << ls] = times(make_float2(s0.x - s2.x, s0.y - s2.y), tw[2 * p << ls]);
      out[3 << ls] = times(make_float2(s1.x - s3.x, s1.y - s3.y), tw[3 * p << ls]);
    }
    __syncthreads();
  }
  if (ls < logN) {
    const int half = N >> 1;
#pragma unroll
    for (int f = 0; f < 2 * kFly; ++f) {
      const int g = threadIdx.x + f * kFftThreads;
      float2* in = v + (g >> (logN - 1)) * (N + kPad) + (g & (half - 1));
      const float2 a = in[0], b = in[half];
      in[0] = make_float2(a.x + b.x, a.y + b.y);
      in[half] = make_float2(a.x - b.x, a.y - b.y);
    }
    __syncthreads();
  }
}

// Forward transform of the rows of a centred real image (row pitch `pitch` >=
// N), image centre to index 0, rows likewise: S[(i + N/2) % N][b].
template <int kFly>
__global__ __launch_bounds__(kFftThreads) void k_m2_image_rows(const float* __restrict__ P, int pitch,
                                                               float2* __restrict__ S, int N, int logN) {
  extern __shared__ float2 lds[];
  const int lines = kElems<kFly> >> logN, h = N >> 1, msk = N - 1;
  float2 *v = lds, *tw = lds + lines * (N + kPad);
  const int i0 = blockIdx.x * lines;
  twiddles(tw, N, -1.0f);
  for (int e = threadIdx.x; e < kElems<kFly>; e += kFftThreads) {
    const int line = e >> logN, j = e & msk, i = i0 + line;
    v[line * (N + kPad) + ((j + h) & msk)] = make_float2(i < N ? P[static_cast<int64_t>(i) * pitch + j] : 0.f, 0.f);
  }
  __syncthreads();
  fft_block<kFly>(v, tw, N, logN, -1.0f);
  for (int e = threadIdx.x; e < kElems<kFly>; e += kFftThreads) {
    const int line = e >> logN, b = e & msk, i = i0 + line;
    if (i < N) S[static_cast<int64_t>((i + h) & msk) * N + b] = v[line * (N + kPad) + b];
  }
}

// Forward transform of the columns, in place.
template <int kFly>
__global__ __launch_bounds__(kFftThreads) void k_m2_image_cols(float2* __restrict__ S, int N, int logN) {
  extern __shared__ float2 lds[];
  const int ll = 2 * 5 + (kFly == 4 ? 2 : 1) - logN, lines = 1 << ll;  // log2 of the lines
  float2 *v = lds, *tw = lds + lines * (N + kPad);
  const int b0 = blockIdx.x * lines;
  twiddles(tw, N, -1.0f);
  for (int e = threadIdx.x; e < kElems<kFly>; e += kFftThreads) {
    const int line = e & (lines - 1), a = e >> ll;
    v[line * (N + kPad) + a] =
        b0 + line < N ? S[static_cast<int64_t>(a) * N + b0 + line] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  fft_block<kFly>(v, tw, N, logN, -1.0f);
  for (int e = threadIdx.x; e < kElems<kFly>; e += kFftThreads) {
    const int line = e & (lines - 1), a = e >> ll;
    if (b0 + line < N) S[static_cast<int64_t>(a) * N + b0 + line] = v[line * (N + kPad) + a];
  }
}

struct Dirs {
  double l0[kChunk], m0[kChunk];
};

// sin(pi y) / (pi y) in FP64 to about 1e-11: the Taylor series over half a
// turn through x^15, the reciprocal by one Newton step.
__device__ __forceinline__ double sinc_pi(double y) {
  const double q = rint(y), x = (y - q) * M_PI, x2 = x * x;
  double p = -1.0 / 1307674368000.0;
  p = fma(p, x2, 1.0 / 6227020800.0);
  p = fma(p, x2, -1.0 / 39916800.0);
  p = fma(p, x2, 1.0 / 362880.0);
  p = fma(p, x2, -1.0 / 5040.0);
  p = fma(p, x2, 1.0 / 120.0);
  p = fma(p, x2, -1.0 / 6.0);
  p = fma(p * x2, x, x);
  const double z = M_PI * y, r = __builtin_amdgcn_rcp(z);
  const double v = p * fma(r, fma(-z, r, 1.0), r);
  const bool odd = 0.5 * q != rint(0.5 * q);
  return fabs(y) < 1e-9 ? 1.0 : odd ? -v : v;
}

// D^(a' du, b' du) of one direction: fac = omega_E dt, fbw = (dnu / nu) |l0|
__device__ __forceinline__ float d_hat(int a, int b, int N, double du, double l0, double m0, double fac, double fbw) {
  const double u0 = (a < N / 2 ? a : a - N) * du, v0 = (b < N / 2 ? b : b - N) * du;
  const double psi = fac * (-v0 * l0 + u0 * m0);  // dPsi / (2 pi)
  const double phi = fbw * sqrt(u0 * u0 + v0 * v0);
  return static_cast<float>(sinc_pi(psi) * sinc_pi(phi));
}

// Rows a = 0 .. N/2 of the Hermitian part of S D^, inverse transformed:
// work[s][a][(j + N/2) % N].  The direction of a one-source launch is read
// from device memory (l0, m0 at ddir) when ddir is not null.
template <int kFly>
__global__ __launch_bounds__(kFftThreads) void k_m2_rows(const float2* __restrict__ S, float2* __restrict__ work, int N,
                                                         int logN, double du, double dt, double frac_bw, Dirs d,
                                                         const double* __restrict__ ddir) {
  extern __shared__ float2 lds[];
  const int lines = kElems<kFly> >> logN, h = N >> 1, msk = N - 1;
  float2 *v = lds, *tw = lds + lines * (N + kPad);
  const int s = blockIdx.y, a0 = blockIdx.x * lines;
  const double l0 = ddir != nullptr ? ddir[0] : d.l0[s], m0 = ddir != nullptr ? ddir[1] : d.m0[s];
  const double fac = kOmegaEarth * dt, fbw = frac_bw * sqrt(l0 * l0 + m0 * m0);
  twiddles(tw, N, 1.0f);
#pragma unroll 2
  for (int e = threadIdx.x; e < kElems<kFly>; e += kFftThreads) {
    const int line = e >> logN, b = e & msk, a = a0 + line;
    float2 x = make_float2(0.f, 0.f);
    if (a <= h) {
      const int an = (N - a) & msk, bn = (N - b) & msk;  // the cell of -a', -b'
      const float2 p = S[static_cast<int64_t>(a) * N + b], q = S[static_cast<int64_t>(an) * N + bn];
      const float dp = d_hat(a, b, N, du, l0, m0, fac, fbw);
      // the model is even, but where a' or b' = -N/2 stands for both signs
      const float dq = a == h || b == h ? d_hat(an, bn, N, du, l0, m0, fac, fbw) : dp;
      x = make_float2(0.5f * (p.x * dp + q.x * dq), 0.5f * (p.y * dp - q.y * dq));
    }
    v[line * (N + kPad) + b] = x;
  }
  __syncthreads();
  fft_block<kFly>(v, tw, N, logN, 1.0f);
  float2* out = work + static_cast<int64_t>(s) * (h + 1) * N;
  for (int e = threadIdx.x; e < kElems<kFly>; e += kFftThreads) {
    const int line = e >> logN, j = e & msk, a = a0 + line;
    if (a <= h) out[static_cast<int64_t>(a) * N + ((j + h) & msk)] = v[line * (N + kPad) + j];
  }
}

// The patches: columns 2 c and 2 c + 1 as real and imaginary part of one
// inverse transform over a.  (Rows 0 and N/2 are real in exact arithmetic.)
template <int kFly>
__global__ __launch_bounds__(kFftThreads) void k_m2_cols(const float2* __restrict__ work, float* __restrict__ P, int N,
                                                         int logN, float scale) {
  extern __shared__ float2 lds[];
  const int ll = 2 * 5 + (kFly == 4 ? 2 : 1) - logN, lines = 1 << ll;  // log2 of the lines
  const int h = N >> 1, msk = N - 1;
  float2 *v = lds, *tw = lds + lines * (N + kPad);
  const int s = blockIdx.y, c0 = blockIdx.x * lines;
  const m2_f32x4* in = reinterpret_cast<const m2_f32x4*>(work + static_cast<int64_t>(s) * (h + 1) * N);
  twiddles(tw, N, 1.0f);
  for (int e = threadIdx.x; e < (h + 1) << ll; e += kFftThreads) {
    const int line = e & (lines - 1), a = e >> ll;
    m2_f32x4 y = {0.f, 0.f, 0.f, 0.f};
    if (c0 + line < h) y = in[static_cast<int64_t>(a) * h + c0 + line];
    float2* z = v + line * (N + kPad);
    if (a == 0 || a == h) {
      z[a] = make_float2(y.x, y.z);
    } else {
      z[a] = make_float2(y.x - y.w, y.y + y.z);
      z[N - a] = make_float2(y.x + y.w, y.z - y.y);
    }
  }
  __syncthreads();
  fft_block<kFly>(v, tw, N, logN, 1.0f);
  float* out = P + static_cast<int64_t>(s) * N * N;
  for (int e = threadIdx.x; e < kElems<kFly>; e += kFftThreads) {
    const int line = e & (lines - 1), i = e >> ll;
    const float2 p = v[line * (N + kPad) + i];
    if (c0 + line < h)
      *reinterpret_cast<m2_f32x2*>(out + static_cast<int64_t>((i + h) & msk) * N + 2 * (c0 + line)) =
          m2_f32x2{p.x * scale, p.y * scale};
  }
}

int log2_exact(int N) {
  int l = 0;
  while ((1 << l) < N) ++l;
  return (1 << l) == N ? l : -1;
}

int validate_grid(int32_t N, double cell) {
  if (N < 16 || N > 4096 || log2_exact(N) < 0) return fail(PSF_EINVAL, "N=%d must be a power of two in 16..4096", N);
  if (!(cell > 0.0) || !std::isfinite(cell) || cell * N / 2 >= 1.0)
    return fail(PSF_EINVAL, "cell %g must be positive and the grid inside the sky", cell);
  return PSF_OK;
}

// Butterflies per thread: 2 where a line fits (N <= 2048), 4 for N = 4096.
size_t fft_lds_bytes(int N, int fly) {
  return (static_cast<size_t>(4 * kFftThreads * fly / N) * (N + kPad) + 3 * N / 4) * sizeof(float2);
}

unsigned fft_blocks(int lines, int N, int fly) {
  const int per = 4 * kFftThreads * fly / N;
  return static_cast<unsigned>((lines + per - 1) / per);
}

template <int kFly>
void launch_spectrum(const float* P, int pitch, float2* S, int N, hipStream_t s) {
  const size_t lds = fft_lds_bytes(N, kFly);
  const dim3 g(fft_blocks(N, N, kFly)), b(kFftThreads);
  hipLaunchKernelGGL(k_m2_image_rows<kFly>, g, b, lds, s, P, pitch, S, N, log2_exact(N));
  hipLaunchKernelGGL(k_m2_image_cols<kFly>, g, b, lds, s, S, N, log2_exact(N));
}

template <int kFly>
void launch_sources(const float2* S, float2* work, float* P, int N, int nq, double du, double dt, double frac_bw,
                    const Dirs& d, const double* ddir, hipStream_t s) {
  const size_t lds = fft_lds_bytes(N, kFly);
  hipLaunchKernelGGL(k_m2_rows<kFly>, dim3(fft_blocks(N / 2 + 1, N, kFly), nq), dim3(kFftThreads), lds, s, S, work, N,
                     log2_exact(N), du, dt, frac_bw, d, ddir);
  hipLaunchKernelGGL(k_m2_cols<kFly>, dim3(fft_blocks(N / 2, N, kFly), nq), dim3(kFftThreads), lds, s, work, P, N,
                     log2_exact(N), static_cast<float>(1.0 / (static_cast<double>(N) * N)));
}

int run_sources(const float2* S, float2* work, float* P, int N, int nq, double cell, double dt, double frac_bw,
                const Dirs& d, const double* ddir, hipStream_t s) {
  const double du = 1.0 / (N * cell);
  if (N <= 2048) launch_sources<2>(S, work, P, N, nq, du, dt, frac_bw, d, ddir, s);
  else launch_sources<4>(S, work, P, N, nq, du, dt, frac_bw, d, ddir, s);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PSF_OK : hip_fail(e, "k_m2_rows launch");
}

// The grid the effective PSF is contracted on: offsets -N/2 .. N/2 - 1, or
// -N/2 .. N/2 (one more row and column, dropped when loaded) where N + 1 is
// one of the patch sizes with a tuned tile family (65, 129, 257).
psf_src effective_grid(int32_t N, double cell) {
  psf_src g{};
  g.l0 = g.m0 = 0.0;
  g.l_first = g.m_first = -(N / 2) * cell;
  g.dl = g.dm = cell;
  g.nl = g.nm = (N == 64 || N == 128 || N == 256) ? N + 1 : N;
  g.out_off = 0;
  return g;
}

struct SpectrumLayout {
  size_t Peff, total;
};

SpectrumLayout spectrum_layout(const psf_obs* o, const PatchPlan& plan, int32_t N) {
  SpectrumLayout L;
  L.Peff = align_up(patch_workspace(o, plan), 256);
  L.total = L.Peff + align_up(static_cast<size_t>(N + 1) * (N + 1) * sizeof(float), 256);
  return L;
}

size_t patch_m2_workspace(int32_t N, int32_t n_src) {
  return static_cast<size_t>(std::min(n_src, kChunk)) * N * N * sizeof(float2);
}

}  // namespace

// One Method-2 patch whose direction (l0, m0) is read from device memory
// when the kernels run (the arguments validated by the caller; work holds
// N^2 complex values).
int method2_patch_device_dir(int32_t N, double cell, const float* S, const double* d_dir, double dt_bin,
                             double dnu_bin, double nu, float* P, float2* work, hipStream_t s) {
  return run_sources(reinterpret_cast<const float2*>(S), work, P, N, 1, cell, dt_bin, dnu_bin / nu, Dirs{}, d_dir, s);
}

}  // namespace psf

using namespace psf;

extern "C" {

int psf_method2_workspace_bytes(const psf_obs* obs, int32_t N, int prec, int32_t n_src, size_t* out) {
  clear_error();
  int st;
  if ((st = validate_obs(obs)) != PSF_OK) return st;
  if ((st = validate_prec(prec)) != PSF_OK) return st;
  if ((st = reject_normalise(prec, "psf_method2")) != PSF_OK) return st;
  if ((st = validate_grid(N, 1e-6)) != PSF_OK) return st;
  if (n_src < 0) return fail(PSF_EINVAL, "n_src < 0");
  if (out == nullptr) return fail(PSF_EINVAL, "out is NULL");
  const psf_src g = effective_grid(N, 1e-6);
  const PatchPlan plan = plan_patch(obs, &g, prec, kTargetWorkgroups);
  *out = std::max(spectrum_layout(obs, plan, N).total, patch_m2_workspace(N, std::max(n_src, 1)));
  return PSF_OK;
}

int psf_method2_spectrum(const psf_obs* obs, int32_t N, double cell, int prec, float* S, void* ws, size_t ws_bytes,
                         void* stream) {
  clear_error();
  int st;
  if ((st = validate_obs(obs)) != PSF_OK) return st;
  if ((st = validate_prec(prec)) != PSF_OK) return st;
  if ((st = reject_normalise(prec, "psf_method2")) != PSF_OK) return st;
  if ((st = validate_grid(N, cell)) != PSF_OK) return st;
  if (S == nullptr) return fail(PSF_EINVAL, "S is NULL");
  const psf_src g = effective_grid(N, cell);
  const PatchPlan plan = plan_patch(obs, &g, prec, kTargetWorkgroups);
  const SpectrumLayout L = spectrum_layout(obs, plan, N);
  if (ws == nullptr || ws_bytes < L.total)
    return fail(PSF_EWORKSPACE, "psf_method2_spectrum needs %zu workspace bytes, got %zu", L.total, ws_bytes);
  if ((st = check_device()) != PSF_OK) return st;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  uint8_t* w = static_cast<uint8_t*>(ws);
  BinRec* rec = reinterpret_cast<BinRec*>(w);
  float2* c = reinterpret_cast<float2*>(w + align_up(static_cast<size_t>(obs->K) * sizeof(BinRec), 256));
  float* partial = reinterpret_cast<float*>(reinterpret_cast<uint8_t*>(c) +
                                            align_up(static_cast<size_t>(obs->K) * sizeof(float2), 256));
  float* Peff = reinterpret_cast<float*>(w + L.Peff);
  // At the phase centre every sample's phase difference is exactly 0, so
  // D_k = 1 and u' = u: the effective PSF.
  if ((st = patch_of(obs, &g, plan, prec, rec, c, partial, Peff, s)) != PSF_OK) return st;
  float2* Sc = reinterpret_cast<float2*>(S);
  if (N <= 2048) launch_spectrum<2>(Peff, g.nm, Sc, N, s);
  else launch_spectrum<4>(Peff, g.nm, Sc, N, s);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PSF_OK : hip_fail(e, "k_m2_image_rows launch");
}

int psf_method2_patch(int32_t N, double cell, const float* S, int32_t n_src, const double* h_dirs, double dt_bin,
                      double dnu_bin, double nu, float* P, void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  int st;
  if ((st = validate_grid(N, cell)) != PSF_OK) return st;
  if (S == nullptr || P == nullptr) return fail(PSF_EINVAL, "S or P is NULL");
  if (n_src < 1 || h_dirs == nullptr) return fail(PSF_EINVAL, "need n_src >= 1 directions");
  if (!(dt_bin >= 0.0) || !(dnu_bin >= 0.0) || !(nu > 0.0) || !std::isfinite(dt_bin) || !std::isfinite(dnu_bin) ||
      !std::isfinite(nu))
    return fail(PSF_EINVAL, "bin duration, bandwidth and frequency must be finite, >= 0 (nu > 0)");
  for (int q = 0; q < n_src; ++q) {
    const double l0 = h_dirs[2 * q], m0 = h_dirs[2 * q + 1];
    if (!std::isfinite(l0) || !std::isfinite(m0) || l0 * l0 + m0 * m0 >= 1.0)
      return fail(PSF_EINVAL, "direction %d outside the sky", q);
  }
  const size_t need = patch_m2_workspace(N, n_src);
  if (ws == nullptr || ws_bytes < need)
    return fail(PSF_EWORKSPACE, "psf_method2_patch needs %zu workspace bytes, got %zu", need, ws_bytes);
  if ((st = check_device()) != PSF_OK) return st;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  float2* work = static_cast<float2*>(ws);
  const int64_t NN = static_cast<int64_t>(N) * N;
  for (int q0 = 0; q0 < n_src; q0 += kChunk) {
    const int nq = std::min(kChunk, n_src - q0);
    Dirs d{};
    for (int q = 0; q < nq; ++q) {
      d.l0[q] = h_dirs[2 * (q0 + q)];
      d.m0[q] = h_dirs[2 * (q0 + q) + 1];
    }
    if ((st = run_sources(reinterpret_cast<const float2*>(S), work, P + q0 * NN, N, nq, cell, dt_bin, dnu_bin / nu, d,
                          nullptr, s)) != PSF_OK)
      return st;
  }
  return PSF_OK;
}

}  // extern "C"
