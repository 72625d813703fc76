// K-a: decorrelation factor of every averaged visibility, and the per-bin
// records the patch contraction consumes; the kernel of one thread per bin.
//
// For bin k (baseline b, samples t in [t0,t1), channels c in [c0,c1)) and
// source direction L = (l0, m0, n0 - 1):
//   A_t = uvw_m[b][t] . L          (metres, FP64)
//   A_k = uvw_c_m[tb] . L
//   phi(t, c) = (A_t nu_c - A_k nu_k) / c          (turns, FP64)
//   D_k = mean exp(-2 pi i phi)                    [section 2.3 averaging;
//                                                   section 3.1 factorisation]
// Both products are rounded separately before the difference, so a
// one-sample bin (uvw_c = uvw_m row, nu_k = nu_c) gives phi = 0 exactly and
// D = 1 exactly, as does the phase centre.
//
// Derivatives for the adjoint: d phi/d l0 = du - dw l0/n0, d phi/d m0 =
// dv - dw m0/n0 (du = (u_t nu_c - u_k nu_k)/c etc.), so
// dD/dl0 = mean(-2 pi i dphi/dl0 exp(-2 pi i phi)).
//
// With c_k = W_k D_k, a_ki = exp(2 pi i u'_k x_i), b_kj = exp(2 pi i v'_k
// y_j) and the pixel grid fixed (x_i = l_i - l0, y_j = m_j - m0):
//   dP_ij/dl0 = 2 Re sum_k a_ki b_kj [W_k dD_k/dl0
//               + 2 pi i c_k (du'_k/dl0 x_i + dv'_k/dl0 y_j - u'_k)]
// and likewise for m0 (with -v'_k), where
//   du'/dl0 = -w (1 - m0^2)/n0^3, du'/dm0 = dv'/dl0 = -w l0 m0/n0^3,
//   dv'/dm0 = -w (1 - l0^2)/n0^3.
// So every derivative patch is a sum of patches of the same form as P with
// c_k replaced by one of five coefficient vectors, weighted by 1, x_i or y_j:
//   e0 = W dD/dl0 - 2 pi i c u'    (weight 1, for l0)
//   e1 = W dD/dm0 - 2 pi i c v'    (weight 1, for m0)
//   e2 = 2 pi i c du'/dl0          (weight x_i, for l0)
//   e3 = 2 pi i c dv'/dl0          (weight y_j for l0; weight x_i for m0)
//   e4 = 2 pi i c dv'/dm0          (weight y_j, for m0)
#pragma once
#include "psf_device.hpp"
#include "psf_kernels.hpp"

namespace psf {

namespace {
// The per-sample factors use the hardware sine and cosine (expi_turns_hw):
// D_k stays within FP32 rounding of the FP64 mean, and D_k = 1 remains exact
// where every phase difference is 0.  The 16-pixel step factors of the
// records, raised to powers by the contraction's recurrence, keep the
// polynomial form.

// Channels per register chunk of bin_sums.  Four rather than eight: 70
// instead of 80 registers, seven waves per SIMD instead of six, which the
// loads of the sample loop need (factors of one source, D only: 0.156
// against 0.168 ms on the uniform-bin workload, 3.52 against 3.91 ms on the
// baseline-dependent bins of 1-8 channels); two channels re-read each
// time row too often (0.196 ms).
constexpr int kChanChunk = 4;
// Channels from which the even form pays: it is level with the other at 8 (10
// x 8 samples, K = 1.5M: 74 us either way, with windows 108 against 88), but
// slower there where few long bins wait for their chains (64 x 8 among smaller
// ones: 65 against 44 us).
constexpr int kEvenBin = 12;

// Sums over one bin's samples: S = sum x e with e = exp(-2 pi i phi) and x
// the sample's window weight (1 without windows), the window sums of the bin
// along time (st) and channel (sc), and for the adjoint G_l = sum x g_l e and
// G_m = sum x g_m e with g = d phi / d(l0, m0).  The bin's channels are taken
// in chunks whose frequencies and channel windows sit in registers, so the
// only memory reads per time row are its uvw (and time window), loaded one
// row ahead.  Samples are summed time-major within a chunk.
struct BinSums {
  float sre, sim, glr, gli, gmr, gmi, st, sc;
};

template <bool kWin, bool kGrad>
__device__ __forceinline__ BinSums bin_sums(const ObsView& o, const BinRef& r, double l0, double m0, double Lw,
                                            double A_k, double nu_k, double uc, double vc, double wc,
                                            double l0_n0, double m0_n0) {
#pragma clang fp contract(off)
  // without derivatives the frequencies are taken over c once per chunk, not
  // the phase once per sample
  const double A_knu = kGrad ? A_k * nu_k : A_k * (nu_k * kInvCLight);
  BinSums s{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const double* row = o.uvw + 3 * (static_cast<int64_t>(r.b) * o.n_t);
  const float* win_tb = kWin && o.win_t != nullptr ? o.win_t + static_cast<int64_t>(r.b) * o.n_t : nullptr;
  const float* win_cb = kWin && o.win_c != nullptr ? o.win_c + static_cast<int64_t>(r.b) * o.n_ch : nullptr;
  for (int cb = r.c0; cb < r.c1; cb += kChanChunk) {
    const int nch = min(kChanChunk, r.c1 - cb);
    double nu[kChanChunk];
    float xc[kChanChunk];
#pragma unroll
    for (int j = 0; j < kChanChunk; ++j) {
      const int c = cb + min(j, nch - 1);  // clamped: always a channel of the bin
      nu[j] = kGrad ? o.freq[c] : o.freq[c] * kInvCLight;
      xc[j] = kWin && win_cb != nullptr ? win_cb[c] : 1.f;
    }
    if constexpr (kWin) {
      // the window sums in channel and time order, from the loaded weights
#pragma unroll
      for (int j = 0; j < kChanChunk; ++j)
        if (j < nch) s.sc += xc[j];
    }
    double u = row[3 * r.t0], v = row[3 * r.t0 + 1], w = row[3 * r.t0 + 2];
    float xt = kWin && win_tb != nullptr ? win_tb[r.t0] : 1.f;
    for (int t = r.t0; t < r.t1; ++t) {
      const int tn = min(t + 1, r.t1 - 1);
      const double un = row[3 * tn], vn = row[3 * tn + 1], wn = row[3 * tn + 2];
      const float xtn = kWin && win_tb != nullptr ? win_tb[tn] : 1.f;
      if (kWin && cb == r.c0) s.st += xt;
      const double A_t = u * l0 + v * m0 + w * Lw;
#pragma unroll
      for (int j = 0; j < kChanChunk; ++j) {
        if (j < nch) {
          const double nu_c = nu[j];
          const double phi = kGrad ? (A_t * nu_c - A_knu) * kInvCLight : A_t * nu_c - A_knu;
          const cf32 e = expi_turns_hw(-phi);
          const float x = kWin ? xt * xc[j] : 1.f;
          if constexpr (kWin) {
            s.sre += x * e.re;
            s.sim += x * e.im;
          } else {
            s.sre += e.re;
            s.sim += e.im;
          }
          if constexpr (kGrad) {
            const double du = (u * nu_c - uc * nu_k) * kInvCLight;
            const double dv = (v * nu_c - vc * nu_k) * kInvCLight;
            const double dw = (w * nu_c - wc * nu_k) * kInvCLight;
            float gl = static_cast<float>(du - dw * l0_n0);
            float gm = static_cast<float>(dv - dw * m0_n0);
            if constexpr (kWin) {
              gl = x * gl;
              gm = x * gm;
            }
            // -2 pi i g e  =  2 pi g (e.im, -e.re); the 2 pi is applied by the caller
            s.glr += gl * e.im;
            s.gli -= gl * e.re;
            s.gmr += gm * e.im;
            s.gmi -= gm * e.re;
          }
        }
      }
      u = un;
      v = vn;
      w = wn;
      xt = xtn;
    }
  }
  return s;
}

// The sums of bin_sums (no derivatives) for a bin of evenly spaced channels
// (half spacing h, in s/m): the channels of a time row are a polynomial in
// z = exp(-4 pi i A_t h) with the channel windows as coefficients, times the
// factor of the row's first channel.  It is summed by Clenshaw's recurrence
// b_j = x_j + 2 Re(z) b_{j+1} - b_{j+2}, sum_j x_j z^j = b_0 - conj(z) b_1:
// two real operations per sample instead of a sine-cosine pair and eight more.
// In FP64, whose rate is that of FP32 here, because the recurrence loses
// digits with the square of the channels at small angles.  Windowed bins take
// kLen channels at a time, the windows (0 beyond the last) of the first
// kWinReg in registers, of the others in this thread's part of LDS (win; the
// registers of four waves per SIMD do not hold 40); without windows all
// channels at once.
constexpr int kWinLen = 40, kWinReg = 20, kWinLds = (kWinLen - kWinReg) / 4;
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <bool kWin, int kLen>
__device__ __forceinline__ BinSums even_sums(const ObsView& o, const BinRef& r, double l0, double m0, double Lw,
                                             double A_k, double nu_k, double h, f32x4_t (*win)[256]) {
#pragma clang fp contract(off)
  constexpr int kReg = kLen < kWinReg ? kLen : kWinReg;
  BinSums s{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const double* row = o.uvw + 3 * (static_cast<int64_t>(r.b) * o.n_t);
  const float* win_tb = kWin && o.win_t != nullptr ? o.win_t + static_cast<int64_t>(r.b) * o.n_t : nullptr;
  const float* win_cb = kWin && o.win_c != nullptr ? o.win_c + static_cast<int64_t>(r.b) * o.n_ch : nullptr;
  const double A_knu = A_k * nu_k;
  for (int cb = r.c0; cb < r.c1; cb += kWin ? kLen : r.c1 - r.c0) {
    const int nch = kWin ? min(kLen, r.c1 - cb) : r.c1 - cb;
    float x[kReg];
    if constexpr (kWin) {
      auto window = [&](int j) {
        const float w = win_cb != nullptr ? win_cb[cb + min(j, nch - 1)] : 1.f;
        if (j < nch) s.sc += w;
        return j < nch ? w : 0.f;
      };
#pragma unroll
      for (int j = 0; j < kReg; ++j) x[j] = window(j);
#pragma unroll
      for (int q = 0; q < (kLen - kReg) / 4; ++q) {
        f32x4_t v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = window(kReg + 4 * q + j);
        win[q][threadIdx.x] = v;
      }
    }
    const double nu = o.freq[cb];
    double u = row[3 * r.t0], v = row[3 * r.t0 + 1], w = row[3 * r.t0 + 2];
    float xt = kWin && win_tb != nullptr ? win_tb[r.t0] : 1.f;
    for (int t = r.t0; t < r.t1; ++t) {
      const int tn = min(t + 1, r.t1 - 1);
      const double un = row[3 * tn], vn = row[3 * tn + 1], wn = row[3 * tn + 2];
      const float xtn = kWin && win_tb != nullptr ? win_tb[tn] : 1.f;
      if (kWin && cb == r.c0) s.st += xt;
      const double A_t = u * l0 + v * m0 + w * Lw;
      const cf32 e = expi_half_turns((A_knu - A_t * nu) * kInvCLight);
      double zc, zs;
      cos_sin_turns(2.0 * (A_t * h), &zc, &zs);
      const double c2 = 2.0 * zc;
      double b0 = 0.0, b1 = 0.0;
      auto step = [&](double xj) {
        const double b = fma(c2, b0, xj - b1);
        b1 = b0;
        b0 = b;
      };
      if constexpr (kWin) {
        const int slot = opaque(threadIdx.x);  // read for every row, not held
#pragma unroll
        for (int q = (kLen - kReg) / 4 - 1; q >= 0; --q) {
          const f32x4_t v = win[q][slot];
#pragma unroll
          for (int j = 3; j >= 0; --j) step(v[j]);
        }
#pragma unroll
        for (int j = kReg - 1; j >= 0; --j) {
          asm("" : "+v"(x[j]));  // converted for every row: 40 registers less than the FP64 values
          step(x[j]);
        }
      } else {
#pragma unroll 4
        for (int j = 0; j < nch; ++j) step(1.0);
      }
      const float gr = xt * static_cast<float>(fma(-b1, zc, b0)), gi = -xt * static_cast<float>(b1 * zs);
      s.sre = __builtin_fmaf(gr, e.re, __builtin_fmaf(-gi, e.im, s.sre));
      s.sim = __builtin_fmaf(gr, e.im, __builtin_fmaf(gi, e.re, s.sim));
      u = un;
      v = vn;
      w = wn;
      xt = xtn;
    }
  }
  return s;
}

// The sums by whichever of the two is the faster: a row costs the recurrence
// as much as 8 to 12 samples by bin_sums.
template <bool kWin>
__device__ __forceinline__ BinSums wide_sums(const ObsView& o, const BinRef& r, double l0, double m0, double Lw,
                                             double A_k, double nu_k, double uc, double vc, double wc, double l0_n0,
                                             double m0_n0, f32x4_t (*win)[256]) {
  const int nc = r.c1 - r.c0;
  const double h =
      nc >= kEvenBin && r.t1 - r.t0 > 1 ? even_half_step(o.freq, r.c0, r.c1, nu_k) : __builtin_nan("");
  if (h == h) {
    if (kWin && nc <= kWinReg) return even_sums<kWin, kWinReg>(o, r, l0, m0, Lw, A_k, nu_k, h, win);
    return even_sums<kWin, kWinLen>(o, r, l0, m0, Lw, A_k, nu_k, h, win);
  }
  return bin_sums<kWin, false>(o, r, l0, m0, Lw, A_k, nu_k, uc, vc, wc, l0_n0, m0_n0);
}
}  // namespace

// The per-bin outputs from the bin's D (and, for the adjoint, its
// derivatives): D, the record the contraction streams (u', v' and the
// 16-pixel steps of both axes), c = W D, and the five adjoint coefficient
// vectors (only where the samples were summed, has_grad).
template <bool kGrad>
__device__ __forceinline__ void finish_bin(const ObsView& o, int64_t k, double l0, double m0, double n0, double dl,
                                           double dm, double nu_k, double uc, double vc, double wc, float dre,
                                           float dim, float dDl_re, float dDl_im, float dDm_re, float dDm_im,
                                           bool has_grad, float2* __restrict__ D_out, BinRec* __restrict__ rec_out,
                                           float2* __restrict__ c_out, float2* __restrict__ coef_out) {
#pragma clang fp contract(off)
  if (D_out != nullptr) D_out[k] = make_float2(dre, dim);
  const double s = nu_k * kInvCLight;
  const double u = uc * s, v = vc * s, w = wc * s;
  const double up = u - w * l0 / n0, vp = v - w * m0 / n0;
  if (rec_out != nullptr) {
    BinRec r;
    r.up = up;
    r.vp = vp;
    const cf32 sa = expi_turns(up * (16.0 * dl)), sb = expi_turns(vp * (16.0 * dm));
    r.step_a = make_float2(sa.re, sa.im);
    r.step_b = make_float2(sb.re, sb.im);
    // records and W D are streamed out (non-temporal stores: they exceed
    // every cache at the sizes that matter, 10.6 GB per source at K = 265M;
    // 5.35 against 5.58 ms per source there)
    static_assert(sizeof(BinRec) == 32 && offsetof(BinRec, vp) == 8 && offsetof(BinRec, step_a) == 16 &&
                      offsetof(BinRec, step_b) == 24,
                  "the record is stored as four 8-byte words");
    double* q = reinterpret_cast<double*>(rec_out + k);
    __builtin_nontemporal_store(r.up, q);
    __builtin_nontemporal_store(r.vp, q + 1);
    __builtin_nontemporal_store(__builtin_bit_cast(double, r.step_a), q + 2);
    __builtin_nontemporal_store(__builtin_bit_cast(double, r.step_b), q + 3);
  }
  const float W = o.W[k];
  const float cre = W * dre, cim = W * dim;
  if (c_out != nullptr)
    __builtin_nontemporal_store(__builtin_bit_cast(double, make_float2(cre, cim)), reinterpret_cast<double*>(c_out + k));
  if (kGrad && coef_out != nullptr && has_grad) {
    // 2 pi i c t = 2 pi t (-Im c, Re c) for real t.  All five vectors are
    // scaled by kAdjointScale (a power of two, exact) so that they stay in
    // the FP16 range of the split-FP16 contraction (|2 pi u' c| reaches a
    // few 1e5 on km baselines at GHz); the reduction undoes the scale.
    const double n03 = n0 * n0 * n0;
    const double two_pi = 6.283185307179586 * kAdjointScale;
    const float tu = static_cast<float>(two_pi * up), tv = static_cast<float>(two_pi * vp);
    const float t2 = static_cast<float>(-two_pi * w * (1.0 - m0 * m0) / n03);
    const float t3 = static_cast<float>(-two_pi * w * l0 * m0 / n03);
    const float t4 = static_cast<float>(-two_pi * w * (1.0 - l0 * l0) / n03);
    const int64_t K = o.K;
    const float Ws = W * static_cast<float>(kAdjointScale);
    coef_out[k] = make_float2(Ws * dDl_re - tu * -cim, Ws * dDl_im - tu * cre);
    coef_out[K + k] = make_float2(Ws * dDm_re - tv * -cim, Ws * dDm_im - tv * cre);
    coef_out[2 * K + k] = make_float2(t2 * -cim, t2 * cre);
    coef_out[3 * K + k] = make_float2(t3 * -cim, t3 * cre);
    coef_out[4 * K + k] = make_float2(t4 * -cim, t4 * cre);
  }
}

// One thread per bin.  Writes any subset of: D, record (u', v', c = W D),
// and the five adjoint coefficient vectors e0..e4 (coef_out, plane e at
// coef_out + e K).  When D_in is given the samples are not read: only the
// record is formed from the caller's D (no coefficients then).
//
// Several sources per launch: grid row y handles source y, whose direction
// is read from device memory at dirs + y * dir_stride (l0, m0 as the first
// two doubles) when dirs is given, and whose records start y * rec_stride
// elements into rec_out and c_out.
//
// wide: wide_sums, for observations that may hold bins it is good for (72
// registers for boxcar averaging, 126 with windows; bin_sums alone takes 66).
// Bins of 20 x 40 samples, K = 2.2M: 1087 -> 331 us, with windows 1574 -> 507
// (arithmetic: 2 or 3 FP64 operations per sample and about 100 per row).
// Nothing is spilled: the windowed kernel held 44 registers in scratch memory,
// which a kernel must have been launched once to have (534 us; with three
// waves per SIMD instead 600).
enum Wide { kNotWide, kWideBoxcar, kWideWindow };
template <bool kGrad, Wide wide>
__global__ __launch_bounds__(256, wide == kWideWindow ? 4 : 1) void k_decorr(ObsView o, double l0, double m0, double dl, double dm,
                                                const double* __restrict__ dirs, int64_t dir_stride,
                                                int64_t rec_stride,
                                                const float2* __restrict__ D_in,
                                                float2* __restrict__ D_out,
                                                BinRec* __restrict__ rec_out,
                                                float2* __restrict__ c_out,
                                                float2* __restrict__ coef_out) {
  // No fused multiply-add in this kernel: the two products of the phase
  // difference must round alike so that identical rows cancel exactly.
#pragma clang fp contract(off)
  __shared__ f32x4_t win[wide == kWideWindow ? kWinLds : 1][256];
  const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= o.K) return;
  if (dirs != nullptr) {
    l0 = dirs[blockIdx.y * dir_stride];
    m0 = dirs[blockIdx.y * dir_stride + 1];
    dl = dirs[blockIdx.y * dir_stride + 4];
    dm = dirs[blockIdx.y * dir_stride + 5];
  }
  // (the same in every lane: scalar registers)
  l0 = uniform(l0), m0 = uniform(m0), dl = uniform(dl), dm = uniform(dm);
  if (rec_out != nullptr) rec_out += blockIdx.y * rec_stride;
  if (c_out != nullptr) c_out += blockIdx.y * rec_stride;
  const BinRef r = locate_bin(o.koff, o.tboff, o.bl_bin, o.n_bl, o.n_t, o.n_ch, k);
  const double n0 = uniform(sqrt(1.0 - l0 * l0 - m0 * m0)), Lw = uniform(n0 - 1.0);
  const double nu_k = bin_freq(o.freq, r.c0, r.c1);
  double uc = o.uvw_c[3 * r.tb + 0], vc = o.uvw_c[3 * r.tb + 1], wc = o.uvw_c[3 * r.tb + 2];

  float dre = 0.f, dim = 0.f;
  float dDl_re = 0.f, dDl_im = 0.f, dDm_re = 0.f, dDm_im = 0.f;
  if (D_in != nullptr) {
    const float2 d = D_in[k];
    dre = d.x;
    dim = d.y;
  } else {
    const double A_k = uc * l0 + vc * m0 + wc * Lw;
    const double l0_n0 = uniform(l0 / n0), m0_n0 = uniform(m0 / n0);
    float inv;
    BinSums bs;
    if (wide == kWideWindow || (wide == kNotWide && (o.win_t != nullptr || o.win_c != nullptr))) {
      // Windowed averaging: sample weight x = win_t[b][t] win_c[b][c], the
      // mean normalised by the window's sum over the bin (D = 0 for a
      // window that sums to 0).  Separable, so the normaliser is the
      // product of the two axis sums.
      if constexpr (wide != kNotWide) {
        bs = wide_sums<true>(o, r, l0, m0, Lw, A_k, nu_k, uc, vc, wc, l0_n0, m0_n0, win);
        // (read again, so that the sums have the registers)
        int64_t tb = r.tb;
        asm volatile("" : "+v"(tb));
        uc = o.uvw_c[3 * tb], vc = o.uvw_c[3 * tb + 1], wc = o.uvw_c[3 * tb + 2];
      } else {
        bs = bin_sums<true, kGrad>(o, r, l0, m0, Lw, A_k, nu_k, uc, vc, wc, l0_n0, m0_n0);
      }
      const float norm = bs.st * bs.sc;
      inv = norm != 0.f ? 1.0f / norm : 0.f;
    } else {
      if constexpr (wide != kNotWide) bs = wide_sums<false>(o, r, l0, m0, Lw, A_k, nu_k, uc, vc, wc, l0_n0, m0_n0, win);
      else bs = bin_sums<false, kGrad>(o, r, l0, m0, Lw, A_k, nu_k, uc, vc, wc, l0_n0, m0_n0);
      inv = 1.0f / static_cast<float>((r.t1 - r.t0) * (r.c1 - r.c0));
    }
    dre = bs.sre * inv;
    dim = bs.sim * inv;
    if constexpr (kGrad) {
      const float sc = 6.283185307179586f * inv;
      dDl_re = bs.glr * sc;
      dDl_im = bs.gli * sc;
      dDm_re = bs.gmr * sc;
      dDm_im = bs.gmi * sc;
    }
  }
  // (formed anew: no registers are held for it)
  const int64_t kf = static_cast<int64_t>(blockIdx.x) * blockDim.x + opaque(threadIdx.x);
  finish_bin<kGrad>(o, kf, l0, m0, n0, dl, dm, nu_k, uc, vc, wc, dre, dim, dDl_re, dDl_im, dDm_re, dDm_im,
                    D_in == nullptr, D_out, rec_out, c_out, coef_out);
}

#ifndef PSF_DECORR_WINDOW
// (compiled by itself, k_decorr_window.hip)
extern template __global__ void k_decorr<false, kWideWindow>(ObsView, double, double, double, double, const double*,
                                                            int64_t, int64_t, const float2*, float2*, BinRec*, float2*,
                                                            float2*);
#endif

}  // namespace psf
