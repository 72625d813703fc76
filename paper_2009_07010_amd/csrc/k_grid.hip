// The gridded form of the patch contraction, for many bins.
//
// P_ij = 2 Re sum_k c_k exp(2 pi i (u'_k x_i + v'_k y_j)) on a regular pixel
// grid is a non-uniform discrete Fourier transform: with x_i = x_h + (i - h) dl
// and h = nl / 2, bin k contributes at the frequency u'_k dl (in turns, modulo
// 1) of a transform of nl modes, and likewise along y.  So instead of
// evaluating every bin at every pixel, each bin is spread with a smooth kernel
// of 9 x 9 cells onto a uv grid of ml x mm cells (at least 1.96 cells per
// pixel), and the patch is the inverse DFT of that grid divided by the
// kernel's transform.  Work per bin: 81 cells instead of nl nm pixels.
//
// Kernel: Kaiser-Bessel of width 9 and shape parameter 2.3 x 9, as a
// polynomial of degree 8 in the bin's offset from its cell per tap (even and
// odd parts shared by mirrored taps).  The transform divided out is that of
// the polynomials as coded, so only aliasing remains: per axis at most 5.1e-8
// of a term (at the patch's edges; 1.3e-7 with the FP32 evaluation, 6e-8 rms),
// which differs from bin to bin and averages out.
//
//   k_grid_init    zero cells; largest |c| (scales the fixed point and the FP16
//                  operands)
//   k_grid_spread  the bins onto the cells (below)
//   k_grid_rows    inverse DFT along the columns of every grid row, FP64,
//                  the nm modes kept, transposed
//   k_grid_cols    inverse DFT along the rows, the nl modes, real part
//
// Spreading runs on the matrix cores: the bins of one wave whose taps lie in
// one window of 16 x 16 cells are a contraction over bins of their row taps
// (16 x bins) and their column taps times c (bins x 16, real and imaginary).
// Successive bins of a baseline lie within a fraction of a cell of each
// other, so a wave takes 64 bins of one baseline, a rectangle of time and
// frequency bins shaped by how fast the track moves along each, which one or
// two windows usually hold; bins outside the current window wait for the
// next one, so any track is spread correctly.  Windows are folded into a
// tile of the workgroup's part of the track in LDS, tiles into the grid, in
// 64-bit fixed point: integer sums do not depend on their order, so the result
// is the same on every run although the workgroups meet in the grid through
// atomics.  The unit is 2^-61 of (a power of two above) sum |c|, which bounds
// every cell: finer than the FP32 sums of a window whatever the weights'
// spread, so what remains is those sums' own rounding.
//
// FUSED, the boxcar case but for long bins, forms D_k in the same kernel: bins
// leave no records in memory (40 bytes each way, 10.6 GB per source at K = 265M).
//
// Measured (one 257 x 257 patch, K = 5.8M in bins of 10 x 4 samples,
// stochastic FP16): 302 us per call, spreading 280, against 1400 us of the
// dense contraction it replaced (FP32 337 against 7540); per source at K =
// 265M of baseline-dependent bins 4.3 ms against 37.  The workgroups' time at
// K = 5.8M: half is the set-up of chunks and their tables (latency), a third the
// samples' factors, a sixth staging and contraction; at one sample per bin
// (K = 116M) staging and contraction are 60% and the factors 30%, bound by
// vector issue (two thirds of the cycles) and LDS (one third), which three
// waves per SIMD overlap only in part.
#include <algorithm>

#include "psf_device.hpp"
#include "psf_grid.hpp"

namespace psf {

namespace {

typedef __bf16 g_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 g_f16x8 __attribute__((ext_vector_type(8)));
typedef float g_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t g_u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint8_t g_lds;

constexpr int kW = 9;             // taps per axis
constexpr int kWin = 16;          // cells per axis of a window
constexpr int kSlack = kWin - kW; // a window holds anchors 0 .. kSlack past its origin
constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kChunkBins = 1 << 14;  // bins of a chunk, at most (one row of frequency bins may be longer)
constexpr int kTabRows = 1024;    // samples of a chunk whose projections sit in LDS
constexpr int kTabFreq = 512;     // frequency bins whose centre frequencies do
constexpr int kGridMaxLevels = 6, kLeastSpan = 1024;  // of spans
constexpr int kCutBlocks = 8;     // workgroups that cut the bins into spans
constexpr int kSparse = 512;      // bins that make a tile worth while
constexpr int kEvenMin = 3, kEvenMax = 16;  // channels per bin summed as evenly spaced
constexpr int kRun = 8;           // batches of 64 bins summed in FP32 before a window is folded (2^9 bins)
constexpr int kInitBlocks = 512;
constexpr int kMargin = 1;        // cells added around a tile's sampled extent

// Operand staging of one wave: 16 rows (taps' cells) x 64 bins.  16-bit
// forms: a plane of hi and one of lo, rows of 128 bytes padded by 16 so that
// eight rows' 16-byte reads fall on distinct banks; FP32: one plane, rows of
// 256 + 16 bytes.
constexpr int kRow16 = 144, kPlane16 = 16 * kRow16, kRow32 = 272;

// The taps' polynomials times kTapScale: tap r and tap 8 - r are
// E_r(f^2) +- f O_r(f^2), f = position - nearest cell in [-1/2, 1/2].
constexpr float kTapScale = 256.0f;
constexpr float kE[5][5] = {{2.002013025e-05f, 6.172497524e-04f, 1.670259167e-03f, 7.180632092e-04f, -4.018611799e-05f},
                            {5.964126438e-03f, 4.019754753e-02f, 1.738595404e-02f, -2.347377595e-03f, -3.952386396e-05f},
                            {1.223278940e-01f, 2.172718942e-01f, -3.498638421e-02f, -2.999314456e-04f, 5.284860381e-04f},
                            {6.036517024e-01f, -8.782624267e-03f, -4.322065413e-02f, 1.082540862e-02f, -1.368907047e-03f},
                            {1.000000000e+00f, -4.986084700e-01f, 1.183041185e-01f, -1.779340580e-02f, 1.820146339e-03f}};
constexpr float kO[4][4] = {{-1.689896308e-04f, -1.282629906e-03f, -1.401485410e-03f, -1.478675258e-04f},
                            {-2.372954227e-02f, -3.653368726e-02f, -1.952710212e-03f, 1.121683628e-03f},
                            {-2.715461552e-01f, -4.635402188e-02f, 2.174760029e-02f, -2.793780062e-03f},
                            {-6.170070171e-01f, 2.074417621e-01f, -3.204887360e-02f, 2.866369672e-03f}};
// 1 / (transform of the kernel at frequency xi), a polynomial in (4 xi)^2
// for |xi| <= 0.2552 (relative error 1.3e-13)
constexpr double kInvHat[12] = {4.05856101315633433e-01, 4.66157209092129265e-01, 2.80608321608683930e-01,
                                1.18036114521012508e-01, 3.90287000662849701e-02, 1.08188056068415379e-02,
                                2.61583858432692246e-03, 5.72886663654686968e-04, 1.06769820665924113e-04,
                                2.69661860537872370e-05, 1.03610339097734577e-07, 1.69455818779958946e-06};

// Windows hold c / 2^ecm times the taps in FP32, kAccBits above their value
// (two tap scales and the coefficients' own); cells hold c in units of
// 2^(esum - kCellBits).  2^ecm exceeds every |Re c|, |Im c|, 2^esum their sum.
constexpr int kCoefBits = 4;
constexpr int kAccBits = 8 + 8 + kCoefBits;
constexpr int kCellBits = 61;

}  // namespace

struct UvGridScale {
  uint32_t maxima[kInitBlocks];  // the init blocks' largest |.|, as bits
  double sums[kInitBlocks];      // and sums of |.|
};

namespace {

// State of one source, behind its grids: whether a bin was not finite (the
// patch is then NaN); the init blocks' maxima and sums; the spreading workgroups' sums
// of Re c (fused form).
struct UvGridState {
  uint32_t poison;
  uint32_t next;  // spans handed out beyond the workgroups' first
  uint32_t pad[62];
  UvGridScale scale;
  double peak[kGridMaxSpans];
  int64_t first[kGridMaxSpans];  // source 0, fused: first bin of every span
};

template <class S>
__device__ __forceinline__ unsigned long long* cells_of(const S& s) {
  return reinterpret_cast<unsigned long long*>(s.work);
}

__device__ __forceinline__ double inv_hat(double xi) {
  const double z = 16.0 * xi * xi;
  double v = kInvHat[11];
#pragma unroll
  for (int q = 10; q >= 0; --q) v = fma(v, z, kInvHat[q]);
  return v;
}

// The nine taps of a bin at offset f from its nearest cell.
__device__ __forceinline__ void taps(float f, float t[kW]) {
  const float g = f * f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float e = kTapScale * kE[r][4], o = kTapScale * kO[r][3];
#pragma unroll
    for (int q = 3; q >= 0; --q) e = __builtin_fmaf(e, g, kTapScale * kE[r][q]);
#pragma unroll
    for (int q = 2; q >= 0; --q) o = __builtin_fmaf(o, g, kTapScale * kO[r][q]);
    t[r] = __builtin_fmaf(f, o, e);
    t[8 - r] = __builtin_fmaf(-f, o, e);
  }
  float e = kTapScale * kE[4][4];
#pragma unroll
  for (int q = 3; q >= 0; --q) e = __builtin_fmaf(e, g, kTapScale * kE[4][q]);
  t[4] = e;
}

__device__ __forceinline__ int wrap(int d, int M) { return d & (M - 1); }  // M: a power of two

// Position of frequency f step (turns) on a torus of M cells: nearest cell
// (0 .. M - 1) and the offset from it.  A frequency that is not finite has an
// offset that is not, in some cell.
__device__ __forceinline__ void torus(double f, double step, int M, int* cell, float* off) {
  const double t = __builtin_amdgcn_fract(f * step) * M;
  const double n = rint(t);
  *off = static_cast<float>(t - n);
  *cell = wrap(static_cast<int>(n), M);
}

typedef const __attribute__((address_space(4))) UvGridSrc karg_gsrc;
__device__ __forceinline__ karg_gsrc& gsrc(int s) {
  typedef const __attribute__((address_space(4))) uint8_t karg_byte;
  return ((karg_gsrc*)((karg_byte*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(UvGridArgs, src)))[s];
}

__device__ __forceinline__ UvGridState* state_of(const UvGridArgs& a, karg_gsrc& s) {
  return reinterpret_cast<UvGridState*>(s.work + (static_cast<size_t>(a.ml) * a.mm + static_cast<size_t>(a.ml) * s.nm) *
                                                   sizeof(double2));
}

// ecm and esum of a source; each wave for itself.
struct Exponents {
  int ecm, esum;
};
__device__ __forceinline__ Exponents exponents(karg_gsrc& s, int n) {
  uint32_t m = 0;
  double sum = 0.0;
  // (a fixed count, so that the loads are under way together)
#pragma unroll
  for (int r = 0; r < kInitBlocks / 64; ++r) {
    const int q = (threadIdx.x & 63) + 64 * r, qc = min(q, n - 1);
    m = max(m, s.scale->maxima[qc]);
    sum += q < n ? s.scale->sums[qc] : 0.0;
  }
  for (int o = 32; o > 0; o >>= 1) {
    m = max(m, static_cast<uint32_t>(__shfl_xor(static_cast<int>(m), o)));
    sum += __shfl_xor(sum, o);
  }
  const int ecm = static_cast<int>(__builtin_amdgcn_readfirstlane(m) >> 23) - 126;
  // (no exponent of its own where the sum is 0 or not finite: the patch is 0 or NaN)
  const int esum = sum > 0.0 && sum < 1e300 ? __builtin_amdgcn_frexp_exp(sum) : ecm;
  return {ecm, __builtin_amdgcn_readfirstlane(esum)};
}

}  // namespace

namespace {

// The bins are handed out in contiguous spans of equal or falling cost: with
// one level, a span per workgroup; with more, a span of half the workgroup's
// even share, one of a quarter and so on, the last two alike, so that
// workgroups that find their spans cheaper take more of the later ones, while
// most bins lie in long spans (whose tracks are cut into fewer chunks).
// First unit of span i, in units of the last level's span.
__host__ __device__ inline int span_units(const UvGridArgs& a, int i) {
  const int q = i / a.n_wg, all = 1 << (a.levels - 1);
  return a.n_wg * (all - (all >> q)) + (i - q * a.n_wg) * (all >> (q + 1) > 0 ? all >> (q + 1) : 1);
}

// What a bin of nt x nc samples costs to spread, from the cycles measured per
// 64 bins: staging and contraction, the samples' factors (a row of evenly
// spaced channels costs little more than one channel), and the set-up of its
// chunk, which holds at most kTabRows samples in time.
__device__ __forceinline__ float bin_cost(int nt, int nc, int nf) {
  const float row = nc >= kEvenMin && nc <= kEvenMax ? 600.f + 20.f * nc : 350.f * nc;
  return 3500.f + nt * (row + 3500.f / nf);
}

// The fused form's spans, equal parts of the cost rather than of the bins:
// the bins of baseline-dependent averaging are of one to hundreds of samples.
// A thread sums consecutive baselines; of kCutBlocks workgroups, each places
// the spans that begin in its share of every thread's baselines.
__device__ void cut_spans(const UvGridArgs& a, int block, int64_t* first) {
  __shared__ double wave_sum[4];
  const ObsView& o = a.o;
  const int per = (o.n_bl + 255) / 256;
  const int b0 = min(o.n_bl, static_cast<int>(threadIdx.x) * per), b1 = min(o.n_bl, b0 + per);
  float w = 0.f;  // of a bin of the baseline last looked at
  auto cost = [&](int b) {
    const int nt = max(1, o.bl_bin[2 * b]), nc = max(1, o.bl_bin[2 * b + 1]);
    w = bin_cost(min(nt, o.n_t), min(nc, o.n_ch), 1 + (o.n_ch - 1) / nc);
    return static_cast<double>(w) * static_cast<double>((b + 1 < o.n_bl ? o.koff[b + 1] : o.K) - o.koff[b]);
  };
  // the first kCutBlocks baselines of the thread (up to 2048 in all) stay in
  // registers: one round of loads
  double own[kCutBlocks], sum = 0.0;
  float own_w[kCutBlocks];
#pragma unroll
  for (int r = 0; r < kCutBlocks; ++r) {
    own[r] = b0 + r < b1 ? cost(b0 + r) : 0.0;
    own_w[r] = w;
  }
#pragma unroll
  for (int r = 0; r < kCutBlocks; ++r) sum += own[r];
  for (int b = b0 + kCutBlocks; b < b1; ++b) sum += cost(b);
  double upto = sum;  // of this thread and those before it
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int step = 1; step < 64; step <<= 1) {
    const double v = __shfl_up(upto, step);
    if (lane >= step) upto += v;
  }
  if (lane == 63) wave_sum[wave] = upto;
  double x = __shfl_up(upto, 1);  // where this thread's first baseline begins
  __syncthreads();
  if (lane == 0) x = 0.0;
  double before = 0.0, all = 0.0;
  for (int q = 0; q < 4; ++q) {
    if (q == wave) before = all;
    all += wave_sum[q];
  }
  x += before;
  const double end = lane == 63 ? before + wave_sum[wave] : upto + before;  // the next thread's x
  const double unit = all / span_units(a, a.n_span);
  // the spans that begin in [x0, x1), the cost of baseline b's bins
  auto place = [&](int b, double x0, double x1, float bin) {
    const int u = static_cast<int>(x0 / unit) - 1;
    int i = 0, q = 0;
    for (; q < a.levels && span_units(a, (q + 1) * a.n_wg) <= u; ++q) i += a.n_wg;
    i += max(0, u - span_units(a, i)) / max(1, 1 << (a.levels - 1) >> (q + 1));
    for (; i < a.n_span; ++i) {
      const double at = span_units(a, i) * unit;
      if (at < x0) continue;
      if (!(at < x1)) break;
      first[i] = o.koff[b] + static_cast<int64_t>((at - x0) / bin);
    }
  };
  double x0 = x, x1 = x;
  float bin = 1.f;
#pragma unroll
  for (int r = 0; r < kCutBlocks; ++r) {
    const double next = b0 + r + 1 == b1 ? end : x + own[r];
    if (r == block) {
      x0 = x;
      x1 = next;
      bin = own_w[r];
    }
    x = next;
  }
  if (b0 + block < b1) place(b0 + block, x0, x1, bin);
  for (int b = b0 + kCutBlocks; b < b1; ++b) {
    const double next = b + 1 < b1 ? x + cost(b) : (cost(b), end);
    if ((b - b0) % kCutBlocks == block) place(b, x, next, w);
    x = next;
  }
}

}  // namespace

// Zeroes the cells and finds the largest and the sum of the |.| of the n
// floats that scale a source: its coefficients' parts, or in the fused form
// the weights (|D| <= 1; one pass, by source 0's blocks, for all sources).
// Block q leaves its own in maxima[q] and sums[q], which later kernels join.
__global__ __launch_bounds__(256) void k_grid_init(UvGridArgs a) {
  karg_gsrc& s = gsrc(blockIdx.y);
  if (static_cast<int>(blockIdx.x) >= a.n_init) {  // kCutBlocks more where fused
    if (blockIdx.y == 0) cut_spans(a, blockIdx.x - a.n_init, state_of(a, s)->first);
    return;
  }
  const int64_t id = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x, step = static_cast<int64_t>(a.n_init) * 256;
  g_u32x4* q = reinterpret_cast<g_u32x4*>(s.work);
  const int64_t ncell = static_cast<int64_t>(a.ml) * a.mm;
  for (int64_t i = id; i < ncell; i += step) q[i] = g_u32x4{0, 0, 0, 0};
  if (id == 0) state_of(a, s)->poison = state_of(a, s)->next = 0;
  if (a.fused && blockIdx.y > 0) return;
  const uint32_t* c = reinterpret_cast<const uint32_t*>(a.fused ? a.o.W : reinterpret_cast<const float*>(s.c));
  const int64_t n = a.fused ? a.o.K : 2 * a.o.K;
  uint32_t m = 0;
  double sum = 0.0;
  auto take = [&](uint32_t v) {
    v &= 0x7fffffffu;
    m = max(m, v);
    sum += static_cast<double>(__builtin_bit_cast(float, v));
  };
  // 16 bytes per load where the array allows, its last n mod 4 words apart
  const bool wide = (reinterpret_cast<uintptr_t>(c) & 15) == 0;
  const int64_t n4 = wide ? n / 4 : 0;
  const g_u32x4* c4 = reinterpret_cast<const g_u32x4*>(c);
#pragma unroll 8
  for (int64_t k = id; k < n4; k += step) {
    const g_u32x4 v = c4[k];
    for (int q = 0; q < 4; ++q) take(v[q]);
  }
  for (int64_t k = 4 * n4 + id; k < n; k += step) take(c[k]);
  for (int o = 32; o > 0; o >>= 1) {
    m = max(m, static_cast<uint32_t>(__shfl_xor(static_cast<int>(m), o)));
    sum += __shfl_xor(sum, o);
  }
  __shared__ uint32_t w[4];
  __shared__ double ws[4];
  if ((threadIdx.x & 63) == 0) {
    w[threadIdx.x >> 6] = m;
    ws[threadIdx.x >> 6] = sum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    s.scale->maxima[blockIdx.x] = max(max(w[0], w[1]), max(w[2], w[3]));
    s.scale->sums[blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
  }
}

namespace {

// How an operand is carried: FP32, split hi + lo in BF16 or FP16, or one
// FP16 value rounded stochastically.
constexpr uint32_t kWeyl = 0x9E3779B1u;
enum Mode : int { kM32, kMBF16, kMFP16, kMSR };
__host__ __device__ constexpr Mode row_mode(int prec) {
  return prec == kFP32 ? kM32 : prec == kSplitBF16 ? kMBF16 : prec == kSplitFP16 ? kMFP16 : kMSR;
}
__host__ __device__ constexpr Mode col_mode(int prec) { return prec == kMixedFP16 ? kMFP16 : row_mode(prec); }

// One axis' nine operand values of a bin into the stage, at rows row0 ..
// row0 + 8, column `lane` (rw: a random word of the bin and axis).
template <Mode M>
__device__ __forceinline__ void stage_taps(g_lds* st, int row0, int lane, const float t[kW], uint32_t rw) {
  if constexpr (M == kM32) {
    typedef __attribute__((address_space(3))) float lds_f32;
    g_lds* p = st + row0 * kRow32 + lane * 4;
#pragma unroll
    for (int r = 0; r < kW; ++r) *reinterpret_cast<lds_f32*>(p + r * kRow32) = t[r];
  } else {
    typedef __attribute__((address_space(3))) uint16_t lds_u16;
    g_lds* p = st + row0 * kRow16 + lane * 2;
#pragma unroll
    for (int r = 0; r < kW; r += 2) {
      const bool two = r + 1 < kW;
      const float v0 = t[r], v1 = two ? t[two ? r + 1 : r] : 0.f;
      uint32_t hi, lo = 0;
      if constexpr (M == kMBF16) {
        hi = pack_bf16x2(v0, v1);
        lo = pack_bf16x2(v0 - bf16_lo_to_f32(hi), v1 - bf16_hi_to_f32(hi));
      } else if constexpr (M == kMFP16) {
        hi = pack_f16x2(v0, v1);
        lo = f16_lo_pair(hi, v0, v1);
      } else {
        // a word of its own for every tap, stepped by the golden ratio
        f16x2_t h = {0, 0};
        h = __builtin_amdgcn_cvt_sr_f16_f32(h, v0, rw + r * kWeyl, false);
        if (two) h = __builtin_amdgcn_cvt_sr_f16_f32(h, v1, rw + (r + 1) * kWeyl, true);
        hi = __builtin_bit_cast(uint32_t, h);
      }
      *reinterpret_cast<lds_u16*>(p + r * kRow16) = static_cast<uint16_t>(hi);
      if (M != kMSR) *reinterpret_cast<lds_u16*>(p + r * kRow16 + kPlane16) = static_cast<uint16_t>(lo);
      if (two) {
        *reinterpret_cast<lds_u16*>(p + (r + 1) * kRow16) = static_cast<uint16_t>(hi >> 16);
        if (M != kMSR) *reinterpret_cast<lds_u16*>(p + (r + 1) * kRow16 + kPlane16) = static_cast<uint16_t>(lo >> 16);
      }
    }
  }
}

// Bytes of a staged operand, and of a wave's stage.
constexpr int operand_bytes(Mode m) { return m == kMSR ? kPlane16 : m == kM32 ? 16 * kRow32 : 2 * kPlane16; }
constexpr int stage_bytes(Mode a, Mode b) { return operand_bytes(a) > operand_bytes(b) ? operand_bytes(a) : operand_bytes(b); }

template <Mode M>
__device__ __forceinline__ void stage_clear(g_lds* st, int lane) {
  typedef __attribute__((address_space(3))) g_u32x4 lds_u32x4;
  constexpr int n = operand_bytes(M), whole = n / 1024;
#pragma unroll
  for (int q = 0; q < whole; ++q)
    *reinterpret_cast<lds_u32x4*>(st + q * 1024 + lane * 16) = g_u32x4{0, 0, 0, 0};
  if (lane < n % 1024 / 16) *reinterpret_cast<lds_u32x4*>(st + whole * 1024 + lane * 16) = g_u32x4{0, 0, 0, 0};
}

// Cells of a workgroup's LDS tile (16 bytes each): what the stages and tables
// leave of a third of a compute unit's LDS (160 KiB in pieces of 1280 bytes).
// Fast tracks, which leave a tile soon, are 3 to 7% slower with 1024.
constexpr int tile_cells(Mode a, Mode b, bool fused) {
  const int used = kWaves * stage_bytes(a, b) + (fused ? (kTabRows + 2 * kTabFreq) * 8 : 24) + 16;
  const int n = (42 * 1280 - used) / 16 / 16 * 16;
  return n < 2048 ? n : 2048;
}
// The side to which a tile grows when its chunk leaves room.
constexpr int tile_side(int cells) {
  int n = 16;
  while ((n + 1) * (n + 1) <= cells) ++n;
  return n;
}

// A wave's LDS operations run in order; this keeps the compiler's order too.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The operand fragments of the staged 64 bins: 16-bit forms two chunks of 32
// bins x (hi, lo), one value each in the stochastic form; FP32 four groups of
// 16 bins.
struct Frags {
  g_u32x4 v[4];
};
template <Mode M>
__device__ __forceinline__ Frags stage_read(const g_lds* st, int lane) {
  typedef const __attribute__((address_space(3))) g_u32x4 lds_u32x4;
  const int lr = lane & 15, lg = lane >> 4;
  Frags f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (M == kM32)
      f.v[q] = *reinterpret_cast<lds_u32x4*>(st + lr * kRow32 + q * 64 + lg * 16);
    else if (M != kMSR || (q & 1) == 0)
      f.v[q] = *reinterpret_cast<lds_u32x4*>(st + (q & 1) * kPlane16 + lr * kRow16 + (q >> 1) * 64 + lg * 16);
  }
  return f;
}

template <Mode M>
__device__ __forceinline__ g_f32x4 mma16(g_u32x4 a, g_u32x4 b, g_f32x4 c) {
  if constexpr (M == kMBF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(g_bf16x8, a), __builtin_bit_cast(g_bf16x8, b), c,
                                                   0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(g_f16x8, a), __builtin_bit_cast(g_f16x8, b), c, 0,
                                                  0, 0);
}

// acc += A B over the staged bins (go: the lanes whose bins take part).
template <Mode MA, Mode MB>
__device__ __forceinline__ g_f32x4 contract_frags(const Frags& a, const Frags& b, uint64_t go, g_f32x4 acc) {
  if constexpr (MA == kM32) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (((go >> (16 * q)) & 0xffff) == 0) continue;  // none of these 16 bins in this window
      const g_f32x4 av = __builtin_bit_cast(g_f32x4, a.v[q]), bv = __builtin_bit_cast(g_f32x4, b.v[q]);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[e], acc, 0, 0, 0);
    }
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      acc = mma16<MB>(a.v[2 * h], b.v[2 * h], acc);
      if (MB != kMSR) acc = mma16<MB>(a.v[2 * h], b.v[2 * h + 1], acc);
      if (MA != kMSR) acc = mma16<MB>(a.v[2 * h + 1], b.v[2 * h], acc);
    }
  }
  return acc;
}

// The 32-bit finaliser of MurmurHash3.
__device__ __forceinline__ uint32_t mix_word(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}

// A workgroup's tile of the grid in LDS.
struct Tile {
  int ox, oy, bx, by;  // origin (cells of the torus) and extent; bx = 0: none
};

struct Cells {
  unsigned long long* g;
  int ml, mm;
};

__device__ __forceinline__ void add_cell(const Cells& c, int i, int j, int part, unsigned long long v) {
  if (v == 0) return;
  __hip_atomic_fetch_add(&c.g[2 * (static_cast<int64_t>(i) * c.mm + j) + part], v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
}

// x scale 2^32 as a 64-bit integer (two's complement), |x scale| < 2^31: the
// FP32 value's own bits, but for values below 2^32, whose fraction is rounded
// to 2^8.
__device__ __forceinline__ unsigned long long to_fixed(float x, float scale) {
  const float y = x * scale;
  const uint32_t hi = static_cast<uint32_t>(static_cast<int>(floorf(y)));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_fractf(y) * 4294967296.0f);
  return static_cast<unsigned long long>(hi) << 32 | lo;
}

// A window's accumulators (origin wx, wy) into the tile, cells outside the
// tile straight into the grid.  A bin whose u', v' or c is not finite leaves
// some accumulator so: the source is poisoned.
__device__ __forceinline__ void fold_window(const Cells& cells, const Tile& t, unsigned long long* tre,
                                            unsigned long long* tim, int wx, int wy, float scale, int lane,
                                            const g_f32x4& re, const g_f32x4& im, UvGridState* state) {
  const int j = lane & 15, i0 = 4 * (lane >> 4);
  const int rx = wrap(wx - t.ox, cells.ml), ry = wrap(wy - t.oy, cells.mm);
  float all = 0.f;  // 0 unless one is not finite
#pragma unroll
  for (int e = 0; e < 4; ++e) all = __builtin_fmaf(0.f, re[e], __builtin_fmaf(0.f, im[e], all));
  if (all != 0.f) state->poison = 1;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const unsigned long long vr = to_fixed(re[e], scale), vi = to_fixed(im[e], scale);
    const int ti = rx + i0 + e, tj = ry + j;
    if (ti < t.bx && tj < t.by) {
      __hip_atomic_fetch_add(&tre[ti * t.by + tj], vr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_fetch_add(&tim[ti * t.by + tj], vi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
      int gi = wx + i0 + e, gj = wy + j;
      if (gi >= cells.ml) gi -= cells.ml;
      if (gj >= cells.mm) gj -= cells.mm;
      add_cell(cells, gi, gj, 0, vr);
      add_cell(cells, gi, gj, 1, vi);
    }
  }
}

__device__ __forceinline__ int first_lane(uint64_t m) { return __builtin_ctzll(m); }
__device__ __forceinline__ int last_lane(uint64_t m) { return 63 - __builtin_clzll(m); }

// Where a window of one axis starts: it holds the anchor a of the first
// waiting bin and extends towards the anchor b of the last.
__device__ __forceinline__ int window_origin(int a, int b, int M) {
  int d = b - a;
  if (d > M / 2) d -= M;
  if (d < -M / 2) d += M;
  const int o = d > kSlack ? a : d < -kSlack ? a - kSlack : a + min(d, 0) - (kSlack - (d < 0 ? -d : d)) / 2;
  return o < 0 ? o + M : o;
}

// What a chunk of one baseline's bins needs: time rows t0 .. t0 + rows of nf
// frequency bins, of which the bins [la, lb) (counted from the baseline's
// first) belong to the workgroup.
struct Chunk {
  int64_t base, la, lb, t0;
  int b, nf, nt, nc, rows;
  int left;   // samples from the chunk's first on (at most 2^30)
  int full;   // samples of a whole bin
  float inv;  // 1 / full
};

// Sum over one bin's samples of exp(-2 pi i phi), phi = (A_t nu_c - A_k nu_k)
// / c: channels in groups of four whose frequencies sit in registers, the
// projections A_t from the chunk's table in LDS (tab, row t of time bin tr at
// tab[t rows + tr]) or, for bins too long for it, from the rows themselves.
// The products round separately, so that identical rows cancel exactly.
template <int NCH>
__device__ __forceinline__ void sum_group(const double* tab, int pitch, int ntu, int ntl, const double nu[4], int nch,
                                          double aknu, float* sre, float* sim) {
#pragma clang fp contract(off)
  constexpr int kRows = NCH == 1 ? 4 : NCH == 2 ? 2 : 1;  // four sine-cosine pairs at a time, for their latency
  auto rows = [&](int t, auto many) {
#pragma clang fp contract(off)
    constexpr int n = decltype(many)::value;
    double at[n];
#pragma unroll
    for (int i = 0; i < n; ++i) at[i] = tab[(t + i) * pitch];
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
      for (int j = 0; j < (NCH == 0 ? 4 : NCH); ++j) {
        const cf32 e = expi_turns_hw(-((at[i] * nu[j] - aknu) * kInvCLight));
        const bool on = t + i < ntl && (NCH != 0 || j < nch);
        *sre += on ? e.re : 0.f;
        *sim += on ? e.im : 0.f;
      }
  };
  int t = 0;
  for (; t + kRows <= ntu; t += kRows) rows(t, std::integral_constant<int, kRows>());
  if (kRows > 1)
    for (; t < ntu; ++t) rows(t, std::integral_constant<int, 1>());
}

// The same sum for n evenly spaced channels about nu_k (half spacing h, in
// s/m): a sample row's channels sum to exp(-2 pi i (A_t - A_k) nu_k / c)
// times the Dirichlet kernel 1 + 2 cos x + ... + 2 cos((n - 1) x / 2) (n odd)
// or 2 cos(x / 2) + 2 cos(3 x / 2) + ... (n even), x = 4 pi A_t h, so that a
// row costs two sine-cosine pairs and three operations per channel pair
// instead of a pair and eight operations per channel.  The cosines step by
// their differences, d <- d - 4 sin^2(x / 2) a, a <- a + d, which loses
// nothing at small x.  From 3 channels (2 save nothing) to 16 (the steps'
// rounding grows with their number): 10 x 4 samples take 490 vector
// instructions per 64 bins with all else, 1270 channel by channel.
// m: (n - 1) / 2, at most mm; SAME: every lane has mm and ntu rows.  Half the
// sum is returned.
template <bool SAME>
__device__ __forceinline__ void sum_even(const double* tab, int pitch, int ntu, int ntl, double nkc, double ak, double h,
                                         bool odd, int m, int mm, float* sre, float* sim) {
  // two rows at a time, for the latency of the sine and cosine
  for (int t = 0; t < ntu; t += 2) {
    float a[2], d[2], q[2], s4[2];
    cf32 e[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const double at = tab[min(t + i, ntu - 1) * pitch];
      e[i] = expi_turns_hw((ak - at) * nkc);
      const cf32 b = expi_half_turns(at * h);
      s4[i] = -4.0f * b.im * b.im;
      a[i] = odd ? 1.0f : b.re;
      d[i] = odd ? -0.5f * s4[i] : 0.0f;
      q[i] = odd ? 0.5f : b.re;
    }
    for (int j = 0; j < mm; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        d[i] = __builtin_fmaf(s4[i], a[i], d[i]);
        a[i] += d[i];
        q[i] += SAME || j < m ? a[i] : 0.0f;
      }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float g = (SAME ? t + i < ntu : t + i < ntl) ? q[i] : 0.0f;
      *sre = __builtin_fmaf(g, e[i].re, *sre);
      *sim = __builtin_fmaf(g, e[i].im, *sim);
    }
  }
}

// Decorrelation factor of this lane's bin (time bin tr of the chunk,
// channels c0 .. c1, centre frequency nuk, half channel spacing h or NaN), as
// k_decorr forms it.
__device__ __forceinline__ cf32 bin_factor(const ObsView& o, const Chunk& ch, const double* tab, bool in, int tr, int c0,
                                           int c1, double nuk, double ak, double h, double l0, double m0, double lw) {
#pragma clang fp contract(off)
  const double aknu = ak * nuk;
  float sre = 0.f, sim = 0.f;
  const int ntl = in ? min(ch.nt, ch.left - tr * ch.nt) : 0;
  if (tab != nullptr && ch.nc == 1) {
    // one channel: its frequency is the bin's centre
    const double nu[4] = {nuk, nuk, nuk, nuk};
    sum_group<1>(tab + tr, ch.rows, ch.nt, ntl, nu, 1, aknu, &sre, &sim);
  } else if (tab != nullptr && ch.nc >= kEvenMin && ch.nc <= kEvenMax && !__any(in && h != h)) {
    const int n = c1 - c0, m = (n - 1) >> 1;
    if (!__any(in && (n != ch.nc || ntl != ch.nt))) {
      const int mm = (ch.nc - 1) >> 1;
      sum_even<true>(tab + tr, ch.rows, ch.nt, ntl, nuk * kInvCLight, ak, h, (ch.nc & 1) != 0, mm, mm, &sre, &sim);
    } else {
      sum_even<false>(tab + tr, ch.rows, ch.nt, ntl, nuk * kInvCLight, ak, h, (n & 1) != 0, m, (ch.nc - 1) >> 1, &sre, &sim);
    }
    sre *= 2.0f;
    sim *= 2.0f;
  } else {
    for (int cb = c0; __any(in && cb < c1); cb += 4) {
      const int nch = in ? min(4, c1 - cb) : 0;  // <= 0: none left for this lane
      double nu[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) nu[j] = o.freq[max(0, min(cb + max(0, min(j, nch - 1)), o.n_ch - 1))];
      const int nl = nch > 0 ? ntl : 0;
      if (tab != nullptr) {
        const uint64_t act = __ballot(nl > 0);
        if (act == __ballot(nl > 0 && nch == 1)) sum_group<1>(tab + tr, ch.rows, ch.nt, nl, nu, nch, aknu, &sre, &sim);
        else if (act == __ballot(nl > 0 && nch == 2)) sum_group<2>(tab + tr, ch.rows, ch.nt, nl, nu, nch, aknu, &sre, &sim);
        else if (act == __ballot(nl > 0 && nch == 4)) sum_group<4>(tab + tr, ch.rows, ch.nt, nl, nu, nch, aknu, &sre, &sim);
        else sum_group<0>(tab + tr, ch.rows, ch.nt, nl, nu, nch, aknu, &sre, &sim);
      } else {
        for (int t = 0; t < nl; ++t) {
          const double* row = o.uvw + 3 * (static_cast<int64_t>(ch.b) * o.n_t + (ch.t0 + tr) * ch.nt + t);
          const double at = row[0] * l0 + row[1] * m0 + row[2] * lw;
          for (int j = 0; j < nch; ++j) {
            const cf32 e = expi_turns_hw(-((at * nu[j] - aknu) * kInvCLight));
            sre += e.re;
            sim += e.im;
          }
        }
      }
    }
  }
  float inv = ch.inv;
  const int n = ntl * (c1 - c0);
  if (__any(in && n != ch.full)) inv = 1.0f / static_cast<float>(max(n, 1));  // short last bins
  return {sre * inv, sim * inv};
}

// The baseline that owns bin k: the last b with koff[b] <= k, found by the
// whole wave, 64 candidates at a time.
__device__ __forceinline__ int owner_of(const int64_t* __restrict__ koff, int n_bl, int64_t k, int lane) {
  int lo = 0, hi = n_bl;
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6;
    const int q = lo + lane * step;
    const uint64_t below = __ballot(q < hi && koff[min(q, n_bl - 1)] <= k);
    lo += (below != 0 ? last_lane(below) : 0) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// Bins [*ka, *kb) of span i.
__device__ __forceinline__ void span_bins(const UvGridArgs& a, int i, int64_t* ka, int64_t* kb) {
  int64_t p, q;
  if (a.fused) {
    const int64_t* first = state_of(a, gsrc(0))->first;
    p = first[i];
    q = i + 1 < a.n_span ? first[i + 1] : a.o.K;
  } else {
    p = span_units(a, i) * a.unit_bins;
    q = span_units(a, i + 1) * a.unit_bins;
  }
  *ka = uniform(min(max(p, int64_t(0)), a.o.K));
  *kb = uniform(min(max(q, *ka), a.o.K));
}

// Waits for this workgroup's LDS traffic only: __syncthreads also waits for
// the atomics into the grid, whose results nobody here reads.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace

// FUSED: the decorrelation factors are formed here from the samples (boxcar
// averaging), else u', v' and c come from records.  Three waves per SIMD, and
// no scratch memory (what is the same in every lane sits in scalar registers):
// a kernel that spills needs an eager launch before it can be captured, to
// have its scratch allocated.
template <int PREC, bool FUSED>
__global__ __launch_bounds__(kThreads, 3) void k_grid_spread(UvGridArgs a) {
  constexpr Mode MA = row_mode(PREC), MB = col_mode(PREC);
  constexpr int kTileCells = tile_cells(MA, MB, FUSED), kTileSide = tile_side(kTileCells), kStage = stage_bytes(MA, MB);
  __shared__ unsigned long long tre[kTileCells], tim[kTileCells];
  __shared__ __attribute__((aligned(16))) uint8_t stage_raw[kWaves * kStage];
  __shared__ double tab[FUSED ? kTabRows : 1], tabnu[FUSED ? kTabFreq : 1], tabh[FUSED ? kTabFreq : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  g_lds* st = (g_lds*)stage_raw + wave * kStage;
  karg_gsrc& s = gsrc(blockIdx.y);
  const BinRec* rec = s.rec;
  const float2* cf = s.c;
  const ObsView& o = a.o;
  double l0 = s.l0, m0 = s.m0, l_first = s.l_first, m_first = s.m_first, dl = s.dl, dm = s.dm;
  if (s.dir != nullptr) {
    l0 = s.dir[0];
    m0 = s.dir[1];
    l_first = s.dir[2];
    m_first = s.dir[3];
    dl = s.dir[4];
    dm = s.dir[5];
  }
  // (the same in every lane: kept in scalar registers)
  l0 = uniform(l0), m0 = uniform(m0), dl = uniform(dl), dm = uniform(dm);
  const double n0 = sqrt(1.0 - l0 * l0 - m0 * m0), lw = uniform(n0 - 1.0), l0n = uniform(l0 / n0), m0n = uniform(m0 / n0);
  // offsets from the source of the pixels that modes (0, 0) stand for;
  // nothing to shift where they are rounding of a grid centred on the source
  const double xh = uniform((l_first + (s.nl / 2) * dl) - l0), yh = uniform((m_first + (s.nm / 2) * dm) - m0);
  const bool shift = !(fabs(xh) <= 1e-12 * fabs(dl) && fabs(yh) <= 1e-12 * fabs(dm));
  UvGridState* state = state_of(a, s);
  const Exponents ex2 = exponents(s, a.n_init);
  const int ecm = ex2.ecm;
  const float fold_scale = uniform(ldexpf(1.0f, ecm - ex2.esum + kCellBits - kAccBits - 32));
  const Cells cells{cells_of(s), a.ml, a.mm};
  Tile tile{0, 0, 0, 0};
  int tab_nc = 0;  // channels per bin that tabnu and tabh are for
  const bool norm = s.norm != 0;
  for (int q = threadIdx.x; q < kTileCells; q += kThreads) tre[q] = tim[q] = 0;
  lds_barrier();

  // The tile into the grid, left zero; every wave has passed a barrier since
  // its last fold.
  auto flush_tile = [&]() {
    for (int i = wave; i < tile.bx; i += kWaves) {
      int gi = tile.ox + i;
      if (gi >= a.ml) gi -= a.ml;
      for (int j = lane; j < tile.by; j += 64) {
        int gj = tile.oy + j;
        if (gj >= a.mm) gj -= a.mm;
        const int e = i * tile.by + j;
        add_cell(cells, gi, gj, 0, tre[e]);
        add_cell(cells, gi, gj, 1, tim[e]);
        tre[e] = tim[e] = 0;
      }
    }
  };

  __shared__ int next_span;
  int64_t ka, kb;
  for (int span = blockIdx.x; span < a.n_span;) {
  span_bins(a, span, &ka, &kb);
  double peak = 0.0;  // this lane's share of sum Re c
  for (int b = owner_of(o.koff, o.n_bl, ka, lane); ka < kb && b < o.n_bl; ++b) {
    Chunk ch;
    ch.b = b;
    ch.base = uniform(o.koff[b]);
    const int64_t kend = uniform(b + 1 < o.n_bl ? min(kb, o.koff[b + 1]) : kb);
    if (kend <= ka) continue;
    ch.nt = uniform(max(1, o.bl_bin[2 * b]));
    ch.nc = uniform(max(1, o.bl_bin[2 * b + 1]));
    ch.nf = 1 + (o.n_ch - 1) / ch.nc;
    ch.la = ka - ch.base;
    ch.lb = kend - ch.base;
    ch.full = min(ch.nt, o.n_t) * min(ch.nc, o.n_ch);
    ch.inv = 1.0f / static_cast<float>(ch.full);
    ka = kend;
    const int64_t tb0 = uniform(o.tboff[b]);
    ch.t0 = ch.la / ch.nf;
    const int64_t t1 = (ch.lb + ch.nf - 1) / ch.nf;
    while (ch.t0 < t1) {
      // Sample the track: 32 times x both ends of the band; the longest
      // prefix whose extent fits the tile is this chunk (of at most kChunkBins
      // bins and as many rows as the table holds).
      int64_t left = t1 - ch.t0;
      left = min(left, static_cast<int64_t>(max(1, kChunkBins / ch.nf)));
      if (FUSED && ch.nt <= kTabRows) left = min(left, static_cast<int64_t>(kTabRows / ch.nt));
      const int nt = static_cast<int>(left);
      const int smp = lane >> 1;
      const int64_t tl = ch.t0 + (static_cast<int64_t>(nt - 1) * smp) / 31;
      double pu, pv;
      if constexpr (FUSED) {
        const int f = (lane & 1) * (ch.nf - 1);
        const double nu = bin_freq(o.freq, f * ch.nc, f * ch.nc + min(ch.nc, o.n_ch - f * ch.nc)) * kInvCLight;
        const double* uc = o.uvw_c + 3 * (tb0 + tl);
        pu = (uc[0] - uc[2] * l0n) * nu;
        pv = (uc[1] - uc[2] * m0n) * nu;
      } else {
        const int64_t ls = min(max(tl * ch.nf + (lane & 1) * (ch.nf - 1), ch.la), ch.lb - 1);
        pu = rec[ch.base + ls].up;
        pv = rec[ch.base + ls].vp;
      }
      pu *= dl * a.ml;
      pv *= dm * a.mm;
      const double ru = of_lane(pu, 0), rv = of_lane(pv, 0);
      const float x = static_cast<float>(pu - ru), y = static_cast<float>(pv - rv);
      const int ln = opaque(lane);
      const float x1 = from_lane(x, ln ^ 1), y1 = from_lane(y, ln ^ 1);
      float xlo = fminf(x, x1), xhi = fmaxf(x, x1), ylo = fminf(y, y1), yhi = fmaxf(y, y1);
#pragma unroll
      for (int q = 2; q < 64; q <<= 1) {
        const float p0 = from_lane(xlo, ln - q), p1 = from_lane(xhi, ln - q);
        const float p2 = from_lane(ylo, ln - q), p3 = from_lane(yhi, ln - q);
        if (lane >= q) {
          xlo = fminf(xlo, p0);
          xhi = fmaxf(xhi, p1);
          ylo = fminf(ylo, p2);
          yhi = fmaxf(yhi, p3);
        }
      }
      const float ex = ceilf(xhi - xlo) + (kW + 1 + 2 * kMargin), ey = ceilf(yhi - ylo) + (kW + 1 + 2 * kMargin);
      const uint64_t fits = __ballot(ex * ey <= kTileCells && ex <= a.ml && ey <= a.mm);
      Tile box{0, 0, 0, 0};
      ch.rows = nt;
      float vt;  // cells per time bin
      const float vf = fmaxf(fabsf(of_lane(x, 1)), fabsf(of_lane(y, 1))) / max(1, ch.nf - 1);  // per frequency bin
      const int sl = fits & 1 ? last_lane(fits) : 0, ss = sl >> 1;
      if (fits & 1) ch.rows = static_cast<int>((static_cast<int64_t>(nt - 1) * ss) / 31) + 1;
      // Where the track leaves a tile within kSparse bins (long baselines, wide
      // bands, long steps in time), a tile saves no atomics: then none, and
      // the chunk as long as it may be (K = 216k of 40 antennas to 8 km, two
      // channels 400 MHz apart, 14 s steps, 150 x 150 pixels: 334 -> 77 us).
      if ((fits & 1) && (ch.rows == nt || ch.rows * ch.nf >= kSparse)) {
        vt = fmaxf(fabsf(of_lane(x, 2 * ss)), fabsf(of_lane(y, 2 * ss))) / max(1, ch.rows - 1);
        box.bx = static_cast<int>(of_lane(ex, sl));
        box.by = static_cast<int>(of_lane(ey, sl));
        const double fx = floor(ru + of_lane(xlo, sl)) - (kW / 2 + kMargin);
        const double fy = floor(rv + of_lane(ylo, sl)) - (kW / 2 + kMargin);
        box.ox = __builtin_amdgcn_readfirstlane(min(max(static_cast<int>(fx - floor(fx / a.ml) * a.ml), 0), a.ml - 1));
        box.oy = __builtin_amdgcn_readfirstlane(min(max(static_cast<int>(fy - floor(fy / a.mm) * a.mm), 0), a.mm - 1));
      } else {
        ch.rows = nt;
        vt = fmaxf(fabsf(of_lane(x, 62)), fabsf(of_lane(y, 62))) / max(1, nt - 1);
      }
      ch.rows = __builtin_amdgcn_readfirstlane(ch.rows);
      // rectangle of time x frequency bins per wave: the fewest windows
      int lt = 0;
      float best = 3.4e38f;
      for (int q = 0; q <= 6; ++q) {
        const int bt = 1 << q, bf = 64 >> q;
        const float cost = static_cast<float>(((ch.rows + bt - 1) >> q) * ((ch.nf + bf - 1) >> (6 - q))) *
                           (1.0f + 0.5f * (bt * vt + bf * vf) * (1.0f / kSlack));
        if (cost < best) {
          best = cost;
          lt = q;
        }
      }
      lt = __builtin_amdgcn_readfirstlane(lt);
      const int bt = 1 << lt, bf = 64 >> lt;

      lds_barrier();  // the previous chunk's folds and table reads are done
      // keep the tile while the chunk lies inside it; else empty it and lay a
      // new one around the chunk
      const int rx = wrap(box.ox - tile.ox, a.ml), ry = wrap(box.oy - tile.oy, a.mm);
      if (box.bx == 0 || rx + box.bx > tile.bx || ry + box.by > tile.by) {
        flush_tile();
        tile = box;
        if (box.bx > 0) {
          tile.bx = max(box.bx, min(min(a.ml, kTileSide), kTileCells / box.by));
          tile.by = max(box.by, min(a.mm, kTileCells / tile.bx));
          tile.ox = wrap(box.ox - (tile.bx - box.bx) / 2, a.ml);
          tile.oy = wrap(box.oy - (tile.by - box.by) / 2, a.mm);
        }
      }
      ch.left = static_cast<int>(min(o.n_t - ch.t0 * ch.nt, int64_t(1) << 30));
      const bool use_tab = FUSED && ch.nt <= kTabRows, use_nu = FUSED && ch.nf <= kTabFreq;
      if constexpr (FUSED) {
#pragma clang fp contract(off)
        if (use_tab) {
          const int n = ch.rows * ch.nt;  // at most kTabRows
          const double* row = o.uvw + 3 * (static_cast<int64_t>(b) * o.n_t + ch.t0 * ch.nt);
          const float rnt = 1.0f / ch.nt;
#pragma unroll
          for (int j = 0; j < kTabRows / kThreads; ++j) {
            const int i = threadIdx.x + j * kThreads;
            const int ic = 3 * min(i, min(n, ch.left) - 1);
            const double at = row[ic] * l0 + row[ic + 1] * m0 + row[ic + 2] * lw;
            const int tr = static_cast<int>((i + 0.5f) * rnt);  // i / nt: exact for such i
            if (i < n) tab[(i - tr * ch.nt) * ch.rows + tr] = at;
          }
        }
        if (use_nu && ch.nc != tab_nc) {
          tab_nc = ch.nc;
          for (int f = threadIdx.x; f < ch.nf; f += kThreads) {
            const int c0 = f * ch.nc, c1 = c0 + min(ch.nc, o.n_ch - c0);
            tabnu[f] = bin_freq(o.freq, c0, c1);
            if (ch.nc >= kEvenMin && ch.nc <= kEvenMax) tabh[f] = even_half_step(o.freq, c0, c1, tabnu[f]);
          }
        }
      }
      lds_barrier();

      // Everything of a bin within the chunk is 32-bit: e = tr nf + f, the
      // workgroup's own bins being [elo, ehi).
      const int64_t first = ch.t0 * ch.nf;
      const int elo = static_cast<int>(max(ch.la - first, int64_t(0)));
      const int ehi = static_cast<int>(min(ch.lb - first, static_cast<int64_t>(ch.rows) * ch.nf));
      const int64_t k0 = ch.base + first;
      const int nqt = (ch.rows + bt - 1) >> lt, nqf = (ch.nf + bf - 1) >> (6 - lt);
      const int nq = nqt * nqf, per = (nq + kWaves - 1) / kWaves;
      const int q0 = wave * per, q1 = min(nq, q0 + per);
      const int tlo = lane & (bt - 1), fl0 = lane >> lt;
      g_f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = {0.f, 0.f, 0.f, 0.f};
      int wx = -1, wy = 0;  // the current window's origin, -1: none
      int run = 0;  // batches in the current window's accumulators
      double pt = 0.0, qtv = 0.0, ak = 0.0;  // the time bin's projections (metres)
      int qt = q0 / nqf, qf = q0 - qt * nqf;
      bool row_new = true;
      // the time bin's centre, loaded a rectangle ahead
      const double* ucs = FUSED ? o.uvw_c + 3 * (tb0 + ch.t0) : nullptr;
      double uc[3] = {0.0, 0.0, 0.0};
      if (FUSED && q0 < q1) {
        const int r = 3 * min((qt << lt) + tlo, ch.rows - 1);
        for (int i = 0; i < 3; ++i) uc[i] = ucs[r + i];
      }
      for (int q = q0; q < q1; ++q) {
        const int tr = (qt << lt) + tlo, f = qf * bf + fl0;
        const int e = tr * ch.nf + f;
        const bool in = f < ch.nf && static_cast<unsigned>(e - elo) < static_cast<unsigned>(ehi - elo);
        const int ec = in ? e : elo;
        double up, vp;
        float2 c0;
        if constexpr (FUSED) {
          const float W = (o.W + k0)[ec];
          const int trc = min(tr, ch.rows - 1);
          if (row_new) {
#pragma clang fp contract(off)
            const double u = uc[0], v = uc[1], w = uc[2];
            ak = u * l0 + v * m0 + w * lw;
            pt = (u - w * l0n) * kInvCLight;
            qtv = (v - w * m0n) * kInvCLight;
            const int r = 3 * min(((qt + 1) << lt) + tlo, ch.rows - 1);
            for (int i = 0; i < 3; ++i) uc[i] = ucs[r + i];
          }
          const int fc = min(f, ch.nf - 1);
          const int c0i = fc * ch.nc, c1i = c0i + min(ch.nc, o.n_ch - c0i);
          const double nu = use_nu ? tabnu[fc] : bin_freq(o.freq, c0i, c1i);
          const cf32 D = bin_factor(o, ch, use_tab ? tab : nullptr, in, trc, c0i, c1i, nu, ak, use_nu ? tabh[fc] : __builtin_nan(""), l0, m0, lw);
          up = pt * nu;
          vp = qtv * nu;
          c0 = make_float2(W * D.re, W * D.im);
          if (norm && in) peak += static_cast<double>(c0.x);
        } else {
          up = (rec + k0)[ec].up;
          vp = (rec + k0)[ec].vp;
          c0 = (cf + k0)[ec];
        }
        row_new = ++qf == nqf;
        if (row_new) {
          qf = 0;
          ++qt;
        }
        int ax, ay;
        float fx, fy;
        torus(up, dl, a.ml, &ax, &fx);
        torus(vp, dm, a.mm, &ay, &fy);
        cf32 c = {ldexpf(c0.x, kCoefBits - ecm), ldexpf(c0.y, kCoefBits - ecm)};
        if (shift) c = cmul(c, expi_turns_hw(up * xh + vp * yh));
        ax = wrap(ax - kW / 2, a.ml);
        ay = wrap(ay - kW / 2, a.mm);
        float tx[kW], ty[kW];
        taps(fx, tx);
        taps(fy, ty);
        // random words of the bin's row and column taps
        const uint32_t kw = static_cast<uint32_t>(k0) + ec;
        const uint32_t rwa = MA == kMSR ? kw * 0xC2B2AE35u : 0u, rwb = MB == kMSR ? mix_word(kw) : 0u;
        uint64_t wait = __ballot(in);
        while (wait != 0) {
          const int fl = first_lane(wait);
          const int fax = __builtin_amdgcn_readlane(ax, fl), fay = __builtin_amdgcn_readlane(ay, fl);
          if (wx < 0 || run == kRun || wrap(fax - wx, a.ml) > kSlack || wrap(fay - wy, a.mm) > kSlack) {
            run = 0;
            if (wx >= 0) {
              fold_window(cells, tile, tre, tim, wx, wy, fold_scale, lane, re, im, state);
              re = im = g_f32x4{0.f, 0.f, 0.f, 0.f};
            }
            const int ll = last_lane(wait);
            wx = window_origin(fax, __builtin_amdgcn_readlane(ax, ll), a.ml);
            wy = window_origin(fay, __builtin_amdgcn_readlane(ay, ll), a.mm);
          }
          // (opaque, or the split operands of both axes, the same in every
          // window of these bins, are formed ahead of the loop, in registers of
          // their own)
          if (MA == kMBF16 || MA == kMFP16)
#pragma unroll
            for (int r = 0; r < kW; ++r) asm volatile("" : "+v"(tx[r]));
          if (MB != kM32) asm volatile("" : "+v"(c.re), "+v"(c.im));
          ++run;
          const int dx = wrap(ax - wx, a.ml), dy = wrap(ay - wy, a.mm);
          const bool go = ((wait >> lane) & 1) != 0 && dx <= kSlack && dy <= kSlack;
          const uint64_t going = __ballot(go);
          wait &= ~going;
          stage_clear<MA>(st, lane);
          wave_order();
          if (go) stage_taps<MA>(st, dx, lane, tx, rwa);
          wave_order();
          const Frags fa = stage_read<MA>(st, lane);
          wave_order();
          stage_clear<MB>(st, lane);
          wave_order();
          float tb[kW];
#pragma unroll
          for (int r = 0; r < kW; ++r) tb[r] = ty[r] * c.re;
          if (go) stage_taps<MB>(st, dy, lane, tb, rwb);
          wave_order();
          const Frags fr = stage_read<MB>(st, lane);
          wave_order();
          re = contract_frags<MA, MB>(fa, fr, going, re);
#pragma unroll
          for (int r = 0; r < kW; ++r) tb[r] = ty[r] * c.im;
          if (go) stage_taps<MB>(st, dy, lane, tb, rwb ^ 0xAAAAAAAAu);
          wave_order();
          const Frags fi = stage_read<MB>(st, lane);
          wave_order();
          im = contract_frags<MA, MB>(fa, fi, going, im);
        }
      }
      if (wx >= 0) fold_window(cells, tile, tre, tim, wx, wy, fold_scale, lane, re, im, state);
      ch.t0 += ch.rows;
    }
  }
  // (not asked for earlier: loads issued after an atomic return after it)
  if (threadIdx.x == 0)
    next_span = a.levels == 1 ? a.n_span
                              : a.n_wg + static_cast<int>(__hip_atomic_fetch_add(&state->next, 1u, __ATOMIC_RELAXED,
                                                                                 __HIP_MEMORY_SCOPE_AGENT));
  if (FUSED && norm) {
    // sum Re c of the span, in a fixed order
    const int ln = opaque(lane);
    for (int q = 32; q > 0; q >>= 1) peak += from_lane(peak, ln ^ q);
    lds_barrier();
    if (lane == 0) tab[wave] = peak;
  }
  lds_barrier();
  if (FUSED && norm && threadIdx.x == 0) {
    double p = 0.0;
    for (int w = 0; w < kWaves; ++w) p += tab[w];
    state->peak[span] = p;
  }
  span = __builtin_amdgcn_readfirstlane(next_span);
  lds_barrier();
  }
  flush_tile();
}

// In-place inverse DFT (sign +) of the M complex values in `v` (LDS), radix
// 2, decimation in frequency: the result is in bit-reversed order.  tw holds
// exp(2 pi i q / M), q < M / 2.
__device__ __forceinline__ void fft_lds(double2* v, const double2* tw, int M) {
  for (int half = M >> 1, sh = 0; half > 0; half >>= 1, ++sh) {
    for (int t = threadIdx.x; t < (M >> 1); t += blockDim.x) {
      const int p = t & (half - 1);
      const int i0 = ((t - p) << 1) + p;
      const double2 x = v[i0], y = v[i0 + half], w = tw[p << sh];
      const double dr = x.x - y.x, di = x.y - y.y;
      v[i0] = make_double2(x.x + y.x, x.y + y.y);
      v[i0 + half] = make_double2(dr * w.x - di * w.y, dr * w.y + di * w.x);
    }
    __syncthreads();
  }
}

__device__ __forceinline__ void fft_twiddles(double2* tw, int M) {
  for (int q = threadIdx.x; q < (M >> 1); q += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * q / M, &sn, &cs);
    tw[q] = make_double2(cs, sn);
  }
}

__device__ __forceinline__ int bit_reverse(int i, int log_m) {
  return static_cast<int>(__brev(static_cast<unsigned>(i)) >> (32 - log_m));
}

// Grid row blockIdx.x: cells to modes 0 .. nm - 1 of the patch's columns
// (mode j - nm / 2), divided by the kernel's transform, to mid[j][row].
__global__ __launch_bounds__(256) void k_grid_rows(UvGridArgs a) {
  extern __shared__ double2 fft_buf[];
  karg_gsrc& s = gsrc(blockIdx.y);
  const int M = a.mm, log_m = 31 - __clz(M), row = blockIdx.x;
  double2* v = fft_buf;
  double2* tw = fft_buf + M;
  const long long* g = reinterpret_cast<const long long*>(cells_of(s)) + 2 * static_cast<int64_t>(row) * M;
  for (int q = threadIdx.x; q < M; q += 256) v[q] = make_double2(static_cast<double>(g[2 * q]), static_cast<double>(g[2 * q + 1]));
  fft_twiddles(tw, M);
  __syncthreads();
  fft_lds(v, tw, M);
  double2* mid = reinterpret_cast<double2*>(s.work) + static_cast<int64_t>(a.ml) * a.mm;
  for (int j = threadIdx.x; j < s.nm; j += 256) {
    const int m = j - s.nm / 2;
    const double2 z = v[bit_reverse(m < 0 ? m + M : m, log_m)];
    const double f = inv_hat(static_cast<double>(m) / M);
    mid[static_cast<int64_t>(j) * a.ml + row] = make_double2(z.x * f, z.y * f);
  }
}

// Patch column blockIdx.x: inverse DFT of mid[column] to its rows' pixels.
__global__ __launch_bounds__(256) void k_grid_cols(UvGridArgs a) {
  extern __shared__ double2 fft_buf[];
  karg_gsrc& s = gsrc(blockIdx.y);
  const int col = blockIdx.x;
  if (col >= s.nm) return;
  const int M = a.ml, log_m = 31 - __clz(M);
  double2* v = fft_buf;
  double2* tw = fft_buf + M;
  const double2* mid = reinterpret_cast<const double2*>(s.work) + static_cast<int64_t>(a.ml) * a.mm +
                       static_cast<int64_t>(col) * M;
  for (int q = threadIdx.x; q < M; q += 256) v[q] = mid[q];
  fft_twiddles(tw, M);
  __syncthreads();
  fft_lds(v, tw, M);
  double scale = ldexp(2.0, exponents(s, a.n_init).esum - kCellBits);
  if (state_of(a, s)->poison != 0) scale = __builtin_nan("");
  const bool norm = a.fused ? s.norm != 0 : s.peak != nullptr;
  double peak = 1.0;
  if (norm && a.fused) {
    // 2 sum Re c: the spreading workgroups' sums, in a fixed order
    double p = 0.0;
    for (int q = threadIdx.x; q < a.n_span; q += 256) p += state_of(a, s)->peak[q];
    for (int q = 32; q > 0; q >>= 1) p += __shfl_xor(p, q);
    __syncthreads();  // the twiddles are read no more
    if ((threadIdx.x & 63) == 0) tw[threadIdx.x >> 6].x = p;
    __syncthreads();
    peak = 2.0 * (((tw[0].x + tw[1].x) + tw[2].x) + tw[3].x);
  } else if (norm) {
    peak = *s.peak;
  }
  for (int i = threadIdx.x; i < s.nl; i += 256) {
    const int m = i - s.nl / 2;
    const double2 z = v[bit_reverse(m < 0 ? m + M : m, log_m)];
    const float p = static_cast<float>(z.x * inv_hat(static_cast<double>(m) / M) * scale);
    // normalised: 0 where the peak is 0 (no weight at all)
    s.P[static_cast<int64_t>(i) * s.nm + col] =
        !norm ? p : peak != 0.0 ? static_cast<float>(static_cast<double>(p) / peak) : 0.0f;
  }
}

// ---------------------------------------------------------------- host side
int grid_axis(int n) {
  int m = 32;
  while (100LL * m < 196LL * n) m <<= 1;
  return m <= kGridMaxAxis ? m : 0;
}

size_t grid_bytes(const GridPlan& g, int nm) {
  return (static_cast<size_t>(g.ml) * g.mm + static_cast<size_t>(g.ml) * nm) * sizeof(double2) +
         sizeof(UvGridState) + kGridAlign;
}

template <int PREC>
static void launch_spread(const UvGridArgs& a, dim3 grid, hipStream_t stream) {
  if (a.fused)
    hipLaunchKernelGGL((k_grid_spread<PREC, true>), grid, dim3(kThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((k_grid_spread<PREC, false>), grid, dim3(kThreads), 0, stream, a);
}

hipError_t launch_grid(int prec, UvGridArgs a, hipStream_t stream) {
  if (a.n_src < 1 || a.n_src > kMaxBatch || a.ml < 32 || a.mm < 32 || a.ml > kGridMaxAxis || a.mm > kGridMaxAxis ||
      (a.ml & (a.ml - 1)) != 0 || (a.mm & (a.mm - 1)) != 0 || a.o.K < 1)
    return hipErrorInvalidValue;
  int nm = 0;
  for (int s = 0; s < a.n_src; ++s) {
    if (a.src[s].nl > a.ml || a.src[s].nm > a.mm) return hipErrorInvalidValue;
    nm = a.src[s].nm > nm ? a.src[s].nm : nm;
    // every source of the fused form is scaled by the weights
    const int m = a.fused ? 0 : s;
    a.src[s].scale = &reinterpret_cast<UvGridState*>(
                          a.src[m].work +
                          (static_cast<size_t>(a.ml) * a.mm + static_cast<size_t>(a.ml) * a.src[m].nm) * sizeof(double2))
                          ->scale;
  }
  const int64_t K = a.o.K;
  // As many workgroups as the chip runs at once (three per compute unit); with
  // fewer than 768 bins each, workgroups of 512 (two rounds of 64 bins per
  // wave) instead, the last of which follow the first that are done, or of 256
  // while those leave compute units idle (K = 26k to 76k: 48-50 -> 39-43 us
  // for 33 to 129 pixels).  Below that, of 128 bins where 256 leave fewer than
  // 160 workgroups (K = 27k: 43 -> 36 us for 65 pixels; at 52k instead 36 -> 39),
  // and, where baselines have fewer than 100 bins, so that successive ones
  // share few windows, as few as 64 while fewer than 380 workgroups (2016
  // baselines of 16 bins: 131 -> 58 us; of 32 bins, in 128 each, 79 -> 60).
  // One span each below 8192 bins per workgroup (K =
  // 5.9M of uneven bins: 195 us against 229 with three levels; six patches of
  // K = 1.45M 1258 against 1356), from there on as many levels as leave the
  // last at least 1024 bins (K = 23.2M, three sources: 1846 us with six levels,
  // 1918 with five, 2150 with one).
  const int resident = 768 / a.n_src;
  const int wanted = K < 100 * static_cast<int64_t>(a.o.n_bl) ? 380 : 160;
  int least = K * a.n_src < 512 * 256 ? 256 : 512;
  while (least > 64 && least < 512 && K * a.n_src < static_cast<int64_t>(wanted) * least) least /= 2;
  a.n_wg = K / resident < 768 ? static_cast<int>((K + least - 1) / least) : resident;
  a.levels = 1;
  if (K / a.n_wg >= 8 * kLeastSpan)
    while (a.levels < kGridMaxLevels && K / a.n_wg >= int64_t(kLeastSpan) << a.levels) ++a.levels;
  a.n_span = a.levels * a.n_wg;
  const int units = span_units(a, a.n_span);
  a.unit_bins = (K + units - 1) / units;
  static_assert(kGridMaxLevels * 768 <= kGridMaxSpans, "a peak and a first bin for every span");
  const unsigned n_src = static_cast<unsigned>(a.n_src);
  const int64_t words = std::max(static_cast<int64_t>(a.ml) * a.mm, K / (a.fused ? 4 : 2));
  a.n_init = static_cast<int>(std::min<int64_t>(kInitBlocks, (words + 255) / 256));
  hipLaunchKernelGGL(k_grid_init, dim3(static_cast<unsigned>(a.n_init + (a.fused ? kCutBlocks : 0)), n_src), dim3(256), 0, stream, a);
  const dim3 sg(static_cast<unsigned>(a.n_wg), n_src);
  switch (prec) {
    case kFP32: launch_spread<kFP32>(a, sg, stream); break;
    case kSplitBF16: launch_spread<kSplitBF16>(a, sg, stream); break;
    case kSplitFP16: launch_spread<kSplitFP16>(a, sg, stream); break;
    case kMixedFP16: launch_spread<kMixedFP16>(a, sg, stream); break;
    case kSRFP16: launch_spread<kSRFP16>(a, sg, stream); break;
    default: return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(k_grid_rows, dim3(static_cast<unsigned>(a.ml), n_src), dim3(256),
                     static_cast<size_t>(a.mm) * 3 / 2 * sizeof(double2), stream, a);
  hipLaunchKernelGGL(k_grid_cols, dim3(static_cast<unsigned>(nm), n_src), dim3(256),
                     static_cast<size_t>(a.ml) * 3 / 2 * sizeof(double2), stream, a);
  return hipGetLastError();
}

}  // namespace psf
