// The shared PSF table (see TableArgs): every star's image interpolated from one polychromatic image,
// and the transpose for the gradient. The products are banded: a block of 16 x 16 focal samples reads a
// K x K window of the table through two [16][K] weight matrices, the same for every block of the star, so
// both directions run as chained FP64 matrix instructions (v_mfma_f64_16x16x4_f64, whose output register
// r of lane group g holds row 4 r + g: an output is the next product's operand as it lies in registers).
//
// The interpolation is FP64 because it is linear in the intensity: a faint sample next to a star's core
// is a sum of terms as large as the core times the weights, and FP32 products would leave 1e-8 of the
// core there, where the FP32 fields squared leave 1e-8 sqrt(core x sample).
#include <algorithm>
#include <cmath>

#include "dlx_internal.h"
#include "wave.h"

namespace dlx {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int iclamp(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// The wave's number in its workgroup, as a scalar (what follows from it stays off the vector units).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// Workgroups go round-robin to the 8 XCDs; renumbered so that a contiguous range runs on one XCD.
__device__ __forceinline__ int xcd_order(int w, int n) {
  const int q = n >> 3, r = n & 7, xcd = w & 7, k = w >> 3;
  return (xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q) + k;
}

__device__ __forceinline__ int floor_div(int a, int b) { return (a >= 0 ? a : a - b + 1) / b; }

// The window of the interpolation kernel at distance t (table samples), zero from W / 2 on.
__device__ __forceinline__ double window(double t, int W, double beta) {
  const double z = 2.0 * t / (double)W;
  const double s = 1.0 - z * z;
  return s > 0.0 ? exp(beta * (sqrt(s) - 1.0)) : (s <= 0.0 ? 0.0 : s);   // NaN stays NaN
}

__device__ __forceinline__ double kernel_weight(double t, int W, double beta) {
  const double w = window(t, W, beta);
  if (t == 0.0) return w;
  return w * sinpi(t) / (3.14159265358979323846 * t);
}

// First table sample of block 0 for a star at offset `pos`, and focal sample 0's distance from it. A
// position that is not finite gets the axis' window and NaN weights.
__device__ __forceinline__ double star_origin(const TableArgs& t, double pos, int& base) {
  const double x = t.c0 - pos / t.tau;
  const double b = ceil(x - 0.5 * (double)t.W);
  const bool ok = fabs(b) < 1e9;
  base = ok ? (int)b : (int)ceil(t.c0 - 0.5 * (double)t.W);
  return ok ? x - b : x - x;
}

// A tilt beyond half a cycle per pupil sample at some wavelength, reduced by that wavelength's period
// lambda / dx (the field of the sampled pupil repeats with it).
__device__ __forceinline__ double reduced(const TableArgs& t, double pos, int l) {
  const double per = t.wl[l].lam / t.dx;
  return pos - rint(pos / per) * per;
}

// wt[fs][axis][a][kPadL + q] = phi(distance of focal sample 16 b + a from table sample h16 b + base + q),
// any b, 0 <= q < K, with zeros around them, so that a shifted window reads zeros where it leaves the K
// samples.
// Block 0 sets range[0], the first table row in use: the largest offset of a star, half the focal grid,
// and W samples on either side (half for the interpolation, half for the derivative's stencil); and where that
// is far out, or a star's tilts are reduced, marks the blocks in use.

// The blocks of 32 x 32 samples that the stars' windows reach, and around them those whose samples go into
// the derivatives there: the band of the derivative's products covers 47 samples more than half its taps. Stars
// that need no more than the rows and columns from lo_sparse on share one square; the others have their own.
__device__ __forceinline__ void mark_blocks(const TableArgs& t, const float* sources, int lo, bool far) {
  const int side = t.Nt / 32, first = lo / 32, last = side - 1 - first, planes = far ? 1 + t.L : 1;
  for (long long i = threadIdx.x; i < (long long)planes * side * side / 4; i += 256) reinterpret_cast<int*>(t.need)[i] = 0;
  for (int i = threadIdx.x; i < planes * side; i += 256) t.need_rows[i] = 0;
  const int lane = threadIdx.x & 63, wave = wave_id(), span = t.h16 * (t.nb - 1) + t.K - 1;
  const double half = 0.5 * t.Nt - 0.5 * (double)(t.No - 1) * t.h16 / 16.0 - t.W - 4.0;   // see range[0]
  const double inner = (half - max(t.lo_sparse, 0)) * t.tau;
  auto outlying = [&](int fs) {   // (a position that is not finite has the axis' window)
    return t.far[fs] || fabs((double)sources[fs * 3]) > inner || fabs((double)sources[fs * 3 + 1]) > inner;
  };
  __shared__ double sm[4];
  double m = 0.0;
  for (int fs = threadIdx.x; fs < t.nfs; fs += 256)
    if (!outlying(fs)) m = fmax(m, fmax(fabs((double)sources[fs * 3]), fabs((double)sources[fs * 3 + 1])));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if (lane == 0) sm[wave] = m;
  __syncthreads();
  const int c0 = max((int)(half - fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3])) / t.tau), 0);
  for (int pass = 0; pass < 2; ++pass) {
    const unsigned char v = pass ? kNeed | kReach : kNeed;
    const int pad = pass ? 0 : t.W / 2 + 64;
    __syncthreads();   // the stores of one pass before the next
    const int b0 = max(floor_div(c0 - pad, 32), first), b1 = side - 1 - b0, nb = b1 - b0 + 1;
    for (int e = threadIdx.x; e < nb * nb; e += 256) t.need[(long long)(b0 + e / nb) * side + b0 + e % nb] = v;
    for (int e = threadIdx.x; e < nb; e += 256) t.need_rows[b0 + e] = v;
    for (int fs = wave; fs < t.nfs; fs += 4) {
      if (!outlying(fs)) continue;
      const int wls = t.far[fs] ? t.L : 1;
      for (int l = 0; l < wls; ++l) {
        double x = sources[fs * 3], y = sources[fs * 3 + 1];
        int plane = 0, jx, jy;
        if (t.far[fs]) {
          x = reduced(t, x, l);
          y = reduced(t, y, l);
          plane = 1 + l;
        }
        star_origin(t, x, jx);
        star_origin(t, y, jy);
        const int x0 = max(floor_div(jx - pad, 32), first), x1 = min(floor_div(jx + span + pad, 32), last);
        const int y0 = max(floor_div(jy - pad, 32), first), y1 = min(floor_div(jy + span + pad, 32), last);
        const int nx = x1 - x0 + 1, ny = y1 - y0 + 1;
        if (nx <= 0 || ny <= 0) continue;
        unsigned char* need = t.need + (long long)plane * side * side;
        for (int e = lane; e < nx * ny; e += 64) need[(long long)(y0 + e / nx) * side + x0 + e % nx] = v;
        for (int e = lane; e < ny; e += 64) t.need_rows[plane * side + y0 + e] = v;
      }
    }
  }
}

// whether the block of 32 x 32 samples at block row i and column j carries `mark` for every wavelength
__device__ __forceinline__ bool block_marked(const TableArgs& t, int i, int j, unsigned char mark) {
  return (t.need[(long long)i * (t.Nt / 32) + j] & mark) != 0;
}

__global__ __launch_bounds__(256) void table_weights_kernel(const TableArgs t, const float* sources) {
  if (blockIdx.x == 0) {
    __shared__ double sm[4];
    __shared__ int sf[4], s_lo;
    double m = 0.0;
    int any = 0;
    for (int fs = threadIdx.x; fs < t.nfs; fs += 256) {
      const double a = sources[fs * 3], b = sources[fs * 3 + 1];
      const bool fin = isfinite(a) && isfinite(b);
      const bool far = fin && (fabs(a) > t.half_min || fabs(b) > t.half_min);
      t.far[fs] = far;
      if (far) {
        any = 1;
        for (int l = 0; l < t.L; ++l) m = fmax(m, fmax(fabs(reduced(t, a, l)), fabs(reduced(t, b, l))));
      } else if (fin) {
        m = fmax(m, fmax(fabs(a), fabs(b)));
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      m = fmax(m, __shfl_xor(m, o, 64));
      any |= __shfl_xor(any, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
      sm[threadIdx.x >> 6] = m;
      sf[threadIdx.x >> 6] = any;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      m = fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]));
      const double half = 0.5 * (double)(t.No - 1) * t.h16 / 16.0 + m / t.tau + t.W + 4.0;
      const double lo = floor((0.5 * t.Nt - half) / 32.0) * 32.0;
      s_lo = lo > 0.0 ? (int)lo : 0;
      sf[0] |= sf[1] | sf[2] | sf[3];
      t.range[0] = s_lo;
      t.range[1] = sf[0];
      t.range[2] = sf[0] || s_lo < t.lo_sparse;
    }
    __syncthreads();
    if (sf[0] || s_lo < t.lo_sparse) mark_blocks(t, sources, s_lo, sf[0] != 0);
    for (int i = threadIdx.x; i < t.n_chunks; i += 256) t.dark_n[i] = 0;
    return;
  }
  const int i = blockIdx.x - 1, fs = i >> 1, axis = i & 1;
  int base;
  const double f = star_origin(t, sources[fs * 3 + axis], base);
  if (threadIdx.x == 0) t.base[i] = base;
  const int KS = wrow(t.K);
  double* w = t.wt + (long long)i * 16 * KS;
  for (int e = threadIdx.x; e < 16 * KS; e += 256) {
    const int a = e / KS, q = e - a * KS - kPadL;
    w[e] = q >= 0 && q < t.K ? kernel_weight(f + (double)(a * t.h16) / 16.0 - (double)q, t.W, t.beta) : 0.0;
  }
}

// w_l |E_l|^2 of one table sample, FP64
__device__ __forceinline__ double power(float er, float ei) {
  return fma((double)er, (double)er, (double)ei * (double)ei);
}

// I = sum_l w_l |E_l|^2 on the rows and columns in use, four columns per thread. HBM- or L2-bound: every
// field of the table is read once.
__global__ __launch_bounds__(256) void table_image_kernel(const TableArgs t) {
  const int lo = t.range[0], n = t.Nt - 2 * lo, nq = n / 4;
  const bool sparse = t.range[2] != 0;
  const long long total = (long long)n * nq;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const int r = (int)(i / nq), c = (int)(i - (long long)r * nq);
    if (sparse && !block_marked(t, (lo + r) >> 5, (lo + 4 * c) >> 5, kNeed)) continue;
    const long long o = (long long)(lo + r) * t.Nt + lo + 4 * c;
    const float* e = t.E + o;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int l = 0; l < t.L; ++l) {
      const f4 er = *reinterpret_cast<const f4*>(e + l * t.e_by_wl);
      const f4 ei = *reinterpret_cast<const f4*>(e + l * t.e_by_wl + t.e_plane);
      const double w = (double)t.wl[l].w;
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] = fma(w, power(er[k], ei[k]), acc[k]);
    }
    *reinterpret_cast<d2*>(t.I + o) = d2{acc[0], acc[1]};
    *reinterpret_cast<d2*>(t.I + o + 2) = d2{acc[2], acc[3]};
  }
}

// Derivatives of the table image at its own samples, Ix[j] = sum_n phi'(n) I[j - n] and likewise along y
// (phi'(n) = (-1)^n / n times the window: the interpolation kernel's derivative at whole distances).
// Samples outside the range in use count as the edge's: only nodes no star's samples touch see them.
constexpr int kMid = 96;   // a band's place, 16 and up to 31 more columns around half the taps
static_assert(kTableMaxW / 2 + 47 < kMid, "");

// s[d + kMid]: weight of the sample d to the right of (or below) the result
__device__ __forceinline__ void band_weights(double* s, const TableArgs& t) {
  if (threadIdx.x < 2 * kMid) {
    const int d = (int)threadIdx.x - kMid, n = d < 0 ? -d : d;
    const double v = n == 0 || n > t.W / 2 ? 0.0 : ((n & 1) ? -1.0 : 1.0) / (double)n * window((double)n, t.W, t.beta);
    s[threadIdx.x] = d < 0 ? v : -v;
  }
}

// The 16 x 16 derivatives at (R, C) of the samples at(row, column), by one wave.
template <class F>
__device__ __forceinline__ void slopes16(const double* s, int H, int R, int C, int lo, int hi, F at, d4& dx, d4& dy) {
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  dx = dy = d4{0.0, 0.0, 0.0, 0.0};
  for (int p0 = 0; 4 * p0 < 16 + 2 * H; p0 += 4) {   // (the weights are zero past the band)
    double v[4], u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = 4 * (p0 + i) + g - H;
      v[i] = at(R + n, iclamp(C + o, lo, hi));
      u[i] = at(iclamp(R + o, lo, hi), C + n);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double w = s[4 * (p0 + i) + g - H - n + kMid];
      dx = mfma_f64(v[i], w, dx);
      dy = mfma_f64(w, u[i], dy);
    }
  }
}

// As products with the banded matrix of the stencil (FP64 matrix instructions, 16 x 16 samples per wave and
// direction): the 2 W loads and products per sample of the plain sum took 174 us for 2112^2 samples and 64
// taps, about 55 us here (18 us of matrix instructions).
__global__ __launch_bounds__(256) void table_slope_kernel(const TableArgs t) {
  __shared__ double s[2 * kMid];
  const int H = t.W / 2;
  band_weights(s, t);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = wave_id(), n = lane & 15, g = lane >> 4;
  const int lo = t.range[0], hi = t.Nt - lo - 1, side = (t.Nt - 2 * lo) / 32;
  const bool sparse = t.range[2] != 0;
  const long long ld = t.Nt;
  for (int tile = blockIdx.x; tile < side * side; tile += gridDim.x) {
    if (sparse && !block_marked(t, lo / 32 + tile / side, lo / 32 + tile % side, kReach)) continue;
    const int R = lo + 32 * (tile / side) + 16 * (wave >> 1), C = lo + 32 * (tile % side) + 16 * (wave & 1);
    d4 dx = d4{0.0, 0.0, 0.0, 0.0}, dy = d4{0.0, 0.0, 0.0, 0.0};
    // along x: rows of I times the band; a lane's two samples 8 p + 2 g and the next are one product's term each
    const double* row = t.I + (R + n) * ld;
    const bool inside = C - H >= lo && C + H + 47 <= hi;
    for (int p0 = 0; 8 * p0 < 16 + 2 * H; p0 += 4) {   // (four loads in flight; the weights are zero past the band)
      d2 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = C - H + 8 * (p0 + i) + 2 * g;
        if (inside)
          __builtin_memcpy(&v[i], row + c, sizeof v[i]);
        else
          v[i] = d2{row[iclamp(c, lo, hi)], row[iclamp(c + 1, lo, hi)]};
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = 8 * (p0 + i) + 2 * g - H - n + kMid;
        dx = mfma_f64(v[i][0], s[k], dx);
        dx = mfma_f64(v[i][1], s[k + 1], dx);
      }
    }
    for (int p0 = 0; 4 * p0 < 16 + 2 * H; p0 += 8) {   // along y: the band times columns of I
      double v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = t.I[iclamp(R - H + 4 * (p0 + i) + g, lo, hi) * ld + C + n];
#pragma unroll
      for (int i = 0; i < 8; ++i) dy = mfma_f64(s[4 * (p0 + i) + g - H - n + kMid], v[i], dy);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      t.Ix[(R + 4 * r + g) * ld + C + n] = (float)dx[r];
      t.Iy[(R + 4 * r + g) * ld + C + n] = (float)dy[r];
    }
  }
}

// A star's weights into LDS: x, then y.
__device__ __forceinline__ void load_weights(const TableArgs& t, int fs, double* w) {
  const int n2 = 16 * wrow(t.K);   // pairs of both axes
  const d2* src = reinterpret_cast<const d2*>(t.wt + (long long)fs * 2 * n2);
  for (int e = threadIdx.x; e < n2; e += 256) reinterpret_cast<d2*>(w)[e] = src[e];
}

// A block of interpolated samples is dark, and interpolated from the fields instead, when one of them lies below
// a bound set by the largest sample of its window, `most`: kDarkPeak of it, as at most 3e-10 of a core reaches the
// samples around it (512^2 pupils, 1 to 32 wavelengths); in the wings, whose rounding errors, 2.5e-10 sqrt(most x
// peak) as interpolated and 1.5e-9 sqrt(sample x peak) from a transform per star, are larger for their light,
// kDarkNull sqrt(most x peak), and nowhere more than kDarkWing of it. Hard-edged pupils' broadband images have no
// such block, or a few in a hundred; those of soft pupils and of a few close wavelengths have many.
constexpr float kDarkPeak = 4e-6f, kDarkNull = 2.5e-7f, kDarkWing = 5e-4f;

// high 32 bits of a sample: in the order of the samples where they are not negative
__device__ __forceinline__ int high_word(double v) { return (int)(__builtin_bit_cast(unsigned long long, v) >> 32); }

__device__ __forceinline__ void add_dark(const TableArgs& t, int chunk, int star, int yb, int xb) {
  if ((threadIdx.x & 63) == 0) t.dark[atomicAdd(t.dark_n + chunk, 1)] = (star * t.nb + yb) * t.nb + xb;
}

// The weights of one wavelength of a star whose tilt is reduced by its period, by one wave into its own LDS.
__device__ __forceinline__ void far_weights(const TableArgs& t, const float* src, int l, double* wx, double* wy,
                                            int& jx, int& jy) {
  const int KS = wrow(t.K);
  const double fx = star_origin(t, reduced(t, src[0], l), jx), fy = star_origin(t, reduced(t, src[1], l), jy);
  for (int e = threadIdx.x & 63; e < 16 * KS; e += 64) {
    const int a = e / KS, q = e - a * KS - kPadL;
    const bool in = q >= 0 && q < t.K;
    const double s = (double)(a * t.h16) / 16.0 - (double)q;
    wx[e] = in ? kernel_weight(fx + s, t.W, t.beta) : 0.0;
    wy[e] = in ? kernel_weight(fy + s, t.W, t.beta) : 0.0;
  }
}

// Star images on the focal grid, plane[f][s][k] = I(u_k - position), FP64 products of the table rounded
// to FP32 at the end. A wave forms 16 columns x 16 NY rows: for each 16 table rows its window touches, the
// product with the column weights (K / 4 instructions), whose output feeds the products with the row
// weights of the NY blocks below each other. Bound by the FP64 matrix rate; the next rows' samples are
// loaded while the current ones' products run, and the workgroups of one part of the focal grid, whatever
// their star, follow each other on one XCD, whose L2 then holds that part of the table. The weights of a
// product with four row groups are read together, and far stars are left to another kernel, so that three
// waves fit a SIMD. 128 stars of 768^2 samples, 28 taps: 270 us, of which the search for dark samples takes 20
// (373 us without it, but with a read and a wait before each product and two waves; 150 us of matrix instructions).
// KP = K / 8.
template <int KP, int NY>
__global__ __launch_bounds__(256, 2) void table_shift_kernel(const TableArgs t, int fs0, int nstar, int nbx, int chunk) {
  constexpr int K = 8 * KP, KS = wrow(K);
  __shared__ __attribute__((aligned(16))) double sh[2 * 16 * KS];
  double *wx = sh, *wy = sh + 16 * KS;
  const int lane = threadIdx.x & 63, wave = wave_id(), n = lane & 15, g = lane >> 4;
  const int lin = xcd_order(blockIdx.x, gridDim.x);
  const int tile = lin / nstar, star = lin - tile * nstar, fs = fs0 + star;
  const int lo = t.range[0], hi = t.Nt - lo - 1;
  const int xb = (tile % nbx) * 4 + wave, yb0 = (tile / nbx) * NY;
  const int ny = t.nb - yb0 < NY ? t.nb - yb0 : NY;
  d4 acc[NY];
#pragma unroll
  for (int y = 0; y < NY; ++y) acc[y] = d4{0.0, 0.0, 0.0, 0.0};
  int top[NY];   // this lane's largest sample in each block's window (high word)
#pragma unroll
  for (int y = 0; y < NY; ++y) top[y] = 0;
  // block y's product with the 16 table rows that start `rel` rows into its window
  auto add_rows = [&](int y, int rel, const d4& d, int m) {
    if (y >= ny || rel <= -16 || rel >= K) return;
    top[y] = max(top[y], m);
    double wr[4];   // read together: a read before each product would be waited for each time
#pragma unroll
    for (int r = 0; r < 4; ++r) wr[r] = wy[n * KS + kPadL + rel + 4 * r + g];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (rel + 4 * r > -4 && rel + 4 * r < K)   // the block's window reaches these four rows
        acc[y] = mfma_f64(wr[r], d[r], acc[y]);
  };

  if (!t.far[fs]) {
    load_weights(t, fs, wx);
    __syncthreads();
    if (xb < t.nb) {
      const int cx = t.base[2 * fs] + t.h16 * xb + 2 * g, ry = t.base[2 * fs + 1] + t.h16 * yb0 + n;
      const int rbs = (t.h16 * (ny - 1) + K + 15) / 16;
      d2 w[KP], v[KP], nx[KP];
#pragma unroll
      for (int p = 0; p < KP; ++p) w[p] = *reinterpret_cast<const d2*>(&wx[n * KS + kPadL + 8 * p + 2 * g]);
      // the window leaves the samples in use only where a block has columns past the focal grid
      const bool inside = cx - 2 * g >= lo && cx - 2 * g + K - 1 <= hi;
      auto load = [&](int rb, d2* o) {
        const double* row = t.I + (long long)iclamp(ry + 16 * rb, lo, hi) * t.Nt;
#pragma unroll
        for (int p = 0; p < KP; ++p)
          __builtin_memcpy(&o[p], row + (inside ? cx + 8 * p : iclamp(cx + 8 * p, lo, hi - 1)), sizeof(d2));
      };
      load(0, v);
      for (int rb = 0; rb < rbs; ++rb) {
        if (rb + 1 < rbs) load(rb + 1, nx);
        d4 d = d4{0.0, 0.0, 0.0, 0.0};
        int m = 0;
#pragma unroll
        for (int p = 0; p < KP; ++p) {
          d = mfma_f64(v[p][0], w[p][0], d);
          d = mfma_f64(v[p][1], w[p][1], d);
          m = max(m, max(high_word(v[p][0]), high_word(v[p][1])));
        }
#pragma unroll
        for (int y = 0; y < NY; ++y) add_rows(y, 16 * rb - t.h16 * y, d, m);
#pragma unroll
        for (int p = 0; p < KP; ++p) v[p] = nx[p];
      }
    }
  } else {   // every wavelength has its own window
    for (int y = 0; y < ny && xb < t.nb; ++y) add_dark(t, chunk, star, yb0 + y, xb);
    return;
  }
  if (xb >= t.nb) return;
  float* o = t.planes + (long long)star * t.No * t.ldg;
  const int x = 16 * xb + n;
  if (x < t.No) {
#pragma unroll
    for (int y = 0; y < NY; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int yy = 16 * (yb0 + y) + 4 * r + g;
        if (y < ny && yy < t.No) o[(long long)yy * t.ldg + x] = (float)acc[y][r];
      }
  }
  // any block dark by the largest sample of all their windows? Only then block by block, by its own
  auto least = [&](int high) {
    const float most = (float)__builtin_bit_cast(double, (unsigned long long)wave_max(high) << 32);
    return (double)fmaxf(kDarkPeak * most, fminf(kDarkNull * __fsqrt_rn(most) * (float)t.root_peak, kDarkWing * most));
  };
  auto below = [&](int y, double bound) {
    bool any = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) any |= acc[y][r] < bound && 16 * (yb0 + y) + 4 * r + g < t.No;
    return any && x < t.No;
  };
  int most = top[0];
#pragma unroll
  for (int y = 1; y < NY; ++y) most = max(most, top[y]);
  const double bound = least(most);
  bool some = false;
#pragma unroll
  for (int y = 0; y < NY; ++y) some |= below(y, bound);
  if (!__any(some)) return;
#pragma unroll
  for (int y = 0; y < NY; ++y) {
    const bool dark = below(y, least(top[y]));
    if (y < ny && __any(dark)) add_dark(t, chunk, star, yb0 + y, xb);
  }
}

// The dark blocks' samples, and all of far stars: sum_l w_l |sum_j phi_j E_l[j]|^2, the fields interpolated with
// the same weights (they have half the image's bandwidth), a far star's with those of its tilt at each wavelength.
// A workgroup per block, its waves share out the wavelengths. Two chains of products per wavelength where
// the image has one for all: bound by the latency of the loads for a few blocks, by the FP64 matrix rate for many
// (80 stars of 256^2 samples, 32 wavelengths, a Gaussian pupil: 3.1 ms; 4.5 us where no block is dark).
template <int KP>
__global__ __launch_bounds__(256, 2) void table_field_kernel(const TableArgs t, const float* sources, int fs0, int chunk) {
  constexpr int K = 8 * KP, KS = wrow(K);
  __shared__ __attribute__((aligned(16))) double wy[16 * KS];
  __shared__ double part[4][4][64];
  const int lane = threadIdx.x & 63, wave = wave_id(), n = lane & 15, g = lane >> 4;
  const int lo = t.range[0], hi = t.Nt - lo - 1, count = t.dark_n[chunk];
  for (int i = blockIdx.x; i < count; i += gridDim.x) {
    const int item = t.dark[i], xb = item % t.nb, yb = item / t.nb % t.nb, star = item / (t.nb * t.nb), fs = fs0 + star;
    const bool far = t.far[fs];
    d2 wx[KP];   // column weights of this lane's samples 8 p + 2 g and the next
    double fy = 0.0;
    if (!far) {
      const double* src = t.wt + (long long)fs * 2 * 16 * KS;
      for (int e = threadIdx.x; e < 8 * KS; e += 256)
        reinterpret_cast<d2*>(wy)[e] = reinterpret_cast<const d2*>(src + 16 * KS)[e];
#pragma unroll
      for (int p = 0; p < KP; ++p) wx[p] = *reinterpret_cast<const d2*>(src + n * KS + kPadL + 8 * p + 2 * g);
    }
    __syncthreads();
    d4 tot = d4{0.0, 0.0, 0.0, 0.0};
    for (int l = wave; l < t.L; l += 4) {
      int jx = t.base[2 * fs], jy = t.base[2 * fs + 1];
      if (far) {   // each weight is needed by one lane, so none goes through LDS
        const double fx = star_origin(t, reduced(t, sources[fs * 3], l), jx) + (double)(n * t.h16) / 16.0;
        fy = star_origin(t, reduced(t, sources[fs * 3 + 1], l), jy) + (double)(n * t.h16) / 16.0;
#pragma unroll
        for (int p = 0; p < KP; ++p)
#pragma unroll
          for (int k = 0; k < 2; ++k) wx[p][k] = kernel_weight(fx - (double)(8 * p + 2 * g + k), t.W, t.beta);
      }
      const float* e = t.E + l * t.e_by_wl;
      const int cx = jx + t.h16 * xb + 2 * g, ry = jy + t.h16 * yb + n;
      d4 fr = d4{0.0, 0.0, 0.0, 0.0}, fi = d4{0.0, 0.0, 0.0, 0.0};
      constexpr bool kAhead = KP <= 6;   // (longer windows leave no registers for the next rows)
      float2 er[KP], ei[KP], nr[kAhead ? KP : 1], ni[kAhead ? KP : 1];
      auto load = [&](int rb, float2* re, float2* im) {
        const float* row = e + (long long)iclamp(ry + 16 * rb, lo, hi) * t.Nt;
#pragma unroll
        for (int p = 0; p < KP; ++p) {
          const int c = iclamp(cx + 8 * p, lo, hi - 1);
          __builtin_memcpy(&re[p], row + c, sizeof re[p]);
          __builtin_memcpy(&im[p], row + c + t.e_plane, sizeof im[p]);
        }
      };
      if constexpr (kAhead) load(0, er, ei);
      for (int rb = 0; 16 * rb < K; ++rb) {
        if constexpr (!kAhead) load(rb, er, ei);
        if constexpr (kAhead)
          if (16 * rb + 16 < K) load(rb + 1, nr, ni);   // while the current rows' products run
        d4 dr = d4{0.0, 0.0, 0.0, 0.0}, di = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int p = 0; p < KP; ++p) {
          dr = mfma_f64((double)er[p].x, wx[p][0], dr);
          di = mfma_f64((double)ei[p].x, wx[p][0], di);
          dr = mfma_f64((double)er[p].y, wx[p][1], dr);
          di = mfma_f64((double)ei[p].y, wx[p][1], di);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * rb + 4 * r < K) {
            const int q = 16 * rb + 4 * r + g;
            const double w = far ? kernel_weight(fy - (double)q, t.W, t.beta) : wy[n * KS + kPadL + q];
            fr = mfma_f64(w, dr[r], fr);
            fi = mfma_f64(w, di[r], fi);
          }
        if constexpr (kAhead) {
#pragma unroll
          for (int p = 0; p < KP; ++p) {
            er[p] = nr[p];
            ei[p] = ni[p];
          }
        }
      }
      const double w = (double)t.wl[l].w;
#pragma unroll
      for (int r = 0; r < 4; ++r) tot[r] = fma(w, fma(fr[r], fr[r], fi[r] * fi[r]), tot[r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][r][lane] = tot[r];
    __syncthreads();   // and the weights are done with
    const int x = 16 * xb + n, y = 16 * yb + 4 * wave + g;   // this wave adds up and writes output register `wave`
    double v = 0.0;
    for (int k = 0; k < 4; ++k) v += part[k][wave][lane];
    if (x < t.No && y < t.No) t.planes[(long long)star * t.No * t.ldg + (long long)y * t.ldg + x] = (float)v;
  }
}

// Binning of the star images (Section 3): per star bs = sum K I over a detector pixel, FP64, and
// binned = sum_s phi_s bs, model = flat binned. One pixel of one frame per thread, with the loads of several
// stars in flight (QT: oversampling, 0 any). Bound by the images it reads: 63 us for 64 frames of 2 stars
// (768^2 samples, 3 x 3 per pixel; 138 us one star and one sample after the other).
template <int QT>
__global__ __launch_bounds__(256) void table_bin_kernel(const TableArgs t, int Qr, int Nd, int f0, const float* sources,
                                                        const float* intrapixel, long long kst, const float* flat,
                                                        float* bs, float* binned, float* model) {
  constexpr int Q2 = QT > 0 ? QT * QT : 1, STARS = QT == 0 ? 1 : QT == 1 ? 8 : QT == 4 ? 1 : 2;
  const int Q = QT > 0 ? QT : Qr;
  const long long npix = (long long)Nd * Nd;
  const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  if (p >= npix) return;
  const int fl = blockIdx.y, f = f0 + fl;
  const int pr = (int)(p / Nd), pc = (int)(p - (long long)pr * Nd);
  const float* kp = intrapixel ? intrapixel + p * kst : nullptr;
  float kw[Q2];
  if constexpr (QT > 0) {
#pragma unroll
    for (int i = 0; i < Q2; ++i) kw[i] = kp ? kp[i] : 1.f;
  }
  const long long star = (long long)t.No * t.ldg;
  const float* e = t.planes + (long long)fl * t.S * star + (long long)(Q * pr) * t.ldg + Q * pc;
  double total = 0.0;
  for (int s0 = 0; s0 < t.S; s0 += STARS) {
    double v[STARS];
    if constexpr (QT > 0) {
      float x[STARS][Q2];
#pragma unroll
      for (int k = 0; k < STARS; ++k) {
        const float* es = e + (long long)min(s0 + k, t.S - 1) * star;   // (past the last star: read again, unused)
#pragma unroll
        for (int i = 0; i < Q2; ++i) x[k][i] = es[(long long)(i / QT) * t.ldg + i % QT];
      }
#pragma unroll
      for (int k = 0; k < STARS; ++k) {
        v[k] = 0.0;
#pragma unroll
        for (int i = 0; i < Q2; ++i)
          v[k] = intrapixel ? fma((double)x[k][i], (double)kw[i], v[k]) : v[k] + (double)x[k][i];
      }
    } else {
      v[0] = 0.0;
      for (int a = 0; a < Q; ++a)
        for (int b = 0; b < Q; ++b) {
          const double x = e[(long long)s0 * star + (long long)a * t.ldg + b];
          v[0] = kp ? fma(x, (double)kp[a * Q + b], v[0]) : v[0] + x;
        }
    }
#pragma unroll
    for (int k = 0; k < STARS; ++k)
      if (s0 + k < t.S) {
        bs[((long long)fl * t.S + s0 + k) * npix + p] = (float)v[k];
        total = fma((double)sources[((long long)f * t.S + s0 + k) * 3 + 2], v[k], total);
      }
  }
  const float bv = (float)total;
  if (binned) binned[(long long)f * npix + p] = bv;
  if (model) model[(long long)f * npix + p] = flat[p] * bv;
}

// The transpose: the seed weights G of frames [f0, f0 + nf) spread onto the table,
//   D_fs[j] = sum_k phi(t_k - j) G_f[k],   H += phi_s D_fs,
// and the position gradient -phi_s / tau sum_j D_fs[j] I'[j] (the derivative field is interpolated with
// the same weights). A workgroup owns 32 table rows x 16 WAVES columns and runs every star of its group in
// two products: its waves share out the blocks of 16 focal columns that reach its columns and contract the
// rows of G with the row weights (V, kept in LDS as it lies in the output registers, which is how the
// second product reads it); then each wave contracts V with the column weights for its 16 columns. Only the
// groups of four focal rows or columns whose taps reach a tile are multiplied. (G holds whole blocks of 16
// rows and columns, zero past the focal grid, so nothing is masked.) The FP64 matrix rate bounds it, with
// two workgroups per CU at about half of it: G comes kAdjRows blocks at a time, one step ahead, and the
// next star's weights during the current star. 128 stars of 768 focal samples onto 832: 480 us (1115 us
// for 32 x 32 samples per wave, each forming its own V from G without a step ahead).
constexpr int kAdjRows = 2;   // blocks of focal rows loaded at a time

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES / 2) void table_adjoint_kernel(const TableArgs t, const float* sources, int f0, int nf,
                                                               int first) {
  extern __shared__ double sh[];
  const int K = t.K, KS = wrow(K), h16 = t.h16, ldg = t.ldg;
  double(*V)[2][4][64] = reinterpret_cast<double(*)[2][4][64]>(sh + 2 * 16 * KS);
  const int lane = threadIdx.x & 63, wave = wave_id(), n = lane & 15, g = lane >> 4;
  // this lane's place in a block of G (row 4 k + g, column n) and in the weights (focal sample 4 k + g,
  // table sample n of a tile that starts at the block's window)
  const unsigned goff = (unsigned)(g * ldg + n);
  const double* wx = sh + g * KS + kPadL + n;
  const double* wy = wx + 16 * KS;
  const int lo = t.range[0], hi = t.Nt - lo - 1;
  constexpr int CW = 16 * WAVES, TH = 64 * WAVES, kPairs = 2048 / TH;
  static_assert(16 * wrow(kTableMaxK) <= kPairs * TH, "the threads stage the weights of any window");
  const int nrt = (t.Nt - 2 * lo) / 32, ncg = (t.Nt - 2 * lo + CW - 1) / CW;
  const int nwg = t.slots / WAVES, lin = xcd_order(blockIdx.x, gridDim.x);
  const int group = lin / nwg, wg = lin - group * nwg;
  const int slot = wg * WAVES + wave;
  const int fs0 = f0 * t.S + group * t.per_group;
  const int fs_end = min((f0 + nf) * t.S, fs0 + t.per_group);
  // this wave's partials of every star start at zero (a far star's are added to by the far pass)
  for (int i = 2 * fs0 + lane; i < 2 * fs_end; i += 64)
    t.pos[((long long)(i >> 1) * t.slots + slot) * 2 + (i & 1)] = 0.0;
  auto next_star = [&](int fs) {
    while (fs < fs_end && t.far[fs]) ++fs;
    return fs;
  };
  // the window's samples that four focal samples 4 k .. 4 k + 3 can reach
  auto first_tap = [&](int k) { return (k * h16) >> 2; };
  auto last_tap = [&](int k) { return (((4 * k + 3) * h16) >> 4) + t.W + 1; };
  const int n2 = 16 * KS;   // weights of both axes, in pairs
  d2 nw[kPairs];
  auto fetch_weights = [&](int fs) {
    const d2* src = reinterpret_cast<const d2*>(t.wt + (long long)fs * 2 * n2);
#pragma unroll
    for (int i = 0; i < kPairs; ++i)
      if ((int)threadIdx.x + TH * i < n2) nw[i] = src[threadIdx.x + TH * i];
  };
  const bool sparse = t.range[2] != 0;
  bool again = false;
  for (int tile = wg; tile < nrt * ncg; tile += nwg) {
    const int R0 = lo + 32 * (tile % nrt), C0 = lo + CW * (tile / nrt);
    const int c = C0 + 16 * wave;   // this wave's columns
    bool live = c <= hi;
    if (sparse) {   // (what no star reaches is neither computed nor read)
      bool any = false;
      for (int k = 0; k < CW; k += 32) any |= C0 + k <= hi && block_marked(t, R0 >> 5, (C0 + k) >> 5, kReach);
      if (!any) continue;
      live = live && block_marked(t, R0 >> 5, c >> 5, kReach);
    }
    const long long t0 = (long long)R0 * t.Nt + (live ? c : lo);   // the tile, and this lane's place in it
    const unsigned o0 = (unsigned)(g * t.Nt + n);
    d4 H[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
    // the blocks of star fs that reach this tile
    int jx, jy, xb0, xb1, yb0, yb1;
    const float* G;
    auto set_star = [&](int fs) {
      jx = t.base[2 * fs];
      jy = t.base[2 * fs + 1];
      G = t.G + (long long)(fs / t.S - f0) * ldg * ldg;
      xb0 = max(0, floor_div(C0 - K - jx, h16) + 1);
      xb1 = min(t.nb - 1, floor_div(min(C0 + CW - 1, hi) - jx, h16));
      yb0 = max(0, floor_div(R0 - K - jy, h16) + 1);
      yb1 = min(t.nb - 1, floor_div(R0 + 31 - jy, h16));
    };
    float nv[4 * kAdjRows];
    auto fetch = [&](int xb, int yc) {   // rows yc .. yc + kAdjRows - 1 (in blocks) of block column xb
      const float* gc = G + 16 * xb;
#pragma unroll
      for (int i = 0; i < kAdjRows; ++i) {
        const float* gr = gc + (long long)(16 * min(yc + i, t.nb - 1)) * ldg;   // uniform
#pragma unroll
        for (int k = 0; k < 4; ++k) nv[4 * i + k] = (gr + (long long)4 * k * ldg)[goff];
      }
    };
    int fs = next_star(fs0);
    if (fs < fs_end) {
      fetch_weights(fs);
      set_star(fs);
      fetch(min(xb0 + wave, t.nb - 1), yb0);
    }
    while (fs < fs_end) {
      const int after = next_star(fs + 1);
      __syncthreads();   // the previous star's weights and V are done with
#pragma unroll
      for (int i = 0; i < kPairs; ++i)
        if ((int)threadIdx.x + TH * i < n2) reinterpret_cast<d2*>(sh)[threadIdx.x + TH * i] = nw[i];
      __syncthreads();
      if (after < fs_end) fetch_weights(after);
      for (int xb = xb0 + wave; xb <= xb1; xb += WAVES) {
        d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
        for (int yc = yb0; yc <= yb1; yc += kAdjRows) {
          float v[4 * kAdjRows];
#pragma unroll
          for (int i = 0; i < 4 * kAdjRows; ++i) v[i] = nv[i];
          const bool last = yc + kAdjRows > yb1;   // one step ahead: more rows, or the wave's next column
          if (!last || xb + WAVES <= xb1) fetch(last ? xb + WAVES : xb, last ? yb0 : yc + kAdjRows);
#pragma unroll
          for (int i = 0; i < kAdjRows; ++i) {
            const int rel = R0 - (jy + h16 * (yc + i));   // the tile's first row in the block's window
            if (yc + i > yb1) continue;
            const int r0 = min(max(rel, -16), K), r1 = min(max(rel + 16, -16), K);   // (unused past either end)
            double w0[4], w1[4];   // read together: a read before each product would be waited for each time
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              w0[k] = wy[4 * k * KS + r0];
              w1[k] = wy[4 * k * KS + r1];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const double a = (double)v[4 * i + k];
              if (first_tap(k) <= rel + 15 && last_tap(k) >= rel) acc[0] = mfma_f64(a, w0[k], acc[0]);
              if (first_tap(k) <= rel + 31 && last_tap(k) >= rel + 16) acc[1] = mfma_f64(a, w1[k], acc[1]);
            }
          }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) V[xb - xb0][i][r][lane] = acc[i][r];
      }
      __syncthreads();
      const double phi = (double)sources[fs * 3 + 2];
      const int cjx = jx, cx0 = xb0, cx1 = xb1;
      if (after < fs_end) {
        set_star(after);
        fetch(min(xb0 + wave, t.nb - 1), yb0);
      }
      d4 D[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
      float gx[8], gy[8];   // read again for every star: kept, they would cost a workgroup per CU
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        gx[k] = (t.Ix + t0 + (long long)(4 * k) * t.Nt)[o0];
        gy[k] = (t.Iy + t0 + (long long)(4 * k) * t.Nt)[o0];
      }
      if (live) {
        const int b1 = min(cx1, floor_div(c + 15 - cjx, h16));
        for (int xb = max(cx0, floor_div(c - K - cjx, h16) + 1); xb <= b1; ++xb) {
          const int rel = c - (cjx + h16 * xb);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (first_tap(r) <= rel + 15 && last_tap(r) >= rel) {
              const double w = wx[4 * r * KS + rel];
              D[0] = mfma_f64(V[xb - cx0][0][r][lane], w, D[0]);
              D[1] = mfma_f64(V[xb - cx0][1][r][lane], w, D[1]);
            }
        }
      }
      double px = 0.0, py = 0.0;
      if (live) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const double d = phi * D[i][r];
            H[i][r] += d;
            px = fma(d, (double)gx[4 * i + r], px);
            py = fma(d, (double)gy[4 * i + r], py);
          }
      }
      px = wave_total(px);
      py = wave_total(py);
      if (lane == 63) {
        double* o = t.pos + ((long long)fs * t.slots + slot) * 2;
        o[0] = (again ? o[0] : 0.0) - px / t.tau;
        o[1] = (again ? o[1] : 0.0) - py / t.tau;
      }
      fs = after;
    }
    again = true;
    if (live) {
      double* h = t.Hpart + group * (long long)t.Nt * t.Nt + t0;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double* q = h + (long long)(16 * i + 4 * r) * t.Nt;
          q[o0] = (first ? 0.0 : q[o0]) + H[i][r];
        }
    }
  }
}

// The same for stars whose tilt is reduced per wavelength, each into that wavelength's own plane of H
// (table_seed_kernel adds the common one). The blocks of 32 x 32 samples that one of these stars reaches at a
// wavelength are shared out over all waves; a wave forms the derivatives of its block from the field, once, and
// the seed weights of every such star there. (One such star among
// 24, 32 wavelengths of 768 focal samples: 3.7 ms; 33 ms one wavelength and one star after the other over the whole table.)
__global__ __launch_bounds__(256) void table_far_kernel(const TableArgs t, const float* sources, int f0, int nf,
                                                        int first) {
  extern __shared__ double sh[];
  __shared__ double s[2 * kMid];
  if (!t.range[1]) return;
  const int KS = wrow(t.K), lane = threadIdx.x & 63, wave = wave_id(), n = lane & 15, g = lane >> 4;
  double *wx = sh + wave * 2 * 16 * KS, *wy = wx + 16 * KS;
  const int lo = t.range[0], hi = t.Nt - lo - 1, side = t.Nt / 32;
  const int slot = blockIdx.x * 4 + wave, waves = gridDim.x * 4;
  band_weights(s, t);
  __syncthreads();
  const long long blocks = (long long)t.L * side * side;
  const unsigned char* need = t.need + (long long)side * side;
  for (long long b0 = slot; b0 < blocks; b0 += 64LL * waves) {   // 64 blocks' marks at a time
    const long long b = b0 + (long long)lane * waves;
    unsigned long long on = __ballot(b < blocks && (need[b < blocks ? b : 0] & kReach) != 0);
    while (on) {
      const int bit = __builtin_ctzll(on);
      on &= on - 1;
      const long long block = b0 + (long long)bit * waves;
      const int l = (int)(block / (side * side)), at = (int)(block - (long long)l * side * side);
      const int R0 = 32 * (at / side), C0 = 32 * (at % side);
      d4 H[2][2], gx[2][2], gy[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          H[i][j] = d4{0.0, 0.0, 0.0, 0.0};
          const float* e = t.E + l * t.e_by_wl;
          const double w = (double)t.wl[l].w;
          slopes16(s, t.W / 2, R0 + 16 * i, C0 + 16 * j, lo, hi, [&](int y, int x) {
            const long long q = (long long)y * t.Nt + x;
            return w * power(e[q], e[q + t.e_plane]);
          }, gx[i][j], gy[i][j]);
        }
      for (int fs = f0 * t.S; fs < (f0 + nf) * t.S; ++fs) {
        if (!t.far[fs]) continue;
        int jx, jy;
        star_origin(t, reduced(t, sources[fs * 3], l), jx);
        star_origin(t, reduced(t, sources[fs * 3 + 1], l), jy);
        const int xb0 = max(0, floor_div(C0 - t.K - jx, t.h16) + 1), xb1 = min(t.nb - 1, floor_div(C0 + 31 - jx, t.h16));
        const int yb0 = max(0, floor_div(R0 - t.K - jy, t.h16) + 1), yb1 = min(t.nb - 1, floor_div(R0 + 31 - jy, t.h16));
        if (xb0 > xb1 || yb0 > yb1) continue;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the previous star's weights are done with
        __builtin_amdgcn_wave_barrier();
        far_weights(t, sources + fs * 3, l, wx, wy, jx, jy);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const float* G = t.G + (long long)(fs / t.S - f0) * t.ldg * t.ldg;
        d4 D[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) D[i][j] = d4{0.0, 0.0, 0.0, 0.0};
        for (int xb = xb0; xb <= xb1; ++xb) {
          const int x = 16 * xb + n;
          const float* gc = G + (x < t.No ? x : t.No - 1);
          d4 V[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
          float nv[4];
          auto fetch = [&](int yb) {
#pragma unroll
            for (int k = 0; k < 4; ++k) nv[k] = gc[(long long)min(16 * yb + 4 * k + g, t.No - 1) * t.ldg];
          };
          fetch(yb0);
          for (int yb = yb0; yb <= yb1; ++yb) {
            double v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = x < t.No && 16 * yb + 4 * k + g < t.No ? (double)nv[k] : 0.0;
            if (yb < yb1) fetch(yb + 1);   // one step ahead
            const int rel = R0 - (jy + t.h16 * yb);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const int ri = rel + 16 * i;
              if (ri > -16 && ri < t.K) {
#pragma unroll
                for (int k = 0; k < 4; ++k) V[i] = mfma_f64(v[k], wy[(4 * k + g) * KS + kPadL + ri + n], V[i]);
              }
            }
          }
          const int rel = C0 - (jx + t.h16 * xb);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int rj = rel + 16 * j;
            if (rj > -16 && rj < t.K) {
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const double w = wx[(4 * r + g) * KS + kPadL + rj + n];
#pragma unroll
                for (int i = 0; i < 2; ++i) D[i][j] = mfma_f64(V[i][r], w, D[i][j]);
              }
            }
          }
        }
        const double phi = (double)sources[fs * 3 + 2];
        double px = 0.0, py = 0.0;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const double d = phi * D[i][j][r];
              H[i][j][r] += d;
              px = fma(d, gx[i][j][r], px);
              py = fma(d, gy[i][j][r], py);
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          px += __shfl_xor(px, o, 64);
          py += __shfl_xor(py, o, 64);
        }
        if (lane < 2) {   // the lanes that zeroed these partials
          double* o = t.pos + ((long long)fs * t.slots + slot) * 2 + lane;
          *o -= (lane ? py : px) / t.tau;
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const long long o = (long long)(R0 + 16 * i + 4 * r + g) * t.Nt + C0 + 16 * j + n;
            float* h = t.H + (1 + l) * (long long)t.Nt * t.Nt;
            h[o] = (float)((first ? 0.0 : (double)h[o]) + H[i][j][r]);
          }
    }
  }
}

// H = sum of the groups' planes, FP32, on the samples in use; with far stars, added to every
// wavelength's own plane
__global__ __launch_bounds__(256) void table_seed_kernel(const TableArgs t) {
  const int lo = t.range[0], n = t.Nt - 2 * lo;
  const long long plane = (long long)t.Nt * t.Nt;
  auto sum = [&](long long o) {
    double v = 0.0;
    for (int k = 0; k < t.groups; ++k) v += t.Hpart[k * plane + o];
    return v;
  };
  if (!t.range[2]) {
    const long long total = (long long)n * n;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
      const long long o = (long long)(lo + i / n) * t.Nt + lo + i % n;
      t.H[o] = (float)sum(o);
    }
    return;
  }
  // only the blocks that a star reaches, at every wavelength (a wavelength's plane starts from its own stars'
  // weights, where it has any) or at some
  const int side = t.Nt / 32, used = n / 32, lane = threadIdx.x & 63;
  for (int b = blockIdx.x; b < used * used; b += gridDim.x) {
    const int bi = lo / 32 + b / used, bj = lo / 32 + b % used;
    const bool here = block_marked(t, bi, bj, kReach);
    for (int l0 = 0; l0 < (t.range[1] ? t.L : 1); l0 += 64) {
      unsigned long long own = 0, all = 1;
      if (t.range[1]) {
        const int l = l0 + lane;
        const unsigned char* m = t.need + ((long long)(1 + (l < t.L ? l : 0)) * side + bi) * side + bj;
        own = __ballot(l < t.L && (*m & kReach) != 0);
        all = here ? __ballot(l < t.L) : own;
      }
      if (!here && !own) continue;
      for (int e = threadIdx.x; e < 1024; e += 256) {
        const long long o = (long long)(32 * bi + e / 32) * t.Nt + 32 * bj + e % 32;
        const double v = here ? sum(o) : 0.0;
        if (here && l0 == 0) t.H[o] = (float)v;
        if (!t.range[1]) continue;
        for (unsigned long long w = all; w; w &= w - 1) {
          const int bit = __builtin_ctzll(w);
          float* h = t.H + (1 + l0 + bit) * plane + o;
          *h = (float)((own >> bit & 1 ? (double)*h : 0.0) + v);
        }
      }
    }
  }
}

// dL/dK from the star images (see kgrad_kernel): v[a][b] = h sum_s phi_s I_s at the pixel's samples.
template <int QT>
__global__ __launch_bounds__(256) void table_kgrad_kernel(const TableArgs t, int Nd, int f0, int nf,
                                                          const float* sources, const float* flat, const float* resid,
                                                          const int* win, int F_img, int Nd_img, double* part,
                                                          double* gpix, int first) {
  constexpr int Q2 = QT * QT;
  __shared__ double sh[Q2][4];
  const long long npix = (long long)Nd * Nd;
  const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  double acc[Q2];
#pragma unroll
  for (int k = 0; k < Q2; ++k) acc[k] = 0.0;
  const int fl0 = gpix ? 0 : blockIdx.y, fl1 = gpix ? nf : blockIdx.y + 1;
  for (int fl = fl0; fl < fl1 && p < npix; ++fl) {
    const int f = f0 + fl;
    const int pr = (int)(p / Nd), pc = (int)(p - (long long)pr * Nd);
    float h = 0.f;
    if (win) {
      const long long nimg = (long long)Nd_img * Nd_img;
      for (int q = 0; q < F_img; ++q) {
        const int ir = pr - win[2 * q], ic = pc - win[2 * q + 1];
        if (ir >= 0 && ir < Nd_img && ic >= 0 && ic < Nd_img) {
          const long long i = (long long)ir * Nd_img + ic;
          h += flat[i] * resid[(long long)q * nimg + i];
        }
      }
    } else {
      h = flat[p] * resid[(long long)f * npix + p];
    }
    for (int s = 0; s < t.S; ++s) {
      const float* e = t.planes + ((long long)fl * t.S + s) * t.No * t.ldg + (long long)(QT * pr) * t.ldg + QT * pc;
      const double w = (double)sources[((long long)f * t.S + s) * 3 + 2] * (double)h;
#pragma unroll
      for (int a = 0; a < QT; ++a)
#pragma unroll
        for (int b = 0; b < QT; ++b) acc[a * QT + b] = fma(w, (double)e[(long long)a * t.ldg + b], acc[a * QT + b]);
    }
  }
  if (gpix) {
    if (p < npix) {
#pragma unroll
      for (int k = 0; k < Q2; ++k) gpix[p * Q2 + k] = (first ? 0.0 : gpix[p * Q2 + k]) + acc[k];
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < Q2; ++k) {
    double v = acc[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < Q2) {
    double v = 0.0;
    for (int w = 0; w < 4; ++w) v += sh[threadIdx.x][w];
    part[((long long)(f0 + blockIdx.y) * gridDim.x + blockIdx.x) * Q2 + threadIdx.x] = v;
  }
}

unsigned blocks(long long n, int per, unsigned most) {
  return (unsigned)std::max<long long>(1, std::min<long long>((n + per - 1) / per, most));
}

}  // namespace

hipError_t launch_table_weights(const TableArgs& t, const float* sources, hipStream_t st) {
  hipLaunchKernelGGL(table_weights_kernel, dim3(1 + 2 * t.nfs), dim3(256), 0, st, t, sources);
  return hipGetLastError();
}

// The polychromatic table image and, for the gradient, its derivatives. n_reg: samples per side the grids
// are sized for (the kernels stride over any more).
hipError_t launch_table_image(const TableArgs& t, int n_reg, bool derivatives, hipStream_t st) {
  const long long n = (long long)n_reg * n_reg;
  if (!derivatives)
    hipLaunchKernelGGL(table_image_kernel, dim3(blocks(n / 4, 256, 1u << 20)), dim3(256), 0, st, t);
  else
    hipLaunchKernelGGL(table_slope_kernel, dim3(blocks(n / 4, 256, 1u << 20)), dim3(256), 0, st, t);
  return hipGetLastError();
}

// Star images of frames [f0, f0 + nf), the chunk's; then its dark blocks (a kernel that leaves at once where
// there are none).
hipError_t launch_table_shift(const TableArgs& t, const float* sources, int f0, int nf, int chunk, hipStream_t st) {
  const int nbx = (t.nb + 3) / 4, nstar = nf * t.S;
  // eight blocks of rows per wave (the fewest instructions) where that still gives a CU four workgroups, four
  // where it gives one (12 stars of 384^2 samples: 20 us, 33 us with one block)
  const long long wg8 = (long long)nbx * ((t.nb + 7) / 8) * nstar, wg4 = (long long)nbx * ((t.nb + 3) / 4) * nstar;
  const int ny = wg8 >= 1024 ? 8 : wg4 >= 256 ? 4 : 1;
  const dim3 grid((unsigned)(nbx * ((t.nb + ny - 1) / ny) * nstar)), blk(256);
  const dim3 fgrid((unsigned)std::min<long long>((long long)t.nb * t.nb * nstar, 512));   // as many as the chip holds
#define DLX_SHIFT(KP)                                                                                              \
  case KP:                                                                                                         \
    if (ny == 8)                                                                                                   \
      hipLaunchKernelGGL((table_shift_kernel<KP, 8>), grid, blk, 0, st, t, f0 * t.S, nstar, nbx, chunk);          \
    else if (ny == 4)                                                                                              \
      hipLaunchKernelGGL((table_shift_kernel<KP, 4>), grid, blk, 0, st, t, f0 * t.S, nstar, nbx, chunk);          \
    else                                                                                                           \
      hipLaunchKernelGGL((table_shift_kernel<KP, 1>), grid, blk, 0, st, t, f0 * t.S, nstar, nbx, chunk);          \
    hipLaunchKernelGGL(table_field_kernel<KP>, fgrid, blk, 0, st, t, sources, f0 * t.S, chunk);                   \
    break
  switch (t.K / 8) {
    DLX_SHIFT(2);
    DLX_SHIFT(3);
    DLX_SHIFT(4);
    DLX_SHIFT(5);
    DLX_SHIFT(6);
    DLX_SHIFT(7);
    DLX_SHIFT(8);
    DLX_SHIFT(9);
    DLX_SHIFT(10);
    default: return hipErrorInvalidValue;
  }
#undef DLX_SHIFT
  static_assert(kTableMinK == 8 * 2 && kTableMaxK == 8 * 10, "every window that can be chosen is compiled");
  return hipGetLastError();
}

hipError_t launch_table_bin(const TableArgs& t, int Q, int Nd, int f0, int nf, const float* sources,
                            const float* intrapixel, long long kst, const float* flat, float* bs, float* binned,
                            float* model, hipStream_t st) {
  const dim3 grid(blocks((long long)Nd * Nd, 256, 1u << 30), nf), blk(256);
#define DLX_TABLE_BIN(QT)                                                                                          \
  hipLaunchKernelGGL(table_bin_kernel<QT>, grid, blk, 0, st, t, Q, Nd, f0, sources, intrapixel, kst, flat, bs, binned, \
                     model)
  switch (Q) {
    case 1: DLX_TABLE_BIN(1); break;
    case 2: DLX_TABLE_BIN(2); break;
    case 3: DLX_TABLE_BIN(3); break;
    case 4: DLX_TABLE_BIN(4); break;
    default: DLX_TABLE_BIN(0); break;
  }
#undef DLX_TABLE_BIN
  return hipGetLastError();
}

// Seed weights of frames [f0, f0 + nf) onto the groups' planes (`first`: overwriting them), and those of
// far stars onto the wavelengths' planes (which leaves at once when there are none).
hipError_t launch_table_adjoint(const TableArgs& t, const float* sources, int f0, int nf, bool first,
                                hipStream_t st) {
  const size_t lds = adjoint_lds(t.waves, t.h16, t.K), far_lds = 4 * 2 * 16 * wrow(t.K) * sizeof(double);
#define DLX_ADJOINT(WAVES)                                                                                           \
  case WAVES:                                                                                                        \
    hipLaunchKernelGGL(table_adjoint_kernel<WAVES>, dim3(t.slots / WAVES * t.groups), dim3(64 * WAVES), lds, st, t, \
                       sources, f0, nf, first ? 1 : 0);                                                              \
    break
  switch (t.waves) {
    DLX_ADJOINT(4);
    DLX_ADJOINT(8);
    default: return hipErrorInvalidValue;
  }
#undef DLX_ADJOINT
  hipLaunchKernelGGL(table_far_kernel, dim3(t.slots / 4), dim3(256), far_lds, st, t, sources, f0, nf, first ? 1 : 0);
  return hipGetLastError();
}

size_t table_weight_count(int K) { return 2 * 16 * (size_t)wrow(K); }

// The table's seed weights, once every frame is in the groups' planes.
hipError_t launch_table_seed(const TableArgs& t, int n_reg, hipStream_t st) {
  hipLaunchKernelGGL(table_seed_kernel, dim3(blocks((long long)n_reg * n_reg, 256, 1u << 20)), dim3(256), 0, st, t);
  return hipGetLastError();
}

hipError_t launch_table_kgrad(const TableArgs& t, int Q, int Nd, int f0, int nf, const float* sources,
                              const float* flat, const float* resid, const int* win, int F_img, int Nd_img,
                              double* part, double* gpix, bool first, hipStream_t st) {
  const dim3 grid(blocks((long long)Nd * Nd, 256, 1u << 30), gpix ? 1 : nf), blk(256);
#define DLX_TKGRAD(QT)                                                                                             \
  hipLaunchKernelGGL(table_kgrad_kernel<QT>, grid, blk, 0, st, t, Nd, f0, nf, sources, flat, resid, win, F_img, \
                     Nd_img, part, gpix, first ? 1 : 0)
  switch (Q) {
    case 1: DLX_TKGRAD(1); break;
    case 2: DLX_TKGRAD(2); break;
    case 3: DLX_TKGRAD(3); break;
    case 4: DLX_TKGRAD(4); break;
    default: return hipErrorInvalidValue;
  }
#undef DLX_TKGRAD
  return hipGetLastError();
}

}  // namespace dlx
