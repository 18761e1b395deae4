#include "table_choice.h"

#include <algorithm>
#include <cmath>

namespace dlx {
namespace {

int ceil_div(int a, int b) { return (a + b - 1) / b; }
int round_up(int a, int b) { return ceil_div(a, b) * b; }

constexpr int kAdjointWgs = 2048;

// Frames per chunk, star groups and device memory of a table whose sizes are set.
void size_arrays(const TableProblem& p, TableShape* s) {
  const size_t ldNo = round_up(p.No, 16), ldNi = round_up(p.Ni, 16), No = p.No, S = p.S, L = p.L, Nt = s->Nt;
  const size_t nd2 = (size_t)p.Nd * p.Nd, nt2 = Nt * Nt, nfs = (size_t)p.F * S;
  const size_t frame = sizeof(float) * (S * No * ldNo + No * ldNo + S * nd2);
  // one grid layer per star of a chunk: at most 65535
  s->chunk = (int)std::max<size_t>(1, std::min<size_t>({(size_t)p.F, kDefaultChunkBudget / frame, 65535 / S}));
  // Star groups of the adjoint, each of two stars or more (a workgroup's start and the sum of the groups'
  // planes cost about half a star): as few as give its workgroups about eight rounds of the chip, and a
  // multiple of the eight XCDs where one is near, as the workgroups of a group share the seed weights of its
  // stars, which one XCD's L2 holds. (128 stars: 16 groups 498 us, 8 groups 584; 24 stars: 8 groups 166 us,
  // 24 groups 183; 20 stars: 10 groups 199 us, 20 groups 208.)
  const int nwg = s->slots / s->waves, stars = s->chunk * p.S;
  const int few = std::min(stars, std::max(2, stars / ceil_div(kAdjointWgs, nwg)));
  s->per_group = few;
  double off = 2.0;
  for (int per = std::min(2, stars); per < 2 * few; ++per) {
    const double ratio = per < few ? (double)few / per : (double)per / few;
    if (ceil_div(stars, per) % 8 == 0 && ratio < off) {
      off = ratio;
      s->per_group = per;
    }
  }
  s->groups = ceil_div(stars, s->per_group);
  // fields, transform buffers, matrices and pupils of every wavelength; seed weights with a plane of each
  // wavelength's own, the groups' planes, the image and its derivatives; the stars' weights and position sums
  const size_t optics = sizeof(float) * 2 * L * (nt2 + 4 * Nt * ldNi + p.Ni * ldNi);
  const size_t table = (4 * (1 + L) + 8 * (size_t)s->groups + 16) * nt2;
  const size_t stars_bytes = nfs * (16 * (size_t)s->slots + 8 * 32 * (size_t)wrow(s->K));
  s->bytes = optics + table + stars_bytes + s->chunk * frame;
}

// whether two adjoint workgroups of eight waves fit a CU
bool adjoint_pair(int h16, int K) { return adjoint_lds(8, h16, K) <= 80 << 10; }

}  // namespace

// The table's pitch, taps and sizes for a problem, or false where one transform pair per star, frame and
// wavelength is the cheaper form. A finer pitch (h16 up) needs fewer taps but more samples to transform;
// the estimate weighs the folded products at their measured rate (85 TFLOP/s executed, after 15 us a
// launch, 121 in split precision; 120 on a table, which leaves out the rows and columns no star reaches) against the FP64 matrix
// instructions of the interpolation and its adjoint (64 cycles of a SIMD each, times 1.7 and 1.8 to 2.0
// measured), the passes over memory and 70 us for the table's seven further launches (388 focal samples, 6
// stars, 2 wavelengths, where the estimates are near: 255 us on a table, 240 without). Of 157 FP32 problems whose
// estimates lie 0.4 to 0.85 apart the slowest took 0.96 of the per-star time on a table, of 125 split ones 1.01;
// 14 further split ones, taken in while the estimate had FP32's rate for them, took up to 1.28 of it (960 pupil, 320 focal
// samples, 38 wavelengths, 3 frames: 2134 us on a table, 1673 without). (512 pupil, 768 focal
// samples, 32 wavelengths: 128 stars 1803 us at h16 = 10, 1686 at 12, 1805 at 13; 24 stars 933 at 9, 994 at 12.)
bool choose_table_shape(const TableProblem& p, TableShape* best) {
  // The table's products are FP32 in both arithmetics (they are a small part of the evaluation). A split
  // plan of few wavelengths keeps its own products: its error in the faintest pixels, 2e-5 to 6e-5 of the
  // residual (2e-6 to 1e-5 where 16 or more wavelengths average it), would make the two forms of one
  // problem differ by as much.
  if (p.bf16x3 && p.L < 16) return false;
  if (p.S > 65535) return false;
  // A band fills the nulls of its wavelengths; one wavelength keeps them, and nearly every block of its image
  // has a sample that would have to be interpolated from the field (5 times the products, see TableArgs).
  if (p.L < 2 || !(p.lmax > p.lmin)) return false;
  const double Ni = p.Ni, No = p.No, L = p.L, nfs = (double)p.F * p.S;
  const double lmin = p.lmin, lmax = p.lmax, n_psf = nfs * L;
  // A focal grid wider than the pupil grid's own field (one period of the sampled tilts) can hold stars whose
  // tilts each wavelength reduces by itself, which cost a table far more than their own transforms (100 pupil
  // and 400 focal samples, 16 wavelengths, 48 stars all over them: 5.7 ms on a table, 1.6 ms without).
  if (No * p.du > lmin / p.dx) return false;
  const double rate = p.bf16x3 ? 121e6 : 85e6, launches = p.bf16x3 ? 150.0 : 60.0;
  const double direct = 4.0 * n_psf * (No * Ni * Ni + No * No * Ni) / rate + launches + n_psf * No * No * 8.0 / 4.5e6;
  double least = 0.85 * direct;
  bool found = false;
  const int nb = ceil_div(p.No, 16);
  for (int h16 = 1; h16 <= 40; ++h16) {
    const double h = h16 / 16.0, tau = p.du / h, sigma = lmin / (2.0 * p.D) / tau;
    if (!(sigma >= 1.2)) continue;
    if (sigma > 4.0 && found) break;
    const int W = (int)std::ceil(2.0 * kTableBeta / (3.14159265358979 * (1.0 - 1.0 / sigma)));
    if (W > kTableMaxW) continue;
    const int K = round_up((int)std::floor(15.0 * h) + W + 1, 8);
    if (K < kTableMinK || K > kTableMaxK) continue;
    // samples in use for stars within the middle of the detector, with the taps and the stencil around them
    const int n_reg = round_up((int)std::ceil(No * h * (nfs > 1 ? 1.25 : 1.02) + 2 * W + 10), 64);
    const double half = 0.5 * (No - 1) * h + 0.5 * lmax / p.dx / tau + W + 6;
    if (half > 16000.0) continue;
    const int Nt = std::max(n_reg, round_up((int)std::ceil(2.0 * half), 64));
    const int waves = table_adjoint_waves(h16, K);
    if (!waves) continue;
    const double n = n_reg, own = std::min(n, No * h + W), cols = 16.0 * waves;   // own: samples a star reaches
    const double fwd = (std::ceil((7 * h16 + K) / 16.0) * K / 4 + 8.0 * (K / 4 + 1)) / 8 * nb * nb;
    const double quads = (17.0 + W + 3 * h) / (h16 / 4.0);   // groups of four focal rows that reach 16 samples
    const double adj = std::min(n / 32, own / 32 + 1) * std::min(std::ceil(n / cols), own / cols + 1) * waves * 2 *
                       quads * (std::ceil(((cols + K - 1) / h16 + 1) / waves) + 1);
    const double est = 4.0 * L * (n * Ni * Ni + n * n * Ni) / 120e6 + 60.0 + L * n * n * 8.0 / 3e6 +
                       nfs * (1.7 * fwd + (adjoint_pair(h16, K) ? 1.8 : 2.0) * adj) * 64.0 / (1024 * 2400.0) +
                       nfs * No * No * 12.0 / 3e6 + 70.0;
    if (est >= least) continue;
    // (stars all over an enlarged plane, as integer dithers are for, use the table about twice as far)
    const int sized = p.dither ? std::min(Nt, round_up((int)std::ceil(2.0 * No * h + 2 * W + 10), 64)) : n_reg;
    TableShape s = {};
    s.Nt = Nt;
    s.n_reg = sized;
    s.h16 = h16;
    s.W = W;
    s.K = K;
    s.waves = waves;
    s.slots = waves * std::min((sized / 32) * ceil_div(sized, 16 * waves), 4096);
    s.tau = tau;
    size_arrays(p, &s);
    if (s.bytes > kTableMaxBytes) continue;
    *best = s;
    least = est;
    found = true;
  }
  return found;
}

}  // namespace dlx
