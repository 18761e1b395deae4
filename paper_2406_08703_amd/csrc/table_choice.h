// The shared PSF table's sizes for a problem (TableArgs says what the table is): which pitch, how many taps,
// and whether a table pays at all. Plain C++ without HIP: built into libdlx, and on its own by the CPU tests,
// which hold every table that can be chosen against the limits of the compiled kernels stated here.
#pragma once

#include <cstddef>

namespace dlx {

constexpr double kTableBeta = 20.0;   // interpolation error about exp(-beta)

// Table samples that a block of 16 focal samples may touch, K (a multiple of 8): the interpolation is compiled
// for kTableMinK to kTableMaxK, and the adjoint stages the weights of one star for no more.
constexpr int kTableMinK = 16, kTableMaxK = 80;
constexpr int kTableMaxW = 72;   // taps: the derivative's band holds half of them on either side

// Row length of a star's weights: K, and zeros on both sides.
constexpr int kPadL = 16;
constexpr int wrow(int K) { return K + kPadL + 18; }

constexpr int kAdjLds = 150 << 10;

// Blocks of focal columns that reach an adjoint workgroup's 16 `waves` table columns, and its LDS: the
// star's weights and 4 KB for each of these blocks.
constexpr int adjoint_blocks(int waves, int h16, int K) { return (16 * waves + K - 2) / h16 + 1; }
constexpr size_t adjoint_lds(int waves, int h16, int K) {
  return sizeof(double) * (2 * 16 * wrow(K) + (size_t)adjoint_blocks(waves, h16, K) * 2 * 4 * 64);
}

// Waves of an adjoint workgroup (16 table columns each): 8, or 4 where the focal blocks that reach 128
// columns do not fit the LDS; 0 where neither does. (Four where eight fit as well is slower, 703 us against
// 665 for 128 stars at h16 = 12: the first product, shared by the waves, covers K columns more than they own.)
constexpr int table_adjoint_waves(int h16, int K) {
  return adjoint_lds(8, h16, K) <= kAdjLds ? 8 : adjoint_lds(4, h16, K) <= kAdjLds ? 4 : 0;
}

constexpr size_t kDefaultChunkBudget = size_t(8) << 30;   // bytes of per-chunk intermediates

// The most device memory a table takes, in all (8.9 GiB for 1024 pupil and 2048 focal samples of 16 wavelengths, 7.9
// for 512, 768, 32 and 128 stars; of 400 problems drawn over 32 to 800 pupil samples and 2 to 40 wavelengths one or two
// need more). A
// constant, so that the form a problem takes does not hang on what else the device holds at the time.
constexpr size_t kTableMaxBytes = size_t(16) << 30;

struct TableProblem {
  int Ni, No, L, S, F;   // pupil and focal samples per side, wavelengths, stars per frame, frames propagated
  int Nd;                // detector pixels per side
  bool bf16x3, dither;
  double D, dx, du;      // pupil diameter and pitch (metres), focal pitch (radians)
  double lmin, lmax;     // metres
};

struct TableShape {
  int Nt;       // table samples per side, for stars anywhere in the pupil grid's own field
  int n_reg;    // those in use for stars within the detector
  int h16, W, K, waves, slots;   // see TableArgs
  double tau;   // pitch, radians
  int chunk;    // frames per chunk
  int groups, per_group;   // star groups of the adjoint
  size_t bytes;            // device memory, to within a few per cent
};

// False where one transform pair per star, frame and wavelength is the cheaper form.
bool choose_table_shape(const TableProblem& p, TableShape* best);

}  // namespace dlx
