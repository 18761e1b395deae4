// Runs choose_table_shape over the problems given on standard input, one per line
//   n_pupil n_focal wavelengths stars frames detector bf16x3 dither diameter focal_pitch lambda_min lambda_max
// and prints for each whether a table was chosen and, if so, its sizes and what the kernels need for them.
// Built by tests/test_table_choice.py (g++, host code only).
#include <cstdio>

#include "table_choice.h"

int main() {
  dlx::TableProblem p;
  int bf = 0, dither = 0;
  while (std::scanf("%d %d %d %d %d %d %d %d %lf %lf %lf %lf", &p.Ni, &p.No, &p.L, &p.S, &p.F, &p.Nd, &bf, &dither, &p.D,
                    &p.du, &p.lmin, &p.lmax) == 12) {
    p.bf16x3 = bf != 0;
    p.dither = dither != 0;
    p.dx = p.D / p.Ni;
    dlx::TableShape s = {};
    if (!dlx::choose_table_shape(p, &s)) {
      std::printf("0\n");
      continue;
    }
    std::printf("1 %d %d %d %d %d %d %d %zu %d %d %d %d %zu\n", s.h16, s.W, s.K, s.waves, s.Nt, s.n_reg, s.slots,
                dlx::adjoint_lds(s.waves, s.h16, s.K), 16 * dlx::wrow(s.K), s.chunk, s.groups, s.per_group, s.bytes);
  }
  return 0;
}
