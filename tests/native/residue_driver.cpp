// Prints the tables of the residue products (csrc/residue.h), one row of integers per line.
#include <cstdio>

#include "../../paper_1702_05167_amd/csrc/residue.h"

int main() {
  static constexpr hsc::ResTables t = hsc::res_tables();
  for (int m = 0; m < hsc::kResMods; ++m) std::printf("%d ", t.p[m]);
  std::printf("\n%d %d %d %a %a\n", hsc::kResSplit, hsc::kResLimbs, hsc::kResBits, t.P_hi, t.P_lo);
  for (int q = 0; q < 4; ++q)
    for (int m = 0; m < hsc::kResMods; ++m) {
      for (int b = 0; b < 16; ++b) std::printf("%d ", t.split[q][m][b]);
      std::printf("\n");
    }
  for (int part = 0; part < 2; ++part)
    for (int g = 0; g < 2; ++g)
      for (int l = 0; l < hsc::kResLimbs; ++l) {
        for (int b = 0; b < 16; ++b) std::printf("%d ", t.crt[part][g][l][b]);
        std::printf("\n");
      }
  for (int m = 0; m < hsc::kResMods; ++m) std::printf("%d ", hsc::res_bias_bits(t.p[m]));
  std::printf("\n");
  for (int m = 0; m < hsc::kResMods; ++m) std::printf("%d ", hsc::kResBias - hsc::res_bias(t.p[m]) / t.p[m]);
  std::printf("\n");
  return 0;
}
