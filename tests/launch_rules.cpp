// Prints the workgroup shape ("qg ks") that each line of standard input launches:
//   f d N bh causal fp8   an MXFP4 forward
//   b d N bh              a BF16 forward
// or, for
//   k d causal fp8 qg ks  whether a kernel of that shape is built ("1" or "0")
#include <cstdio>

#include "../paper_2609_04105_amd/csrc/launch_rules.hpp"

int main() {
  char kind;
  int d, n, bh, causal = 0, fp8 = 0;
  while (std::scanf(" %c %d %d %d", &kind, &d, &n, &bh) == 4) {
    if (kind == 'k') {
      int qg, ks;
      if (std::scanf("%d %d", &qg, &ks) != 2) return 1;
      std::printf("%d\n", fp4attn::directp_launches(d, n != 0, bh != 0, fp4attn::Shape{qg, ks}));
      continue;
    }
    if (kind == 'f' && std::scanf("%d %d", &causal, &fp8) != 2) return 1;
    const fp4attn::Shape s = kind == 'f' ? fp4attn::directp_shape(d, n, bh, causal != 0, fp8 != 0) : fp4attn::bf16_shape(d, n, bh);
    std::printf("%d %d\n", s.qg, s.ks);
  }
  return 0;
}
