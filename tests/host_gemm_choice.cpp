// Prints the kernel that csrc/gemm_choice.h gives each call of a list: reads
// lines "M N K cus fused mx amax statistic" and writes a name for each.
#include <cstdio>

#include "../paper_2407_17353_amd/csrc/gemm_choice.h"

int main() {
  long M, N, K;
  int cus, fused, mx, amax, stat;
  while (scanf("%ld %ld %ld %d %d %d %d %d", &M, &N, &K, &cus, &fused, &mx, &amax, &stat) == 8) {
    const scalify::GemmChoice c =
        scalify::gemm_choice(M, N, K, cus, fused != 0, mx != 0, amax != 0, stat != 0);
    const char* mid[] = {"mid256", "mid128", "pair"};
    const char* kind[] = {"big", "fused8", mid[c.mid], "wave"};
    printf("%s%s\n", kind[c.kind], c.tiles > (long)c.resident * cus ? "-rounds" : "");
  }
}
