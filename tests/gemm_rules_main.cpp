// The host-side choices of goq_gemm (goq_gemm_rules.h), one launch per line of stdin:
//     bw fp16 staged n  tokens out in  tokens out in ..   ->   32 or 64
#include <cstdio>
#include "../paper_2605_26092_amd/csrc/goq_gemm_rules.h"

int main()
{
    int bw, fp16, staged, n;
    while (scanf("%d %d %d %d", &bw, &fp16, &staged, &n) == 4) {
        GoqTileProblem p[8];
        for (int i = 0; i < n; ++i) {
            int in;
            if (scanf("%d %d %d", &p[i].tokens, &p[i].out, &in) != 3) return 1;
            p[i].gn = in / GOQ_N;
        }
        printf("%d\n", goq_narrow_tiles(bw, fp16 != 0, staged != 0, n, p) ? 32 : 64);
    }
    return 0;
}
