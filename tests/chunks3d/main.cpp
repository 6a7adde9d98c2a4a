// Prints chunks3d for cases "tiles nz K grad per_cu" on 256 CUs.
#include <cstdio>

#include "../../paper_1810_05268_amd/csrc/wv_chunks3d.h"

int main()
{
    long long tiles;
    int nz, K, grad, per_cu;
    while (std::scanf("%lld %d %d %d %d", &tiles, &nz, &K, &grad, &per_cu) == 5)
        std::printf("%d\n", wv::chunks3d(tiles, nz, K, grad != 0, per_cu, 256));
    return 0;
}
