// Builds 2-D programs and prints what each holds.
//   stdin: cases of "K T M comp rows nact" and nact action triples
//   stdout, a line a case: ops, and those of them that are no groups of steps
#include <cstdio>

#include "../../paper_1810_05268_amd/csrc/wv_prog2d.h"

using namespace wv;

struct Codes {
    int advance = 1, store = 2, restore = 3, reverse = 5;
};

int main()
{
    int K, T, M, comp, rows, nact;
    while (std::scanf("%d %d %d %d %d %d", &K, &T, &M, &comp, &rows, &nact) == 6) {
        std::vector<int32_t> acts(3 * nact);
        for (auto &v : acts)
            if (std::scanf("%d", &v) != 1) return 2;
        // every store keeps both levels: as many fields as any schedule has
        std::vector<char> need2(nact, 1);
        Prog2d p(K, T);
        p.schedule(acts, need2, M, comp != 0, rows != 0, Codes{});
        if (!p.valid) return 1;
        size_t other = 0;
        for (const BatchOp &op : p.ops) other += !Prog2d::steps(op);
        std::printf("%zu %zu\n", p.ops.size(), other);
    }
    return 0;
}
