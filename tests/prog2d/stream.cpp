// Takes 2-D programs op by op and compares them with the whole ones.
//   stdin: cases of "K T M comp rows nact" and nact action triples
//   stdout, a line a case: ops, and the most of them held at a time; exit code 1 where a
//   streamed op differs, or one follows a sink that returned false.
#include <cstdio>
#include <cstring>

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
        std::vector<char> need2(nact, 1);
        Prog2d whole(K, T);
        whole.schedule(acts, need2, M, comp != 0, rows != 0, Codes{});
        size_t n = 0, held = 0;
        bool same = true;
        Prog2d p(K, T);
        p.stream(acts, need2, M, comp != 0, rows != 0, Codes{}, [&](const BatchOp &op) {
            held = std::max(held, p.ops.size());
            same = same && n < whole.ops.size() && std::memcmp(&op, &whole.ops[n], sizeof op) == 0;
            ++n;
            return true;
        });
        if (!same || n != whole.ops.size() || p.advances != whole.advances || !p.ops.empty()) return 1;
        size_t taken = 0;
        Prog2d q(K, T);
        q.stream(acts, need2, M, comp != 0, rows != 0, Codes{}, [&](const BatchOp &) { return ++taken < (n + 1) / 2; });
        if (taken != (n + 1) / 2) return 1;
        std::printf("%zu %zu\n", n, held);
    }
    return 0;
}
