// Runs 2-D programs symbolically: every buffer holds the name of the level in it, and each
// step must read the levels it is meant to, from buffers it does not write.
//   stdin: cases of "K T M comp rows nact" and nact action triples; exit code 1 with a message
//   on the first wrong read.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>

#include "../../paper_1810_05268_amd/csrc/wv_prog2d.h"

using namespace wv;

struct Codes {
    int advance = 1, store = 2, restore = 3, reverse = 5;
};

static int g_case = -1;
#define NEED(cond, ...)                                   \
    do {                                                  \
        if (!(cond)) {                                    \
            std::printf("case %d: ", g_case);             \
            std::printf(__VA_ARGS__);                     \
            std::printf(" [%s]\n", #cond);                \
            std::exit(1);                                 \
        }                                                 \
    } while (0)

static std::string U(int n) { return n <= 0 ? "0" : "u" + std::to_string(n); }

int main()
{
    int K, T, M, comp, rows, nact;
    while (std::scanf("%d %d %d %d %d %d", &K, &T, &M, &comp, &rows, &nact) == 6) {
        ++g_case;
        std::vector<int32_t> acts(3 * nact);
        for (auto &v : acts)
            if (std::scanf("%d", &v) != 1) return 2;
        int N = 0;
        for (int i = 0; i < nact; ++i)
            if (acts[3 * i] == 5) N = std::max(N, acts[3 * i + 1]);
        // stores whose checkpoint the schedule later advances from
        std::vector<char> need2(nact, 0);
        std::map<int, int> holder;
        for (int i = 0; i < nact; ++i) {
            if (acts[3 * i] == 2) holder[acts[3 * i + 2]] = i;
            if (acts[3 * i] == 3 && acts[3 * i + 2] > 0) {
                int j = i + 1;
                while (j < nact && acts[3 * j] == 4) ++j;
                if (j < nact && acts[3 * j] == 1) need2[holder[acts[3 * i + 2]]] = 1;
            }
        }
        Prog2d p(K, T);
        p.schedule(acts, need2, M, comp != 0, rows != 0, Codes{});
        NEED(p.valid, "program not valid");
        std::map<int, std::string> mem, arena;   // buffers; streams by offset word
        mem[kBufZ] = "0";
        mem[kBufL] = mem[kBufL + 1] = "L";       // lam^N = lam^{N+1} = 0
        auto lam = [&](int k) { return k >= N ? std::string("L") : "l" + std::to_string(k); };
        std::set<int> gathered, reversed;
        int next_k = N;
        auto in_range = [&](int id) {
            return id == kBufZ || id == kBufDB || (id >= kBufL && id < kBufL + 4) ||
                   (id >= kBufU && id < kBufU + tile2d_ring(K)) || (id >= kBufUB && id < kBufUB + tile2d_decoded(K)) ||
                   (id >= kBufSlot + 2 && id < kBufSlot + 2 * M && !comp);
        };
        for (const BatchOp &op : p.ops) {
            switch (op.kind) {
            case kOpStep: {
                NEED(op.ns >= 1 && op.ns <= T, "group of %d steps", op.ns);
                NEED(mem[op.a] == U(op.n) && mem[op.b] == U(op.n - 1), "steps from %d read %s %s", op.n, mem[op.a].c_str(),
                     mem[op.b].c_str());
                std::set<int> outs;
                for (int j = 0; j < op.ns; ++j) {
                    if (op.e >> j & 1) NEED(gathered.insert(op.n + j).second, "row %d twice", op.n + j);
                    if (op.c[j] == kBufNone) continue;
                    NEED(in_range(op.c[j]) && op.c[j] != kBufZ, "buffer %d", op.c[j]);
                    NEED(op.c[j] != op.a && op.c[j] != op.b && outs.insert(op.c[j]).second, "writes what it reads");
                    mem[op.c[j]] = U(op.n + j + 1);
                }
                NEED(op.e >> op.ns == 0, "row past the group");
                NEED(op.c[op.ns - 1] != kBufNone, "last level dropped");
                break;
            }
            case kOpAdj: {
                NEED(op.ns >= 1 && op.ns <= T && op.n == next_k, "reverse group %d x %d, expected %d", op.n, op.ns, next_k);
                NEED(mem[op.a] == lam(op.n) && mem[op.b] == lam(op.n + 1), "adjoint levels at %d", op.n);
                for (int j = 0; j < op.ns; ++j) {
                    NEED(in_range(op.c[j]) && mem[op.c[j]] == U(op.n - j), "reverse step %d reads %s", op.n - j,
                         mem[op.c[j]].c_str());
                    reversed.insert(op.n - j);
                }
                NEED(op.d[0] != op.a && op.d[0] != op.b && op.d[1] != op.a && op.d[1] != op.b && op.d[0] != op.d[1],
                     "adjoint writes what it reads");
                next_k = op.n - op.ns;
                mem[op.d[0]] = lam(next_k);
                if (op.ns > 1) mem[op.d[1]] = lam(next_k + 1);
                break;
            }
            case kOpGather:
                NEED(rows && mem[op.a] == U(op.n), "row %d from %s", op.n, mem[op.a].c_str());
                NEED(gathered.insert(op.n).second, "row %d twice", op.n);
                break;
            case kOpEnc:
                NEED(op.ns >= 1 && op.ns <= tile2d_jobs(K), "%d fields", op.ns);
                for (int j = 0; j < op.ns; ++j) {
                    std::string v = mem[op.c[j]];
                    NEED(v[0] == 'u' || v == "0", "encodes %s", v.c_str());
                    if (op.d[j] != kBufNone) v += "-" + mem[op.d[j]];
                    if (op.y[j] >= 0) NEED(v == U(op.y[j]), "size of %d is that of %s", op.y[j], v.c_str());
                    const int end = j + 1 < op.ns ? op.x[j + 1] : op.n;
                    NEED(end > op.x[j] && end <= op.x[j] + 2, "offset words %d -> %d", op.x[j], end);
                    for (auto it = arena.lower_bound(op.x[j]); it != arena.end();) it = arena.erase(it);   // a stack
                    arena[op.x[j]] = v;
                }
                break;
            case kOpDec:
                NEED(op.ns >= 1 && op.ns <= tile2d_jobs(K), "%d streams", op.ns);
                for (int j = 0; j < op.ns; ++j) {
                    NEED(arena.count(op.x[j]), "decodes nothing at %d", op.x[j]);
                    std::string v = arena[op.x[j]];
                    NEED(in_range(op.c[j]) && op.c[j] != kBufZ, "buffer %d", op.c[j]);
                    if (op.d[j] != kBufNone) {   // u^k - (u^k - u^{k-1})
                        const std::string head = mem[op.d[j]] + "-";
                        NEED(v.compare(0, head.size(), head) == 0, "%s less %s", mem[op.d[j]].c_str(), v.c_str());
                        v = v.substr(head.size());
                    }
                    mem[op.c[j]] = v;
                }
                break;
            case kOpCopy:
                NEED(in_range(op.b) && mem.count(op.a), "copy");
                mem[op.b] = mem[op.a];
                break;
            case kOpResid:
                NEED(mem[op.a] == U(N), "residual after %s", mem[op.a].c_str());
                if (rows)
                    for (int n = 1; n <= N; ++n) NEED(gathered.count(n), "row %d missing", n);
                break;
            case kOpMisfit: break;
            default: NEED(false, "kind %d", op.kind);
            }
        }
        NEED(next_k == 0 && (int)reversed.size() == N, "%d reverse steps left", next_k);
        NEED((int)gathered.size() == (rows ? N : 0), "%d rows", (int)gathered.size());
    }
    std::printf("%d programs\n", g_case + 1);
    return 0;
}
