// Runs 2-D programs symbolically on the field arrays a run reserves (Prog2d::rings).  What one
// op does is concurrent on the device, so its reads are taken before any of its writes, it
// writes no array twice, and none that it reads.
//   stdin: cases of "K T chunks M comp nact" and nact action triples, or "K T 0 0 0 n": n steps of
//   a forward run; T = 0: steps that march, which may write the level they read last
//   stdout: a line a case with the arrays; exit code 1 with a message on the first fault
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
#define NEED(cond)                                                     \
    do {                                                               \
        if (!(cond)) {                                                 \
            std::printf("case %d op %ld: %s\n", g_case, nop, #cond);   \
            std::exit(1);                                              \
        }                                                              \
    } while (0)

static std::string U(int n) { return n <= 0 ? "0" : "u" + std::to_string(n); }

int main()
{
    int K, T, chunks, M, comp, nact;
    while (std::scanf("%d %d %d %d %d %d", &K, &T, &chunks, &M, &comp, &nact) == 6) {
        ++g_case;
        long nop = 0;
        const bool forward = M == 0;
        std::vector<int32_t> acts(forward ? 0 : 3 * nact);
        for (auto &v : acts)
            if (std::scanf("%d", &v) != 1) return 2;
        int N = forward ? nact : 0;
        for (size_t i = 0; i < acts.size() / 3; ++i)
            if (acts[3 * i] == 5) N = std::max(N, acts[3 * i + 1]);
        std::vector<char> need2(acts.size() / 3, 0);   // stores that the schedule later advances from
        std::map<int, size_t> holder;
        for (size_t i = 0; i < need2.size(); ++i) {
            if (acts[3 * i] == 2) holder[acts[3 * i + 2]] = i;
            if (acts[3 * i] == 3 && acts[3 * i + 2] > 0) {
                size_t j = i + 1;
                while (j < need2.size() && acts[3 * j] == 4) ++j;
                if (j < need2.size() && acts[3 * j] == 1) need2[holder[acts[3 * i + 2]]] = 1;
            }
        }
        const bool march = T == 0;
        if (march) T = 1;
        const Rings2d R = Prog2d::rings(K, T, chunks ? chunks : 1, 256, !forward, march);
        NEED(R.steps == T && R.march == march && R.jobs >= 1 && R.jobs <= kEncJobs && R.jobs <= kTileSteps);
        NEED(kBufU + R.levels <= kBufUB && kBufUB + R.decoded <= kBufSlot);
        std::map<int, std::string> mem{{kBufZ, "0"}, {kBufL, "L"}, {kBufL + 1, "L"}}, arena;
        auto lam = [&](int k) { return k >= N ? std::string("L") : "l" + std::to_string(k); };
        auto writable = [&](int id) {
            return (id >= kBufU && id < kBufU + R.levels) ||
                   (!forward && (id == kBufDB || (id >= kBufL && id < kBufL + R.lam) ||
                                 (id >= kBufUB && id < kBufUB + R.decoded) ||
                                 (!comp && id >= kBufSlot + 2 && id < kBufSlot + 2 + 2 * M)));
        };
        int next_k = N;
        std::set<int> gathered;
        auto sink = [&](const BatchOp &op) {
            ++nop;
            std::set<int> reads, writes;
            std::map<int, std::string> after;
            auto rd = [&](int id) {
                NEED(mem.count(id));
                reads.insert(id);
                return mem[id];
            };
            auto wr = [&](int id, const std::string &v) {
                NEED(writable(id));
                NEED(writes.insert(id).second);
                after[id] = v;
            };
            switch (op.kind) {
            case kOpStep:
                NEED(op.ns >= 1 && op.ns <= T && op.c[op.ns - 1] != kBufNone);
                NEED(rd(op.a) == U(op.n) && rd(op.b) == U(op.n - 1));
                for (int j = 0; j < op.ns; ++j) {
                    if (op.e >> j & 1) NEED(gathered.insert(op.n + j).second);
                    if (op.c[j] != kBufNone) wr(op.c[j], U(op.n + j + 1));
                }
                break;
            case kOpAdj:
                NEED(op.ns >= 1 && op.ns <= T && op.n == next_k);
                NEED(rd(op.a) == lam(op.n) && rd(op.b) == lam(op.n + 1));
                for (int j = 0; j < op.ns; ++j) NEED(rd(op.c[j]) == U(op.n - j));
                next_k -= op.ns;
                wr(op.d[0], lam(next_k));
                if (op.ns > 1) wr(op.d[1], lam(next_k + 1));
                break;
            case kOpGather:
                NEED(rd(op.a) == U(op.n) && gathered.insert(op.n).second);
                break;
            case kOpEnc:
                NEED(op.ns >= 1 && op.ns <= R.jobs);
                for (int j = 0; j < op.ns; ++j) {
                    std::string v = rd(op.c[j]);
                    if (op.d[j] != kBufNone) v += "-" + rd(op.d[j]);
                    NEED(op.y[j] < 0 || v == U(op.y[j]));
                    const int end = j + 1 < op.ns ? op.x[j + 1] : op.n;
                    NEED(end > op.x[j] && end <= op.x[j] + 2);
                    arena.erase(arena.lower_bound(op.x[j]), arena.end());   // a stack
                    arena[op.x[j]] = v;
                }
                break;
            case kOpDec:
                NEED(op.ns >= 1 && op.ns <= R.jobs);
                for (int j = 0; j < op.ns; ++j) {
                    NEED(arena.count(op.x[j]));
                    std::string v = arena[op.x[j]];
                    if (op.d[j] != kBufNone) {   // u^k - (u^k - u^{k-1})
                        const std::string head = rd(op.d[j]) + "-";
                        NEED(v.compare(0, head.size(), head) == 0);
                        v = v.substr(head.size());
                    }
                    wr(op.c[j], v);
                }
                break;
            case kOpCopy: wr(op.b, rd(op.a)); break;
            case kOpResid:
                NEED(rd(op.a) == U(N) && (int)gathered.size() == N);
                break;
            case kOpMisfit: break;
            default: NEED(false);
            }
            if (march && (op.kind == kOpStep || op.kind == kOpAdj) && op.a != op.b) {
                reads.erase(op.b);   // each lane its own point
                if (op.kind == kOpAdj) NEED(op.c[0] != op.b);
            }
            for (int id : writes) NEED(!reads.count(id));
            for (const auto &[id, v] : after) mem[id] = v;
            return true;
        };
        Prog2d p(R);
        if (forward) {
            for (int n = 0; n < N; ++n) p.step(n, true);
            p.flush_rows(N);
            for (const BatchOp &op : p.ops) sink(op);
            NEED(mem[p.u] == U(N) && mem[p.up] == U(N - 1) && (int)gathered.size() == N);
        } else {
            p.stream(acts, need2, M, comp != 0, true, Codes{}, sink);
            NEED(p.valid && next_k == 0);
        }
        std::printf("%d %d %d\n", R.jobs, R.levels, R.decoded);
    }
    return 0;
}
