// The program of a 2-D OT2 run: what the solo executor and the batched solver launch
// op by op (the latter several other ops than steps at once).  Host only.
//
// A schedule's steps, checkpoint writes, reads and reverse steps are collected and emitted in
// groups: up to `steps` forward or reverse steps in one pass over the tiles (a level goes
// to memory only if something reads it: a checkpoint, a reverse step, the next group), the
// checkpoint fields written between two groups in one encode, those read in one decode.
// Grouping changes no arithmetic and no order of any point's updates.
#pragma once

#include <algorithm>
#include <utility>
#include <vector>

#include "wv_internal.h"

namespace wv {

class Prog2d {
public:
    std::vector<BatchOp> ops;
    bool valid = true;
    long advances = 0, stores = 0, restores = 0, reverses = 0, decodes = 0, fields = 0;
    int max_depth = 0;
    int u = kBufZ, up = kBufZ;            // buffers of u^n and u^{n-1} (kBufNone: not decoded)
    int lam = kBufL, lamp = kBufL + 1;    // buffers of lam^k and lam^{k+1}

    // Whether an op is a group of steps.  Of the others a reversal of nt steps has at most so
    // many, whatever its slots: every state is reached for storing or reversing at most once
    // from a restore, so there are at most nt stores (a copy or a field of an encode for each of
    // their two levels), 2 nt + 1 restores (a decode each, and one for the second level), nt data
    // rows, and the residual and the misfit.  Groups of steps grow as nt^2 with one slot.
    static bool steps(const BatchOp &op) { return op.kind == kOpStep || op.kind == kOpAdj; }
    static int most_other_ops(int nt) { return 10 * nt + 64; }

    // What a run of order 2 K works with, in groups of up to T steps, on fields of so many codec
    // chunks.  A forward run holds the two levels a group starts from and the two it leaves; steps
    // that march (T = 1) write over the older level they read, which leaves more of their operands
    // in the L2.  A gradient run also holds the levels that wait for an encode or for their reverse
    // steps, and the checkpoints decoded for those: with so many arrays no schedule of 60 or 301
    // steps at 1 to 301 slots, in tiles, has over 0.3 % more launches than with any number.
    // Fields are encoded and decoded several at a time: one of 552 x 552 points is 75 chunks of
    // 256 lanes, which leave the chip idle, and larger ones save launches and the scan's one
    // workgroup (40 steps of 4000 x 3000 points with 8 states' memory: 4.8 ms by eights and 5.9 one
    // by one at order 2, 8.8 by fours and 9.3 at order 8).  From 64 chunks a CU on (8192 x 8192
    // points, 268 MB an array) arrays count: each goes alone, and at most four levels wait for
    // reverse steps (groups of eight, at orders 2 and 4: up to 4 % more launches).
    static Rings2d rings(int K, int T, long long chunks, int cus, bool gradient, bool march)
    {
        const int lam = march ? 2 : (T > 1 ? 4 : 3);
        if (!gradient) return {T, 1, lam, 0, 0, march};
        const int jobs = (int)std::min<long long>(tile2d_jobs(K), (64LL * cus + chunks - 1) / chunks);
        const int most = jobs > 1 ? std::max(T, jobs) : std::min(T, 4);
        return {T, jobs, most + (march ? 1 : (T > 1 ? 4 : 2)), most, lam, march};
    }

    explicit Prog2d(const Rings2d &r) : T(r.steps), NU(r.levels), ND(r.decoded), NE(r.jobs), march(r.march) {}

    // with as many buffers as any run of order 2 K has
    Prog2d(int K, int group) : Prog2d(Rings2d{group, tile2d_jobs(K), tile2d_ring(K), tile2d_decoded(K), 4, false}) {}

    // u^{n+1} from the current state, into dest if given (kept); gather: its data row is wanted
    void step(int n, bool gather, int dest = kBufNone)
    {
        if ((int)pend.size() == T) flush_steps();   // what they left to encode can wait
        int out = dest;
        if (dest != kBufNone && busy(dest)) {
            flush_adj();
            flush();
            if (busy(dest)) out = kBufNone;   // the state itself starts there: stored by a copy
        }
        if (out == kBufNone) out = free_level();
        if (pend.empty()) {
            base_u = u;
            base_up = up;
            base_row = carry;
            carry = false;
        }
        // u^{n-1} leaves the state: nothing can ask for it any more
        if (pend.size() >= 2 && !pend[pend.size() - 2].keep) pend[pend.size() - 2].out = kBufNone;
        pend.push_back({n, out, gather, dest == out});
        up = u;
        u = out;
    }

    // steps and encodes collected so far; u and up are in memory afterwards
    void flush()
    {
        flush_steps();
        flush_enc();
    }

    // and the last level's data row (row index n of u = u^n)
    void flush_rows(int n)
    {
        flush();
        if (carry) {
            BatchOp op = blank(kOpGather);
            op.a = u;
            op.n = n;
            ops.push_back(op);
        }
        carry = false;
    }

    void flush_adj()
    {
        if (adj.empty()) return;
        flush_dec();
        for (size_t i = 0; i < adj.size(); i += T) {
            BatchOp op = blank(kOpAdj);
            op.n = adj[i].first;
            op.ns = (int)std::min(adj.size() - i, (size_t)T);
            op.a = lam;
            op.b = lamp;
            for (int j = 0; j < op.ns; ++j) op.c[j] = adj[i + j].second;
            int fr[2] = {lamp, kBufNone}, nf = 0;
            for (int q = 0; q < 4 && nf < 2 && !march; ++q)
                if (kBufL + q != lam && kBufL + q != lamp) fr[nf++] = kBufL + q;
            op.d[0] = fr[0];
            op.d[1] = op.ns > 1 ? fr[1] : kBufNone;
            lamp = op.ns > 1 ? fr[1] : lam;
            lam = fr[0];
            ops.push_back(op);
        }
        adj.clear();
    }

    // the reversal that acts prescribe (action triples; codes as the executor's), with
    // M slots, plain or compressed; need2 flags the stores that keep both levels; rows: the
    // first sweep gathers data rows (a gradient of a given residual wants none).  The whole
    // program: nt^2 / (2 T) groups of steps with one slot
    template <typename Codes>
    void schedule(const std::vector<int32_t> &acts, const std::vector<char> &need2, int M, bool comp, bool rows,
                  Codes code)
    {
        std::vector<BatchOp> all;
        stream(acts, need2, M, comp, rows, code, [&](const BatchOp &op) {
            all.push_back(op);
            return true;
        });
        ops.swap(all);
    }

    // The same op by op, none of them kept: sink(op) takes each as the schedule reaches it, and
    // ends the program when it returns false.
    template <typename Codes, typename Sink>
    void stream(const std::vector<int32_t> &acts, const std::vector<char> &need2, int M, bool comp, bool rows,
                Codes code, Sink sink)
    {
        auto drain = [&]() {
            for (BatchOp &op : ops)
                if (!sink(op)) return false;
            ops.clear();
            return true;
        };
        std::vector<char> slot2((size_t)M + 2, 0);
        int hot_slot = -1, hot_k = -1, hot_buf = kBufNone, pend_slot = -1, cur_n = 0;
        bool up_pending = false, hot_db = false, started = false;
        int gathered = 0;
        // reverse steps collected before they run: a group, or, where their states are decoded,
        // as many groups as one decode serves
        const int collect = comp ? std::max(T, NE / T * T) : T;
        const size_t nact = acts.size() / 3;
        for (size_t i = 0; i < nact && valid; ++i) {
            const int op = acts[3 * i], a = acts[3 * i + 1], b = acts[3 * i + 2];
            if (op == code.advance) {
                if (up == kBufNone) {   // advancing from a restore: the second level is needed now
                    if (!up_pending) {  // cannot happen: need2 marks these checkpoints
                        valid = false;
                        break;
                    }
                    if (!hot_db) {
                        flush_dec();     // it is rebuilt from the first level
                        push_dec(kBufDB, hot_buf, 2 * pend_slot + 1);
                        hot_db = true;
                        decodes++;
                    }
                    up = kBufDB;
                    up_pending = false;
                }
                // an uncompressed state that the next action stores is written into its slot
                int last = kBufNone, prev = kBufNone;
                if (!comp && i + 1 < nact && acts[3 * (i + 1)] == code.store && acts[3 * (i + 1) + 1] == b &&
                    acts[3 * (i + 1) + 2] >= 1) {
                    last = kBufSlot + 2 * acts[3 * (i + 1) + 2];
                    if (need2[i + 1] && b - a >= 2) prev = last + 1;
                }
                for (int n = a; n < b; ++n) {
                    step(n, rows && n + 1 > gathered, n == b - 1 ? last : (n == b - 2 ? prev : kBufNone));
                    if (n + 1 > gathered) gathered = n + 1;
                    if (!drain()) return;
                }
                cur_n = b;
                advances += b - a;
            } else if (op == code.store) {
                slot2[b] = need2[i];
                if (need2[i] && up == kBufNone) {
                    valid = false;
                    break;
                }
                if (comp) {
                    const int base = 2 * b;
                    push_enc(u, kBufNone, base, need2[i] ? base + 1 : base + 2, a, need2[i] ? 2 : 1);
                    if (need2[i]) push_enc(u, up, base + 1, base + 2, -1, 1);
                    if (hot_slot == b) hot_slot = -1;
                } else {
                    copy(u, kBufSlot + 2 * b);
                    if (need2[i]) copy(up, kBufSlot + 2 * b + 1);
                }
                stores++;
                fields += need2[i] ? 2 : 1;
                if (b > max_depth) max_depth = b;
            } else if (op == code.restore) {
                flush_rows(cur_n);
                up_pending = false;
                if (b == 0) {
                    u = up = kBufZ;
                } else if (comp) {
                    if (hot_slot != b || hot_k != a) {
                        u = up = kBufNone;
                        const int id = free_decoded();
                        push_dec(id, kBufNone, 2 * b);
                        hot_buf = id;
                        hot_slot = b;
                        hot_k = a;
                        hot_db = false;
                        decodes++;
                    }
                    // u^{k-1} is decoded by the advance that needs it
                    u = hot_buf;
                    up = kBufNone;
                    up_pending = slot2[b] != 0;
                    pend_slot = b;
                } else {
                    u = kBufSlot + 2 * b;
                    up = slot2[b] ? u + 1 : kBufNone;
                }
                cur_n = a;
                restores++;
            } else if (op == code.reverse) {
                flush_rows(cur_n);
                if (!started) {
                    started = true;
                    flush_dec();
                    BatchOp r = blank(kOpResid);
                    r.a = u;
                    ops.push_back(r);
                    ops.push_back(blank(kOpMisfit));
                }
                adj.push_back({a, u});
                reverses++;
                if ((int)adj.size() >= collect) flush_adj();
            }
            if (!drain()) return;
        }
        if (!valid) return;
        flush_adj();
        flush();
        (void)drain();
    }

private:
    struct Step {
        int n, out;
        bool gather, keep;
    };
    struct Enc {
        int field, sub, base, next, k;
    };
    struct Dec {
        int dest, sub, base;
    };
    const int T, NU, ND, NE;
    const bool march;
    std::vector<Step> pend;
    int base_u = kBufNone, base_up = kBufNone;
    bool base_row = false, carry = false;   // the base's / the current level's data row is still to be gathered
    std::vector<std::pair<int, int>> adj;   // collected reverse steps (k, buffer of u^k)
    std::vector<Enc> enc;
    std::vector<Dec> dec;

    static BatchOp blank(int kind)
    {
        BatchOp op{};
        op.kind = kind;
        op.a = op.b = kBufNone;
        for (int j = 0; j < kTileSteps; ++j) op.c[j] = op.d[j] = kBufNone;
        return op;
    }

    // whether the current state is in the buffer, or something collected still reads or writes it
    bool busy(int id) const { return id == u || id == up || wanted(id); }

    bool wanted(int id) const
    {
        if (!pend.empty() && (id == base_u || id == base_up)) return true;
        for (const Step &p : pend)
            if (p.out == id) return true;
        for (const auto &r : adj)
            if (r.second == id) return true;
        for (const Enc &e : enc)
            if (e.field == id || e.sub == id) return true;
        for (const Dec &x : dec)
            if (x.dest == id || x.sub == id) return true;
        return false;
    }

    // where the next level goes
    int free_level()
    {
        for (int t = 0;; ++t) {
            if (march && up >= kBufU && up < kBufU + NU && !wanted(up)) return up;
            for (int i = 0; i < NU; ++i)
                if (!busy(kBufU + i)) return kBufU + i;
            // the level that leaves the state with this step, if it is only passed through
            if (pend.size() >= 2 && !pend[pend.size() - 2].keep) return up;
            if (t == 0) flush_adj();
            else flush();
        }
    }

    // where the next checkpoint is decoded (the state has just left, so that the flushes free all)
    int free_decoded()
    {
        for (;;) {
            for (int i = 0; i < ND; ++i)
                if (!busy(kBufUB + i)) return kBufUB + i;
            flush_adj();
            flush_dec();
        }
    }

    void need(int id)
    {
        for (Step &p : pend)
            if (p.out == id) p.keep = true;
    }

    void flush_steps()
    {
        if (pend.empty()) return;
        flush_dec();
        BatchOp op = blank(kOpStep);
        op.n = pend[0].n;
        op.ns = (int)pend.size();
        op.a = base_u;
        op.b = base_up;
        op.e = base_row ? 1 : 0;
        for (int j = 0; j < op.ns; ++j) {
            op.c[j] = (j >= op.ns - 2 || pend[j].keep) ? pend[j].out : kBufNone;
            if (pend[j].gather && j + 1 < op.ns) op.e |= 2 << j;
        }
        carry = pend.back().gather;
        ops.push_back(op);
        pend.clear();
    }

    void flush_enc()
    {
        if (enc.empty()) return;
        flush_steps();
        flush_dec();               // streams about to be overwritten
        BatchOp op = blank(kOpEnc);
        op.ns = (int)enc.size();
        for (int j = 0; j < op.ns; ++j) {
            op.c[j] = enc[j].field;
            op.d[j] = enc[j].sub;
            op.x[j] = enc[j].base;
            op.y[j] = enc[j].k;
        }
        op.n = enc.back().next;    // every other job's next is the base of the one after it
        ops.push_back(op);
        enc.clear();
    }

    // room: jobs that have to fit this group together
    void push_enc(int field, int sub, int base, int next, int k, int room)
    {
        if (!enc.empty() && (enc.back().next != base || (int)enc.size() + room > NE)) flush();
        need(field);
        if (sub != kBufNone) need(sub);
        enc.push_back({field, sub, base, next, k});
    }

    void flush_dec()
    {
        if (dec.empty()) return;
        BatchOp op = blank(kOpDec);
        op.ns = (int)dec.size();
        for (int j = 0; j < op.ns; ++j) {
            op.c[j] = dec[j].dest;
            op.d[j] = dec[j].sub;
            op.x[j] = dec[j].base;
        }
        ops.push_back(op);
        dec.clear();
    }

    void push_dec(int dest, int sub, int base)
    {
        flush();                   // the stream may be one just collected; steps may still read dest
        if ((int)dec.size() == NE) flush_dec();
        dec.push_back({dest, sub, base});
    }

    void copy(int src, int dst)
    {
        if (src == dst) return;
        need(src);
        flush();
        for (const auto &r : adj)
            if (r.second == dst) {
                flush_adj();
                break;
            }
        BatchOp op = blank(kOpCopy);
        op.a = src;
        op.b = dst;
        ops.push_back(op);
    }
};

}  // namespace wv
