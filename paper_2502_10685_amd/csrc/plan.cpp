// Host planner of libpauliprop.
//
// The observable is propagated in the Heisenberg picture, so gates are taken
// g_m first.  Two schedules are built from the same list:
//
// Dense: the paper divides a circuit into operators of non-CX gates U_k and
// CX gates V_k and groups each U_k by wire, so that all single-qubit gates of
// one wire act as one composed map (Sec. III-A, Sec. III-C, eq. (5)).  Here a
// wire's run of single-qubit gates between two CX gates touching that wire
// becomes one U1 op, whatever other wires do in between (gates on disjoint
// qubits commute).  For n too large for one workgroup's LDS the ops are
// packed into passes over k-qubit tiles: a greedy list scheduler takes every
// gate whose predecessors on its wires are done and whose qubits lie in the
// pass's qubit set, and grows the set (up to k qubits) with the earliest
// ready gate when nothing else fits.
//
// Sparse: one pass per rotation, carrying the Clifford gates that precede it
// (in Heisenberg order), so every Clifford is fused into a rotation's pass.
#include "plan.h"

#include <algorithm>

#include "lds_tile.h"

namespace pp {

// Heisenberg maps on the (X, Y, Z) weights, rows = output letter.
unsigned gate_smask(int op) {
    auto bit = [](int r, int c) { return 1u << (3 * r + c); };
    switch (op) {
    case 0: return bit(0, 2) | bit(1, 1) | bit(2, 0);                                  // H
    case 1: return bit(0, 1) | bit(1, 0) | bit(2, 2);                                  // S
    case 3: return bit(0, 0) | bit(1, 1) | bit(1, 2) | bit(2, 1) | bit(2, 2);          // RX
    case 4: return bit(0, 0) | bit(0, 2) | bit(1, 1) | bit(2, 0) | bit(2, 2);          // RY
    default: return bit(0, 0) | bit(0, 1) | bit(1, 0) | bit(1, 1) | bit(2, 2);         // RZ
    }
}

// boolean product after * before
unsigned smask_compose(unsigned after, unsigned before) {
    unsigned out = 0;
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            bool v = false;
            for (int t = 0; t < 3; ++t)
                v = v || (((after >> (3 * r + t)) & 1u) && ((before >> (3 * t + c)) & 1u));
            if (v) out |= 1u << (3 * r + c);
        }
    return out;
}

DensePlan plan_dense(const GateList &g, int k, int low, bool compose, bool reorder) {
    PlanOptions o;
    o.compose = compose;
    o.group = compose;
    o.reorder = reorder;
    return plan_dense_opts(g, k, low, o);
}

namespace {

unsigned op_digits(const DOp &d) { return d.kind == DOP_CX ? (1u << d.a) | (1u << d.b) : (1u << d.a); }

}  // namespace

int group_shape(const DOp *m, int count, int lo) {
    if (count < 2 || count > 3 || m[0].kind != DOP_CX) return 0;
    const int dir = m[0].a == lo ? 0 : 1;
    for (int j = 1; j < count; ++j)
        if (m[j].kind != DOP_U1) return 0;
    int code;
    if (count == 2) {
        code = m[1].a == lo ? 0 : 1;
    } else {
        if ((m[1].a == lo) == (m[2].a == lo)) return 0;
        code = m[1].a == lo ? 2 : 3;
    }
    return 1 + 4 * dir + code;
}

namespace {

// A GROUP of one of the eight shapes carries the map indices of its U1
// members in its header (map: the first, reserved: the second, or the
// first again), so a sweep can load its maps as soon as it decodes the
// header.
void set_shape_maps(DOp &h, const DOp *members) {
    if (!h.perm) return;
    h.map = members[1].map;
    h.reserved = h.ngates > 2 ? members[2].map : members[1].map;
}

// Regroups a run of ops: repeatedly takes the first remaining op and every
// later op whose digits stay within one pair of digits and that does not
// share a digit with an op it would move past (ops on disjoint digits
// commute).  Groups of two or more ops get a GROUP header.
std::vector<DOp> group_ops(const std::vector<DOp> &in, int k) {
    std::vector<DOp> out;
    out.reserve(in.size() + in.size() / 2);
    std::vector<char> used(in.size(), 0);
    const unsigned all = (1u << k) - 1u;
    for (size_t i = 0; i < in.size(); ++i) {
        if (used[i]) continue;
        unsigned pair = op_digits(in[i]), skipped = 0;
        DOp mem[kMaxGroupOps];
        int count = 1;
        mem[0] = in[i];
        used[i] = 1;
        for (size_t j = i + 1; j < in.size() && count < kMaxGroupOps; ++j) {
            if (used[j]) continue;
            const unsigned d = op_digits(in[j]);
            if (d & skipped) {
                skipped |= d;
            } else if (__builtin_popcount(pair | d) <= 2) {
                pair |= d;
                mem[count++] = in[j];
                used[j] = 1;
                continue;
            } else {
                skipped |= d;
            }
            // nothing can join any more
            if (!((__builtin_popcount(pair) == 2 ? pair : all) & ~skipped)) break;
        }
        if (count > 1 && __builtin_popcount(pair) == 1) {
            if (k < 2) {  // a one-digit tile has no pair: keep the ops as they are
                out.insert(out.end(), mem, mem + count);
                continue;
            }
            pair |= 1u << (pair == 1u ? 1 : 0);  // any second digit completes the block
        }
        if (count > 1) {
            DOp h{};
            h.kind = DOP_GROUP;
            h.a = (uint8_t)__builtin_ctz(pair);
            h.b = (uint8_t)(31 - __builtin_clz(pair));
            h.ngates = (uint8_t)count;
            h.perm = (uint16_t)group_shape(mem, count, h.a);
            set_shape_maps(h, mem);
            out.push_back(h);
        }
        out.insert(out.end(), mem, mem + count);
    }
    return out;
}

// Orders the ops of a k = kSegTileDigits pass into register segments: the
// same greedy rule as group_ops with up to three digits per segment.  Each
// segment opens with a SEG header naming its digit triple (a < b < smask)
// and the number of entries that follow (GROUP headers included); inside a
// segment ops on a common digit pair are packed into GROUP ops.  A triple
// with spare digits is completed with the previous segment's digits (no
// re-layout between the two) and otherwise with digits 2..5 when the
// segment avoids digits 0 and 1 (a layout that can be loaded from and
// stored to HBM directly).
std::vector<DOp> segment_ops(const std::vector<DOp> &in, int k) {
    std::vector<DOp> out;
    std::vector<char> used(in.size(), 0);
    unsigned prev = 0;
    for (size_t i = 0; i < in.size(); ++i) {
        if (used[i]) continue;
        unsigned set = op_digits(in[i]), skipped = 0;
        std::vector<DOp> mem{in[i]};
        used[i] = 1;
        for (size_t j = i + 1; j < in.size(); ++j) {
            if (used[j]) continue;
            const unsigned d = op_digits(in[j]);
            if (d & skipped) {
                skipped |= d;
                continue;
            }
            if (__builtin_popcount(set | d) <= 3) {
                set |= d;
                mem.push_back(in[j]);
                used[j] = 1;
            } else {
                skipped |= d;
            }
        }
        if (__builtin_popcount(set | prev) == 3) set |= prev;
        const unsigned pref = (set & 3u) ? 0u : 0x3cu;
        for (int q = 0; q < k && __builtin_popcount(set) < 3; ++q)
            if ((pref >> q) & 1u) set |= 1u << q;
        for (int q = 0; q < k && __builtin_popcount(set) < 3; ++q) set |= 1u << q;
        prev = set;
        const std::vector<DOp> body = group_ops(mem, k);
        // SEG headers count at most 255 entries; a GROUP stays with its members
        size_t b = 0;
        while (b < body.size()) {
            size_t e = b;
            while (e < body.size()) {
                const size_t unit = body[e].kind == DOP_GROUP ? 1 + body[e].ngates : 1;
                if (e + unit - b > 255) break;
                e += unit;
            }
            DOp h{};
            h.kind = DOP_SEG;
            h.a = (uint8_t)__builtin_ctz(set);
            h.b = (uint8_t)__builtin_ctz(set & (set - 1));
            h.smask = (uint16_t)(31 - __builtin_clz(set));
            h.ngates = (uint8_t)(e - b);
            out.push_back(h);
            out.insert(out.end(), body.begin() + b, body.begin() + e);
            b = e;
        }
    }
    return out;
}

// Digits an op's LDS sweep covers that matter for the wave split: a lone U1
// on digit a is swept with digit a - 1 (digit 1 for a = 0), which is digit 5
// only when a is.
unsigned sweep_digits(const DOp &d) {
    return d.kind == DOP_U1 ? 1u << d.a : (1u << d.a) | (1u << d.b);
}

// Workgroup barriers between consecutive LDS ops of a pass if the waves of a
// 256-thread sweep split the tile by digit D: one is skipped only between
// two ops that both avoid D.
int split_barriers(const std::vector<DOp> &ops, int D) {
    int count = 0;
    bool have_prev = false, prev_avoids = false;
    for (size_t i = 0; i < ops.size();) {
        const DOp &d = ops[i];
        if (d.kind == DOP_SEG) {
            ++i;
            continue;
        }
        const bool avoids = !((sweep_digits(d) >> D) & 1u);
        if (have_prev && !(prev_avoids && avoids)) ++count;
        have_prev = true;
        prev_avoids = avoids;
        i += d.kind == DOP_GROUP ? 1 + d.ngates : 1;
    }
    return count;
}

// 6-digit tiles: the kernels that sweep them with 256 threads give each wave
// the quarter of the tile whose digit 5 is the wave's index and skip the
// workgroup barrier between two consecutive ops that avoid digit 5.  This
// renames the tile digits of the pass so that the digit among 2..5 that
// costs the fewest barriers becomes digit 5 (the digits above it move down
// by one; digits 0 and 1, the two lowest qubits that give the tile its
// 128-byte runs in HBM, keep their places), then marks every op after which
// the barrier can go.
void split_waves(std::vector<DOp> &ops, DensePass &ps) {
    int best = 5, best_count = split_barriers(ops, 5);
    for (int D = 2; D < 5; ++D) {
        const int c = split_barriers(ops, D);
        if (c < best_count) {
            best = D;
            best_count = c;
        }
    }
    if (best != 5) {
        uint8_t to[8];
        for (int d = 0; d < 8; ++d) to[d] = (uint8_t)(d < best ? d : (d == best ? 5 : (d <= 5 ? d - 1 : d)));
        for (size_t i = 0; i < ops.size();) {
            DOp &h = ops[i];
            if (h.kind == DOP_SEG) {
                uint8_t t[3] = {to[h.a], to[h.b], to[h.smask]};
                std::sort(t, t + 3);
                h.a = t[0];
                h.b = t[1];
                h.smask = t[2];
                ++i;
            } else if (h.kind == DOP_GROUP) {
                const uint8_t a = to[h.a], b = to[h.b];
                h.a = std::min(a, b);
                h.b = std::max(a, b);
                for (int j = 1; j <= h.ngates; ++j) {
                    DOp &m = ops[i + j];
                    m.a = to[m.a];
                    if (m.kind == DOP_CX) m.b = to[m.b];
                }
                h.perm = (uint16_t)group_shape(&ops[i + 1], h.ngates, h.a);
                set_shape_maps(h, &ops[i + 1]);
                i += 1 + h.ngates;
            } else {
                h.a = to[h.a];
                if (h.kind == DOP_CX) h.b = to[h.b];
                ++i;
            }
        }
        uint8_t q[8];
        for (int d = 0; d < ps.k; ++d) q[to[d]] = ps.qubit[d];
        for (int d = 0; d < ps.k; ++d) ps.qubit[d] = q[d];
    }
}

// Marks the barriers of a 6-digit pass (ops [begin, end)) that its sweeps can
// skip.
void tag_barriers(std::vector<DOp> &ops, size_t begin, size_t end) {
    for (size_t i = begin; i < end; ++i)
        if (ops[i].kind != DOP_SEG) ops[i].perm &= (uint16_t)~kSkipBarrier;
    DOp *prev = nullptr;
    for (size_t i = begin; i < end;) {
        DOp &d = ops[i];
        if (d.kind == DOP_SEG) {
            ++i;
            continue;
        }
        const bool avoids = !((sweep_digits(d) >> 5) & 1u);
        if (prev && avoids && !((sweep_digits(*prev) >> 5) & 1u)) prev->perm |= (uint16_t)kSkipBarrier;
        prev = &d;
        i += d.kind == DOP_GROUP ? 1 + d.ngates : 1;
    }
}

// Tiles of 7 and 6 digits run as record chains: a group becomes groups of one CX and at
// most one map per digit behind it, the lower digit's first (maps on different
// digits commute).  Then a unit (group or lone op) on digits above 1 that
// commutes with every unit before it comes first, and one that commutes with
// every unit behind it last: those two are applied between registers and HBM,
// where the 128-byte runs need digits 0 and 1 across the lanes.
// Appends the ops to `ops`; ends receives the end of every piece of at most
// kTileUnits units.
struct ChainUnit {
    int begin, count;  // its ops
    unsigned digits;
};
void chain_order(const std::vector<DOp> &in, std::vector<DOp> &ops, std::vector<int> &ends) {
    std::vector<DOp> body;
    std::vector<ChainUnit> units;
    body.reserve(in.size());
    units.reserve(in.size());
    auto open = [&] { units.push_back({(int)body.size(), 0, 0u}); };
    auto add = [&](const DOp &m) {
        body.push_back(m);
        ChainUnit &u = units.back();
        u.digits |= op_digits(m);
        if (++u.count > 1) {  // two maps: the lower digit's first
            DOp &a = body[body.size() - 2], &b = body.back();
            if (a.kind == DOP_U1 && b.kind == DOP_U1 && b.a < a.a) std::swap(a, b);
        }
    };
    for (size_t i = 0; i < in.size();) {
        open();
        if (in[i].kind != DOP_GROUP) {
            add(in[i++]);
            continue;
        }
        const DOp &head = in[i];
        bool lo = false, hi = false;
        for (int j = 1; j <= head.ngates; ++j) {
            const DOp &m = in[i + (size_t)j];
            bool &seen = m.a == head.a ? lo : hi;
            if (m.kind == DOP_CX ? units.back().count > 0 : seen) {
                open();
                lo = hi = false;
            }
            if (m.kind == DOP_U1) seen = true;
            add(m);
        }
        i += 1 + (size_t)head.ngates;
    }
    for (size_t first = 0; first < units.size(); first += kTileUnits) {
        ChainUnit *u = units.data() + first;
        const size_t count = std::min(units.size() - first, (size_t)kTileUnits);
        unsigned seen = 0;
        for (size_t i = 0; i < count; ++i) {
            if (!(u[i].digits & (3u | seen))) {
                std::rotate(u, u + i, u + i + 1);
                break;
            }
            seen |= u[i].digits;
        }
        seen = 0;
        for (size_t i = count; i-- > 1;) {  // never the first again
            if (!(u[i].digits & (3u | seen))) {
                std::rotate(u + i, u + i + 1, u + count);
                break;
            }
            seen |= u[i].digits;
        }
        for (size_t i = 0; i < count; ++i) {
            const DOp *m = body.data() + u[i].begin;
            if (u[i].count > 1) {
                DOp h{};
                h.kind = DOP_GROUP;
                h.a = (uint8_t)__builtin_ctz(u[i].digits);
                h.b = (uint8_t)(31 - __builtin_clz(u[i].digits));
                h.ngates = (uint8_t)u[i].count;
                h.perm = (uint16_t)group_shape(m, u[i].count, h.a);
                set_shape_maps(h, m);
                ops.push_back(h);
            }
            ops.insert(ops.end(), m, m + u[i].count);
        }
        ends.push_back((int)ops.size());
    }
}

void group_all(DensePlan &P, bool segments, bool chain) {
    std::vector<DOp> ops;
    std::vector<DensePass> passes;
    std::vector<int> ends;
    ops.reserve(2 * P.ops.size());
    for (DensePass &ps : P.passes) {
        const std::vector<DOp> in(P.ops.begin() + ps.op_begin, P.ops.begin() + ps.op_end);
        std::vector<DOp> out =
            (segments && !P.resident && ps.k == kSegTileDigits) ? segment_ops(in, ps.k) : group_ops(in, ps.k);
        if (!P.resident && ps.k == 6) split_waves(out, ps);
        int begin = (int)ops.size();
        ends.clear();
        if (!P.resident && chain && !out.empty()) {
            chain_order(out, ops, ends);
        } else {
            ops.insert(ops.end(), out.begin(), out.end());
            ends.push_back((int)ops.size());
        }
        for (int end : ends) {
            if (!P.resident && ps.k == 6) tag_barriers(ops, (size_t)begin, (size_t)end);
            ps.op_begin = begin;
            ps.op_end = begin = end;
            passes.push_back(ps);
            ps.ngates = 0;  // counted in the first piece
        }
    }
    P.ops = std::move(ops);
    P.passes = std::move(passes);
}

// Builds the passes of one direction over a gate list, front first.
class Scheduler {
public:
    DensePlan P;
    int64_t remaining;  // gates not scheduled

    Scheduler(const GateList &gates, int k_, int low, const PlanOptions &opts)
        : g(gates), o(opts), n(gates.n), k(k_), gb(opts.g_begin), ge(opts.g_end < 0 ? gates.m : opts.g_end) {
        remaining = m = ge - gb;
        P.roff.push_back(0);
        P.k = k;
        P.resident = k >= n;
        lowmask = low >= 32 ? 0xffffffffu : ((1u << std::min(low, n)) - 1u);
        if (!P.resident && o.reorder) build_runs();
    }

    // The only pass of a resident schedule: every gate.
    void whole() {
        DensePass pass;
        pass.k = n;
        int local[32];
        for (int q = 0; q < n; ++q) local[q] = q;
        for (int j = 0; j < n && j < 8; ++j) pass.qubit[j] = (uint8_t)j;
        sched.resize((size_t)m);
        for (int64_t h = 0; h < m; ++h) sched[(size_t)h] = h;
        emit_ops(local, n);
        pass.op_begin = 0;
        pass.op_end = (int)P.ops.size();
        pass.ngates = m;
        P.passes.push_back(pass);
    }

    // The next tiled pass; false if there is none.
    bool pass() {
        uint32_t S = lowmask;
        sched.clear();
        if (!o.reorder) {
            // keep the Heisenberg gate order: a pass is a maximal run of
            // consecutive gates whose qubits fit in k
            int64_t h = m - remaining;
            while (h < m && __builtin_popcount(S | wires(h)) <= k) {
                S |= wires(h);
                sched.push_back(h++);
            }
        }
        for (; o.reorder;) {
            absorb(
                S, head,
                [&](int q, const Run &r) {
                    sched.insert(sched.end(), one[(size_t)q].begin() + r.begin, one[(size_t)q].begin() + r.end);
                },
                [&](int64_t h) { sched.push_back(h); });
            if (__builtin_popcount(S) >= k) break;
            // grow the tile by the wires of one ready gate: the one whose
            // greedy completion of the tile schedules the most gates
            // (earliest on ties); without lookahead simply the earliest.
            // Looking only one gate ahead packed 7 % fewer gates per pass
            // into the 6-qubit tiles of random circuits.
            int64_t best = -1, best_gain = -1;
            for (int q = 0; q < n; ++q) {
                const uint32_t w = next_wires(head, q);
                if (!w || __builtin_popcount(S | w) > k) continue;
                const Run &r = wire[q][head.run[q]];
                const int64_t h = at_cx(head, q) ? r.cx : one[(size_t)q][(size_t)r.begin];
                const int64_t gain = o.lookahead ? rollout(S | w) : 0;
                if (gain > best_gain || (gain == best_gain && h < best)) {
                    best = h;
                    best_gain = gain;
                }
            }
            if (best < 0) break;
            S |= wires(best);
        }
        if (sched.empty()) return false;
        remaining -= (int64_t)sched.size();
        // pad the qubit set to exactly k qubits with the lowest unused ones
        for (int q = 0; q < n && __builtin_popcount(S) < k; ++q) S |= 1u << q;
        DensePass pass;
        pass.k = k;
        int local[32];
        int j = 0;
        for (int q = 0; q < n; ++q)
            if ((S >> q) & 1u) {
                pass.qubit[j] = (uint8_t)q;
                local[q] = j++;
            }
        pass.op_begin = (int)P.ops.size();
        emit_ops(local, k);
        pass.op_end = (int)P.ops.size();
        pass.ngates = (int64_t)sched.size();
        P.passes.push_back(pass);
        return true;
    }

    // What a scheduler of the same gates in the other direction has taken is no
    // longer there.
    void give_up(const Scheduler &other) {
        for (int q = 0; q < n; ++q) last.run[q] = (int32_t)runs[(size_t)q].size() - 1 - other.head.run[q];
        last.taken = other.head.taken;
        remaining = other.remaining;
    }

private:
    // A wire's gates in processing order, as runs of single-qubit gates with a
    // CX (or the end) behind each.
    struct Run {
        int32_t begin, end;    // in one[q]
        int32_t partner = -1;  // the CX behind it: the other wire, that wire's
        int32_t prun = 0;      // run before it, and its position
        int64_t cx = 0;
    };
    // How far each wire is: its run, and whether that run's gates are taken.
    struct Heads {
        int32_t run[32];
        uint32_t taken;
    };

    const GateList &g;
    const PlanOptions &o;
    const int n, k;
    const int64_t gb, ge;
    int64_t m;
    uint32_t lowmask;
    std::vector<std::vector<Run>> runs;
    const Run *wire[32] = {};               // runs[q]
    std::vector<std::vector<int64_t>> one;  // positions of the single-qubit gates
    Heads head{}, last{};  // last: each wire's last run, and whether its gates are gone
    std::vector<int64_t> sched;  // positions of the pass's gates, in order
    std::vector<int32_t> map_of, open, at;

    // position h in processing order <-> gate index
    size_t gate_of(int64_t h) const { return (size_t)(o.forward ? gb + h : ge - 1 - h); }

    uint32_t wires(int64_t h) const {
        const size_t gi = gate_of(h);
        uint32_t w = 1u << g.q0[gi];
        if (g.op[gi] == 2) w |= 1u << g.q1[gi];
        return w;
    }

    void build_runs() {
        runs.resize((size_t)n);
        one.resize((size_t)n);
        for (auto &r : runs) r.push_back({0, 0});
        for (int64_t h = 0; h < m; ++h) {
            const size_t gi = gate_of(h);
            const int32_t a = g.q0[gi];
            std::vector<Run> &ra = runs[(size_t)a];
            if (g.op[gi] != 2) {
                one[(size_t)a].push_back(h);
                ++ra.back().end;
                continue;
            }
            const int32_t b = g.q1[gi];
            std::vector<Run> &rb = runs[(size_t)b];
            const int32_t ia = (int32_t)ra.size() - 1, ib = (int32_t)rb.size() - 1;
            ra.back().partner = b;
            ra.back().prun = ib;
            rb.back().partner = a;
            rb.back().prun = ia;
            ra.back().cx = rb.back().cx = h;
            ra.push_back({(int32_t)one[(size_t)a].size(), (int32_t)one[(size_t)a].size()});
            rb.push_back({(int32_t)one[(size_t)b].size(), (int32_t)one[(size_t)b].size()});
        }
        for (int q = 0; q < n; ++q) {
            wire[q] = runs[(size_t)q].data();
            last.run[q] = (int32_t)runs[(size_t)q].size() - 1;
        }
    }

    // Whether nothing is left of wire q's run.
    bool at_cx(const Heads &hd, int q) const {
        const Run &r = wire[q][hd.run[q]];
        return ((hd.taken >> q) & 1u) || r.begin == r.end || (hd.run[q] == last.run[q] && ((last.taken >> q) & 1u));
    }

    // Takes every gate whose wires lie in S2 and that is next on all of them,
    // until none is; returns their number.  take_run and take_cx are told of
    // them in order.
    template <class TakeRun, class TakeCx>
    int64_t absorb(uint32_t S2, Heads &hd, TakeRun take_run, TakeCx take_cx) const {
        int64_t got = 0;
        for (bool prog = true; prog;) {
            prog = false;
            for (uint32_t left = S2; left; left &= left - 1u) {
                const int q = __builtin_ctz(left);
                for (;;) {
                    const Run &r = wire[q][hd.run[q]];
                    if (!at_cx(hd, q)) {
                        take_run(q, r);
                        got += r.end - r.begin;
                        hd.taken |= 1u << q;
                    }
                    const int t = r.partner;
                    if (hd.run[q] >= last.run[q] || !((S2 >> t) & 1u) || hd.run[t] != r.prun || !at_cx(hd, t)) break;
                    take_cx(r.cx);
                    ++got;
                    hd.run[q]++;
                    hd.run[t]++;
                    hd.taken &= ~((1u << q) | (1u << t));
                    prog = true;
                }
            }
        }
        return got;
    }
    int64_t count(uint32_t S2, Heads &hd) const {
        return absorb(S2, hd, [](int, const Run &) {}, [](int64_t) {});
    }

    // Wires of the gate next on wire q if it is next on all of them (0: none);
    // a CX is found on its lower wire.
    uint32_t next_wires(const Heads &hd, int q) const {
        if (!at_cx(hd, q)) return 1u << q;
        if (hd.run[q] >= last.run[q]) return 0u;
        const Run &r = wire[q][hd.run[q]];
        const int t = r.partner;
        if (t < q || hd.run[t] != r.prun || !at_cx(hd, t)) return 0u;
        return (1u << q) | (1u << t);
    }

    // Gates a pass would take if its qubit set started as S0 and were then
    // completed to k qubits greedily, each step adding the wires of the
    // ready gate after which the most gates become schedulable.
    int64_t rollout(uint32_t S0) const {
        Heads hd = head, h2, best = head;
        uint32_t S2 = S0;
        int64_t total = count(S2, hd);
        while (__builtin_popcount(S2) < k) {
            int64_t bg = -1;
            uint32_t bw = 0;
            for (int q = 0; q < n; ++q) {
                const uint32_t w = next_wires(hd, q);
                if (!w || __builtin_popcount(S2 | w) > k) continue;
                h2 = hd;
                const int64_t gg = count(S2 | w, h2);
                if (gg > bg) {
                    bg = gg;
                    bw = w;
                    best = h2;
                }
            }
            if (bg < 0) break;
            S2 |= bw;
            total += bg;
            hd = best;
        }
        return total;
    }

    // Ops of the gates of sched, in that order, on digits local[q]; composed
    // maps have their gates' recipes in one piece.
    void emit_ops(const int *local, int digits) {
        const int map_base = P.nmaps();
        int maps = 0;
        map_of.assign(sched.size(), -1);
        open.assign((size_t)digits, -1);
        at.clear();  // gates per map, then where its next one goes
        for (size_t i = 0; i < sched.size(); ++i) {
            const size_t gi = gate_of(sched[i]);
            const uint8_t op = g.op[gi];
            DOp d{};
            d.ngates = 1;
            if (op == 2) {
                d.kind = DOP_CX;
                d.a = (uint8_t)local[g.q0[gi]];
                d.b = (uint8_t)local[g.q1[gi]];
                open[d.a] = -1;
                open[d.b] = -1;
                P.ops.push_back(d);
                continue;
            }
            const int dg = local[g.q0[gi]];
            const bool rot = op >= 3;
            if (o.compose && open[(size_t)dg] >= 0 && P.ops[(size_t)open[(size_t)dg]].ngates < 255) {
                DOp &u = P.ops[(size_t)open[(size_t)dg]];
                u.ngates++;
                u.smask = (uint16_t)smask_compose(gate_smask(op), u.smask);
                if (rot) u.perm = 0;
                map_of[i] = (int32_t)u.map - map_base;
            } else {
                d.kind = DOP_U1;
                d.a = (uint8_t)dg;
                d.smask = (uint16_t)gate_smask(op);
                d.perm = rot ? 0 : 1;
                d.map = (uint32_t)(map_base + maps);
                map_of[i] = maps++;
                at.push_back(0);
                open[(size_t)dg] = (int32_t)P.ops.size();
                P.ops.push_back(d);
            }
            ++at[(size_t)map_of[i]];
        }
        int32_t end = (int32_t)P.rop.size();
        for (int32_t &first : at) {
            const int32_t gates = first;
            first = end;
            end += gates;
            P.roff.push_back(end);
        }
        P.rop.resize((size_t)end);
        P.rparam.resize((size_t)end);
        P.rgate.resize((size_t)end);
        for (size_t i = 0; i < sched.size(); ++i) {
            if (map_of[i] < 0) continue;
            const size_t gi = gate_of(sched[i]), r = (size_t)at[(size_t)map_of[i]]++;
            P.rop[r] = g.op[gi];
            P.rparam[r] = g.op[gi] >= 3 ? g.param[gi] : -1;
            P.rgate[r] = (int32_t)gi;
        }
    }
};

}  // namespace

DensePlan plan_dense_opts(const GateList &g, int k, int low, const PlanOptions &o) {
    Scheduler s(g, k, low, o);
    if (s.P.resident) s.whole();
    else while (s.remaining > 0 && s.pass()) {}
    if (o.group && o.compose) group_all(s.P, o.segments, o.chain);
    return std::move(s.P);
}

std::string plan_check(const DensePlan &P, int n) {
    int expect = 0;
    for (size_t p = 0; p < P.passes.size(); ++p) {
        const DensePass &ps = P.passes[p];
        if (ps.op_begin != expect || ps.op_end < ps.op_begin) return "passes do not tile the op list";
        expect = ps.op_end;
        const int k = ps.k;
        if (k < 1 || k > n || (k < n && k > 8)) return "bad tile size";
        // ascending, except that a 6-digit tile may carry any of its qubits
        // but the two lowest as digit 5
        uint64_t seen = 0;
        for (int j = 0; j < k && j < 8; ++j) {
            if (ps.qubit[j] >= n || ((seen >> ps.qubit[j]) & 1u)) return "tile qubits not distinct";
            seen |= 1ull << ps.qubit[j];
        }
        const int ordered = (!P.resident && k == 6) ? 5 : k;
        for (int j = 1; j < ordered && j < 8; ++j)
            if (ps.qubit[j] <= ps.qubit[j - 1]) return "tile qubits not ascending";
        if (ordered < k && ps.qubit[5] < ps.qubit[1]) return "a lowest qubit moved to digit 5";
        const bool segmented = ps.op_begin < ps.op_end && P.ops[ps.op_begin].kind == DOP_SEG;
        if (segmented && (P.resident || k != kSegTileDigits)) return "SEG header outside a register-tile pass";
        int seg_end = ps.op_begin;
        unsigned triple = 0;
        for (int i = ps.op_begin; i < ps.op_end; ++i) {
            const DOp &d = P.ops[i];
            if (d.kind == DOP_SEG) {
                if (!segmented || i != seg_end) return "SEG header inside a segment";
                if (!(d.a < d.b && d.b < d.smask && d.smask < k) || d.ngates < 1 || i + d.ngates >= ps.op_end)
                    return "bad SEG header";
                triple = (1u << d.a) | (1u << d.b) | (1u << d.smask);
                seg_end = i + 1 + d.ngates;
                continue;
            }
            if (segmented && i >= seg_end) return "op outside every SEG";
            if (segmented) {
                const unsigned dg = d.kind == DOP_CX ? (1u << d.a) | (1u << d.b) : (1u << d.a);
                if (d.kind != DOP_GROUP && (dg & ~triple)) return "op digit outside its SEG triple";
                if (d.kind == DOP_GROUP && i + d.ngates >= seg_end) return "GROUP crosses a SEG boundary";
            }
            if (d.kind == DOP_GROUP) {
                if (d.a == d.b || d.a >= k || d.b >= k || d.ngates < 2 || i + d.ngates >= ps.op_end)
                    return "bad GROUP header";
                for (int j = i + 1; j <= i + d.ngates; ++j) {
                    const DOp &m = P.ops[j];
                    if (m.kind == DOP_GROUP || m.kind == DOP_SEG) return "nested GROUP";
                    if (segmented && (op_digits(m) & ~triple)) return "op digit outside its SEG triple";
                    if (m.a != d.a && m.a != d.b) return "GROUP member outside its pair";
                    if (m.kind == DOP_CX && ((m.b != d.a && m.b != d.b) || m.a == m.b)) return "GROUP CX outside its pair";
                    if (m.kind == DOP_U1 && m.map >= (uint32_t)P.nmaps()) return "map index out of range";
                }
                const unsigned shape = (unsigned)group_shape(&P.ops[(size_t)i + 1], d.ngates, d.a);
                if ((d.perm & ~kSkipBarrier) != shape) return "GROUP shape tag";
                if (shape && (d.map != P.ops[(size_t)i + 2].map ||
                              d.reserved != P.ops[(size_t)i + (d.ngates > 2 ? 3 : 2)].map))
                    return "GROUP shape maps";
                i += d.ngates;
                continue;
            }
            if (d.a >= k || (d.kind == DOP_CX && (d.b >= k || d.a == d.b))) return "op digit outside the tile";
            if (d.kind == DOP_U1 && d.map >= (uint32_t)P.nmaps()) return "map index out of range";
        }
        // a skipped workgroup barrier: only in 6-digit tiled passes, between
        // two ops that both avoid digit 5, so never after a pass's last op
        // (the streaming kernel reads the tile out after that barrier)
        const DOp *prev = nullptr;
        for (int i = ps.op_begin; i < ps.op_end;) {
            const DOp &d = P.ops[i];
            if (d.kind == DOP_SEG) {
                ++i;
                continue;
            }
            if (prev && (prev->perm & kSkipBarrier) && ((sweep_digits(d) >> 5) & 1u))
                return "barrier skipped before an op on digit 5";
            if ((d.perm & kSkipBarrier) && (P.resident || k != 6 || ((sweep_digits(d) >> 5) & 1u)))
                return "barrier skipped after an op on digit 5";
            prev = &d;
            i += d.kind == DOP_GROUP ? 1 + d.ngates : 1;
        }
        if (prev && (prev->perm & kSkipBarrier)) return "barrier skipped after a pass's last op";
    }
    if (expect != (int)P.ops.size()) return "ops outside every pass";
    return "";
}

uint32_t pass_reg_entry(const DensePlan &P, const DensePass &ps) {
    if (ps.op_begin < ps.op_end && P.ops[ps.op_begin].kind == DOP_SEG) {
        const DOp &h = P.ops[ps.op_begin];
        const uint32_t t = (1u << h.a) | (1u << h.b) | (1u << h.smask);
        if (!(t & 3u)) return t;
    }
    return 0x38u;
}

bool plan_segmented(const DensePlan &P) {
    for (const DensePass &ps : P.passes)
        if (!P.resident && ps.k == kSegTileDigits && ps.op_begin < ps.op_end && P.ops[ps.op_begin].kind != DOP_SEG)
            return false;
    return true;
}

void plan_append(DensePlan &all, const DensePlan &part) {
    if (all.roff.empty()) all.roff.push_back(0);
    const int op_off = (int)all.ops.size();
    const uint32_t map_off = (uint32_t)all.nmaps();
    const int32_t rec_off = (int32_t)all.rop.size();
    for (DOp d : part.ops) {
        if (d.kind == DOP_U1) d.map += map_off;
        if (d.kind == DOP_GROUP && (d.perm & ~kSkipBarrier)) {  // a shape's map indices
            d.map += map_off;
            d.reserved += map_off;
        }
        all.ops.push_back(d);
    }
    for (size_t i = 1; i < part.roff.size(); ++i) all.roff.push_back(part.roff[i] + rec_off);
    all.rop.insert(all.rop.end(), part.rop.begin(), part.rop.end());
    all.rparam.insert(all.rparam.end(), part.rparam.begin(), part.rparam.end());
    all.rgate.insert(all.rgate.end(), part.rgate.begin(), part.rgate.end());
    for (DensePass ps : part.passes) {
        ps.op_begin += op_off;
        ps.op_end += op_off;
        all.passes.push_back(ps);
    }
    all.k = part.k;
    all.resident = part.resident;
}

void build_chain(DensePlan &P, std::vector<int> *begin, bool ends) {
    const bool tiled = !P.resident && ends;
    std::vector<int> order;  // new map index -> old
    std::vector<uint32_t> renum((size_t)P.nmaps(), 0);
    // maps are numbered pair member by pair member, the lower digit first
    auto take = [&](uint32_t old) {
        renum[old] = (uint32_t)order.size();
        order.push_back((int)old);
    };
    for (const DensePass &ps : P.passes) {
        const size_t first_rec = P.chain.size();
        if (begin) begin->push_back((int)first_rec);
        // a record that only moves the tile between its layout in HBM (pair
        // k - 2, k - 1 in registers) and LDS
        auto pass_through = [&] {
            ChainOp r{};
            const int b = ps.k - 1, a = b - 1;
            r.word = (uint32_t)(b * (b - 1) / 2 + a);
            r.map = (uint32_t)order.size();
            for (int k = 0; k < 4; ++k)
                r.read[k] = r.write[k] = (uint32_t)sw((1 + k % 2) << (2 * (k < 2 ? a : b))) * (uint32_t)sizeof(double);
            return r;
        };
        bool ends_high = false;  // the last unit's pair avoids digits 0 and 1
        for (int i = ps.op_begin; i < ps.op_end;) {
            const DOp &h = P.ops[(size_t)i];
            int lo, hi, first = i, count = 1;
            if (h.kind == DOP_GROUP) {
                lo = h.a;
                hi = h.b;
                first = i + 1;
                count = h.ngates;
            } else {
                int other = h.kind == DOP_CX ? h.b : (h.a == 0 ? 1 : h.a - 1);
                if (tiled && h.kind == DOP_U1 && h.a == 2) other = 3;  // away from digits 0 and 1
                lo = std::min<int>(h.a, other);
                hi = std::max<int>(h.a, other);
            }
            i = first + count;
            ends_high = lo >= 2;
            if (tiled && P.chain.size() == first_rec && !ends_high) P.chain.push_back(pass_through());
            // a record holds a CX and one map per digit behind it; longer
            // groups become several records (one in twelve on random circuits)
            unsigned cx = 0;
            int64_t mlo = -1, mhi = -1;
            auto flush = [&] {
                ChainOp r{};
                r.word = (uint32_t)(hi * (hi - 1) / 2 + lo) |
                         (((unsigned)(mlo >= 0) + 2 * (unsigned)(mhi >= 0)) << kChainKindShift);
                r.map = (uint32_t)order.size();
                if (mlo >= 0) take((uint32_t)mlo);
                if (mhi >= 0) take((uint32_t)mhi);
                // bits of e: x, z of the lower digit, x, z of the higher; CX
                // conjugation is (x_c, z_c ^ z_t, x_t ^ x_c, z_t), its own
                // inverse, with the sign of (X, Z) <-> -(Y, Y)
                for (int k = 0; k < 4; ++k)
                    r.read[k] = r.write[k] = (uint32_t)sw((1 + k % 2) << (2 * (k < 2 ? lo : hi))) * (uint32_t)sizeof(double);
                if (cx) {
                    const int c = cx == 1 ? 0 : 2, t = 2 - c;
                    r.read[c] ^= r.write[t];
                    r.read[t + 1] ^= r.write[c + 1];
                    r.word |= (kChainFlip6 >> 2) | (kChainFlip6 >> (cx == 1 ? 1 : 0));
                }
                P.chain.push_back(r);
                cx = 0;
                mlo = mhi = -1;
            };
            for (int j = first; j < first + count; ++j) {
                const DOp &m = P.ops[(size_t)j];
                if (m.kind == DOP_CX) {
                    if (cx || mlo >= 0 || mhi >= 0) flush();
                    cx = m.a == lo ? 1u : 2u;
                } else {
                    int64_t &slot = m.a == lo ? mlo : mhi;
                    if (slot >= 0) flush();
                    slot = m.map;
                }
            }
            flush();
        }
        if (tiled && (!ends_high || P.chain.size() < first_rec + 2)) {
            while (P.chain.size() < first_rec + 1) P.chain.push_back(pass_through());
            P.chain.push_back(pass_through());
        }
    }
    // six qubits: a wave's sweep of a pair below digit 5 stays in the quarter
    // of the tile whose digit 5 is the wave's index (lane_order)
    if (P.k == 6)
        for (size_t i = 0; i + 1 < P.chain.size(); ++i)
            if ((P.chain[i].word & 0xffu) < 10u && (P.chain[i + 1].word & 0xffu) < 10u)
                P.chain[i].word |= 1u << kChainNoBarrierBit;
    if (begin) begin->push_back((int)P.chain.size());
    P.nchain = (int)P.chain.size();
    // the recipes in the new order, and the ops' indices
    std::vector<int32_t> roff{0}, rparam, rgate;
    std::vector<uint8_t> rop;
    roff.reserve(P.roff.size());
    rop.reserve(P.rop.size());
    rparam.reserve(P.rparam.size());
    rgate.reserve(P.rgate.size());
    for (int old : order) {
        rop.insert(rop.end(), P.rop.begin() + P.roff[(size_t)old], P.rop.begin() + P.roff[(size_t)old + 1]);
        rparam.insert(rparam.end(), P.rparam.begin() + P.roff[(size_t)old], P.rparam.begin() + P.roff[(size_t)old + 1]);
        rgate.insert(rgate.end(), P.rgate.begin() + P.roff[(size_t)old], P.rgate.begin() + P.roff[(size_t)old + 1]);
        roff.push_back((int32_t)rop.size());
    }
    P.roff = std::move(roff);
    P.rop = std::move(rop);
    P.rparam = std::move(rparam);
    P.rgate = std::move(rgate);
    for (DOp &d : P.ops) {
        if (d.kind == DOP_U1) d.map = renum[d.map];
        if (d.kind == DOP_GROUP && (d.perm & ~kSkipBarrier)) {
            d.map = renum[d.map];
            d.reserved = renum[d.reserved];
        }
    }
}

void record_offsets(const ChainOp &r, const DensePass &ps, int dbytes, bool after, uint32_t out[4]) {
    int b = 1;
    while (b * (b + 1) / 2 <= (int)(r.word & 0xffu)) ++b;
    const int a = (int)(r.word & 0xffu) - b * (b - 1) / 2;
    for (int k = 0; k < 4; ++k)
        out[k] = (uint32_t)(((uint64_t)(1 + k % 2) << (2 * ps.qubit[k < 2 ? a : b])) * (uint64_t)dbytes);
    if (!after && (r.word & (kChainFlip6 >> 2))) {  // the CX's letter map, as in build_chain
        const int c = r.word & (kChainFlip6 >> 1) ? 0 : 2, t = 2 - c;
        const uint32_t w[4] = {out[0], out[1], out[2], out[3]};
        out[c] ^= w[t];
        out[t + 1] ^= w[c + 1];
    }
}

DensePlan plan_meet(const GateList &g, int k, int low, int64_t g_end, bool segments, std::vector<int> *rec) {
    const bool chains = k == g.n || chain_tiles(k, g.n, segments);
    std::vector<int> hrec, frec;
    PlanOptions o;
    o.g_end = g_end;
    o.segments = segments;
    o.chain = chains;
    PlanOptions f = o;
    f.forward = true;
    DensePlan P, F;
    if (k == g.n) {
        int64_t ncx = 0;
        for (int64_t i = 0; i < g_end; ++i) ncx += g.op[(size_t)i] == 2;
        int64_t s = ncx ? 0 : g_end / 2;
        for (int64_t seen = 0; ncx && seen < ncx / 2; ++s) seen += g.op[(size_t)s] == 2;
        o.g_begin = s;
        f.g_end = s;
        P = plan_dense_opts(g, k, low, o);
        F = plan_dense_opts(g, k, low, f);
    } else {
        // a pass from either end in turn, until they meet
        Scheduler back(g, k, low, o), front(g, k, low, f);
        for (Scheduler *s = &back, *t = &front; s->remaining > 0 && s->pass(); std::swap(s, t)) t->give_up(*s);
        group_all(back.P, o.segments, o.chain);
        group_all(front.P, f.segments, f.chain);
        P = std::move(back.P);
        F = std::move(front.P);
    }
    if (chains) build_chain(P, &hrec);
    if (chains) build_chain(F, &frec);
    const int base = P.nmaps();
    const size_t hpass = P.passes.size();
    plan_append(P, F);
    for (ChainOp r : F.chain) {
        r.map += (uint32_t)base;
        P.chain.push_back(r);
    }
    P.fwd_from = base;
    if (k == g.n) {  // the ops of both, for the self-check and the statistics
        P.passes.front().op_end = P.passes.back().op_end;
        P.passes.front().ngates += P.passes.back().ngates;
        P.passes.resize(1);
        return P;
    }
    P.fwd_pass = (int)hpass;
    if (rec && chains) {
        *rec = hrec;
        rec->pop_back();
        for (int v : frec) rec->push_back(v + P.nchain);
    }
    return P;
}

DensePlan plan_reversed_forward(const DensePlan &P) {
    DensePlan R;
    R.k = P.k;
    for (size_t p = P.passes.size(); p-- > (size_t)P.fwd_pass;) {
        DensePass ps = P.passes[p];
        const int begin = (int)R.ops.size();
        for (int i = ps.op_end; i-- > ps.op_begin;) {
            DOp d = P.ops[(size_t)i];
            if (d.kind == DOP_GROUP || d.kind == DOP_SEG) continue;
            d.perm = 0;
            R.ops.push_back(d);
        }
        ps.op_begin = begin;
        ps.op_end = (int)R.ops.size();
        R.passes.push_back(ps);
    }
    return R;
}

GradPlan plan_gradient(const GateList &g, int k_heis, int k_fwd, int low, int64_t every, bool segments) {
    GradPlan G;
    const int64_t m = g.m;
    if (every <= 0) every = m > 0 ? m : 1;
    for (int64_t b = 0; b < m; b += every) G.bounds.push_back(b);
    G.bounds.push_back(m);
    if (G.bounds.size() == 1) G.bounds.push_back(m);  // m == 0: one empty segment
    std::vector<int32_t> slot((size_t)m, -1), param_of;
    for (int64_t gi = 0; gi < m; ++gi)
        if (g.op[(size_t)gi] >= 3) {
            slot[(size_t)gi] = (int32_t)param_of.size();
            param_of.push_back(g.param[(size_t)gi]);
        }
    G.nslots = (int)param_of.size();
    G.param_off.assign((size_t)g.n_params + 1, 0);
    for (int32_t p : param_of) ++G.param_off[(size_t)p + 1];
    for (int32_t p = 0; p < g.n_params; ++p) G.param_off[(size_t)p + 1] += G.param_off[(size_t)p];
    G.param_slot.resize(param_of.size());
    {
        std::vector<int32_t> at(G.param_off.begin(), G.param_off.end() - 1);
        for (size_t j = 0; j < param_of.size(); ++j) G.param_slot[(size_t)at[(size_t)param_of[j]]++] = (int32_t)j;
    }
    G.heis.roff.push_back(0);
    G.fwd.roff.push_back(0);
    for (size_t s = 0; s + 1 < G.bounds.size(); ++s) {
        PlanOptions h;
        h.g_begin = G.bounds[s];
        h.g_end = G.bounds[s + 1];
        h.segments = segments;
        h.chain = chain_tiles(k_heis, g.n, segments);
        G.heis_pass_begin.push_back((int)G.heis.passes.size());
        plan_append(G.heis, plan_dense_opts(g, k_heis, low, h));
        PlanOptions f;
        f.forward = true;
        f.segments = false;
        f.g_begin = G.bounds[s];
        f.g_end = G.bounds[s + 1];
        G.fwd_pass_begin.push_back((int)G.fwd.passes.size());
        G.fwd_map_begin.push_back(G.fwd.nmaps());
        plan_append(G.fwd, plan_dense_opts(g, k_fwd, low, f));
    }
    G.heis_pass_begin.push_back((int)G.heis.passes.size());
    G.fwd_pass_begin.push_back((int)G.fwd.passes.size());
    G.fwd_map_begin.push_back(G.fwd.nmaps());
    build_chain(G.fwd, &G.fwd_chain_begin, false);
    for (size_t r = 0; r < G.fwd.rgate.size(); ++r) G.rslot.push_back(slot[(size_t)G.fwd.rgate[r]]);
    if (G.heis.resident || chain_tiles(k_heis, g.n, segments)) build_chain(G.heis, &G.heis_chain_begin);
    return G;
}

SparsePlan plan_sparse(const GateList &g) {
    SparsePlan P;
    const int64_t m = g.m;
    SparsePassDesc cur{};
    cur.g_begin = 0;
    cur.rot_op = -1;
    int ng = 0;
    for (int64_t h = 0; h < m; ++h) {
        const int64_t gi = m - 1 - h;
        const uint8_t op = g.op[gi];
        if (op <= 2) {
            const uint32_t b = op == 2 ? (uint32_t)g.q1[gi] : 0u;
            P.codes.push_back((uint32_t)op | ((uint32_t)g.q0[gi] << 8) | (b << 16));
            ++ng;
            continue;
        }
        cur.g_end = (int32_t)P.codes.size();
        cur.rot_op = op;
        cur.rot_q = g.q0[gi];
        cur.rot_param = g.param[gi];
        cur.ngates = ng + 1;
        P.passes.push_back(cur);
        cur = SparsePassDesc{};
        cur.g_begin = (int32_t)P.codes.size();
        cur.rot_op = -1;
        ng = 0;
    }
    if (ng > 0) {
        cur.g_end = (int32_t)P.codes.size();
        cur.rot_op = -1;
        cur.rot_q = 0;
        cur.rot_param = 0;
        cur.ngates = ng;
        P.passes.push_back(cur);
    }
    return P;
}

// ------------------------------------------------------------ Clifford frame
namespace {

// i^r X^x Z^z (Pauli operators in product form; r mod 4)
struct RawPauli {
    uint64_t x, z;
    int r;
};

RawPauli raw_mul(const RawPauli &A, const RawPauli &B) {
    // X^x1 Z^z1 X^x2 Z^z2 = (-1)^|z1 & x2| X^(x1^x2) Z^(z1^z2)
    return RawPauli{A.x ^ B.x, A.z ^ B.z, (A.r + B.r + 2 * __builtin_popcountll(A.z & B.x)) & 3};
}

// Heisenberg image of a Pauli string's bits under one Clifford code (signs
// not needed here): H swaps x_q and z_q, S^dag . S adds x_q to z_q,
// CX(a -> b) adds x_a to x_b and z_b to z_a.
void heis_bits(uint64_t &x, uint64_t &z, uint32_t code) {
    const int op = code & 0xff, a = (code >> 8) & 0xff, b = (code >> 16) & 0xff;
    const uint64_t xa = (x >> a) & 1ull, za = (z >> a) & 1ull;
    if (op == 0) {
        const uint64_t f = (xa ^ za) << a;
        x ^= f;
        z ^= f;
    } else if (op == 1) {
        z ^= xa << a;
    } else {
        x ^= xa << b;
        z ^= ((z >> b) & 1ull) << a;
    }
}

}  // namespace

FramePlan plan_frame(const GateList &g, const SparsePlan &sp) {
    const int n = g.n;
    FramePlan F;
    // rows of D: DX[j] = D X_j D^dag, DZ[j] = D Z_j D^dag; D starts as the
    // identity and becomes D g for every Clifford g processed
    std::vector<RawPauli> DX(n), DZ(n);
    for (int j = 0; j < n; ++j) {
        DX[j] = RawPauli{1ull << j, 0, 0};
        DZ[j] = RawPauli{0, 1ull << j, 0};
    }
    for (const SparsePassDesc &p : sp.passes) {
        for (int i = p.g_begin; i < p.g_end; ++i) {
            // D g G g^dag D^dag for the generators G that g moves:
            // H: X <-> Z; S: X -> iXZ; CX(c -> t): X_c -> X_c X_t, Z_t -> Z_c Z_t
            const uint32_t code = sp.codes[(size_t)i];
            const int op = code & 0xff, a = (code >> 8) & 0xff, b = (code >> 16) & 0xff;
            if (op == 0) {
                std::swap(DX[a], DZ[a]);
            } else if (op == 1) {
                RawPauli y = raw_mul(DX[a], DZ[a]);
                y.r = (y.r + 1) & 3;
                DX[a] = y;
            } else {
                DX[a] = raw_mul(DX[a], DX[b]);
                DZ[b] = raw_mul(DZ[a], DZ[b]);
            }
        }
        FramePassDesc d{};
        d.ngates = p.ngates;
        d.rot_param = -1;
        if (p.rot_op >= 3) {
            RawPauli P;
            if (p.rot_op == 3) {
                P = DX[p.rot_q];
            } else if (p.rot_op == 5) {
                P = DZ[p.rot_q];
            } else {  // Y = i X Z
                P = raw_mul(DX[p.rot_q], DZ[p.rot_q]);
                P.r = (P.r + 1) & 3;
            }
            // P = i^r X^x Z^z = i^(r - |x & z|) (Hermitian Pauli of x, z);
            // the factor is +-1 because P is Hermitian
            const int a = __builtin_popcountll(P.x & P.z) & 3;
            const int e = (P.r - a) & 3;
            d.pmask = (P.z << n) | P.x;
            d.sign = e == 0 ? 1 : -1;
            d.a = a;
            d.rot_param = p.rot_param;
        }
        F.passes.push_back(d);
    }
    // x part of the actual string D^dag S D of a stored key, bit by bit: the
    // map is linear in the key bits, so column b is the image of the b-th
    // generator (x_b for b < n, z_(b-n) above) under every code in order
    std::vector<uint64_t> colx((size_t)2 * n);
    for (int b = 0; b < 2 * n; ++b) {
        uint64_t x = b < n ? 1ull << b : 0, z = b < n ? 0 : 1ull << (b - n);
        for (uint32_t code : sp.codes) heis_bits(x, z, code);
        colx[(size_t)b] = x;
    }
    F.xrows.assign((size_t)n, 0);
    for (int j = 0; j < n; ++j)
        for (int b = 0; b < 2 * n; ++b)
            if ((colx[(size_t)b] >> j) & 1ull) F.xrows[(size_t)j] |= 1ull << b;
    return F;
}

}  // namespace pp
