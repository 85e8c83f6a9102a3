// Register-resident tile pass (rtile.hpp): the host scheduler of a fused run
// and the kernel for complex128 and complex64 states.
#include <algorithm>
#include <cstring>

#include "gates.hpp"
#include "rtile.hpp"

namespace sv {

// ---------------------------------------------------------------------------
// host: layouts and scheduling
// ---------------------------------------------------------------------------

namespace {

// Where each tile-local bit sits: reg[k] is the tile-local bit of register
// bit k, thr[i] that of thread bit i.
struct Layout {
    std::vector<int> reg, thr;
    int reg_of[kTileMaxLog], thr_of[kTileMaxLog];
    bool operator==(const Layout &o) const { return reg == o.reg && thr == o.thr; }
};

// The lowest five lane bits take tile-local bits of different residues
// modulo 5 where the register bits leave them: rt_slot then puts 32
// consecutive lanes on 32 different slots modulo 32.  Of equal residues the
// lowest bit comes first, so a load or store layout keeps the state's lowest
// index bits on lane bits.
Layout make_layout(int m, uint32_t rmask, bool block) {
    Layout L;
    std::vector<int> rest;
    for (int q = 0; q < m; ++q)
        if ((rmask >> q) & 1u)
            L.reg.push_back(q);
        else
            rest.push_back(q);
    if (block) {
        L.thr = rest;  // 2..5 first: a 64-amplitude block is 16 lanes of 4 registers
    } else {
        uint32_t seen = 0;
        std::vector<int> later;
        for (int q : rest) {
            if ((int)L.thr.size() < 5 && !((seen >> (q % 5)) & 1u)) {
                seen |= 1u << (q % 5);
                L.thr.push_back(q);
            } else {
                later.push_back(q);
            }
        }
        L.thr.insert(L.thr.end(), later.begin(), later.end());
    }
    for (int q = 0; q < kTileMaxLog; ++q)
        L.reg_of[q] = L.thr_of[q] = -1;
    for (size_t k = 0; k < L.reg.size(); ++k)
        L.reg_of[L.reg[k]] = (int)k;
    for (size_t i = 0; i < L.thr.size(); ++i)
        L.thr_of[L.thr[i]] = (int)i;
    return L;
}

// A tile-local condition split into its register and thread parts.
struct Cond {
    uint32_t rm = 0, rv = 0, tm = 0, tv = 0;
};
Cond split_cond(const Layout &L, uint32_t lm, uint32_t lv) {
    Cond c;
    for (int q = 0; q < kTileMaxLog; ++q) {
        if (!((lm >> q) & 1u))
            continue;
        const uint32_t v = (lv >> q) & 1u;
        if (L.reg_of[q] >= 0) {
            c.rm |= 1u << L.reg_of[q];
            c.rv |= v << L.reg_of[q];
        } else {
            c.tm |= 1u << L.thr_of[q];
            c.tv |= v << L.thr_of[q];
        }
    }
    return c;
}

uint32_t regs_where(int nb, uint32_t rm, uint32_t rv) {
    uint32_t s = 0;
    for (uint32_t r = 0; r < (1u << nb); ++r)
        if ((r & rm) == rv)
            s |= 1u << r;
    return s;
}

// One schedulable operation: a pair gate, a diagonal gate, or a block of
// diagonal gates.  nd: tile-local bits it mixes, dg: bits it only reads.
struct Unit {
    int first, count;
    bool phase, diag;
    int bit;
    uint32_t nd, dg;
};

struct Deferred {
    uint32_t nd = 0, dg = 0;
    bool free(const Unit &u) const { return !(u.nd & (nd | dg)) && !(u.dg & nd); }
    void add(const Unit &u) {
        nd |= u.nd;
        dg |= u.dg;
    }
};

// Units a segment's register bits are chosen by, and at most deferred from one
// segment to the next: on a state of one tile a run is the whole circuit, and
// looking through all of it for every segment took 10 s for 64,000 gates.
constexpr size_t kSegmentWindow = 1024;

// The bits that pair gates among the units mix.
uint32_t pair_bits(const std::vector<Unit> &units) {
    uint32_t b = 0;
    for (const Unit &u : units)
        b |= u.nd;
    return b;
}

// Pair gates a segment with the register bits of rmask would take; bits:
// pair_bits (once all of them are deferred, no further pair gate is free).
int taken(const std::vector<Unit> &units, uint32_t rmask, uint32_t bits) {
    Deferred d;
    int n = 0;
    for (const Unit &u : units) {
        if (d.free(u) && (u.diag || ((rmask >> u.bit) & 1u))) {
            n += u.diag ? 0 : 1;
        } else {
            d.add(u);
            if (!(bits & ~d.nd))
                break;
        }
    }
    return n;
}

// The register bits of the next segment, one at a time: the bit that lets
// the segment take the most pair gates.  allowed: bits it may choose from;
// fixed bits are kept.  Bits left over go to the highest allowed positions,
// so a layout kept for the store leaves the low bits to the lanes.
uint32_t choose_regs(const std::vector<Unit> &units, int m, int nb, uint32_t fixed, uint32_t allowed) {
    const uint32_t bits = pair_bits(units);
    uint32_t r = fixed;
    int cur = taken(units, r, bits);
    while (__builtin_popcount(r) < nb) {
        int best = -1, best_n = cur;
        for (int q = 0; q < m; ++q) {
            if (!((allowed >> q) & 1u) || ((r >> q) & 1u))
                continue;
            const int n = taken(units, r | (1u << q), bits);
            if (n > best_n) {
                best_n = n;
                best = q;
            }
        }
        if (best < 0)
            break;
        r |= 1u << best;
        cur = best_n;
    }
    for (int q = m - 1; q >= 0 && __builtin_popcount(r) < nb; --q)
        if ((allowed >> q) & 1u)
            r |= 1u << q;
    return r;
}

// Slot terms of a layout's thread bits; a thread bit beyond the tile's leads
// past the tile's slots (2^top of them).
void thread_terms(uint32_t *t, const Layout &L, uint32_t comp, int top) {
    const int tb = (int)L.thr.size();
    for (int i = 0; i < kRtMaxThreadBits; ++i)
        t[i] = (i < tb ? rt_slot(1u << L.thr[i]) : 1u << (top + i - tb)) * comp;
}

RtIO make_io(const TileMap &tm, const Layout &L, uint32_t comp, int top) {
    RtIO io;
    memset(&io, 0, sizeof(io));
    auto global = [&](int q) { return (uint8_t)(q < (int)tm.a ? q : (int)tm.hpos[q - (int)tm.a]); };
    for (size_t i = 0; i < L.thr.size(); ++i)
        io.tq[i] = global(L.thr[i]);
    thread_terms(io.slot, L, comp, top);
    for (size_t k = 0; k < L.reg.size(); ++k)
        io.rq[k] = global(L.reg[k]);
    return io;
}

// comp: bytes of a component; dual: a further register bit tells psi and
// lambda apart
RtOp exchange_op(const Layout &from, const Layout &to, uint32_t comp, int m, bool dual) {
    RtOp o;
    memset(&o, 0, sizeof(o));
    o.w[0] = kRtExch * 8;
    o.w[5] = rt_jump(kRtEntryExch);
    static const int at[kRtMaxNB] = {2, 3, 4, 6, 7};
    thread_terms(o.t, to, comp, dual ? m + 1 : m);
    for (size_t k = 0; k < to.reg.size(); ++k) {
        o.w[at[k]] = rt_slot(1u << from.reg[k]) * comp;
        o.w[8 + k] = rt_slot(1u << to.reg[k]) * comp;
    }
    if (dual)
        o.w[at[to.reg.size()]] = o.w[8 + to.reg.size()] = (1u << m) * comp;
    return o;
}

void set_matrix(RtOp &o, int tile_dt, const double *m) {
    for (int k = 0; k < 8; ++k)
        if (tile_dt == SV_C128)
            o.m[k] = m[k];
        else
            o.f[k] = (float)m[k];
}

} // namespace

RtGateInfo rt_gate_info(int kind, bool from_param, const double *m, bool diag) {
    RtGateInfo g;
    const int k = kind & ~SV_G_ADJOINT;
    g.kind = kRtGen;
    g.unit_a = 0;
    g.grad = kRtNoGrad;
    g.sign = 1;
    g.slot = -1;
    if (diag) {
        g.kind = kRtDiag;
        g.unit_a = k == SV_G_P || k == SV_G_Z || (!from_param && m[0] == 1.0 && m[1] == 0.0);
    } else if (from_param) {
        g.kind = k == SV_G_RX ? kRtCross : kRtReal;  // RY is real; the other kinds are diagonal
    } else {
        const bool real = m[1] == 0.0 && m[3] == 0.0 && m[5] == 0.0 && m[7] == 0.0;
        if (real && m[0] == 0.0 && m[2] == 1.0 && m[4] == 1.0 && m[6] == 0.0)
            g.kind = kRtSwap;
        else if (real)
            g.kind = kRtReal;
        else if (m[1] == 0.0 && m[7] == 0.0 && m[2] == 0.0 && m[4] == 0.0)
            g.kind = kRtCross;
    }
    return g;
}

RtPass build_rt_pass(const TileMap &tm, uint64_t fixed_mask, int tile_dt, const TileGate *t, int count,
                     RtGateInfo *info, const std::vector<SweepPat> &pats, int nb, int coal, bool block, bool dual,
                     RtProgram &prog, double *slow) {
    *slow = 0.0;
    // nr: register bits of the layouts; nb: with the bit telling psi and lambda apart
    const int m = (int)tm.m, nr = nb - (dual ? 1 : 0);
    RtPass pass;
    memset(&pass, 0, sizeof(pass));
    pass.nb = (uint32_t)nb;
    pass.first = (uint32_t)prog.ops.size();
    pass.acc_first = (uint32_t)prog.acc.size();
    auto outer_mask = [&](int k) { return t[k].diag ? t[k].o_mask : t[k].hi_mask; };
    auto outer_vals = [&](int k) { return t[k].diag ? t[k].o_vals : t[k].hi_vals; };
    for (int k = 0; k < count; ++k)
        if (!(outer_mask(k) & ~fixed_mask))
            pass.always = 1;
    std::vector<Unit> units;
    for (int k = 0; k < count;) {
        Unit u;
        u.first = k;
        u.count = 1;
        u.phase = t[k].diag && t[k].sweep_phase && m >= 7;  // narrower runs have no phase patterns
        if (u.phase)
            u.count = std::max(1, (int)t[k].sweep_len);
        u.diag = info[k].kind == kRtDiag;
        u.bit = t[k].l_target;
        u.nd = u.dg = 0;
        for (int q = k; q < k + u.count; ++q) {
            u.dg |= t[q].l_mask;
            if (t[q].l_target >= 0)
                (u.diag ? u.dg : u.nd) |= 1u << t[q].l_target;
        }
        units.push_back(u);
        k += u.count;
    }
    const uint32_t comp = tile_dt == SV_C128 ? 8 : 4;
    size_t lds = 16;

    // phase patterns as a preparation and the multiplications by its factors
    struct Part {
        Cond c;
        RtPat p;
    };
    auto put_pats = [&](const std::vector<Part> &v) {
        for (const Part &a : v)
            prog.pats.push_back(a.p);
    };
    auto prepare = [&](size_t np, size_t r_first, size_t r_count) {
        RtOp o;
        memset(&o, 0, sizeof(o));
        o.w[0] = kRtPrep * 8;
        o.w[1] = (uint32_t)np;
        o.w[2] = (uint32_t)prog.pats.size();
        o.w[3] = (uint32_t)r_first;
        o.w[4] = (uint32_t)r_count;
        prog.ops.push_back(o);
        lds = std::max(lds, np * sizeof(RtPat) + ((size_t)16 << nb));
    };
    auto factor = [&](uint32_t regs, size_t first, size_t cnt, uint32_t reg) {
        RtOp f;
        memset(&f, 0, sizeof(f));
        f.w[0] = kRtFactor * 8;
        f.w[1] = regs;
        f.w[5] = rt_jump(kRtEntryMul);
        f.w[12] = (uint32_t)first;
        f.w[13] = (uint32_t)cnt;
        f.w[14] = reg;
        prog.ops.push_back(f);
    };
    auto emit_phases = [&](const Part *parts, size_t np) {
        std::vector<Part> ts, rs, xs;
        for (size_t i = 0; i < np; ++i) {
            const Part &a = parts[i];
            (!a.c.rm ? ts : !a.c.tm ? rs : xs).push_back(a);
        }
        for (Part &a : rs) {
            a.p.cm = a.c.rm;
            a.p.cv = a.c.rv;
        }
        std::stable_sort(xs.begin(), xs.end(), [](const Part &a, const Part &b) {
            return a.c.rm != b.c.rm ? a.c.rm < b.c.rm : a.c.rv < b.c.rv;
        });
        prepare(np, ts.size(), rs.size());
        put_pats(ts);
        put_pats(rs);
        put_pats(xs);
        if (!ts.empty())
            factor(regs_where(nb, 0, 0), 0, ts.size(), 0);
        if (!rs.empty()) {
            RtOp f;
            memset(&f, 0, sizeof(f));
            f.w[0] = kRtTable * 8;
            f.w[5] = rt_jump(kRtEntryTab);
            prog.ops.push_back(f);
        }
        for (size_t i = 0; i < xs.size();) {
            size_t e = i;
            while (e < xs.size() && xs[e].c.rm == xs[i].c.rm && xs[e].c.rv == xs[i].c.rv)
                ++e;
            factor(regs_where(nb, xs[i].c.rm, xs[i].c.rv), ts.size() + rs.size() + i, e - i, 0);
            i = e;
        }
    };
    // complex64: one factor per amplitude.  Phases under one register bit and
    // thread bits come as a factor per register bit (one asked to be 0 adds
    // its phase to every register and takes it off where the bit is 1); a
    // block with phases under several register bits and thread bits sums all
    // of its phases once for each set of registers that they do not tell apart.
    auto emit_block = [&](const Part *parts, size_t np) {
        std::vector<Part> ts, rs, xs[kRtMaxNB];
        bool split = true, bits = false;
        for (size_t i = 0; i < np; ++i) {
            Part a = parts[i];
            if (!a.c.rm) {
                ts.push_back(a);
            } else if (!a.c.tm) {
                a.p.cm = a.c.rm;
                a.p.cv = a.c.rv;
                rs.push_back(a);
            } else {
                split &= !(a.c.rm & (a.c.rm - 1));
                if (!a.c.rv) {
                    ts.push_back(a);
                    a.p.count |= kRtPatNegative;
                }
                xs[__builtin_ctz(a.c.rm)].push_back(a);
                bits = true;
            }
        }
        if (!split) {
            std::vector<Part> all(parts, parts + np);
            for (Part &a : all) {
                a.p.cm |= a.c.rm << kRtRegBit;
                a.p.cv |= a.c.rv << kRtRegBit;
            }
            prepare(np, 0, 0);
            put_pats(all);
            uint32_t todo = regs_where(nb, 0, 0);
            while (todo) {
                const uint32_t r = (uint32_t)__builtin_ctz(todo);
                uint32_t same = todo;
                bool any = false;
                for (size_t i = 0; i < np; ++i) {
                    const uint32_t in = regs_where(nb, parts[i].c.rm, parts[i].c.rv);
                    same &= (in >> r) & 1u ? in : ~in;
                    any |= (in >> r) & 1u;
                }
                if (any) {
                    factor(same, 0, np, r);
                    *slow += 8.0 * (double)np + 60.0;  // a pattern's test and addition; sine, cosine, decoding
                }
                todo &= ~same;
            }
            return;
        }
        // all under one register bit (a QFT's target): the others keep their
        // amplitudes
        uint32_t one = parts[0].c.rm & parts[0].c.rv;
        for (size_t i = 1; i < np; ++i)
            one &= parts[i].c.rm & parts[i].c.rv;
        if (one & (one - 1))
            one = 0;
        if (one) {
            const int k = __builtin_ctz(one);
            for (size_t i = rs.size(); i-- > 0;)
                if (rs[i].c.rm == one) {  // no other register bit: a phase of the lane
                    rs[i].p.cm = rs[i].p.cv = 0;
                    xs[k].push_back(rs[i]);
                    rs.erase(rs.begin() + (long)i);
                }
        }
        size_t count = ts.size() + rs.size();
        for (const std::vector<Part> &x : xs)
            count += x.size();
        prepare(count, ts.size(), rs.size());
        put_pats(ts);
        put_pats(rs);
        if (one && rs.empty()) {
            const std::vector<Part> &x = xs[__builtin_ctz(one)];
            put_pats(x);
            factor(regs_where(nb, one, one), 0, x.size(), 0);
            return;
        }
        if (rs.empty() && !bits) {
            factor(regs_where(nb, 0, 0), 0, ts.size(), 0);
            return;
        }
        RtOp f;
        memset(&f, 0, sizeof(f));
        f.w[0] = kRtBlock * 8;
        f.w[5] = rt_jump(one             ? kRtEntryOneBit + (uint32_t)__builtin_ctz(one)
                         : !bits      ? kRtEntryTab
                         : rs.empty() ? kRtEntryBitsOnly
                                      : kRtEntryBits);
        f.w[13] = (uint32_t)ts.size();
        size_t at = ts.size() + rs.size();
        for (int k = 0; k < nb; ++k) {
            f.t[k] = (uint32_t)at;
            f.t[8 + k] = (uint32_t)xs[k].size();
            at += xs[k].size();
            put_pats(xs[k]);
        }
        prog.ops.push_back(f);
    };

    // the gradient term of parameterised gate k: over its pairs, or over the
    // amplitudes a diagonal gate multiplies (registers of psi)
    auto emit_grad = [&](int k, const Layout &L) {
        const RtGateInfo &g = info[k];
        if (g.grad == kRtNoGrad)
            return;
        const Cond c = split_cond(L, t[k].l_mask, t[k].l_vals);
        RtOp o;
        memset(&o, 0, sizeof(o));
        o.w[0] = kRtGrad * 8;
        o.w[2] = c.tm;
        o.w[3] = c.tv;
        uint64_t om = outer_mask(k), ov = outer_vals(k), ob = 0;
        const int lt = t[k].l_target;
        o.m[0] = o.m[1] = g.sign;
        if (g.grad == kRtGradRY || g.grad == kRtGradRX) {
            const int b = L.reg_of[lt];
            o.w[5] = rt_jump((g.grad == kRtGradRY ? kRtEntryGradY : kRtEntryGradX) + (uint32_t)b);
            for (uint32_t p = 0; p < (1u << (nr - 1)); ++p) {
                const uint32_t i = ((p >> b) << (b + 1)) | (p & ((1u << b) - 1u));
                if ((i & c.rm) == c.rv)
                    o.w[1] |= 1u << p;
            }
        } else {
            const bool rz = g.grad == kRtGradRZ;
            o.w[5] = rt_jump(kRtEntryGradD);
            const uint32_t regs = regs_where(nr, c.rm, c.rv);
            if (lt >= 0 && L.reg_of[lt] >= 0) {
                const uint32_t one = regs_where(nr, 1u << L.reg_of[lt], 1u << L.reg_of[lt]);
                o.w[1] = rz ? regs & ~one : 0u;
                o.w[12] = regs & one;
                o.m[0] = o.m[1] = (rz ? 1.0 : 2.0) * g.sign;
            } else {
                o.w[1] = regs;
                o.m[0] = rz ? (double)g.sign : 0.0;
                o.m[1] = (rz ? -1.0 : -2.0) * g.sign;
                if (lt >= 0)
                    o.w[4] = 1u << L.thr_of[lt];
                else
                    ob = 1ull << t[k].target;
            }
        }
        o.w[6] = (uint32_t)om;
        o.w[7] = (uint32_t)(om >> 32);
        o.w[8] = (uint32_t)ov;
        o.w[9] = (uint32_t)(ov >> 32);
        o.w[10] = (uint32_t)ob;
        o.w[11] = (uint32_t)(ob >> 32);
        o.w[13] = (uint32_t)prog.acc.size() - pass.acc_first;
        prog.acc.push_back(g.slot);
        prog.ops.push_back(o);
    };

    auto emit = [&](const Unit &u, const Layout &L) {
        RtOp o;
        memset(&o, 0, sizeof(o));
        const int k = u.first;
        // conj(lambda_j) psi_j stays the same through a block of diagonal
        // gates of unit modulus, so its terms may all be taken before it
        for (int q = k; q < k + u.count; ++q)
            emit_grad(q, L);
        if (u.phase) {
            const TileGate &h = t[k];
            const uint32_t np = h.sweep_cls[3 + (m - 6)];
            std::vector<Part> parts;
            for (uint32_t i = 0; i < np; ++i) {
                const SweepPat &sp = pats[h.pat0 + i];
                Part a;
                a.c = split_cond(L, sp.lmask, sp.lvals);
                for (uint32_t f = 0; f < sp.count; f += kRtPatMembers) {
                    a.p = RtPat{a.c.tm, a.c.tv, sp.first + f, std::min(kRtPatMembers, sp.count - f)};
                    parts.push_back(a);
                }
            }
            for (size_t p0 = 0; p0 < parts.size(); p0 += kRtMaxPats)
                if (comp == 4)
                    emit_block(&parts[p0], std::min<size_t>(kRtMaxPats, parts.size() - p0));
                else
                    emit_phases(&parts[p0], std::min<size_t>(kRtMaxPats, parts.size() - p0));
            for (int q = k; q < k + u.count; ++q)
                info[q].op = info[q].op2 = -1;
            return;
        }
        const Cond c = split_cond(L, t[k].l_mask, t[k].l_vals);
        uint64_t om = outer_mask(k), ov = outer_vals(k), ob = 0;
        o.w[2] = c.tm;
        o.w[3] = c.tv;
        set_matrix(o, tile_dt, t[k].m);
        info[k].op2 = -1;
        auto put = [&]() {
            o.w[6] = (uint32_t)om;
            o.w[7] = (uint32_t)(om >> 32);
            o.w[8] = (uint32_t)ov;
            o.w[9] = (uint32_t)(ov >> 32);
            o.w[10] = (uint32_t)ob;
            o.w[11] = (uint32_t)(ob >> 32);
            prog.ops.push_back(o);
            return (int32_t)prog.ops.size() - 1;
        };
        if (u.diag) {
            o.w[0] = kRtDiag * 8;
            o.w[5] = rt_jump(kRtEntryMul);
            o.w[1] = regs_where(nb, c.rm, c.rv);
            const bool unit_a = info[k].unit_a != 0;
            const int lt = t[k].l_target;
            if (lt >= 0 && L.reg_of[lt] >= 0) {
                const uint32_t one = regs_where(nb, 1u << L.reg_of[lt], 1u << L.reg_of[lt]), regs = o.w[1];
                if (!unit_a) {  // the registers with the bit clear, as an operation of its own
                    o.w[1] = regs & ~one;
                    info[k].op2 = put();
                }
                o.w[0] = kRtDiag * 8 + 1;
                o.w[1] = regs & one;
            } else if (lt >= 0) {
                const uint32_t b = 1u << L.thr_of[lt];
                if (unit_a) {  // only the lanes with the bit set
                    o.w[2] |= b;
                    o.w[3] |= b;
                    o.w[0] = kRtDiag * 8 + 1;
                } else {
                    o.w[4] = b;
                }
            } else {  // target outside the tile
                const uint64_t b = 1ull << t[k].target;
                if (unit_a) {
                    om |= b;
                    ov |= b;
                    o.w[0] = kRtDiag * 8 + 1;
                } else {
                    ob = b;
                }
            }
        } else {
            const int b = L.reg_of[u.bit];
            o.w[0] = (uint32_t)info[k].kind * 8 + (uint32_t)b;
            for (uint32_t p = 0; p < (1u << (nb - 1)); ++p) {
                const uint32_t i = ((p >> b) << (b + 1)) | (p & ((1u << b) - 1u));
                if ((i & c.rm) == c.rv)
                    o.w[1] |= 1u << p;
            }
            o.w[5] = rt_jump(o.w[0] + (c.rm ? 0u : kRtEntryFull));
        }
        info[k].op = put();
    };

    const uint32_t all = (1u << m) - 1u;
    // load and store layouts: the low bits on lanes (complex states), or
    // bits 0 and 1 in registers and 2..5 on lanes (fixed-point blocks)
    const uint32_t io_fixed = block ? 3u : 0u;
    const uint32_t io_allowed = all & ~(block ? 63u : (1u << std::min(coal, m - nr)) - 1u);
    auto io_ok = [&](uint32_t r) { return (r & io_fixed) == io_fixed && !(r & ~(io_allowed | io_fixed)); };
    std::vector<Unit> open;  // the next units of the window, deferred ones first
    size_t ahead = 0;        // the first unit beyond it
    auto fill = [&]() {
        while (open.size() < kSegmentWindow && ahead < units.size())
            open.push_back(units[ahead++]);
    };
    fill();
    uint32_t r = choose_regs(open, m, nr, io_fixed, io_allowed);
    Layout cur = make_layout(m, r, block);
    pass.in = make_io(tm, cur, comp, dual ? m + 1 : m);
    bool exch = false;
    while (true) {
        Deferred d;
        std::vector<Unit> rest;
        auto take = [&](const Unit &u) {
            if (d.free(u) && (u.diag || ((r >> u.bit) & 1u))) {
                emit(u, cur);
            } else {
                d.add(u);
                rest.push_back(u);
            }
        };
        for (const Unit &u : open)
            take(u);
        while (rest.size() < kSegmentWindow && ahead < units.size())
            take(units[ahead++]);
        open.swap(rest);
        fill();
        if (open.empty())
            break;
        r = choose_regs(open, m, nr, 0u, all);
        // a last segment takes register bits a store layout may have, if they do
        const int npair = (int)std::count_if(open.begin(), open.end(), [](const Unit &u) { return !u.diag; });
        const uint32_t bits = pair_bits(open);
        bool last = ahead == units.size() && taken(open, r, bits) == npair;
        if (last) {
            const uint32_t rs = choose_regs(open, m, nr, io_fixed, io_allowed);
            last = taken(open, rs, bits) == npair;
            if (last)
                r = rs;
        }
        const Layout next = make_layout(m, r, last && block);
        prog.ops.push_back(exchange_op(cur, next, comp, m, dual));
        exch = true;
        cur = next;
    }
    if (!io_ok(r) || (block && !(cur == make_layout(m, r, true)))) {
        uint32_t keep = 0;
        if (!block)
            keep = r & io_allowed;
        const Layout next = make_layout(m, choose_regs({}, m, nr, io_fixed | keep, io_allowed), block);
        prog.ops.push_back(exchange_op(cur, next, comp, m, dual));
        exch = true;
        cur = next;
    }
    pass.out = make_io(tm, cur, comp, dual ? m + 1 : m);
    pass.count = (uint32_t)prog.ops.size() - pass.first;
    if (exch)
        lds = std::max(lds, ((size_t)(dual ? 2 : 1) << m) * comp);
    pass.lds = (uint32_t)((lds + 15) / 16 * 16);
    pass.acc_count = (uint32_t)prog.acc.size() - pass.acc_first;
    return pass;
}

// ---------------------------------------------------------------------------
// device
// ---------------------------------------------------------------------------

// One workgroup of 2^(m - NB) lanes per tile.  128 registers per lane keep
// four wavefronts per SIMD: four complex128 tiles of 2^12 (or complex64 tiles
// of 2^13) amplitudes per CU, so one tile's exchanges and copies overlap the
// others' arithmetic.
//
// Measured against the LDS tiles of k_tile on one MI355X (complex128 unless
// noted): 28-qubit layered circuit of 315 gates 40.1 -> 27.8 ms (16 passes of
// 1.64 ms; a read and write of the 4 GiB state takes 1.28 ms), 24-qubit
// ansatz forward 8.2 -> 3.7 ms, 29-qubit QFT in complex64 25.8 -> 9.3 ms, 200
// gates on one 12-qubit tile 194 -> 120 us.  A real gate on a resident tile
// costs about 375 cycles per tile and CU (256 of them FP64 instructions), a
// general one 630 (512), X 296; complex64 tiles 615, 1140 and 370 for twice
// the amplitudes.  Tiles of 2^13 complex128 amplitudes (512 lanes) save one
// pass of 17 on the layered circuit but run 4% slower in all, 2^11 ones 25%
// slower.
template <typename R, int NB>
__global__ __launch_bounds__(kRtMaxThreads, 4) void k_rtile(cplx_t<R> *__restrict__ psi, TileMap tm, RtPass p,
                                                            const RtOp *__restrict__ ops,
                                                            const RtPat *__restrict__ pats,
                                                            const SweepMember *__restrict__ mems,
                                                            DeviceGates gates) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const uint64_t base = expand_index<uint64_t>(tm.outer, tm.tile0 + blockIdx.x);
    if (!p.always && !tile_touched(base, gates))
        return;
    const int tb = (int)tm.m - NB;
    RtRegs<R, NB> v;
    const cplx_t<R> *src = psi + (base | rt_thread_offset(p.in, threadIdx.x, tb));
    SV_RT_FOR(1 << NB, r) {
        const cplx_t<R> a = ld_stream<R>(src + rt_reg_offset<NB>(p.in, r));
        v.x[r] = rt_own(a.x);
        v.y[r] = rt_own(a.y);
    });
    const uint32_t slot = rt_xor_terms(threadIdx.x, p.in.slot);
    rt_run<R, NB>(v, lds, slot, base, ops + p.first, p.count, pats, mems);
    cplx_t<R> *dst = psi + (base | rt_thread_offset(p.out, rt_fresh(threadIdx.x), tb));
    SV_RT_FOR(1 << NB, r) {
        cplx_t<R> a;
        a.x = rt_own(v.x[r]);
        a.y = rt_own(v.y[r]);
        st_stream<R>(dst + rt_reg_offset<NB>(p.out, r), a);
    });
}

template <typename R, int NB>
static int launch_rt(void *psi, const TileMap &tm_in, const RtPass &p, const RtDevice &d, const DeviceGates &gates,
                     hipStream_t st) {
    TileMap tm = tm_in;
    const unsigned lanes = 1u << ((int)tm.m - NB);
    for (uint64_t t0 = 0; t0 < tm.ntiles; t0 += kMaxGridBlocks) {
        tm.tile0 = t0;
        const dim3 grid((unsigned)std::min(kMaxGridBlocks, tm_in.ntiles - t0));
        hipLaunchKernelGGL((k_rtile<R, NB>), grid, dim3(lanes), p.lds, st, reinterpret_cast<cplx_t<R> *>(psi), tm, p, d.ops,
                           d.pats, gates.mm, gates);
        SV_LAUNCH_CHECK();
    }
    return SV_OK;
}

int launch_rt_pass(int dtype, void *psi, const TileMap &tm, const RtPass &p, const RtDevice &d,
                   const DeviceGates &gates, hipStream_t st) {
    if (!rt_tile_ok(dtype, (int)tm.m, false))
        return fail(SV_EINVAL, "register tiles of 2^%u amplitudes", tm.m);
    if (dtype == SV_C128)
        return p.nb == 4 ? launch_rt<double, 4>(psi, tm, p, d, gates, st)
                         : launch_rt<double, 3>(psi, tm, p, d, gates, st);
    return p.nb == 5 ? launch_rt<float, 5>(psi, tm, p, d, gates, st) : launch_rt<float, 4>(psi, tm, p, d, gates, st);
}

// The reverse sweep on register tiles: a lane holds the same amplitudes of psi
// and lambda (2^(NB-1) each), every operation un-applies its gate on both, and
// a parameterised gate's gradient term is summed over its pairs first: per
// lane in registers, then over the wavefront, into the wavefront's accumulator
// of that gate.  Each workgroup strides over the tiles and writes its
// accumulators' sums (wavefronts in index order) once at the end.  Measured
// against k_adj_tile, which kept both tiles in LDS (MI355X, complex128): the
// 24-qubit, 768-angle ansatz step 33.7 -> 19.2 ms, its sweep 28.5 -> 14.4 ms;
// what bounds it now is FP64 arithmetic on two states (tiles of 2^11
// amplitudes of each, four per CU).
__global__ __launch_bounds__(kRtMaxThreads, 4) void k_radj(double2 *__restrict__ psi, double2 *__restrict__ lam,
                                                           TileMap tm, RtPass p, const RtOp *__restrict__ ops,
                                                           const RtPat *__restrict__ pats,
                                                           const SweepMember *__restrict__ mems,
                                                           const int32_t *__restrict__ acc, DeviceGates gates,
                                                           double *__restrict__ partials, int stride) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    using R = double;
    constexpr int NB = rt_nb<R>(), H = 1 << (NB - 1);
    double *accl = reinterpret_cast<double *>(lds + p.lds);
    const uint32_t nw = blockDim.x >> 6;
    const int tb = (int)tm.m - NB + 1;
    for (uint32_t k = threadIdx.x; k < rt_acc_slots(p) * nw; k += blockDim.x)
        accl[k] = 0.0;
    __syncthreads();
    for (uint64_t t = blockIdx.x; t < tm.ntiles; t += gridDim.x) {
        const uint64_t base = expand_index<uint64_t>(tm.outer, t);
        if (!p.always && !tile_touched(base, gates))
            continue;  // uniform
        RtRegs<R, NB> v;
        const uint64_t src = base | rt_thread_offset(p.in, rt_fresh(threadIdx.x), tb);
        SV_RT_FOR(H, r) {
            const uint64_t k = src + rt_reg_offset<NB - 1>(p.in, r);
            const cplx_t<R> a = ld_stream<R>(psi + k), b = ld_stream<R>(lam + k);
            v.x[r] = rt_own(a.x);
            v.y[r] = rt_own(a.y);
            v.x[r + H] = rt_own(b.x);
            v.y[r + H] = rt_own(b.y);
        });
        const uint32_t slot = rt_xor_terms(rt_fresh(threadIdx.x), p.in.slot);
        rt_run<R, NB, true>(v, lds, slot, base, ops + p.first, p.count, pats, mems, accl, p.acc_count);
        const uint64_t dst = base | rt_thread_offset(p.out, rt_fresh(threadIdx.x), tb);
        SV_RT_FOR(H, r) {
            const uint64_t k = dst + rt_reg_offset<NB - 1>(p.out, r);
            cplx_t<R> a, b;
            a.x = rt_own(v.x[r]);
            a.y = rt_own(v.y[r]);
            b.x = rt_own(v.x[r + H]);
            b.y = rt_own(v.y[r + H]);
            st_stream<R>(psi + k, a);
            st_stream<R>(lam + k, b);
        });
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < p.acc_count; k += blockDim.x) {
        double s = 0.0;
        for (uint32_t q = 0; q < nw; ++q)
            s += accl[k * nw + q];
        partials[(size_t)acc[p.acc_first + k] * stride + blockIdx.x] = s;
    }
}

static unsigned rt_adjoint_lanes(const TileMap &tm) { return 1u << ((int)tm.m - rt_nb<double>() + 1); }

size_t rt_adjoint_lds(const TileMap &tm, const RtPass &p) {
    return p.lds + (size_t)rt_acc_slots(p) * (rt_adjoint_lanes(tm) / 64) * sizeof(double);
}

int rt_adjoint_lds_limit(size_t lds) {
    SV_HIP_TRY(hipFuncSetAttribute((const void *)k_radj, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    return SV_OK;
}

int launch_rt_adjoint(void *psi, void *lam, const TileMap &tm, const RtPass &p, const RtDevice &d,
                      const DeviceGates &gates, unsigned grid, double *partials, int stride, hipStream_t st) {
    if (!rt_tile_ok(SV_C128, (int)tm.m, true))
        return fail(SV_EINVAL, "register tiles of 2^%u amplitudes", tm.m);
    hipLaunchKernelGGL(k_radj, dim3(grid), dim3(rt_adjoint_lanes(tm)), rt_adjoint_lds(tm, p), st,
                       (double2 *)psi, (double2 *)lam, tm, p, d.ops, d.pats, gates.mm, d.acc, gates, partials, stride);
    SV_LAUNCH_CHECK();
    return SV_OK;
}

} // namespace sv
