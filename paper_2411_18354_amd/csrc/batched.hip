// Batched execution of many independent circuits of uneven width in one
// persistent launch, and their batched adjoint gradients.
//
// Every workgroup repeatedly takes the next circuit from a device work queue
// (an atomic counter; circuits ordered by decreasing cost so the longest ones
// start first) and runs it alone, so no barrier ever spans workgroups and
// every workgroup leaves the loop once the queue is empty.
//  - A circuit follows its fused plan (the same planner and register tiles as
//    single circuits, rtile.hpp; some complex64 batches LDS tiles, below): a
//    fused run visits the state tile by tile,
//    a tile being the 2^m amplitudes that share the index bits outside the
//    run's qubit set S, held in the workgroup's registers while the run's
//    operations act on it; other gates are pair loops over the state.  A
//    workgroup barrier separates passes.  A state of at most one tile is read
//    and written once per pass, mostly once in all.
//  - Small states (resident_below; on LDS tiles those of one tile) are read
//    into LDS, all gates are applied there, and written back.
// Each gate visits only the amplitude pairs whose controls hold: the pair
// index is built by inserting the target bit (0) and the control bits (their
// values) into the iteration counter, lowest position first (Sec. III-B).
#include <algorithm>
#include <atomic>
#include <cstring>
#include <numeric>
#include <string>
#include <thread>

#include "circuit.hpp"
#include "gates.hpp"
#include "pauli.hpp"
#include "rtile.hpp"
#include "tile_adj.hpp"

namespace sv {

int validate_circuit_gate(int n, int nparams, const sv_gate_t &g, int index);
int validate_unitary_gate(const sv_gate_t &g, int index);

// Workgroups of 256 lanes, four per CU (128 registers per lane),
// with the exchange buffer of the widest tile (2^12 complex128 or 2^13
// complex64 amplitudes; one component of each) before the work-item slot.
// Bound by the tiles' arithmetic once every workgroup has work; with LDS
// tiles (two workgroups of 512 lanes per CU, two barriers per operation) the
// LDS bound it.  512 circuits of widths 10-20, 100-400 gates, complex128:
// 21.9 ms with LDS tiles, 11.5 ms (10.0 with the split and helpers of today);
// 300 of widths 10-18, 100-300 gates, complex64: 1.89 and 1.04 ms; 400 of
// widths 8-12, 50-200 gates, gate by gate in LDS or on register tiles:
// complex128 0.25 and 0.16 ms, complex64 0.23 and 0.20.
constexpr int kBatchThreads = 256, kBatchThreadBits = 8;
constexpr unsigned kBatchPerCu = 4;
constexpr size_t kBatchSlot = 128;  // reduction scratch, work item and ticket
constexpr size_t kBatchExchange = 32768;
// Complex64 batches with angles, or lambda states to take gradients with, keep
// LDS tiles, 512 lanes, as a parameterised complex64 circuit alone does: a
// tile's gates in program order, one rounding per gate and amplitude.  Register
// tiles reorder commuting gates, which moves a complex64 state by
// single-precision rounding, and with it expectation values and gradients,
// which are given in double.
constexpr int kLdsThreads = 512;
__host__ __device__ constexpr int batch_threads(bool lds) { return lds ? kLdsThreads : kBatchThreads; }
// One-shot batches of states that all fit there run on the same kernel.
constexpr int kLdsTileBits = 13;  // 64 KiB of complex64: the tile, or a resident state
constexpr size_t kLdsBytes = 65536 + sizeof(double) * diag_table_doubles(kLdsTileBits);
// amplitudes per lane in flight when a tile pair is written back (tiles are
// loaded by direct HBM-to-LDS copies)
constexpr int kLdsCopy = 2;

struct BGate {
    double m[8];      // matrix of a fixed gate
    int32_t kind;     // matrix recomputed from params[param] when param >= 0
    int32_t param;    // index into the concatenated parameter array, or -1
    int32_t target;
    int32_t pad;
    uint64_t cmask, cvals;
};

// One pass of a circuit's fused plan.  The reverse sweep has two of its own:
// lambda = H psi before the others (one partial sum: the loss) and the sums
// over the partials after them; states below 2^kSweepLdsBelow amplitudes take
// one pass for the gates, with psi and lambda in LDS.
constexpr int32_t kPassGate = 0, kPassTiles = 1, kPassPauli = 2, kPassSums = 3, kPassSmall = 4;
constexpr int kSweepLdsBelow = 5;  // fewer amplitudes than a lane's registers hold
struct BPass {
    TileMap tm;       // fused: the tiles' qubit set
    RtPass rt;        // fused: the register tiles' operations
    int32_t kind;     // kPassTiles: tile descriptors [first, first + count); kPassGate: gate `gate`; ..
    int32_t gate;     // single: index among the circuit's gates
    int32_t first, count;
    // adjoint: gradient sums the pass leaves per chunk, chunk k's at
    // part + k * nacc in the batch's partial sums
    int32_t nacc;
    int64_t part;
    // circuits split over several workgroups: the pass's chunks are tickets
    // [chunk0, chunk0 + nchunks) of the circuit, each chunk_len tiles (fused)
    // or pairs (single gate)
    int32_t chunk0, nchunks;
    uint64_t chunk_len;
};

// A parameterised gate inside a fused run: its descriptor's matrix (and
// phases) is recomputed from the angle before each batched run.
struct BTileJob {
    int32_t kind, param, tile;
    int32_t op[2];    // the operations holding its matrix, or -1
};

struct BCirc {
    void *psi;
    void *lam;           // adjoint only
    int32_t n;
    int32_t first_pass, npasses;  // the fused plan (adjoint: of the reverse sweep)
    int32_t first_gate;  // gates [first_gate, first_gate + ngates), in program order
    int32_t ngates;
    int32_t first_param, nparams;  // adjoint: gradient slots
    int32_t first_term, nterms;    // adjoint: Hamiltonian terms
    int32_t first_gen;             // adjoint: first generator
    int32_t first_slot, nslots;    // adjoint: partial sums, grouped by parameter, the loss last
    int32_t first_csr;             // adjoint: each parameter's range among them
    int32_t group;       // >= 0 when split over workgroups (its ticket counters)
    int32_t nchunks;     // split: tickets over all passes
};

// Adjoint: a gate's gradient term (or the loss) as `count` partial sums at
// first, first + stride, ...
struct BSlot {
    int64_t first;
    int32_t stride, count;
};

// Insert the target bit (0) and the control bits (their values) into x,
// lowest position first.  I: uint32_t when every index fits 32 bits.
template <typename I> __device__ __forceinline__ I insert_bits(I x, I positions, I vals) {
    while (positions) {
        const int p = sizeof(I) == 8 ? __builtin_ctzll((uint64_t)positions) : __builtin_ctz((uint32_t)positions);
        positions &= positions - 1;
        const I lo = x & (((I)1 << p) - 1);
        x = ((x >> p) << (p + 1)) | (((vals >> p) & (I)1) << p) | lo;
    }
    return x;
}

// The gate's matrix (angle from params when parameterised), or its conjugate
// transpose for the reverse sweep.
template <typename R>
__device__ __forceinline__ Mat2<R> bgate_mat(const BGate &g, const double *params, bool adjoint) {
    double m[8];
    if (g.param >= 0)
        gate_matrix(g.kind, params[g.param], nullptr, m);
    else
        for (int k = 0; k < 8; ++k)
            m[k] = g.m[k];
    if (adjoint)
        return Mat2<R>{(R)m[0], (R)-m[1], (R)m[4], (R)-m[5], (R)m[2], (R)-m[3], (R)m[6], (R)-m[7]};
    return Mat2<R>{(R)m[0], (R)m[1], (R)m[2], (R)m[3], (R)m[4], (R)m[5], (R)m[6], (R)m[7]};
}

constexpr int kBatchPairUnroll = 4;  // pairs per lane per step of a pair loop

// Apply one gate (target, controls) to amplitudes held at base[0 .. 2^nbits)
// (LDS or global), controls below nbits enumerated, controls at or above
// nbits already known to hold: the iteration indices [lo, min(hi, pairs)).
template <typename R, typename I, int THREADS>
__device__ __forceinline__ void gate_on_block_i(cplx_t<R> *base, int nbits, int target, uint64_t cmask,
                                                uint64_t cvals, const Mat2<R> &mm, uint64_t lo, uint64_t hi) {
    const uint64_t lowm = (nbits >= 64) ? ~0ull : ((1ull << nbits) - 1);
    const I cm = (I)(cmask & lowm);
    const I pos = cm | ((I)1 << target);
    const uint64_t all = 1ull << (nbits - 1 - __popcll((uint64_t)cm));
    const I npairs = (I)(hi < all ? hi : all);
    const I st = (I)1 << target;
    const I cv = (I)(cvals & cm);
    constexpr int U = kBatchPairUnroll;  // 2U loads in flight
    for (I i0 = (I)lo + threadIdx.x; i0 < npairs; i0 += (I)U * THREADS) {
        cplx_t<R> x[U], y[U];
        I p1[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const I i = i0 + (I)u * THREADS;
            p1[u] = insert_bits<I>(i, pos, cv);
            if (i < npairs) {
                x[u] = base[p1[u]];
                y[u] = base[p1[u] | st];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + (I)u * THREADS < npairs) {
                apply_pair<R>(mm, x[u], y[u]);
                base[p1[u]] = x[u];
                base[p1[u] | st] = y[u];
            }
        }
    }
}

// 32-bit index arithmetic whenever the block's indices fit (always for LDS
// tiles; for global memory up to n = 32).
template <typename R, int THREADS>
__device__ __forceinline__ void gate_on_block(cplx_t<R> *base, int nbits, int target, uint64_t cmask, uint64_t cvals,
                                              const Mat2<R> &mm, uint64_t lo, uint64_t hi) {
    if (nbits <= 32)
        gate_on_block_i<R, uint32_t, THREADS>(base, nbits, target, cmask, cvals, mm, lo, hi);
    else
        gate_on_block_i<R, uint64_t, THREADS>(base, nbits, target, cmask, cvals, mm, lo, hi);
}

// A split circuit's words: the next ticket, the chunks completed, and whether
// a wait has given up.
constexpr int kGroupWords = 3;

// Device tables of a run.
struct BatchTables {
    const BCirc *circs;
    const BGate *gates;
    const BPass *passes;
    const TileGate *tiles;
    const RtOp *ops;
    const RtPat *pats;
    const SweepPat *lpats;  // LDS tiles: phase patterns
    const SweepMember *mems;
    const double *params;
    unsigned int *gstate;  // split circuits: kGroupWords each
    uint64_t limit;        // clock ticks a wait may see no chunk completed
    unsigned int *err;     // counts waits that did
    double *part;          // adjoint: partial sums
};
// The adjoint's others.
struct SweepTables {
    const DTerm *terms;
    const double *gens;
    const int32_t *gen_of;
    const int32_t *tslot;  // LDS tiles: generator of every tile descriptor, or -1
    const BSlot *slots;
    const int32_t *csr;
    double *grad, *loss;
    uint64_t *stamps;      // start and end clock of every circuit, or none
};

// Tiles [lo, hi) of a fused pass over the state in global memory.
template <typename R>
__device__ __forceinline__ void fused_tiles(cplx_t<R> *psi, const BPass &p, const BatchTables &d, unsigned char *lds,
                                            uint64_t lo, uint64_t hi) {
    constexpr int NB = rt_nb<R>();
    const DeviceGates dg{d.tiles + p.first, p.count};
    const int tb = (int)p.tm.m - NB;
    for (uint64_t tt = lo; tt < hi; ++tt) {
        const uint64_t base = expand_index<uint64_t>(p.tm.outer, tt);
        if (!p.rt.always && !tile_touched(base, dg))
            continue;  // uniform
        RtRegs<R, NB> v;
        const uint32_t tid = rt_fresh(threadIdx.x);
        const bool in = (tid >> tb) == 0;
        const cplx_t<R> *src = psi + (base | rt_thread_offset(p.rt.in, in ? tid : 0u, tb));
        SV_RT_FOR(1 << NB, r) {
            const cplx_t<R> a = src[rt_reg_offset<NB>(p.rt.in, r)];
            v.x[r] = rt_own(a.x);
            v.y[r] = rt_own(a.y);
        });
        rt_run<R, NB, false, true>(v, lds, rt_xor_terms(tid, p.rt.in.slot), base, d.ops + p.rt.first, p.rt.count,
                                   d.pats, d.mems, nullptr, 0, tb);
        const uint32_t tod = rt_fresh(threadIdx.x);
        if ((tod >> tb) == 0) {
            cplx_t<R> *dst = psi + (base | rt_thread_offset(p.rt.out, tod, tb));
            SV_RT_FOR(1 << NB, r) {
                cplx_t<R> a;
                a.x = rt_own(v.x[r]);
                a.y = rt_own(v.y[r]);
                dst[rt_reg_offset<NB>(p.rt.out, r)] = a;
            });
        }
    }
}

// The same on LDS tiles.
template <typename R>
__device__ __forceinline__ void lds_tiles(cplx_t<R> *psi, const BPass &p, const BatchTables &d, unsigned char *buf,
                                          uint64_t lo, uint64_t hi) {
    const DeviceGates dg{d.tiles + p.first, p.count, d.lpats, d.mems};
    cplx_t<R> *lds = reinterpret_cast<cplx_t<R> *>(buf);
    const uint32_t T = 1u << p.tm.m;
    for (uint64_t tt = lo; tt < hi; ++tt) {
        const uint64_t base = expand_index<uint64_t>(p.tm.outer, tt);
        if (!tile_touched(base, dg))
            continue;  // uniform
        tile_load_dma<R, kLdsThreads>(lds, psi, base, p.tm, T);
        __syncthreads();
        tile_run<R, kLdsThreads, false>(lds, base, p.tm, dg);  // at its register limit
        tile_store<R, kLdsThreads, false, 1>(psi, lds, base, p.tm, T);
        __syncthreads();
    }
}

// States held in LDS for the whole circuit, gate by gate, rather than on
// register tiles: those a wavefront's registers would hold many times over.
// Above that register tiles win however few of their lanes have amplitudes,
// as most operations need no barrier.  Ansatz circuits of three layers, LDS
// against register tiles, 32 and 600 at once: complex128 n=5 61 and 79 us
// against 53 and 70, n=8 89 and 119 against 56 and 74, n=9 101 and 143 against
// 59 and 75; complex64 n=6 71 and 92 against 74 and 95, n=8 90 and 120 against
// 66 and 91, n=10 112 and 160 against 70 and 92.
// A plan costs the host about 1.5 us a gate on one thread, though, where a
// resident state needs none: 400 circuits of 8 to 12 qubits and 150 gates take
// 0.16 ms on register tiles and 0.25 in LDS, and their plan 7 ms on 16 threads.
// So kept batches plan them, which about a hundred runs earn back, and one-shot
// batches, which would plan at every call (9.0 ms instead of 1.2), do not: on
// the LDS kernel where every state fits it, else up to the exchange buffer's
// 32 KiB.
constexpr int resident_below(bool dbl, bool once) { return once ? (dbl ? 12 : 13) : dbl ? 5 : 7; }

template <typename R, int THREADS>
__device__ void run_circuit_resident(const BCirc &c, const BatchTables &d, unsigned char *buf) {
    cplx_t<R> *psi = reinterpret_cast<cplx_t<R> *>(c.psi);
    const uint64_t N = 1ull << c.n;
    cplx_t<R> *lds = reinterpret_cast<cplx_t<R> *>(buf);
    for (uint64_t k = threadIdx.x; k < N; k += THREADS)
        lds[k] = psi[k];
    __syncthreads();
    for (int i = 0; i < c.ngates; ++i) {
        const BGate &g = d.gates[c.first_gate + i];
        gate_on_block<R, THREADS>(lds, c.n, g.target, g.cmask, g.cvals, bgate_mat<R>(g, d.params, false), 0, ~0ull);
        __syncthreads();
    }
    for (uint64_t k = threadIdx.x; k < N; k += THREADS)
        psi[k] = lds[k];
}

// ----------------------------------------------------------------- adjoint
//
// One circuit's gradients: lambda = H psi (and the loss), the reverse sweep
// (the fused plan of the inverse circuit on register tiles holding psi and
// lambda, as the single-circuit sweep has them, and single gates as pair
// loops), then the sums.  Every chunk of a pass leaves its gradient terms as
// partial sums (per wavefront, wavefronts in index order), which the last
// pass adds in chunk and pass order: results are reproducible, and a circuit's
// passes split over workgroups exactly as in the forward run.
// Before, one workgroup of 512 or 1024 lanes took a whole circuit with both
// tiles in LDS: bound by the LDS, and by few workgroups.  Ansatz circuits of
// three layers, complex128: 160 of 15 qubits 4.71 -> 1.17 ms, 160 of 13 1.31 ->
// 0.36 ms, 4 of 15 4.39 -> 0.27 ms, 600 of 8 0.63 -> 0.12 ms.  Complex64 keeps
// its LDS tiles and gains from the split alone, forward and gradients together:
// 160 of 15 qubits (two layers) 1.88 -> 1.30 ms, 4 of 15 (four) 3.27 -> 0.62 ms,
// 4 of 8 0.25 -> 0.13 ms.

// Tiles [lo, hi) of a fused reverse pass (complex128).
__device__ __forceinline__ void sweep_tiles(double2 *psi, double2 *lam, const BPass &p, const BatchTables &d,
                                            unsigned char *lds, uint64_t lo, uint64_t hi, int chunk) {
    using R = double;
    constexpr int NB = rt_nb<R>(), H = 1 << (NB - 1), NW = kBatchThreads / 64;
    const DeviceGates dg{d.tiles + p.first, p.count};
    const int tb = (int)p.tm.m - NB + 1;
    double *accl = reinterpret_cast<double *>(lds + kBatchExchange);
    for (uint32_t k = threadIdx.x; k < rt_acc_slots(p.rt) * NW; k += kBatchThreads)
        accl[k] = 0.0;
    __syncthreads();
    for (uint64_t tt = lo; tt < hi; ++tt) {
        const uint64_t base = expand_index<uint64_t>(p.tm.outer, tt);
        if (!p.rt.always && !tile_touched(base, dg))
            continue;  // uniform
        RtRegs<R, NB> v;
        const uint32_t tid = rt_fresh(threadIdx.x);
        const uint64_t src = base | rt_thread_offset(p.rt.in, (tid >> tb) == 0 ? tid : 0u, tb);
        SV_RT_FOR(H, r) {
            const cplx_t<R> a = psi[src + rt_reg_offset<NB - 1>(p.rt.in, r)];
            v.x[r] = rt_own(a.x);
            v.y[r] = rt_own(a.y);
        });
        __builtin_amdgcn_sched_barrier(0);
        SV_RT_FOR(H, r) {
            const cplx_t<R> a = lam[src + rt_reg_offset<NB - 1>(p.rt.in, r)];
            v.x[r + H] = rt_own(a.x);
            v.y[r + H] = rt_own(a.y);
        });
        rt_run<R, NB, true, true>(v, lds, rt_xor_terms(tid, p.rt.in.slot), base, d.ops + p.rt.first, p.rt.count,
                                  d.pats, d.mems, accl, p.rt.acc_count, tb);
        const uint32_t tod = rt_fresh(threadIdx.x);
        if ((tod >> tb) == 0) {
            const uint64_t dst = base | rt_thread_offset(p.rt.out, tod, tb);
            SV_RT_FOR(H, r) {
                const uint64_t k = dst + rt_reg_offset<NB - 1>(p.rt.out, r);
                cplx_t<R> a, b;
                a.x = rt_own(v.x[r]);
                a.y = rt_own(v.y[r]);
                b.x = rt_own(v.x[r + H]);
                b.y = rt_own(v.y[r + H]);
                psi[k] = a;
                lam[k] = b;
            });
        }
    }
    __syncthreads();
    double *part = d.part + p.part + (int64_t)chunk * p.nacc;
    for (uint32_t k = threadIdx.x; k < p.rt.acc_count; k += kBatchThreads) {
        double sum = 0.0;
        for (int q = 0; q < NW; ++q)
            sum += accl[k * NW + q];
        part[k] = sum;
    }
}

// The same on LDS tiles.
template <typename R>
__device__ __forceinline__ void lds_sweep_tiles(cplx_t<R> *psi, cplx_t<R> *lam, const BPass &p, const BatchTables &d,
                                                const SweepTables &a, unsigned char *buf, uint64_t lo, uint64_t hi,
                                                int chunk) {
    const DeviceGates dg{d.tiles + p.first, p.count};
    const int32_t *gs = a.tslot + p.first;
    const uint32_t T = 1u << p.tm.m;
    cplx_t<R> *tp = reinterpret_cast<cplx_t<R> *>(buf), *tl = tp + T;
    double *accl = reinterpret_cast<double *>(tl + T);
    const int npg = adj_acc_zero(dg, gs, accl);
    for (uint64_t tt = lo; tt < hi; ++tt) {
        const uint64_t base = expand_index<uint64_t>(p.tm.outer, tt);
        if (!adj_tile_touched(base, dg))
            continue;  // uniform
        tile_load_dma<R, kLdsThreads>(tp, psi, base, p.tm, T);
        tile_load_dma<R, kLdsThreads>(tl, lam, base, p.tm, T);
        __syncthreads();
        adj_tile_run<R, kLdsThreads>(tp, tl, base, T, dg, gs, a.gens, accl);
        tile_store2<R, kLdsThreads, false, kLdsCopy>(psi, lam, tp, tl, base, p.tm, T);
        __syncthreads();
    }
    double *part = d.part + p.part + (int64_t)chunk * p.nacc;
    for (int k = threadIdx.x; k < npg; k += kLdsThreads)
        part[k] = adj_acc_sum(accl, k);
}

// One gate of the reverse sweep on the amplitudes at psi and lam (global
// memory or LDS): gradient term (when parameterised) and un-apply, the pairs
// [lo, min(hi, pairs)).  Returns the workgroup's sum of the term.
template <typename R, int THREADS>
__device__ __forceinline__ double sweep_gate(int n, const BGate &g, const double *gen, const double *params,
                                          cplx_t<R> *psi, cplx_t<R> *lam, uint64_t lo, uint64_t hi,
                                          double *scratch) {
    const Mat2<R> ud = bgate_mat<R>(g, params, true);
    const uint64_t pos = g.cmask | (1ull << g.target);
    const uint64_t all = 1ull << (n - 1 - __popcll(g.cmask));
    const uint64_t npairs = hi < all ? hi : all;
    const uint64_t st = 1ull << g.target;
    double acc = 0.0;
    for (uint64_t it = lo + threadIdx.x; it < npairs; it += THREADS) {
        const uint64_t p1 = insert_bits<uint64_t>(it, pos, g.cvals);
        cplx_t<R> x = psi[p1], y = psi[p1 | st], lx = lam[p1], ly = lam[p1 | st];
        if (gen) {
            const double xr = x.x, xi = x.y, yr = y.x, yi = y.y;
            const double axr = gen[0] * xr - gen[1] * xi + gen[2] * yr - gen[3] * yi;
            const double axi = gen[0] * xi + gen[1] * xr + gen[2] * yi + gen[3] * yr;
            const double ayr = gen[4] * xr - gen[5] * xi + gen[6] * yr - gen[7] * yi;
            const double ayi = gen[4] * xi + gen[5] * xr + gen[6] * yi + gen[7] * yr;
            acc += 2.0 * ((double)lx.x * axr + (double)lx.y * axi + (double)ly.x * ayr + (double)ly.y * ayi);
        }
        apply_pair<R>(ud, x, y);
        apply_pair<R>(ud, lx, ly);
        psi[p1] = x;
        psi[p1 | st] = y;
        lam[p1] = lx;
        lam[p1 | st] = ly;
    }
    return gen ? block_sum(acc, scratch) : 0.0;  // uniform
}

// The other passes.
template <typename R, int THREADS>
__device__ __forceinline__ void sweep_other(const BCirc &c, int ci, const BPass &p, const BGate *gates,
                                         const double *params, double *parts, SweepTables d, unsigned char *buf,
                                         double *scratch, uint64_t lo, uint64_t hi, int chunk,
                                         const unsigned int *gave_up) {
    cplx_t<R> *psi = reinterpret_cast<cplx_t<R> *>(c.psi);
    cplx_t<R> *lam = reinterpret_cast<cplx_t<R> *>(c.lam);
    const uint64_t N = 1ull << c.n;
    double *part = parts + p.part + (int64_t)chunk * p.nacc;
    const int tid = (int)threadIdx.x;
    if (p.kind == kPassGate) {
        const int gs = d.gen_of[c.first_gate + p.gate];
        const double sum = sweep_gate<R, THREADS>(c.n, gates[c.first_gate + p.gate], gs >= 0 ? d.gens + 8 * gs : nullptr,
                                         params, psi, lam, lo, hi, scratch);
        if (gs >= 0 && tid == 0)
            part[0] = sum;
    } else if (p.kind == kPassPauli) {
        if (d.stamps && chunk == 0 && tid == 0)
            d.stamps[2 * ci] = wall_clock64();
        const uint64_t end = hi < N ? hi : N;
        double lp = 0.0;
        for (uint64_t k = lo + tid; k < end; k += THREADS) {
            const cplx_t<R> at = psi[k];
            cplx_t<R> v = at;
            uint64_t X = 0;
            double ar = 0.0, ai = 0.0;
            for (int j = 0; j < c.nterms; ++j) {
                const DTerm T = d.terms[c.first_term + j];
                const uint64_t x = (uint64_t)T.idx;  // the term's x mask (stored in idx for the batch)
                if (x != X) {  // uniform
                    X = x;
                    v = psi[k ^ X];
                }
                double cr = 0.0, cim = 0.0;
                add_term<uint32_t>(T, k ^ X, cr, cim);
                ar += cr * (double)v.x - cim * (double)v.y;
                ai += cr * (double)v.y + cim * (double)v.x;
            }
            cplx_t<R> o;
            o.x = (R)ar;
            o.y = (R)ai;
            lam[k] = o;
            lp += (double)at.x * ar + (double)at.y * ai;
        }
        const double sum = block_sum(lp, scratch);
        if (tid == 0)
            part[0] = sum;
    } else if (p.kind == kPassSmall) {
        cplx_t<R> *tp = reinterpret_cast<cplx_t<R> *>(buf), *tl = tp + N;
        if ((uint64_t)tid < N) {
            tp[tid] = psi[tid];
            tl[tid] = lam[tid];
        }
        __syncthreads();
        for (int f = c.ngates - 1; f >= 0; --f) {
            const int gs = d.gen_of[c.first_gate + f];
            const double sum = sweep_gate<R, THREADS>(c.n, gates[c.first_gate + f], gs >= 0 ? d.gens + 8 * gs : nullptr,
                                             params, tp, tl, 0, ~0ull, scratch);
            if (gs >= 0 && tid == 0)
                part[gs - c.first_gen] = sum;
            __syncthreads();
        }
        if ((uint64_t)tid < N) {
            psi[tid] = tp[tid];
            lam[tid] = tl[tid];
        }
    } else {  // kPassSums: over the chunks, then over the gates that share a parameter
        // (NaN where a wait has given up: partial sums of half-written states
        // look like any others)
        const bool undefined = gave_up && __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int s = tid; s < c.nslots; s += THREADS) {
            const BSlot a = d.slots[c.first_slot + s];
            double *q = parts + a.first;
            double sum = 0.0;
#pragma unroll 8
            for (int k = 0; k < a.count; ++k)
                sum += q[(int64_t)k * a.stride];
            q[0] = sum;
        }
        __syncthreads();
        for (int j = tid; j <= c.nparams; j += THREADS) {
            const int s0 = d.csr[c.first_csr + j], s1 = d.csr[c.first_csr + j + 1];
            double sum = 0.0;
#pragma unroll 4
            for (int s = s0; s < s1; ++s)
                sum += parts[d.slots[c.first_slot + s].first];
            sum = undefined ? __builtin_nan("") : sum;
            if (j < c.nparams)
                d.grad[c.first_param + j] = sum;
            else
                d.loss[ci] = sum;
        }
        if (d.stamps && tid == 0)
            d.stamps[2 * ci + 1] = wall_clock64();
    }
}

// Wait (lane 0 polling, the workgroup held at a barrier) until the circuit's
// completed chunks are at least target, then make other workgroups' writes
// visible to this one.  The wait is bounded: once no chunk has completed for
// `limit` clock ticks it gives up, counts that in *err and marks the circuit
// (the results of that run are then undefined), before the workgroup counts
// any chunk it goes on to compute.
__device__ __forceinline__ void wait_count(unsigned int *done, unsigned int target, uint64_t limit,
                                           unsigned int *err) {
    if (threadIdx.x == 0) {
        unsigned int seen = __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint64_t t0 = seen < target ? wall_clock64() : 0;
        while (seen < target) {
            __builtin_amdgcn_s_sleep(2);
            const unsigned int now = __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (now != seen) {
                seen = now;
                t0 = wall_clock64();
            } else if (wall_clock64() - t0 > limit) {
                atomicAdd(err, 1u);
                __hip_atomic_store(done + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the CU's and the XCD's caches refetch
    }
    __syncthreads();
}

// A circuit's passes.  Alone (group < 0) a workgroup runs them in order, a
// barrier between.
// A circuit split over several workgroups: every workgroup that joins it
// takes chunk tickets from the circuit's counter: the chunks of all passes
// are numbered in program order, and a chunk of pass p starts once the
// circuit's completion count has reached the first ticket of p.  Chunks of
// p and later cannot complete before that, so the count then says that every
// chunk of the earlier passes is written.  The holder of the lowest unfinished
// ticket never waits, so the circuit progresses whatever the number of
// workgroups that have joined (one is enough); a workgroup that finds the
// tickets used up goes back to the work queue.  Each tile or pair is
// computed exactly as by one workgroup, so results do not depend on the
// split.  (One loop for both: the tile code is in the kernel once.)
template <typename R, bool ADJ, bool LDS>
__device__ __forceinline__ void run_circuit(int ci, const BatchTables &d, const SweepTables &a, unsigned char *buf,
                                            double *scratch, int *slot) {
    const BCirc &c = d.circs[ci];
    cplx_t<R> *psi = reinterpret_cast<cplx_t<R> *>(c.psi);
    const BPass *passes = d.passes + c.first_pass;
    const bool split = c.group >= 0;  // uniform
    unsigned int *next = d.gstate + kGroupWords * c.group, *done = next + 1;
    int pi = 0, ready = -1;
    for (;;) {
        uint64_t lo = 0, hi = ~0ull;
        int chunk = 0;  // of its pass
        if (split) {
            if (threadIdx.x == 0)
                *slot = (int)__hip_atomic_fetch_add(next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int k = __builtin_amdgcn_readfirstlane(*slot);
            __syncthreads();
            if (k >= c.nchunks)
                break;
            while (k >= passes[pi].chunk0 + passes[pi].nchunks)
                ++pi;  // tickets only grow
            if (ready != pi) {
                wait_count(done, (unsigned int)passes[pi].chunk0, d.limit, d.err);
                ready = pi;
            }
            chunk = k - passes[pi].chunk0;
            lo = (uint64_t)chunk * passes[pi].chunk_len;
            hi = lo + passes[pi].chunk_len;
        } else if (pi >= c.npasses) {
            break;
        }
        const BPass &p = passes[pi];
        if (p.kind == kPassTiles) {  // uniform
            const uint64_t end = hi < p.tm.ntiles ? hi : p.tm.ntiles;
            if constexpr (ADJ && LDS)
                lds_sweep_tiles<R>(psi, reinterpret_cast<cplx_t<R> *>(c.lam), p, d, a, buf, lo, end, chunk);
            else if constexpr (ADJ)
                sweep_tiles(psi, reinterpret_cast<double2 *>(c.lam), p, d, buf, lo, end, chunk);
            else if constexpr (LDS)
                lds_tiles<R>(psi, p, d, buf, lo, end);
            else
                fused_tiles<R>(psi, p, d, buf, lo, end);
        } else if constexpr (ADJ) {
            sweep_other<R, batch_threads(LDS)>(c, ci, p, d.gates, d.params, d.part, a, buf, scratch, lo, hi, chunk,
                                               split ? done + 1 : nullptr);
        } else {
            const BGate &g = d.gates[c.first_gate + p.gate];
            gate_on_block<R, batch_threads(LDS)>(psi, c.n, g.target, g.cmask, g.cvals,
                                                 bgate_mat<R>(g, d.params, false), lo, hi);
        }
        if (split) {
            // Publish the chunk: every wavefront waits until its own stores
            // have reached the L2 (a workgroup barrier alone does not wait
            // for them), then lane 0's device-scope release writes the L2
            // back once and counts the chunk.  (A release in every wavefront
            // writes the L2 back once for each: a 256-circuit batch of width
            // 16 ran 2.95 ms against 2.15 ms this way.)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (threadIdx.x == 0)
                __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            __syncthreads();
            ++pi;
        }
    }
}

// Angles of the parameterised gates inside fused runs, into their tile
// descriptors (matrix, and phases of diagonal ones) and register operations.
__global__ void k_batch_tile_params(const BTileJob *__restrict__ jobs, int njobs, const double *__restrict__ params,
                                    TileGate *__restrict__ tiles, SweepMember *__restrict__ mems,
                                    RtOp *__restrict__ ops) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= njobs)
        return;
    const BTileJob j = jobs[i];
    double m[8];
    gate_matrix(j.kind, params[j.param], nullptr, m);
    TileGate &t = tiles[j.tile];
    for (int k = 0; k < 8; ++k)
        t.m[k] = m[k];
    if (t.diag) {
        diag_phases(m, t.ph, &t.unit);
        for (int s = 0; s < 2; ++s)  // the phase-sweep members holding ph (forward plans)
            if (mems && t.mem[s] >= 0)
                mems[t.mem[s]].theta = t.ph[s];
    }
    if (ops)
        for (int s = 0; s < 2; ++s)
            if (j.op[s] >= 0)
                rt_set_matrix(ops[j.op[s]], m);
}

// ADJ: the adjoint gradients, else the forward run.  LDS: on LDS tiles.  tail:
// LDS bytes before the work-item slot.  resident: states of fewer qubits are
// held in LDS, gate by gate.
template <typename R, bool ADJ, bool LDS>
__global__ __launch_bounds__(batch_threads(LDS), 4) void k_batched(
    const BCirc *__restrict__ circs, const int32_t *__restrict__ items, int nitems, int nlisted,
    const BGate *__restrict__ gates, const BPass *__restrict__ passes, const TileGate *__restrict__ tiles, const RtOp *__restrict__ ops,
    const RtPat *__restrict__ pats, const SweepPat *__restrict__ lpats, const SweepMember *__restrict__ mems,
    const double *__restrict__ params, unsigned int *__restrict__ queue, unsigned int *gstate, uint64_t limit, unsigned int *err,
    uint64_t *__restrict__ stamps, double *part, SweepTables a, uint32_t tail, int resident) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    // the exchange buffer first: its addresses step by xor
    unsigned char *buf = lds_raw;
    double *scratch = reinterpret_cast<double *>(lds_raw + tail);
    int *item = reinterpret_cast<int *>(scratch + batch_threads(LDS) / 64);
    int *ticket = item + 1;
    const BatchTables d{circs, gates, passes, tiles, ops, pats, lpats, mems, params, gstate, limit, err, part};
    for (;;) {
        if (threadIdx.x == 0)
            *item = (int)atomicAdd(queue, 1u);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(*item);  // uniform: descriptors are scalar loads
        __syncthreads();
        if (it >= nitems)
            break;
        const uint64_t t0 = !ADJ && stamps ? wall_clock64() : 0;
        const int ci = items[it];  // one that is split appears once per workgroup that may join it
        if (!ADJ && circs[ci].n < resident)  // uniform
            run_circuit_resident<R, batch_threads(LDS)>(circs[ci], d, buf);
        else
            run_circuit<R, ADJ, LDS>(ci, d, a, buf, scratch, ticket);
        __syncthreads();
        if (!ADJ && stamps && it < nlisted && threadIdx.x == 0) {
            stamps[2 * it] = t0;
            stamps[2 * it + 1] = wall_clock64();
        }
    }
}

__global__ void k_zero_u32(unsigned int *p) { *p = 0u; }

__global__ void k_zero_words(unsigned int *p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count)
        p[i] = 0u;
}

// ----------------------------------------------------------------- host

// One circuit's tables, built independently of the others (so circuits can
// be planned in parallel) and concatenated afterwards.
struct CircBuild {
    BCirc bc;
    std::vector<BGate> gates;
    std::vector<BPass> passes;     // the plan (circuit-local indices; adjoint: of the reverse sweep)
    std::vector<TileGate> tiles;
    PlanRt rt;                     // register tile operations (circuit-local)
    std::vector<SweepMember> mems; // members of their phase patterns
    bool lds = false;              // LDS tiles
    int resident = 0;              // forward: states of fewer qubits have no plan
    std::vector<SweepPat> lpats;   // their phase patterns
    std::vector<int32_t> tslot;    // adjoint: gradient slot of every tile descriptor, or -1
    std::vector<BTileJob> jobs;    // tile and operation indices circuit-local
    // adjoint: per gradient slot (a parameterised gate; numbered in the order
    // of the reverse sweep), then for the loss: its parameter (circuit-local;
    // the loss: nparams) and where its partial sums are
    struct Sum {
        int32_t param, pass, acc;
    };
    std::vector<Sum> sums;
    std::vector<double> gens;      // generators of the parameterised gates
    std::vector<int32_t> gen_of;   // per gate: index into gens / 8, or -1
    std::vector<DTerm> terms;
    double cost = 0.0;
    int err = SV_OK;
    std::string msg;
};

struct BatchArgs {
    const sv_state_t *states, *lams;
    int ncirc;
    const sv_gate_t *gates;
    const int64_t *gate_off, *param_off;
    int64_t nparams_total;
    const sv_pauli_t *terms;
    const int64_t *term_off;
    bool once = false;  // run once: planning has to pay at once
};

// The fused plan of one circuit's gates (those of the reverse sweep when
// out->rt.dual) into out's passes, tiles and jobs.
static int plan_passes(int n, int dtype, const sv_gate_t *gates, int ngates, int nparams, int32_t param0, int m_cap,
                       CircBuild *out) {
    std::vector<PlanPass> pp;
    std::vector<SweepPat> pats;
    if (out->lds)  // (a reverse sweep applies diagonal gates without patterns)
        SV_TRY(circuit_plan_tiles(n, dtype, gates, ngates, nparams, m_cap, &pp, &out->tiles,
                                  out->rt.dual ? nullptr : &out->lpats, out->rt.dual ? nullptr : &out->mems));
    else
        SV_TRY(circuit_plan_tiles(n, dtype, gates, ngates, nparams, m_cap, &pp, &out->tiles, &pats, &out->mems,
                                  &out->rt));
    for (const PlanPass &q : pp) {
        BPass b;
        memset(&b, 0, sizeof(b));
        b.kind = q.fused ? kPassTiles : kPassGate;
        b.gate = q.gate;
        b.first = q.first;
        b.count = q.count;
        if (q.fused) {
            if (q.tm.m > (uint32_t)m_cap)
                return fail(SV_EINVAL, "tile width %u beyond the batch limit", q.tm.m);
            b.tm = q.tm;
            if (out->lds) {
                b.tm.tab = 1;  // the launch reserves the tables
            } else {
                if (!q.rt || q.rp.lds > kBatchExchange)
                    return fail(SV_EINVAL, "fused pass beyond the batch's register tiles");
                b.rt = q.rp;
                b.nacc = (int32_t)q.rp.acc_count;
            }
        }
        out->passes.push_back(b);
    }
    if (out->lds) {
        for (size_t t = 0; t < out->tiles.size(); ++t) {
            const sv_gate_t &g = gates[out->tiles[t].src_gate];
            if (g.param >= 0)
                out->jobs.push_back(BTileJob{g.kind, param0 + g.param, (int32_t)t, {-1, -1}});
        }
        return SV_OK;
    }
    for (const ParamJob &j : out->rt.jobs)
        if (j.tile_slot >= 0)
            out->jobs.push_back(BTileJob{j.kind, param0 + j.param, j.tile_slot, {j.op[0], j.op[1]}});
    return SV_OK;
}

// The reverse sweep of circuit c: its passes, generators and partial sums.
static int build_sweep(const BatchArgs &A, int c, int dtype, int m_cap, CircBuild *out) {
    BCirc &bc = out->bc;
    const int64_t g0 = A.gate_off[c], p0 = A.param_off[c];
    const int G = bc.ngates;
    // inverses in reverse order, planned like a forward circuit; a lane's
    // registers hold psi and lambda, so tiles are half as wide
    std::vector<sv_gate_t> rev(G);
    std::vector<int32_t> slot_of(G, -1);  // per gate of rev
    out->gen_of.assign(G, -1);
    for (int r = 0; r < G; ++r) {
        const sv_gate_t &g = A.gates[g0 + G - 1 - r];
        rev[r] = g;
        rev[r].kind ^= SV_G_ADJOINT;
        if (g.param < 0)
            continue;
        double a[8];
        gate_generator(g.kind, a);
        if (g.kind & SV_G_ADJOINT) {
            for (int q = 1; q < 8; q += 2)
                a[q] = -a[q];
            std::swap(a[2], a[4]);
            std::swap(a[3], a[5]);
        }
        slot_of[r] = out->gen_of[G - 1 - r] = (int32_t)out->sums.size();
        out->gens.insert(out->gens.end(), a, a + 8);
        out->sums.push_back({g.param, -1, 0});
    }
    auto extra = [&](int32_t kind, int32_t nacc) {
        BPass b;
        memset(&b, 0, sizeof(b));
        b.kind = kind;
        b.nacc = nacc;
        out->passes.push_back(b);
    };
    extra(kPassPauli, 1);
    if (G > 0 && bc.n < kSweepLdsBelow && !out->lds) {
        extra(kPassSmall, (int32_t)out->sums.size());
        for (size_t k = 0; k < out->sums.size(); ++k) {
            out->sums[k].pass = 1;
            out->sums[k].acc = (int32_t)k;
        }
    } else if (G > 0) {
        out->rt.dual = true;
        SV_TRY(plan_passes(bc.n, dtype, rev.data(), G, bc.nparams, (int32_t)p0, m_cap, out));
        out->tslot.assign(out->tiles.size(), -1);
        for (size_t pi = 1; pi < out->passes.size(); ++pi) {
            BPass &b = out->passes[pi];
            if (b.kind == kPassTiles) {
                auto place = [&](int32_t slot, int32_t k) {
                    out->sums[slot].pass = (int32_t)pi;
                    out->sums[slot].acc = k;
                };
                if (out->lds) {
                    for (int t = b.first; t < b.first + b.count; ++t) {
                        out->tslot[t] = slot_of[out->tiles[t].src_gate];
                        if (out->tslot[t] >= 0)
                            place(out->tslot[t], b.nacc++);
                    }
                    continue;
                }
                for (int32_t k = 0; k < b.nacc; ++k)
                    place(out->rt.prog.acc[b.rt.acc_first + k], k);
                continue;
            }
            const int32_t sl = slot_of[b.gate];
            b.gate = G - 1 - b.gate;  // forward index
            if (sl >= 0) {
                b.nacc = 1;
                out->sums[sl].pass = (int32_t)pi;
            }
        }
    }
    for (const CircBuild::Sum &u : out->sums)
        if (u.pass < 0)
            return fail(SV_EINVAL, "a gradient term without a pass");
    out->sums.push_back({bc.nparams, 0, 0});
    extra(kPassSums, 0);
    return SV_OK;
}

// Tables of circuit c: its gates in program order, and either the forward
// fused plan (passes, tile descriptors, parameter jobs; none when the state
// is LDS-resident) or, for the adjoint, the reverse sweep's, with generators
// and the Hamiltonian.
static int build_circuit(const BatchArgs &A, int c, int dtype, bool adjoint, CircBuild *out) {
    const sv_state_t &s = A.states[c];
    const int64_t g0 = A.gate_off[c], g1 = A.gate_off[c + 1];
    const int64_t p0 = A.param_off ? A.param_off[c] : 0, p1 = A.param_off ? A.param_off[c + 1] : 0;
    BCirc &bc = out->bc;
    memset(&bc, 0, sizeof(bc));
    bc.group = -1;
    bc.psi = s.data;
    bc.lam = adjoint ? A.lams[c].data : nullptr;
    bc.n = s.n;
    // one workgroup's LDS or registers
    const int m_cap = (out->lds ? kLdsTileBits : rt_nb_of(dtype) + kBatchThreadBits) - (adjoint ? 1 : 0);
    bc.ngates = (int32_t)(g1 - g0);
    bc.first_param = (int32_t)p0;
    bc.nparams = (int32_t)(p1 - p0);
    if (bc.ngates > 0) {
        for (int64_t i = g0; i < g1; ++i) {
            SV_TRY(validate_circuit_gate(s.n, (int)(p1 - p0), A.gates[i], (int)(i - g0)));
            if (adjoint)
                SV_TRY(validate_unitary_gate(A.gates[i], (int)(i - g0)));
        }
    }
    if (adjoint)
        SV_TRY(build_sweep(A, c, dtype, m_cap, out));
    else if (bc.ngates > 0 && s.n >= out->resident)
        SV_TRY(plan_passes(s.n, dtype, A.gates + g0, bc.ngates, (int)(p1 - p0), (int32_t)p0, m_cap, out));
    bc.npasses = (int32_t)out->passes.size();
    double work = 0.0;
    out->gates.reserve(bc.ngates);
    for (int k = 0; k < bc.ngates; ++k) {
        const sv_gate_t &g = A.gates[g0 + k];
        BGate b;
        memset(&b, 0, sizeof(b));
        if (g.param < 0)
            gate_matrix(g.kind, g.theta, g.U, b.m);
        else
            for (int q = 0; q < 8; ++q)
                b.m[q] = g.U[q];
        b.kind = g.kind;
        b.param = g.param >= 0 ? (int32_t)(p0 + g.param) : -1;
        b.target = g.target;
        b.cmask = g.ctrl_mask;
        b.cvals = g.ctrl_vals;
        out->gates.push_back(b);
        work += std::ldexp(1.0, s.n - popcount64(g.ctrl_mask));
    }
    if (adjoint) {
        const int64_t t0 = A.term_off[c], t1 = A.term_off[c + 1];
        if (t0 < 0 || t1 <= t0)
            return fail(SV_EINVAL, "needs at least one term");
        const uint64_t full = (1ull << s.n) - 1;
        bc.nterms = (int32_t)(t1 - t0);
        for (int64_t j = t0; j < t1; ++j) {
            if ((A.terms[j].x_mask | A.terms[j].z_mask) & ~full)
                return fail(SV_EINVAL, "term %lld acts on qubits >= n", (long long)(j - t0));
            DTerm d;
            d.coef = A.terms[j].coef;
            d.z = A.terms[j].z_mask;
            d.ny = popcount64(A.terms[j].x_mask & A.terms[j].z_mask) & 3;
            d.idx = (int32_t)A.terms[j].x_mask;  // x mask (n <= 31 in batches)
            out->terms.push_back(d);
        }
        work *= 2.0;
    }
    out->cost = work;
    return SV_OK;
}

struct BatchHost {
    std::vector<BCirc> circs;
    std::vector<BGate> gates;
    std::vector<BPass> passes;
    std::vector<TileGate> tiles;
    RtProgram prog;
    bool lds = false;              // LDS tiles
    int resident = 0;
    std::vector<SweepPat> lpats;
    std::vector<int32_t> tslot;
    std::vector<SweepMember> mems;
    std::vector<BTileJob> jobs;
    std::vector<BSlot> slots;
    std::vector<int32_t> csr;
    int64_t npart = 0;             // partial sums
    size_t lds_bytes = 0;          // exchange buffer or tiles, then gradient accumulators of a pass
    std::vector<int32_t> order;    // work items in queue order (each a circuit), then helpers'
    int nlisted = 0;               // the former
    int ngroups = 0;               // circuits split over workgroups
    double chunk_work = 0.0;       // amplitudes times gates (or terms) of the largest chunk
    std::vector<double> gens;
    std::vector<int32_t> gen_of;
    std::vector<DTerm> terms;
};

// A chunk wait gives up once no chunk of its circuit has completed for the
// "batch_wait_ms" knob and the time the largest chunk can take at kSlowestRate
// amplitudes times gates (terms) a second.  (A workgroup reaches 1e9 to 1e10;
// a chunk's gates and Hamiltonian terms have no bound, so it may take long.)
// Only a workgroup stalled from outside, the device preempted or a fault
// elsewhere, can take longer than both.
constexpr double kSlowestRate = 1e8;

// A circuit that costs more than the batch's mean load per workgroup is
// split into that many workgroups' worth of work items (rounded; at most the
// "batch_split" knob, and the tiles or pair steps of its largest pass): else
// the widest circuits, started first, still run long after the rest of the
// batch is done.  A split circuit's passes are cut into chunk tickets of whole
// tiles (fused passes) or whole pair-loop steps (single gates),
// kChunksPerWorker per joining workgroup.  Measured on the 4096-circuit batch
// (widths 10-20), with LDS tiles: splitting also the circuits above a quarter
// or a half of the mean load, or into items of half of it, was slower, and so
// were 8 or 16 chunks per workgroup.
//  - Rounded: rounded up, the items outnumber the workgroups, and the last
//    circuits' items all wait for a second turn (128 circuits of 16 qubits:
//    1094 items for 1024 workgroups, 1.46 ms, against 1.23 ms); rounded down,
//    circuits of nearly twice the mean stay whole (512 of widths 10-20: 12.8
//    ms, against 11.1 ms).
//  - A knob of 64: 64 circuits of widths 10-18 took 1.27 ms with at most 16
//    workgroups each, 0.52 ms with 64; four of width 18 0.91 and 0.39 ms; the
//    512 circuits the same.  Workgroups beyond a pass's tiles would only wait
//    (the 64 circuits: 0.64 ms without that limit).
// Workgroups that find nothing else to do help: after the circuits' own work
// items the queue lists every ticketed circuit again, costliest first, once for
// each further workgroup its chunks have work for (a circuit that is done by
// then costs one ticket).  Circuits from half the mean load on have tickets,
// cut for at least kMinShares workgroups.  Without helpers the last circuits ran
// on their own shares while the rest of the chip was done: 512 circuits of
// widths 10-20 10.9 -> 10.05 ms, mean workgroups busy 867 -> 939 of 1024; 300 in
// complex64 1.16 -> 1.09 ms.  Tickets from a fifth of the mean on: 10.15 ms;
// chunks for eight: 10.75.
constexpr int kChunksPerWorker = 4, kMinShares = 4;

static void split_circuits(BatchHost *h, int dtype, bool adjoint, const std::vector<double> &cost,
                           std::vector<int32_t> *workers, std::vector<int32_t> *helpers) {
    const int gmax = tuning().batch_split;
    if (gmax <= 1)
        return;
    DeviceInfo di;
    const double P = (double)(h->lds ? 2 : kBatchPerCu) * (device_info(&di) == SV_OK ? di.num_cus : 256);  // persistent workgroups
    double W = 0.0;
    for (double c : cost)
        W += c;
    const double load = W / P;
    const int kc = kChunksPerWorker;
    const int m_cap = (h->lds ? kLdsTileBits : rt_nb_of(dtype) + kBatchThreadBits) - (adjoint ? 1 : 0);
    for (size_t c = 0; c < h->circs.size(); ++c) {
        BCirc &bc = h->circs[c];
        if (bc.npasses == 0 || bc.n <= m_cap || !(cost[c] > 0.5 * load))
            continue;  // LDS-resident, empty, one workgroup's registers, or short enough
        // a pass's tiles or pairs, and how many of them a workgroup takes at least
        auto extent = [&](const BPass &p, uint64_t *total, uint64_t *unit) {
            *total = *unit = 1;
            if (p.kind == kPassTiles) {
                *total = p.tm.ntiles;
            } else if (p.kind == kPassPauli) {
                *total = 1ull << bc.n;
                *unit = (uint64_t)kBatchPairUnroll * batch_threads(h->lds);
            } else if (p.kind == kPassGate) {
                const BGate &gt = h->gates[bc.first_gate + p.gate];
                *total = 1ull << (bc.n - 1 - popcount64(gt.cmask));
                *unit = (uint64_t)kBatchPairUnroll * batch_threads(h->lds);
            }
            return (*total + *unit - 1) / *unit;
        };
        uint64_t total, unit, most = 0;
        for (int pi = 0; pi < bc.npasses; ++pi)
            if (h->passes[bc.first_pass + pi].kind <= kPassTiles)
                most = std::max(most, extent(h->passes[bc.first_pass + pi], &total, &unit));
        const int limit = (int)std::min<uint64_t>((uint64_t)gmax, most);
        const int g = std::max(1, (int)std::min<double>(limit, std::floor(cost[c] / load + 0.5)));
        const int shares = std::max(g, std::min(limit, kMinShares));  // chunks are cut for
        if (limit < 2 || (int64_t)bc.npasses * shares * kc > (1 << 30))
            continue;
        int64_t k = 0;
        for (int pi = 0; pi < bc.npasses; ++pi) {
            BPass &p = h->passes[bc.first_pass + pi];
            const uint64_t steps = extent(p, &total, &unit);
            const uint64_t want = std::max<uint64_t>(1, std::min<uint64_t>(steps, (uint64_t)shares * kc));
            const uint64_t len = (steps + want - 1) / want * unit;
            p.chunk0 = (int32_t)k;
            p.nchunks = (int32_t)((total + len - 1) / len);
            p.chunk_len = len;
            k += p.nchunks;
            const double amps = (double)std::min(len, total);
            const double work = p.kind == kPassTiles   ? std::ldexp(amps, (int)p.tm.m) * std::max<double>(p.count, p.rt.count)
                                : p.kind == kPassPauli ? amps * bc.nterms
                                                       : 2.0 * amps;
            h->chunk_work = std::max(h->chunk_work, work);
        }
        bc.group = h->ngroups++;
        bc.nchunks = (int32_t)k;  // at most npasses * 4 * 64
        (*workers)[c] = g;
        (*helpers)[c] = std::min(limit, shares * kc) - g;
    }
}

// Where the passes of a circuit leave their partial sums, and the list of
// them by parameter.
static void place_sums(const std::vector<CircBuild::Sum> &sums, BCirc *bc, BatchHost *h) {
    BPass *ps = &h->passes[bc->first_pass];
    for (int pi = 0; pi < bc->npasses; ++pi) {
        ps[pi].part = h->npart;
        h->npart += (int64_t)ps[pi].nacc * (bc->group >= 0 ? ps[pi].nchunks : 1);
        const size_t acc = (size_t)(h->lds ? ps[pi].nacc : rt_acc_slots(ps[pi].rt)) * (batch_threads(h->lds) / 64) * sizeof(double);
        if (ps[pi].kind == kPassTiles)
            h->lds_bytes = std::max(h->lds_bytes, (h->lds ? ((size_t)2 << ps[pi].tm.m) * sizeof(float2) : kBatchExchange) + acc);
    }
    bc->first_slot = (int32_t)h->slots.size();
    bc->nslots = (int32_t)sums.size();
    bc->first_csr = (int32_t)h->csr.size();
    std::vector<int32_t> at(bc->nparams + 2, 0);
    for (const CircBuild::Sum &u : sums)
        ++at[u.param + 1];
    std::partial_sum(at.begin(), at.end(), at.begin());
    h->csr.insert(h->csr.end(), at.begin(), at.end());
    h->slots.resize(h->slots.size() + sums.size());
    for (const CircBuild::Sum &u : sums) {  // in the sweep's order where gates share a parameter
        const BPass &p = ps[u.pass];
        h->slots[bc->first_slot + at[u.param]++] = BSlot{p.part + u.acc, p.nacc, bc->group >= 0 ? p.nchunks : 1};
    }
}

// Checks the batch description, plans every circuit (in parallel over host
// threads for large batches) and concatenates the tables; circuits are
// ordered by decreasing cost per workgroup for the work queue.
static int build_batch(const BatchArgs &A, bool adjoint, BatchHost *h, int *dtype) {
    if (A.ncirc < 1 || !A.states || !A.gate_off || (A.gate_off[A.ncirc] > 0 && !A.gates))
        return fail(SV_EINVAL, "bad batch description (ncirc %d)", A.ncirc);
    if (adjoint && (!A.term_off || !A.terms || !A.lams || !A.param_off))
        return fail(SV_EINVAL, "batched adjoint needs lambda states, param offsets, terms and term offsets");
    *dtype = A.states[0].dtype;
    int64_t total_gates = 0;
    for (int c = 0; c < A.ncirc; ++c) {
        const sv_state_t &s = A.states[c];
        int r = validate_state(&s);
        if (r != SV_OK)
            return fail(r, "circuit %d: %s", c, sv_last_error());
        if (s.dtype != *dtype)
            return fail(SV_EINVAL, "circuit %d: all states of a batch need one dtype", c);
        if (adjoint) {
            r = validate_state(&A.lams[c]);
            if (r != SV_OK)
                return fail(r, "circuit %d (lambda): %s", c, sv_last_error());
            if (A.lams[c].n != s.n || A.lams[c].dtype != s.dtype || A.lams[c].data == s.data)
                return fail(SV_EINVAL, "circuit %d: lambda must be a distinct state of the same shape", c);
            if (s.n > 31)
                return fail(SV_EINVAL, "circuit %d: batched adjoint supports n <= 31", c);
        }
        const int64_t g0 = A.gate_off[c], g1 = A.gate_off[c + 1];
        if (g0 < 0 || g1 < g0 || g1 - g0 > INT32_MAX)
            return fail(SV_EINVAL, "circuit %d: bad gate offsets", c);
        const int64_t p0 = A.param_off ? A.param_off[c] : 0, p1 = A.param_off ? A.param_off[c + 1] : 0;
        if (p0 < 0 || p1 < p0 || p1 > A.nparams_total)
            return fail(SV_EINVAL, "circuit %d: bad parameter offsets", c);
        total_gates += g1 - g0;
    }
    if (total_gates > INT32_MAX)
        return fail(SV_EINVAL, "batch holds %lld gates (at most 2^31 - 1)", (long long)total_gates);
    std::vector<CircBuild> cb(A.ncirc);
    int widest = 0;
    for (int c = 0; c < A.ncirc; ++c)
        widest = std::max(widest, (int)A.states[c].n);
    const int lds_bits = kLdsTileBits - (*dtype == SV_C128 ? 1 : 0);
    const bool angles = A.gates && std::any_of(A.gates, A.gates + A.gate_off[A.ncirc],
                                               [](const sv_gate_t &g) { return g.param >= 0; });
    h->lds = (*dtype == SV_C64 && (A.lams || angles)) || (A.once && !adjoint && widest <= lds_bits);
    h->resident = h->lds ? lds_bits + 1 : resident_below(*dtype == SV_C128, A.once);
    h->lds_bytes = h->lds ? (adjoint ? 0 : kLdsBytes) : kBatchExchange;
    auto work = [&](int lo, int hi) {
        for (int c = lo; c < hi; ++c) {
            CircBuild &b = cb[c];
            b.lds = h->lds;
            b.resident = h->resident;
            b.err = build_circuit(A, c, *dtype, adjoint, &b);
            if (b.err != SV_OK) {
                b.msg = sv_last_error();  // error text is per thread
                return;
            }
        }
    };
    unsigned nth = std::min(16u, std::max(1u, std::thread::hardware_concurrency()));
    if (total_gates < 2000)  // one thread plans these in 3 ms
        nth = 1;
    nth = std::min<unsigned>(nth, (unsigned)A.ncirc);
    if (nth <= 1) {
        work(0, A.ncirc);
    } else {
        int dev = 0;
        const bool have_dev = hipGetDevice(&dev) == hipSuccess;
        std::vector<std::thread> pool;
        std::atomic<int> next{0};
        constexpr int kChunk = 4;
        for (unsigned t = 0; t < nth; ++t)
            pool.emplace_back([&, have_dev, dev] {
                if (have_dev)
                    (void)hipSetDevice(dev);  // planner queries use the caller's device
                for (;;) {
                    const int lo = next.fetch_add(kChunk);
                    if (lo >= A.ncirc)
                        break;
                    work(lo, std::min(A.ncirc, lo + kChunk));
                }
            });
        for (auto &t : pool)
            t.join();
    }
    std::vector<double> cost(A.ncirc);
    size_t nops = 0, ntiles = 0, nmems = 0;
    for (const CircBuild &b : cb) {
        nops += b.rt.prog.ops.size();
        ntiles += b.tiles.size();
        nmems += b.mems.size();
    }
    h->gates.reserve((size_t)total_gates);
    h->prog.ops.reserve(nops);
    h->tiles.reserve(ntiles);
    h->mems.reserve(nmems);
    for (int c = 0; c < A.ncirc; ++c) {
        CircBuild &b = cb[c];
        if (b.err != SV_OK)
            return fail(b.err, "circuit %d: %s", c, b.msg.c_str());
        b.bc.first_gate = (int32_t)h->gates.size();
        b.bc.first_term = (int32_t)h->terms.size();
        b.bc.first_pass = (int32_t)h->passes.size();
        const int32_t tbase = (int32_t)h->tiles.size(), obase = (int32_t)h->prog.ops.size();
        const uint32_t pbase = (uint32_t)h->prog.pats.size(), mbase = (uint32_t)h->mems.size();
        for (BPass p : b.passes) {
            if (p.kind == kPassTiles) {
                p.first += tbase;
                p.rt.first += (uint32_t)obase;
            }
            h->passes.push_back(p);
        }
        for (BTileJob j : b.jobs) {
            j.tile += tbase;
            for (int s = 0; s < 2; ++s)
                if (j.op[s] >= 0)
                    j.op[s] += obase;
            h->jobs.push_back(j);
        }
        for (RtOp &o : b.rt.prog.ops)
            if (o.w[0] >> 3 == kRtPrep)
                o.w[2] += pbase;
        h->prog.ops.insert(h->prog.ops.end(), b.rt.prog.ops.begin(), b.rt.prog.ops.end());
        for (RtPat p : b.rt.prog.pats) {
            p.first += mbase;
            h->prog.pats.push_back(p);
        }
        const uint32_t lbase = (uint32_t)h->lpats.size();
        for (TileGate &t : b.tiles)
            if (t.diag) {
                t.pat0 += lbase;
                for (int s = 0; s < 2; ++s)
                    if (t.mem[s] >= 0)
                        t.mem[s] += (int32_t)mbase;
            }
        for (SweepPat p : b.lpats) {
            p.first += mbase;
            h->lpats.push_back(p);
        }
        h->tiles.insert(h->tiles.end(), b.tiles.begin(), b.tiles.end());
        h->mems.insert(h->mems.end(), b.mems.begin(), b.mems.end());
        const int32_t gbase = (int32_t)(h->gens.size() / 8);  // generators before this circuit's
        b.bc.first_gen = gbase;
        for (int32_t t : b.tslot)
            h->tslot.push_back(t >= 0 ? t + gbase : -1);
        for (int32_t g : b.gen_of)
            h->gen_of.push_back(g >= 0 ? g + gbase : -1);
        h->gates.insert(h->gates.end(), b.gates.begin(), b.gates.end());
        h->gens.insert(h->gens.end(), b.gens.begin(), b.gens.end());
        h->terms.insert(h->terms.end(), b.terms.begin(), b.terms.end());
        h->circs.push_back(b.bc);
        cost[c] = b.cost;
    }
    std::vector<int32_t> workers(A.ncirc, 1);
    std::vector<int32_t> helpers(A.ncirc, 0);
    split_circuits(h, *dtype, adjoint, cost, &workers, &helpers);
    if (adjoint)
        for (int c = 0; c < A.ncirc; ++c)
            place_sums(cb[c].sums, &h->circs[c], h);
    std::vector<int32_t> circ(A.ncirc);
    std::iota(circ.begin(), circ.end(), 0);
    std::stable_sort(circ.begin(), circ.end(),
                     [&](int a, int b) { return cost[a] / workers[a] > cost[b] / workers[b]; });
    for (int c : circ)
        h->order.insert(h->order.end(), (size_t)workers[c], c);
    h->nlisted = (int)h->order.size();
    std::stable_sort(circ.begin(), circ.end(), [&](int a, int b) { return cost[a] > cost[b]; });
    for (bool more = true; more;) {
        more = false;
        for (int c : circ)
            if (helpers[c] > 0) {
                h->order.push_back(c);
                more |= --helpers[c] > 0;
            }
    }
    return SV_OK;
}

struct BatchDevice {
    void *block = nullptr;  // the tables below, one allocation
    BCirc *circs = nullptr;
    BGate *gates = nullptr;
    BPass *passes = nullptr;
    TileGate *tiles = nullptr;
    RtOp *ops = nullptr;
    RtPat *pats = nullptr;
    SweepMember *mems = nullptr;
    BTileJob *jobs = nullptr;
    int njobs = 0;
    bool lds = false;
    int resident = 0;
    SweepPat *lpats = nullptr;
    int32_t *tslot = nullptr;
    BSlot *slots = nullptr;
    int32_t *csr = nullptr;
    double *part = nullptr;
    size_t lds_bytes = 0;
    int32_t *order = nullptr, *gen_of = nullptr;
    int nitems = 0, nlisted = 0;
    double *gens = nullptr;
    DTerm *terms = nullptr;
    unsigned int *queue = nullptr;
    // split circuits: kGroupWords each, then the count of waits that gave up
    unsigned int *gstate = nullptr;
    int ngroups = 0;
    uint64_t wait_limit = 0;  // clock ticks
};

// Stream-ordered release when async (after the kernels enqueued on st),
// otherwise an immediate free.
static void batch_release(BatchDevice *d, bool async, hipStream_t st) {
    if (d->block)
        (void)(async ? hipFreeAsync(d->block, st) : hipFree(d->block));
    *d = BatchDevice();
}

static int upload_batch(const BatchHost &h, bool async, hipStream_t st, BatchDevice *d) {
    TableBlock tb;
    tb.add(&d->circs, h.circs);
    tb.add(&d->gates, h.gates);
    tb.add(&d->passes, h.passes);
    tb.add(&d->tiles, h.tiles);
    tb.add(&d->ops, h.prog.ops);
    tb.add(&d->pats, h.prog.pats);
    tb.add(&d->mems, h.mems);
    tb.add(&d->jobs, h.jobs);
    tb.add(&d->slots, h.slots);
    tb.add(&d->csr, h.csr);
    tb.add(&d->lpats, h.lpats);
    tb.add(&d->tslot, h.tslot);
    tb.add(&d->order, h.order);
    tb.add(&d->gen_of, h.gen_of);
    tb.add(&d->gens, h.gens);
    tb.add(&d->terms, h.terms);
    tb.add((void **)&d->queue, nullptr, sizeof(unsigned int));
    const int words = h.ngroups > 0 ? kGroupWords * h.ngroups + 1 : 0;
    tb.add((void **)&d->gstate, nullptr, words * sizeof(unsigned int));
    tb.add((void **)&d->part, nullptr, (size_t)h.npart * sizeof(double));
    int r = tb.upload(&d->block, async, st);
    d->njobs = (int)h.jobs.size();
    d->lds = h.lds;
    d->resident = h.resident;
    d->lds_bytes = h.lds_bytes;
    d->nitems = (int)h.order.size();
    d->nlisted = h.nlisted;
    d->ngroups = h.ngroups;
    if (r == SV_OK && h.ngroups > 0) {
        hipLaunchKernelGGL(k_zero_words, dim3((words + 255) / 256), dim3(256), 0, st, d->gstate, words);
        if (!async)
            r = hipStreamSynchronize(st) == hipSuccess ? SV_OK : fail(SV_EHIP, "clearing the batch counters failed");
        int dev = 0, khz = 0;
        if (r == SV_OK && (hipGetDevice(&dev) != hipSuccess ||
                           hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess ||
                           khz <= 0))
            r = fail(SV_EHIP, "device reports no constant-rate clock");
        const int ms = tuning().batch_wait_ms;  // 0: give up at once
        d->wait_limit = ms ? (uint64_t)((double)khz * (ms + 1e3 * h.chunk_work / kSlowestRate)) : 0;
    }
    if (r != SV_OK)
        batch_release(d, async, st);
    return r;
}

// One persistent launch: the forward run, or (grad) the adjoint.
static int launch_batch(int dtype, const BatchDevice &d, const double *params, double *grad, double *loss,
                        hipStream_t s, uint64_t *stamps) {
    constexpr size_t kLdsPerWorkgroup = 160 * 1024;  // gfx950, with the opt-in limit raised
    const size_t lds = d.lds_bytes + kBatchSlot;
    if (lds > kLdsPerWorkgroup)
        return fail(SV_ENOTSUP, "a fused reverse pass needs %zu bytes of LDS", lds);
    DeviceInfo di;
    const unsigned cus = device_info(&di) == SV_OK ? (unsigned)di.num_cus : 256u;
    const unsigned per_cu = std::min<unsigned>(d.lds ? 2 : kBatchPerCu, (unsigned)(kLdsPerWorkgroup / lds));
    const unsigned grid = std::min<unsigned>(cus * per_cu, (unsigned)d.nitems);
    if (d.njobs > 0)
        hipLaunchKernelGGL(k_batch_tile_params, dim3((d.njobs + 255) / 256), dim3(256), 0, s, d.jobs, d.njobs, params,
                           d.tiles, d.lds && grad ? nullptr : d.mems, d.lds ? nullptr : d.ops);
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, s, d.queue);
    if (d.ngroups > 0)  // not the count of waits after them
        hipLaunchKernelGGL(k_zero_words, dim3((kGroupWords * d.ngroups + 255) / 256), dim3(256), 0, s, d.gstate,
                           kGroupWords * d.ngroups);
    const SweepTables a{d.terms, d.gens, d.gen_of, d.tslot, d.slots, d.csr, grad, loss, stamps};
    auto go = [&](auto fn) -> int {
        if (lds > 65536)
            SV_HIP_TRY(hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(fn, dim3(grid), dim3(batch_threads(d.lds)), lds, s, d.circs, d.order, d.nitems, d.nlisted, d.gates, d.passes,
                           d.tiles, d.ops, d.pats, d.lpats, d.mems, params, d.queue, d.gstate, d.wait_limit,
                           d.gstate ? d.gstate + kGroupWords * d.ngroups : nullptr, stamps, d.part, a, (uint32_t)d.lds_bytes,
                           d.resident);
        SV_LAUNCH_CHECK();
        return SV_OK;
    };
    if (dtype == SV_C128)
        return grad    ? go(k_batched<double, true, false>)
               : d.lds ? go(k_batched<double, false, true>)
                       : go(k_batched<double, false, false>);
    if (d.lds)
        return grad ? go(k_batched<float, true, true>) : go(k_batched<float, false, true>);
    return go(k_batched<float, false, false>);  // gradients: LDS tiles
}

} // namespace sv

// A planned batch resident on one device (the C ABI's opaque sv_batch_t).
struct sv_batch {
    int dtype = 0, ncirc = 0, device = 0;
    int64_t nparams_total = 0;
    bool has_adjoint = false;
    sv::BatchDevice fwd, adj;
    std::vector<int32_t> items; // the forward run's work items (circuits), in queue order
    hipEvent_t done = nullptr;  // end of the last run
    uint64_t *stamps = nullptr; // per-circuit start/end clock of later runs (measurement), or none
};

using namespace sv;

extern "C" {

int sv_batch_create(const sv_state_t *states, const sv_state_t *lam_states, int ncirc, const sv_gate_t *gates,
                    const int64_t *gate_offsets, const int64_t *param_offsets, int64_t nparams_total,
                    const sv_pauli_t *terms, const int64_t *term_offsets, sv_batch_t **out) {
    clear_error();
    if (!out)
        return fail(SV_EINVAL, "out is NULL");
    *out = nullptr;
    const bool adj = lam_states != nullptr;
    BatchArgs A{states, lam_states, ncirc, gates, gate_offsets, param_offsets, nparams_total, terms, term_offsets};
    BatchHost hf, ha;
    int dtype = 0;
    SV_TRY(build_batch(A, false, &hf, &dtype));
    if (adj)
        SV_TRY(build_batch(A, true, &ha, &dtype));
    sv_batch *b = new sv_batch();
    b->dtype = dtype;
    b->ncirc = ncirc;
    b->nparams_total = nparams_total;
    b->has_adjoint = adj;
    int r = hipGetDevice(&b->device) == hipSuccess ? SV_OK : fail(SV_EHIP, "no current device");
    b->items.assign(hf.order.begin(), hf.order.begin() + hf.nlisted);
    if (r == SV_OK)
        r = upload_batch(hf, false, nullptr, &b->fwd);
    if (r == SV_OK && adj)
        r = upload_batch(ha, false, nullptr, &b->adj);
    if (r != SV_OK) {
        batch_release(&b->fwd, false, nullptr);
        batch_release(&b->adj, false, nullptr);
        delete b;
        return r;
    }
    *out = b;
    return SV_OK;
}

static int batch_check(sv_batch_t *b, const double *params_dev) {
    if (!b)
        return fail(SV_EINVAL, "batch is NULL");
    if (b->nparams_total > 0 && !params_dev)
        return fail(SV_EINVAL, "params_dev is NULL");
    int dev = 0;
    SV_HIP_TRY(hipGetDevice(&dev));
    if (dev != b->device)
        return fail(SV_EINVAL, "batch was created on device %d, current device is %d", b->device, dev);
    return SV_OK;
}

static int batch_done(sv_batch_t *b, hipStream_t st) {
    if (!b->done)
        SV_HIP_TRY(hipEventCreateWithFlags(&b->done, hipEventDisableTiming));
    SV_HIP_TRY(hipEventRecord(b->done, st));
    return SV_OK;
}

int sv_batch_run(sv_batch_t *b, const double *params_dev, sv_stream_t st) {
    clear_error();
    SV_TRY(batch_check(b, params_dev));
    SV_TRY(launch_batch(b->dtype, b->fwd, params_dev, nullptr, nullptr, (hipStream_t)st, b->stamps));
    return batch_done(b, (hipStream_t)st);
}

int sv_batch_adjoint(sv_batch_t *b, const double *params_dev, double *grad_dev, double *loss_dev, sv_stream_t st) {
    clear_error();
    SV_TRY(batch_check(b, params_dev));
    if (!b->has_adjoint)
        return fail(SV_EINVAL, "batch was created without lambda states and terms");
    if (!grad_dev || !loss_dev)
        return fail(SV_EINVAL, "grad_dev and loss_dev are required");
    SV_TRY(launch_batch(b->dtype, b->adj, params_dev, grad_dev, loss_dev, (hipStream_t)st, b->stamps));
    return batch_done(b, (hipStream_t)st);
}

int sv_batch_set_timing(sv_batch_t *b, uint64_t *stamps_dev, double *ns_per_tick) {
    clear_error();
    if (!b)
        return fail(SV_EINVAL, "batch is NULL");
    b->stamps = stamps_dev;
    if (ns_per_tick) {
        int khz = 0;
        SV_HIP_TRY(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, b->device));
        if (khz <= 0)
            return fail(SV_EHIP, "device reports no constant-rate clock");
        *ns_per_tick = 1e6 / (double)khz;
    }
    return SV_OK;
}

int sv_batch_info(sv_batch_t *b, int64_t *nitems, int32_t *item_circuit, int64_t cap, uint64_t *wait_timeouts) {
    clear_error();
    if (!b)
        return fail(SV_EINVAL, "batch is NULL");
    const int64_t n = (int64_t)b->items.size();
    if (nitems)
        *nitems = n;
    if (item_circuit) {
        if (cap < n)
            return fail(SV_EINVAL, "item_circuit holds %lld entries, the batch has %lld items", (long long)cap,
                        (long long)n);
        std::copy(b->items.begin(), b->items.end(), item_circuit);
    }
    if (wait_timeouts) {
        *wait_timeouts = 0;
        for (const BatchDevice *d : {&b->fwd, &b->adj})
            if (d->ngroups > 0) {
                if (b->done)
                    SV_HIP_TRY(hipEventSynchronize(b->done));
                unsigned int v = 0;
                SV_HIP_TRY(hipMemcpy(&v, d->gstate + kGroupWords * d->ngroups, sizeof(v), hipMemcpyDeviceToHost));
                *wait_timeouts += v;
            }
    }
    return SV_OK;
}

int sv_batch_destroy(sv_batch_t *b) {
    clear_error();
    if (!b)
        return SV_OK;
    if (b->done) {
        (void)hipEventSynchronize(b->done);
        (void)hipEventDestroy(b->done);
    }
    batch_release(&b->fwd, false, nullptr);
    batch_release(&b->adj, false, nullptr);
    delete b;
    return SV_OK;
}

int sv_apply_circuits_batched(const sv_state_t *states, int ncirc, const sv_gate_t *gates, const int64_t *gate_offsets,
                              const double *params_dev, const int64_t *param_offsets, int64_t nparams_total,
                              sv_stream_t st) {
    clear_error();
    BatchArgs A{states, nullptr, ncirc, gates, gate_offsets, param_offsets, nparams_total, nullptr, nullptr, true};
    BatchHost h;
    int dtype = 0;
    SV_TRY(build_batch(A, false, &h, &dtype));
    if (nparams_total > 0 && !params_dev)
        return fail(SV_EINVAL, "params_dev is NULL");
    BatchDevice d;
    hipStream_t s = (hipStream_t)st;
    SV_TRY(upload_batch(h, true, s, &d));
    const int r = launch_batch(dtype, d, params_dev, nullptr, nullptr, s, nullptr);
    batch_release(&d, true, s);
    return r;
}

int sv_adjoint_grad_batched(const sv_state_t *psi_states, const sv_state_t *lam_states, int ncirc,
                            const sv_gate_t *gates, const int64_t *gate_offsets, const double *params_dev,
                            const int64_t *param_offsets, int64_t nparams_total, const sv_pauli_t *terms,
                            const int64_t *term_offsets, double *grad_dev, double *loss_dev, sv_stream_t st) {
    clear_error();
    if (!lam_states || !grad_dev || !loss_dev || !param_offsets)
        return fail(SV_EINVAL, "batched adjoint needs lambda states, param offsets, grad_dev and loss_dev");
    BatchArgs A{psi_states, lam_states, ncirc, gates, gate_offsets, param_offsets, nparams_total, terms,
                term_offsets, true};
    BatchHost h;
    int dtype = 0;
    SV_TRY(build_batch(A, true, &h, &dtype));
    if (nparams_total > 0 && !params_dev)
        return fail(SV_EINVAL, "params_dev is NULL");
    BatchDevice d;
    hipStream_t s = (hipStream_t)st;
    SV_TRY(upload_batch(h, true, s, &d));
    const int r = launch_batch(dtype, d, params_dev, grad_dev, loss_dev, s, nullptr);
    batch_release(&d, true, s);
    return r;
}

} // extern "C"
