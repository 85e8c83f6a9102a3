// Descriptors of the register tile pass (rtile.hpp), shared by the planner,
// the circuit driver and the kernels.
#pragma once

#include "tile.hpp"

namespace sv {

constexpr int kRtMaxThreadBits = 9;  // workgroups of up to 512 lanes
constexpr int kRtMaxThreads = 1 << kRtMaxThreadBits;
constexpr int kRtMaxNB = 5;
// Register bits: 16 complex128 or 32 complex64 amplitudes per lane; half as
// many where a pass has no more tiles than the chip has CUs.  Such a pass is
// bound by the latency of each operation, which twice the wavefronts with
// half the work each hide better (complex64 QFT n=12 45.0 -> 34.5 us, n=20
// 88.1 -> 78.7; complex128 n=10 28.4 -> 24.3 us, even from n=12 on).
template <typename R> constexpr int rt_nb() { return sizeof(R) == 8 ? 4 : 5; }
inline int rt_nb_of(int tile_dt) { return tile_dt == SV_C128 ? 4 : 5; }
constexpr uint64_t kRtFewTiles = 256;
// Tiles of 64 to 512 lanes; narrower ones stay with the LDS tiles.  dual: the
// reverse sweep, whose lanes hold psi and lambda together (the top register
// bit tells them apart, so a layout has one register bit less).
inline bool rt_tile_ok(int tile_dt, int m, bool dual) {
    const int t = m - rt_nb_of(tile_dt) + (dual ? 1 : 0);
    return t >= 6 && t <= kRtMaxThreadBits;
}
inline int rt_pass_nb(int tile_dt, int m, bool dual, uint64_t ntiles) {
    const int nb = rt_nb_of(tile_dt);
    return !dual && ntiles <= kRtFewTiles && m - nb < kRtMaxThreadBits ? nb - 1 : nb;
}

// Operation kinds (RtOp::w[0] = kind * 8 + a small number).
constexpr uint32_t kRtReal = 0;    // pair gate, real entries (number: the register bit)
constexpr uint32_t kRtCross = 1;   // pair gate, real diagonal, imaginary off-diagonal
constexpr uint32_t kRtGen = 2;     // pair gate, any entries
constexpr uint32_t kRtSwap = 3;    // X
constexpr uint32_t kRtDiag = 4;    // registers times entry a of a diagonal gate, or entry d where the lane's
                                   // or the tile's target bit is 1 (number 1: d everywhere)
constexpr uint32_t kRtFactor = 5;  // registers times a factor per lane, exp(i sum of phases)
constexpr uint32_t kRtTable = 6;   // registers times the prepared table's factors (complex128)
constexpr uint32_t kRtExch = 7;    // to another layout
constexpr uint32_t kRtPrep = 8;    // phases of a block of diagonal gates in this tile
constexpr uint32_t kRtGrad = 9;    // gradient term of a parameterised gate (reverse sweep)
constexpr uint32_t kRtBlock = 10;  // complex64 tiles: registers times the prepared block's factors

struct RtOp {
    uint32_t w[16];
    //  w[0] kind and number, w[1] pairs or registers, w[5] rt_jump
    //  gates: w[2] w[3] condition on the thread index (mask, value), w[4] thread bit of a diagonal
    //    gate's target, w[6] w[7] and w[8] w[9] condition on the tile's base index (low and high
    //    words), w[10] w[11] base-index bit of a diagonal gate's target
    //  kRtFactor: w[12] first and w[13] number of its patterns, w[14] the register number they
    //    are asked about beside the thread index
    //  kRtBlock: w[12] first and w[13] number of the patterns of thread bits alone; t[k] first and
    //    t[8 + k] number of those of register bit k and thread bits
    //  kRtPrep: w[1] patterns, w[2] first pattern, w[3] first and w[4] number of the R patterns
    //  kRtExch: register terms as rt_apply takes them
    //  kRtGrad: as a gate; w[12] the registers subtracted (diagonal gates), w[13] its accumulator;
    //    m[0] the term's factor, or m[1] where the lane's or the tile's target bit is 1 (both
    //    precisions: double)
    union {
        double m[8];    // matrix, complex128 tiles
        float f[8];     // matrix, complex64 tiles
        uint32_t t[16]; // exchange: slot terms of the new thread bits (bytes)
    };
};
static_assert(sizeof(RtOp) == 128, "descriptor layout");

// A phase pattern in a layout: the sum of its members' phases (those whose
// outer predicate holds) is added where (index & cm) == cv, the index being
// the register number for R patterns and the thread index (the register
// number above it, from kRtRegBit on) otherwise.  A
// pattern with more than kRtPatMembers members is split, so that the lanes
// share the members of a long one; one preparation holds at most kRtMaxPats
// (twice that where kRtBlock lists a pattern once more with its sign changed,
// which still fits the smallest exchange buffer of batches, 32 KiB).
constexpr uint32_t kRtPatMembers = 4, kRtMaxPats = 1000, kRtPatNegative = 1u << 31;
constexpr int kRtRegBit = kRtMaxThreadBits;
struct RtPat {
    uint32_t cm, cv, first, count;  // count: | kRtPatNegative to subtract the phases
};

// Where a layout's amplitudes live in global memory: the qubits of its
// thread and register bits, and the slot terms (bytes) of its thread bits (those
// beyond the tile's give the lanes of a wider workgroup slots of their own).
struct RtIO {
    uint8_t tq[12], rq[8];  // (whole words: kernels read them as such)
    uint32_t slot[kRtMaxThreadBits];
};

struct RtPass {
    RtIO in, out;
    uint32_t first, count;  // operations
    uint32_t always;        // every launched tile is touched
    uint32_t nb;            // register bits
    uint32_t lds;           // bytes of dynamic LDS (dual: accumulators not included)
    uint32_t acc_first, acc_count;  // dual: gradient accumulators (RtProgram::acc)
};

// Accumulators in LDS: whole groups of four.
__host__ __device__ inline uint32_t rt_acc_slots(const RtPass &p) { return (p.acc_count + 3u) & ~3u; }

// Host-side program of a circuit's fused passes.
struct RtProgram {
    std::vector<RtOp> ops;
    std::vector<RtPat> pats;
    std::vector<int32_t> acc;  // gradient slot of every accumulator
};

// Device copies.
struct RtDevice {
    RtOp *ops;
    RtPat *pats;
    int32_t *acc;
};

// Gradient terms 2 Re <lambda|A|psi> by generator A: -i/2 Y, -i/2 X, -i/2 Z and
// diag(0, i).
constexpr uint8_t kRtNoGrad = 0, kRtGradRY = 1, kRtGradRX = 2, kRtGradRZ = 3, kRtGradP = 4;

// Structure of a gate's matrix, known on the host for every angle.
struct RtGateInfo {
    uint8_t kind;     // kRtReal .. kRtDiag
    uint8_t unit_a;   // diagonal: entry a is exactly 1
    uint8_t grad;     // gradient term to take: kRtNoGrad ..
    int8_t sign;      // its sign (-1: the gate was given with the adjoint flag)
    int32_t slot;     // its gradient slot
    int32_t op = -1, op2 = -1;  // out: its operations (matrix slots); -1 inside a phase block
};
RtGateInfo rt_gate_info(int kind, bool from_param, const double *mat, bool diag);

// Schedule one fused run (descriptors tiles[0 .. count), with the marks of
// mark_diag_sweeps and the patterns of build_sweep_patterns) over the tile
// map tm and append its operations.  coal: the state's lowest index bits
// that stay thread bits where tiles are loaded and stored (whole 128-byte
// lines); block: fixed-point tiles, loaded and stored with tile-local bits 0
// and 1 in registers and 2..5 on the lowest lane bits instead.
// nb: register bits (rt_pass_nb, or rt_nb_of).  dual: the reverse sweep's passes.
// fixed_mask: outer index bits every launched tile has with the required
// values.  *slow: instructions, roughly, of complex64 blocks that sum their
// phases once for each set of registers.
RtPass build_rt_pass(const TileMap &tm, uint64_t fixed_mask, int tile_dt, const TileGate *tiles, int count,
                     RtGateInfo *info, const std::vector<SweepPat> &pats, int nb, int coal, bool block, bool dual,
                     RtProgram &prog, double *slow);

// One pass over a complex128 or complex64 state.
int launch_rt_pass(int dtype, void *psi, const TileMap &tm, const RtPass &p, const RtDevice &d,
                   const DeviceGates &gates, hipStream_t st);

// One pass of the reverse sweep over complex128 psi and lambda (dual program): partials
// [slot * stride + workgroup] receive every accumulator's sum per workgroup of
// the grid.
int launch_rt_adjoint(void *psi, void *lam, const TileMap &tm, const RtPass &p, const RtDevice &d,
                      const DeviceGates &gates, unsigned grid, double *partials, int stride, hipStream_t st);
// Dynamic LDS of such a pass, and the per-kernel limit raised to lds bytes.
size_t rt_adjoint_lds(const TileMap &tm, const RtPass &p);
int rt_adjoint_lds_limit(size_t lds);

} // namespace sv
