// Register-resident tile pass: a fused run applied to tiles whose amplitudes
// live in registers, 2^NB per lane (16 complex128 or 32 complex64: 64 vector
// registers), for the whole run.
//
// What bounds a long run is the work inside the tile.  With the tile in LDS
// (k_tile) every operation reads and writes all of it there: 64 KiB each way
// for a complex128 tile of 2^12 amplitudes, at least 1024 cycles at 128 B per
// clock, plus a barrier, against 512 cycles for a general FP64 pair update
// and 256 for a real or axis rotation.  Here a gate whose target is one of the
// NB "register bits" of the current layout touches registers only.  Gates on
// other targets wait until an exchange through LDS has given their targets
// register positions; the host schedules a run as segments, each with the NB
// register bits that serve most of the gates that may come next (gates pass
// each other only where they commute).
//
// A layout places every tile-local index bit: NB of them number a lane's
// registers, the rest are bits of the thread index (6 lane bits, then
// wavefront bits).  A control on a thread bit is a lane predicate, one on a
// register bit selects registers (a mask formed on the host), one outside the
// tile is a predicate on the tile's base index.  The exchange writes one
// component of every amplitude, meets at a barrier and reads it back in the
// new layout, so it needs only half the tile's bytes of LDS; the slot of
// amplitude j is j with its upper bits folded onto the lowest five (rt_slot),
// which keeps a wavefront's accesses on different banks for the lane-bit
// choices of RtLayout.
#pragma once

#include <utility>

#include "reduce.hpp"
#include "rtile_ops.hpp"
#include "rtile_plan.hpp"

namespace sv {

// Slot of amplitude j in the exchange buffer; linear over xor.
__host__ __device__ constexpr uint32_t rt_slot(uint32_t j) { return j ^ ((j >> 5) & 31u) ^ ((j >> 10) & 31u); }

#ifdef __HIPCC__

// f(integral constant) for 0 .. N - 1: register arrays are only ever indexed
// by constants of the source.
template <typename F, int... I>
__device__ __forceinline__ void rt_unrolled(const F &f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F> __device__ __forceinline__ void rt_for(const F &f) {
    rt_unrolled(f, std::make_integer_sequence<int, N>());
}
#define SV_RT_FOR(N, i) rt_for<(N)>([&](auto i) __attribute__((always_inline))

// A matrix formed on the device into an operation (of complex128 tiles: a
// parameterised complex64 circuit has none).
__device__ __forceinline__ void rt_set_matrix(RtOp &o, const double *m) {
    for (int k = 0; k < 8; ++k)
        o.m[k] = m[k];
}

template <typename R> __device__ __forceinline__ Mat2<R> rt_mat(const RtOp &o) {
    if constexpr (sizeof(R) == 8)
        return Mat2<R>{o.m[0], o.m[1], o.m[2], o.m[3], o.m[4], o.m[5], o.m[6], o.m[7]};
    else
        return Mat2<R>{o.f[0], o.f[1], o.f[2], o.f[3], o.f[4], o.f[5], o.f[6], o.f[7]};
}

// A value the compiler may not take as known: keeps what depends on it where
// it is written instead of hoisted out of the operation loop, where it would
// occupy registers beside the tile's for the whole run.
__device__ __forceinline__ uint32_t rt_fresh(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Two values of which it may take anything.
template <typename R> __device__ __forceinline__ void rt_unset(R &a, R &b) { asm volatile("" : "=v"(a), "=v"(b)); }

// Coefficients of phase_factor's polynomials (tile.hpp): 2/pi, pi/2 in two
// parts, the sine series from 1/17! down to 1, the cosine series from 1/16!
// down to 1.  Read from memory as uniform operands, for the reason above.
static __device__ const double kRtSeries[21] = {
    0.63661977236758134, 1.5707963267948966, 6.123233995736766e-17,
    1.0 / 355687428096000.0, 1.0 / 1307674368000.0, 1.0 / 6227020800.0, 1.0 / 39916800.0, 1.0 / 362880.0,
    1.0 / 5040.0, 1.0 / 120.0, 1.0 / 6.0, 1.0,
    1.0 / 20922789888000.0, 1.0 / 87178291200.0, 1.0 / 479001600.0, 1.0 / 3628800.0, 1.0 / 40320.0, 1.0 / 720.0,
    1.0 / 24.0, 1.0 / 2.0, 1.0};

// exp(i (th + e)) as phase_factor evaluates it, by polynomials of fewer terms
// (errors below 1e-11) for a factor that is rounded to single precision.
template <bool SHORT = false>
__device__ __forceinline__ void rt_phase_factor(double th, double e, double *fr, double *fi) {
    const double *c = kRtSeries;
    asm volatile("" : "+s"(c));
    const double k = rint(th * c[0]);
    double rd = fma(-k, c[1], th);
    rd = fma(-k, c[2], rd) + e;
    constexpr int first = SHORT ? 6 : 3, firstc = SHORT ? 15 : 12;
    const double r2 = rd * rd;
    double ps = c[first], pc = c[firstc];
#pragma unroll
    for (int i = first + 1; i < 12; ++i)
        ps = fma(ps, -r2, c[i]);
#pragma unroll
    for (int i = firstc + 1; i < 21; ++i)
        pc = fma(pc, -r2, c[i]);
    const double s = rd * ps, co = pc;
    const int q = (int)k & 3;  // |k| is far below 2^31
    *fi = q == 0 ? s : q == 1 ? co : q == 2 ? -s : -co;
    *fr = q == 0 ? co : q == 1 ? -s : q == 2 ? -co : s;
}

// One phase pattern of the current tile, kept in LDS: where the index and the
// low half of c are its high half, hi + lo is added.  hi is a multiple of
// 2^-47, so sums of less than 64 are exact, and lo the rest of the phase.  (A
// lane's phases reach the size of several turns: summed as they are, nine
// qubits' round off 6e-16, more than three times what multiplying the nine
// factors one by one does; this way 6e-17.)
struct RtPhase {
    uint32_t c;
    float lo;
    double hi;
};

__device__ __forceinline__ double rt_phase_hi(double th) { return (th + 48.0) - 48.0; }  // |th| <= pi

// Sum of the phases of patterns [first, first + count) that index idx selects,
// and *e its small part.
__device__ __forceinline__ double rt_phase_sum(const RtPhase *ph, uint32_t first, uint32_t count, uint32_t idx,
                                               double *e) {
    double t0 = 0.0, t1 = 0.0;
    float l0 = 0.0f, l1 = 0.0f;
    const uint32_t end = first + (count & ~1u);
#pragma unroll 2
    for (uint32_t p = first; p < end; p += 2) {
        const RtPhase q0 = ph[p], q1 = ph[p + 1];
        const bool on0 = (idx & q0.c) == q0.c >> 16, on1 = (idx & q1.c) == q1.c >> 16;  // (idx is below 2^16)
        t0 += on0 ? q0.hi : 0.0;
        t1 += on1 ? q1.hi : 0.0;
        l0 += on0 ? q0.lo : 0.0f;
        l1 += on1 ? q1.lo : 0.0f;
    }
    if (count & 1u) {  // uniform
        const RtPhase q = ph[end];
        const bool on = (idx & q.c) == q.c >> 16;
        t0 += on ? q.hi : 0.0;
        l0 += on ? q.lo : 0.0f;
    }
    *e = (double)(l0 + l1);
    return t0 + t1;
}

// The factor of those phases.
template <bool SHORT>
__device__ __forceinline__ void rt_phases(const RtPhase *ph, uint32_t first, uint32_t count, uint32_t idx, double *fr,
                                          double *fi) {
    if (SHORT && count == 0) {  // uniform
        *fr = 1.0;
        *fi = 0.0;
        return;
    }
    double e;
    const double t = rt_phase_sum(ph, first, count, idx, &e);
    rt_phase_factor<SHORT>(t, e, fr, fi);
}

// A block of diagonal gates multiplies every amplitude by exp(i theta), theta
// the sum of the block's phases its index selects.  The phases split by the
// register condition they carry: those without one (T patterns) sum to one
// phase per lane, those without a thread condition (R patterns) to one per
// register number, shared by all lanes, and the rest to one phase per lane
// for each distinct register condition; so an amplitude costs a few complex
// products and a lane a few sines and cosines, however many gates the block
// has.  This operation sums every pattern's members for the tile and forms
// the R patterns' table of factors; kRtFactor and kRtTable operations follow
// (each a product with the amplitudes), or, on complex64 tiles, one kRtBlock or
// kRtFactor operation, as single precision has no roundings to spare: with a
// product for each, the QFT's error was 4% (n = 20) to 7% (n = 29) larger than
// with one factor for the sum of all phases.
template <typename R, int NB>
__device__ __forceinline__ void rt_prep(unsigned char *lds, uint64_t base, const uint32_t (&w)[16],
                                        const RtPat *__restrict__ pats, const SweepMember *__restrict__ mems) {
    const uint32_t tid = rt_fresh(threadIdx.x), np = w[1];
    double2 *fr = reinterpret_cast<double2 *>(lds);
    RtPhase *ph = reinterpret_cast<RtPhase *>(fr + (1 << NB));
    __syncthreads();  // the buffer's last readers are done
    for (uint32_t p = tid; p < np; p += blockDim.x) {
        // (a byte offset below 2^32 from a uniform base: no 64-bit lane address)
        const RtPat q = *reinterpret_cast<const RtPat *>(reinterpret_cast<const char *>(pats) +
                                                         (uint32_t)((w[2] + p) * sizeof(RtPat)));
        double hi = 0.0;
        float lo = 0.0f;
#pragma unroll 1
        for (uint32_t k = 0; k < (q.count & ~kRtPatNegative); ++k) {
            const SweepMember mm = mems[q.first + k];
            const double th = (base & mm.om) == mm.ov ? mm.theta : 0.0, h = rt_phase_hi(th);
            hi += h;
            lo += (float)(th - h);
        }
        const bool minus = (q.count & kRtPatNegative) != 0;
        RtPhase a;
        a.c = q.cm | q.cv << 16;
        a.lo = minus ? -lo : lo;
        a.hi = minus ? -hi : hi;
        ph[p] = a;
    }
    __syncthreads();
    if (w[4]) {  // uniform
        if (tid < (1u << NB)) {
            double2 f;
            rt_phases<sizeof(R) == 4>(ph, w[3], w[4], tid, &f.x, &f.y);
            fr[tid] = f;
        }
        __syncthreads();
    }
}

// xor of the terms of a thread index's set bits
__device__ __forceinline__ uint32_t rt_xor_terms(uint32_t tid, const uint32_t *t) {
    uint32_t a = 0;
#pragma unroll
    for (int i = 0; i < kRtMaxThreadBits; ++i)
        a ^= ((tid >> i) & 1u) ? t[i] : 0u;
    return a;
}

// A run's operations on the tile in registers.  slot: the lane's byte offset
// in the exchange buffer in the current layout.  GRAD: the reverse sweep; accl
// holds one accumulator per parameterised gate and wavefront (accl[k * nw +
// wavefront]; acc_count gates rounded up to four).  Terms come in the order of
// their accumulators, and four at a time are summed over the wavefront.  tb: thread bits of the tile; in a wider workgroup (PART) the
// lanes beyond them only take part in the exchanges, on slots of their own.
template <typename R, int NB, bool GRAD = false, bool PART = false>
__device__ __forceinline__ void rt_run(RtRegs<R, NB> &v, unsigned char *lds, uint32_t slot, uint64_t base,
                                       const RtOp *__restrict__ ops, uint32_t count,
                                       const RtPat *__restrict__ pats, const SweepMember *__restrict__ mems,
                                       double *accl = nullptr, uint32_t acc_count = 0, int tb = kRtMaxThreadBits) {
    const uint32_t tid = threadIdx.x;
    // LDS byte address of the buffer
    const uint32_t buf = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const RtPhase *ph = reinterpret_cast<const RtPhase *>(reinterpret_cast<double2 *>(lds) + (1 << NB));
    // gradient terms not yet summed: this lane's last one, and two before it
    // folded (lanes of either value of bit 0 hold one of them)
    double one_term = 0.0, two_terms = 0.0;
    auto take = [&](uint32_t k, double t) __attribute__((always_inline)) {
        if (k & 1u) {  // uniform
            const double a = fold_pair<0>(one_term, t, tid);
            if (k & 2u) {
                double s = row_sum_over4(fold_pair<1>(two_terms, a, tid));
                s += __shfl_xor(s, 16);
                s += __shfl_xor(s, 32);
                if ((tid & 63u) < 4u)
                    accl[((k & ~3u) + (tid & 3u)) * (blockDim.x >> 6) + (tid >> 6)] += s;
            }
            two_terms = a;
        }
        one_term = t;
    };
    for (uint32_t i = 0; i < count; ++i) {
        const RtOp &o = ops[i];
        uint32_t w[16];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            w[k] = o.w[k];
        const uint32_t kind = w[0] >> 3;
        const Mat2<R> m = rt_mat<R>(o);
        // the factor of operations with one; others leave it unset in half-size
        // lanes, whose few tiles wait on every instruction (200 gates on one
        // 12-qubit tile 120.9 -> 117.5 us; full lanes gain nothing)
        R fr = (R)0, fi = (R)0;
        if constexpr (NB < rt_nb<R>())
            rt_unset(fr, fi);
        uint64_t lanes = ~0ull;
        uint32_t next = slot;
        // every path meets at rt_apply (lanes 0: nothing to do): paths of
        // their own around it would split the amplitudes' live ranges
        const bool gate = kind <= kRtDiag || (GRAD && kind == kRtGrad);
        if (gate) {
            const uint64_t om = (uint64_t)w[7] << 32 | w[6], ov = (uint64_t)w[9] << 32 | w[8];
            lanes = __ballot((tid & w[2]) == w[3]);
            if ((base & om) != ov)
                lanes = 0;
        }
        // complex64: the factors (left unset on every path of its own, where
        // that costs no moves)
        RtPhases<NB> bl;
        auto no_bits = [&]() __attribute__((always_inline)) {
            if constexpr (sizeof(R) == 4)
                SV_RT_FOR(NB, b) { rt_unset(bl.ur[b], bl.ui[b]); });
        };
        if (kind == kRtDiag) {
            const uint64_t ob = (uint64_t)w[11] << 32 | w[10];
            const bool one = (tid & w[4]) != 0 || (base & ob) != 0 || (w[0] & 7u) != 0;
            if constexpr (sizeof(R) == 4) {
                bl.gr = one ? m.dr : m.ar;
                bl.gi = one ? m.di : m.ai;
            } else {
                fr = one ? m.dr : m.ar;
                fi = one ? m.di : m.ai;
            }
            no_bits();
        } else if (gate) {
            if constexpr (sizeof(R) == 4)
                rt_unset(bl.gr, bl.gi);
            no_bits();
        } else if (sizeof(R) == 4 && kind == kRtBlock) {
            if constexpr (sizeof(R) == 4) {
                rt_phases<true>(ph, w[12], w[13], tid, &bl.gr, &bl.gi);
                SV_RT_FOR(NB, b) { rt_phases<true>(ph, o.t[b], o.t[8 + b], tid, &bl.ur[b], &bl.ui[b]); });
            }
        } else {
            if (kind == kRtFactor) {
                if constexpr (sizeof(R) == 4)
                    rt_phases<true>(ph, w[12], w[13], tid | w[14] << kRtRegBit, &bl.gr, &bl.gi);
                else
                    rt_phases<false>(ph, w[12], w[13], tid, &fr, &fi);
            } else {
                if constexpr (sizeof(R) == 4)
                    rt_unset(bl.gr, bl.gi);
                if (kind == kRtExch) {
                    next = rt_xor_terms(rt_fresh(tid), o.t);
                } else if (kind == kRtPrep) {
                    rt_prep<R, NB>(lds, base, w, pats, mems);
                    lanes = 0;
                }
            }
            no_bits();
        }
        uint32_t sa = buf + slot, na = buf + next;
        if (PART && kind != kRtExch)
            lanes &= __ballot((tid >> tb) == 0);
        if constexpr (GRAD) {
            double g[4] = {0.0, 0.0, 0.0, 0.0};
            rt_apply_grad(v, w, m, fr, fi, lanes, buf, sa, na, g);
            if (kind == kRtGrad) {  // uniform
                const uint64_t ob = (uint64_t)w[11] << 32 | w[10];
                const bool one = (tid & w[4]) != 0 || (base & ob) != 0;
                take(w[13], (one ? m.ai : m.ar) * ((g[0] + g[1]) - (g[2] + g[3])));
            }
        } else if constexpr (sizeof(R) == 4) {
            rt_apply(v, w, m, lanes, buf, sa, na, bl);
        } else {
            rt_apply(v, w, m, fr, fi, lanes, buf, sa, na);
        }
        slot = next;
    }
    if constexpr (GRAD)
        for (uint32_t k = acc_count; k & 3u; ++k)
            take(k, 0.0);
}

// A component in registers of its own.  Amplitudes are loaded and stored as
// whole 16- or 8-byte values; without these moves the compiler keeps each one
// in adjacent registers through the run, and the aligned groups no longer fit.
__device__ __forceinline__ double rt_own(double v) {
    double o;
    asm("v_mov_b64 %0, %1" : "=v"(o) : "v"(v));
    return o;
}
__device__ __forceinline__ float rt_own(float v) {
    float o;
    asm("v_mov_b32 %0, %1" : "=v"(o) : "v"(v));
    return o;
}

// Byte i of a descriptor's byte array: by whole words, which are scalar loads
// where the descriptor lies in memory.
__device__ __forceinline__ uint32_t rt_byte(const uint8_t *b, int i) {
    return reinterpret_cast<const uint32_t *>(b)[i >> 2] >> (8 * (i & 3)) & 63u;
}

// The lane's part of a global amplitude index, and one register's.
__device__ __forceinline__ uint64_t rt_thread_offset(const RtIO &io, uint32_t tid, int bits) {
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < kRtMaxThreadBits; ++i)
        if (i < bits) {  // uniform
            const uint64_t q = 1ull << rt_byte(io.tq, i);
            const uint32_t on = 0u - ((tid >> i) & 1u);
            lo |= on & (uint32_t)q;
            hi |= on & (uint32_t)(q >> 32);
        }
    return (uint64_t)hi << 32 | lo;
}
template <int NB> __device__ __forceinline__ uint64_t rt_reg_offset(const RtIO &io, int r) {
    uint64_t a = 0;
#pragma unroll
    for (int k = 0; k < NB; ++k)
        if ((r >> k) & 1)
            a |= 1ull << rt_byte(io.rq, k);
    return a;
}

#endif  // __HIPCC__

} // namespace sv
