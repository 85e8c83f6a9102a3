// Pauli-sum expectation values <psi|H|psi> and the product H psi.
//
// For one x mask X != 0 the amplitudes pair up as (k, k ^ X); with b the
// lowest set bit of X and k running over indices with bit b clear, the two
// contributions of a pair to <psi|P|psi> are complex conjugates (P is
// Hermitian), so the term is 2 Re( conj(psi_k) i^{ny} (-1)^{z.(k^X)}
// psi_{k^X} ) summed over half the indices: one read of every amplitude per
// x-mask group, enumerated with the same index expansion as the gate
// kernels.  Diagonal terms (X = 0) sum |psi_k|^2 (-1)^{z.k}.  Terms of a
// group are evaluated together in one pass.  Reductions are deterministic
// (reduce.hpp).  Fixed-point states (SV_CQ16, SV_CQ32) are read through
// their codes: each amplitude is code * 2^scale of its 64-amplitude block,
// which double holds exactly, so an expectation of a fixed-point state is
// that of the decoded state with the same double arithmetic.
//
// Tile passes.  A tile is the 2^m amplitudes (m = min(n, 12)) whose indices
// agree outside a qubit set T made of the lowest qubits (as many as fill a
// 128-byte line: kLow) and others.  A term whose x mask lies inside T pairs
// amplitudes of one tile only, so one read of the state into LDS serves every
// such term: the terms are split into tile sets (the first is qubits 0..m-1;
// the others take the remaining x masks' upper qubits, first fit, then are
// filled up to m with the lowest unused qubits), and one pass per set (<= 64
// terms) evaluates them all.  Diagonal terms join the first set.  Groups whose
// x mask has too many upper qubits keep the one-pass-per-group kernel.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <numeric>
#include <utility>

#include "pauli.hpp"

namespace sv {

constexpr int kMaxT = 16;        // terms evaluated per pass
constexpr int kExpectLoads = 4;  // visits per lane loaded together

int make_pauli_plan(int n, const sv_pauli_t *terms, int nterms, PauliPlan *p) {
    if (nterms < 1 || !terms)
        return fail(SV_EINVAL, "need at least one term (nterms %d, terms %p)", nterms, (const void *)terms);
    const uint64_t full = (n >= 64) ? ~0ull : ((1ull << n) - 1);
    std::vector<int> idx(nterms);
    std::iota(idx.begin(), idx.end(), 0);
    for (int j = 0; j < nterms; ++j)
        if ((terms[j].x_mask | terms[j].z_mask) & ~full)
            return fail(SV_EINVAL, "term %d acts on qubits >= n=%d", j, n);
    std::stable_sort(idx.begin(), idx.end(), [&](int a, int b) { return terms[a].x_mask < terms[b].x_mask; });
    p->groups.clear();
    p->terms.clear();
    for (int k = 0; k < nterms; ++k) {
        const sv_pauli_t &t = terms[idx[k]];
        const bool start = p->groups.empty() || p->groups.back().x != t.x_mask || p->groups.back().count == kMaxT;
        if (start)
            p->groups.push_back(DGroup{t.x_mask, (int32_t)p->terms.size(), 0});
        DTerm d;
        d.coef = t.coef;
        d.z = t.z_mask;
        d.ny = popcount64(t.x_mask & t.z_mask) & 3;
        d.idx = idx[k];
        p->terms.push_back(d);
        p->groups.back().count++;
    }
    return SV_OK;
}

int pauli_upload(const PauliPlan &p, size_t partial_doubles, hipStream_t st, PauliDevice *d) {
    *d = PauliDevice();
    d->nterms = (int)p.terms.size();
    d->ngroups = (int)p.groups.size();
    auto alloc = [&](void **ptr, size_t bytes) -> int {
        hipError_t e = hipMallocAsync(ptr, bytes, st);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            *ptr = nullptr;
            return fail(SV_ENOMEM, "device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
        }
        return SV_OK;
    };
    int r = alloc((void **)&d->terms, p.terms.size() * sizeof(DTerm));
    if (r == SV_OK)
        r = alloc((void **)&d->groups, p.groups.size() * sizeof(DGroup));
    if (r == SV_OK && partial_doubles)
        r = alloc((void **)&d->partials, partial_doubles * sizeof(double));
    if (r != SV_OK) {
        pauli_release(d, st);
        return r;
    }
    SV_HIP_TRY(hipMemcpyAsync(d->terms, p.terms.data(), p.terms.size() * sizeof(DTerm), hipMemcpyHostToDevice, st));
    SV_HIP_TRY(
        hipMemcpyAsync(d->groups, p.groups.data(), p.groups.size() * sizeof(DGroup), hipMemcpyHostToDevice, st));
    return SV_OK;
}

void pauli_release(PauliDevice *d, hipStream_t st) {
    if (d->terms)
        (void)hipFreeAsync(d->terms, st);
    if (d->groups)
        (void)hipFreeAsync(d->groups, st);
    if (d->partials)
        (void)hipFreeAsync(d->partials, st);
    *d = PauliDevice();
}

// Amplitude sources for the expectation passes: what is loaded of amplitude k
// (raw), and the amplitude as two doubles.
template <typename R> struct CplxAmps {
    static constexpr int kLow = sizeof(R) == 8 ? 3 : 4;  // qubits of a 128-byte line
    using Raw = cplx_t<R>;
    const Raw *__restrict__ psi;
    __device__ Raw raw(uint64_t k) const { return psi[k]; }
    static __device__ void decode(const Raw &v, double &re, double &im) {
        re = (double)v.x;
        im = (double)v.y;
    }
    __device__ void get(uint64_t k, double &re, double &im) const { decode(raw(k), re, im); }
};

// SV_CQ16: one 32-bit word per amplitude, re in the low half.
struct Q16Amps {
    static constexpr int kLow = 5;
    struct Raw {
        uint32_t w;
        int s;
    };
    const uint32_t *__restrict__ codes;
    const int8_t *__restrict__ scales;
    __device__ Raw raw(uint64_t k) const { return Raw{codes[k], scales[k >> 6]}; }
    static __device__ void decode(const Raw &v, double &re, double &im) {
        re = ldexp((double)(int16_t)(v.w & 0xffffu), v.s);
        im = ldexp((double)(int16_t)(v.w >> 16), v.s);
    }
    __device__ void get(uint64_t k, double &re, double &im) const { decode(raw(k), re, im); }
};

// SV_CQ32: two 32-bit words per amplitude (re, im).
struct Q32Amps {
    static constexpr int kLow = 4;
    struct Raw {
        uint2 w;
        int s;
    };
    const uint2 *__restrict__ codes;
    const int8_t *__restrict__ scales;
    __device__ Raw raw(uint64_t k) const { return Raw{codes[k], scales[k >> 6]}; }
    static __device__ void decode(const Raw &v, double &re, double &im) {
        re = ldexp((double)(int32_t)v.w.x, v.s);
        im = ldexp((double)(int32_t)v.w.y, v.s);
    }
    __device__ void get(uint64_t k, double &re, double &im) const { decode(raw(k), re, im); }
};

// A group's terms as a kernel argument.
struct GroupTerms {
    uint64_t z[kMaxT];
    int32_t ny[kMaxT];
};

// One pass for one group (<= kMaxT terms sharing the x mask X).
// partials[(first + j) * kMaxPartials + block] receives the workgroup's sum
// of <P_j> contributions.
template <typename A>
__global__ __launch_bounds__(kRedThreads) void k_expect_group(const A amps, uint64_t count, uint64_t X, uint32_t b,
                                                              const GroupTerms terms, int first, int nt,
                                                              double *__restrict__ partials) {
    __shared__ double red[kRedThreads / 64];
    uint64_t z[kMaxT];
    int ny[kMaxT];
    double acc[kMaxT];
#pragma unroll
    for (int j = 0; j < kMaxT; ++j) {
        acc[j] = 0.0;
        z[j] = terms.z[j];
        ny[j] = terms.ny[j];
    }
    // Each lane visits i0, i0 + stride, i0 + 2 stride, ...; kExpectLoads of
    // those visits load before any of them is summed, so enough bytes are in
    // flight for the narrow formats too.  The lane's summation order is that
    // of the visits.
    const uint64_t stride = (uint64_t)gridDim.x * kRedThreads;
    const uint64_t lowb = (1ull << b) - 1;
    const uint64_t i0 = (uint64_t)blockIdx.x * kRedThreads + threadIdx.x;
    if (X == 0) {
        for (uint64_t i = i0; i < count; i += kExpectLoads * stride) {
            double vr[kExpectLoads], vi[kExpectLoads];
#pragma unroll
            for (int u = 0; u < kExpectLoads; ++u)  // visits past the end load the last amplitude, unused
                amps.get(min(i + u * stride, count - 1), vr[u], vi[u]);
#pragma unroll
            for (int u = 0; u < kExpectLoads; ++u) {
                const uint64_t iu = i + u * stride;
                if (iu < count) {
                    const double pr = vr[u] * vr[u] + vi[u] * vi[u];
#pragma unroll
                    for (int j = 0; j < kMaxT; ++j)
                        if (j < nt)
                            acc[j] += odd_parity(z[j] & iu) ? -pr : pr;
                }
            }
        }
    } else {
        for (uint64_t i = i0; i < count; i += kExpectLoads * stride) {
            double ur[kExpectLoads], ui[kExpectLoads], vr[kExpectLoads], vi[kExpectLoads];
#pragma unroll
            for (int u = 0; u < kExpectLoads; ++u) {  // visits past the end load the last pair, unused
                const uint64_t iu = min(i + u * stride, count - 1);
                const uint64_t k = ((iu >> b) << (b + 1)) | (iu & lowb);  // bit b cleared
                amps.get(k, ur[u], ui[u]);
                amps.get(k ^ X, vr[u], vi[u]);
            }
#pragma unroll
            for (int u = 0; u < kExpectLoads; ++u) {
                const uint64_t iu = i + u * stride;
                if (iu < count) {
                    const uint64_t k2 = (((iu >> b) << (b + 1)) | (iu & lowb)) ^ X;
                    // w = conj(u) * v
                    const double wr = ur[u] * vr[u] + ui[u] * vi[u];
                    const double wi = ur[u] * vi[u] - ui[u] * vr[u];
#pragma unroll
                    for (int j = 0; j < kMaxT; ++j)
                        if (j < nt) {
                            const double r = re_ipow(ny[j], wr, wi);
                            acc[j] += odd_parity(z[j] & k2) ? -r : r;
                        }
                }
            }
        }
    }
    const double scale = X == 0 ? 1.0 : 2.0;
#pragma unroll
    for (int j = 0; j < kMaxT; ++j) {
        if (j < nt) {  // uniform
            const double s = block_sum(acc[j], red);
            if (threadIdx.x == 0)
                partials[(size_t)(first + j) * kMaxPartials + blockIdx.x] = scale * s;
        }
    }
}

constexpr int kTileBits = 12;                                 // tile: 2^12 amplitudes, 64 KiB of double2
constexpr int kTileTerms = 64;                                // terms per tile pass: one lane each
constexpr int kTileThreads = 256;
constexpr int kTilePerLane = (1 << kTileBits) / kTileThreads;  // amplitudes per lane and tile

// A term of a tile pass, its masks split at the tile's qubit set T.
struct TTerm {
    uint64_t zh;      // z outside T: the sign set by the tile's fixed bits
    uint32_t xl, zl;  // x (inside T, nonzero unless diagonal) and z on T, as tile-local bits
    int32_t ny;       // |x & z| mod 4: the power of i
    int32_t slot;     // the term's position in the plan: its row of partials
};

// One tile pass.  Tile-local bit r < L is qubit r; bit L + q is the q-th
// lowest qubit of himask; the tile number's bit r is the r-th lowest qubit of
// frmask.  Terms in order: the diagonal ones by the upper four bits of zl (ends in
// end); those whose x mask is one of kRegMasks in tile-local bits 8 - 4 p ..
// 11 - 4 p, by p and mask; the others.
constexpr int kRegMasks[7] = {1, 2, 4, 8, 3, 6, 12};  // one bit or two neighbours
struct TilePass {
    uint64_t himask, frmask;
    int32_t m, L, nfree, nt;
    int32_t end[37];    // ends: 16 of diagonal terms, then 7 of each p
    TTerm t[kTileTerms];
};

// The bits of v, lowest first, placed at the set bits of mask, lowest first.
__device__ __forceinline__ uint64_t deposit_bits(uint64_t v, uint64_t mask) {
    uint64_t out = 0;
    while (mask) {
        if (v & 1ull)
            out |= mask & (~mask + 1ull);
        v >>= 1;
        mask &= mask - 1ull;
    }
    return out;
}

// LDS slot of a tile's amplitude l: linear over xor, and without bank
// conflicts whichever four bits of l number a lane's registers.
__device__ __forceinline__ uint32_t tile_slot(uint32_t l) { return l ^ ((l >> 4) & 15u); }

// s + x, with what that rounds off added to e.
__device__ __forceinline__ void add_exact(double &s, double &e, double x) {
    const double t = s + x, b = t - s;
    e += (s - (t - b)) + (x - b);
    s = t;
}
// s + e (infinite sums leave no e)
__device__ __forceinline__ double with_rest(double s, double e) { return s + (e == e ? e : 0.0); }

// The pass's terms.  Lane j holds term j's masks; acck of lane i is the sum
// of term 16 k + (i & 15) over its row of lanes in this tile.
struct TileTerms {
    uint32_t txl, tzl;
    int tny, tend;          // tend: the pass's ends
    uint64_t tzh;
    uint64_t minus;         // bit j: term j changes sign in this tile (z outside the tile)
    double acc0, acc1, acc2, acc3;
    double v0, v1, v2, v3;  // values of the last four terms
};

// Value of term j in this lane (the lane's part of the sum over the tile).
// Every fourth term the four are summed.
__device__ __forceinline__ void tile_push(TileTerms &T, int j, double v, uint32_t lane) {
    T.v0 = T.v1;
    T.v1 = T.v2;
    T.v2 = T.v3;
    T.v3 = v;
    if ((j & 3) == 3) {  // uniform
        double c = row_sum_over4(
            fold_pair<1>(fold_pair<0>(T.v0, T.v1, lane), fold_pair<0>(T.v2, T.v3, lane), lane));
        if ((lane >> 2 & 3u) == ((uint32_t)j >> 2 & 3u)) {
            c = (T.minus >> (j & 48) >> (lane & 15u)) & 1ull ? -c : c;
            // (one addend each: an index would put the sums into scratch memory)
            T.acc0 += j < 16 ? c : 0.0;
            T.acc1 += j >> 4 == 1 ? c : 0.0;
            T.acc2 += j >> 4 == 2 ? c : 0.0;
            T.acc3 += j >= 48 ? c : 0.0;
        }
    }
}

// Walsh transform over the register bits: v[s] <- sum_r (-1)^{popc(s & r)} v[r].
__device__ __forceinline__ void walsh16(double (&v)[kTilePerLane]) {
#pragma unroll
    for (int h = 1; h < kTilePerLane; h <<= 1)
#pragma unroll
        for (int r = 0; r < kTilePerLane; ++r)
            if (!(r & h)) {
                const double a = v[r], b = v[r | h];
                v[r] = a + b;
                v[r | h] = a - b;
            }
}

// A lane's 16 amplitudes t_r: sum over the pairs (r, r ^ X), the lowest bit of
// X clear in r, of (-1)^{zr.r} Re or Im conj(t_r) t_{r^X}.
template <int X>
__device__ __forceinline__ double reg_pairs(const double (&tr)[kTilePerLane], const double (&ti)[kTilePerLane], bool im,
                                            uint32_t zr) {
    constexpr int low = X & -X;
    double s = 0.0, q = 0.0;
    if (!im && zr == 0) {  // uniform; a product of X only
#pragma unroll
        for (int r = 0; r < kTilePerLane; ++r)
            if (!(r & low)) {
                s = __builtin_fma(tr[r], tr[r ^ X], s);
                q = __builtin_fma(ti[r], ti[r ^ X], q);
            }
        return s + q;
    }
#pragma unroll
    for (int r = 0; r < kTilePerLane; ++r)
        if (!(r & low)) {
            const double sg = (__popc(zr & (uint32_t)r) & 1) ? -1.0 : 1.0;  // uniform
            const double w = im ? tr[r] * ti[r ^ X] - ti[r] * tr[r ^ X] : tr[r] * tr[r ^ X] + ti[r] * ti[r ^ X];
            s = __builtin_fma(sg, w, s);
        }
    return s;
}

// f(std::integral_constant<int, I>) for the numbers of the sequence.
template <typename F, int... I>
__device__ __forceinline__ void unrolled(const F &f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}

// Every tile of the pass into LDS once, then, once the next tile's loads
// are issued, every term of the pass over it (each adds, over the pairs
// (l, l ^ xl) with the lowest bit of xl clear in l, twice
// (-1)^{zl.(l^xl)} Re(i^ny conj(t_l) t_{l^xl})):
//  - diagonal terms from a Walsh transform of the lane's |t|^2: the lane's sum
//    over l = tid | (r << 8) is (-1)^{zl.tid} times its coefficient at zl >> 8;
//  - terms whose x mask is one bit or two neighbours of a group of four
//    tile-local bits: the tile is read from LDS once per group, that group's
//    bits numbering a lane's registers, and their pairs are in registers;
//  - the other terms' pairs from LDS.
// A pass over 2^26 amplitudes takes 0.23 ms in complex128 and 0.16 in complex64
// with few terms (reading the state alone 0.18 and 0.14); a further term adds
// 1 to 7 us from registers (bound by FP64 arithmetic, two wavefronts per SIMD),
// 20 from LDS (by its bandwidth).  With both amplitudes of every pair read from
// LDS for every term, a sum over the wavefront for each, and six low qubits in
// every tile, the 51 terms of a chain model took four passes and 1.45 ms
// (complex64 1.35), now three and 0.86 (0.77); 20 strings of up to four
// operators 1.08 -> 0.78 ms.
template <typename A>
__global__ __launch_bounds__(kTileThreads, 2) void k_expect_tile(const A amps, const TilePass P,
                                                                 double *__restrict__ partials) {
    __shared__ double2 tile[1 << kTileBits];
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t M = 1u << P.m;
    const int L = P.L, nt = P.nt;
    const uint64_t ntiles = 1ull << P.nfree, himask = P.himask, frmask = P.frmask;
    // index bits on the tile's qubits of the lane's amplitudes l = tid | (r << 8):
    // those of tid, and those of r's bits (uniform)
    const uint32_t lt = min(tid, M - 1);
    const uint64_t off = (lt & ((1u << L) - 1)) | deposit_bits(lt >> L, himask);
    uint64_t rb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        rb[k] = 8 + k < P.m ? deposit_bits(1ull << (8 + k - L), himask) : 0;
    TileTerms T;
    T.txl = T.tzl = 0;
    T.tny = 0;
    T.tzh = 0;
    T.minus = 0;
    T.tend = lane < 37 ? P.end[lane] : 0;
    T.v0 = T.v1 = T.v2 = T.v3 = 0.0;
    // the same over the wavefront's tiles, and what adding them rounded off: a
    // term's rows may all have one sign in every tile and cancel between rows
    // (neighbours among qubits 4 to 7 had ten times the error of one sum per
    // wavefront and tile)
    double sum0 = 0.0, sum1 = 0.0, sum2 = 0.0, sum3 = 0.0, rest0 = 0.0, rest1 = 0.0, rest2 = 0.0, rest3 = 0.0;
    if ((int)lane < nt) {
        T.txl = P.t[lane].xl;
        T.tzl = P.t[lane].zl;
        T.tny = P.t[lane].ny;
        T.tzh = P.t[lane].zh;
    }
    typename A::Raw raw[kTilePerLane];
    auto load = [&](uint64_t t) {
        const uint64_t at = deposit_bits(t, frmask) | off;
#pragma unroll
        for (int r = 0; r < kTilePerLane; ++r)  // (past a small tile's end: an amplitude of it, unused)
            raw[r] = amps.raw(at | (r & 1 ? rb[0] : 0) | (r & 2 ? rb[1] : 0) | (r & 4 ? rb[2] : 0) | (r & 8 ? rb[3] : 0));
    };
    uint64_t tl = blockIdx.x;
    if (tl < ntiles)
        load(tl);
    for (; tl < ntiles; tl += gridDim.x) {
        const uint64_t base = deposit_bits(tl, frmask);
        __syncthreads();  // every read of the previous tile is done
        double wc[kTilePerLane];
#pragma unroll
        for (int r = 0; r < kTilePerLane; ++r) {
            const uint32_t l = tid | ((uint32_t)r << 8);
            double re = 0.0, im = 0.0;
            if (l < M)
                A::decode(raw[r], re, im);
            tile[tile_slot(l)] = make_double2(re, im);
            wc[r] = re * re + im * im;
        }
        __syncthreads();
        if (tl + gridDim.x < ntiles)
            load(tl + gridDim.x);
        T.minus = __ballot(odd_parity(T.tzh & base));
        T.acc0 = T.acc1 = T.acc2 = T.acc3 = 0.0;
        int j = 0;
        if (__builtin_amdgcn_readlane(T.tend, 15)) {
            walsh16(wc);
            unrolled([&](auto q) __attribute__((always_inline)) {
#pragma unroll 1
                for (const int end = __builtin_amdgcn_readlane(T.tend, q); j < end; ++j) {
                    const uint32_t zl = (uint32_t)__builtin_amdgcn_readlane((int)T.tzl, j);
                    tile_push(T, j, (__popc(zl & tid) & 1) ? -wc[q] : wc[q], lane);
                }
            }, std::make_integer_sequence<int, kTilePerLane>());
        }
#pragma unroll 1
        for (int p = 0; p < 3; ++p) {
            if (j == __builtin_amdgcn_readlane(T.tend, 16 + 7 * p + 6))
                continue;  // uniform
            const int sh = 8 - 4 * p;
            // tid's bits around the register bits sh .. sh + 3
            const uint32_t l0 = ((tid >> sh) << (sh + 4)) | (tid & ((1u << sh) - 1u));
            double tr[kTilePerLane], ti[kTilePerLane];
#pragma unroll
            for (int r = 0; r < kTilePerLane; ++r) {
                const double2 t = tile[tile_slot(l0) ^ tile_slot((uint32_t)r << sh)];
                tr[r] = t.x;
                ti[r] = t.y;
            }
            unrolled([&](auto k) __attribute__((always_inline)) {
                constexpr int X = kRegMasks[k];
#pragma unroll 1
                for (const int end = __builtin_amdgcn_readlane(T.tend, 16 + 7 * p + k); j < end; ++j) {
                    // (not known to the compiler, which would otherwise form
                    // every kind of product ahead of the loop)
#pragma unroll
                    for (int r = 0; r < kTilePerLane; ++r)
                        asm volatile("" : "+v"(tr[r]), "+v"(ti[r]));
                    const uint32_t zl = (uint32_t)__builtin_amdgcn_readlane((int)T.tzl, j);
                    const int ny = __builtin_amdgcn_readlane(T.tny, j);
                    const double s = reg_pairs<X>(tr, ti, ny & 1, (zl >> sh) & 15u);
                    // Re(i^ny w): ny = 0, 1, 2, 3 give Re w, -Im w, -Re w, Im w
                    const bool neg =
                        (ny == 1 || ny == 2) != (bool)(__popc(zl & (l0 ^ ((uint32_t)X << sh))) & 1);
                    tile_push(T, j, neg ? -2.0 * s : 2.0 * s, lane);
                }
            }, std::make_integer_sequence<int, 7>());
        }
#pragma unroll 1
        for (; j < nt; ++j) {
            const uint32_t xl = (uint32_t)__builtin_amdgcn_readlane((int)T.txl, j);
            const uint32_t zl = (uint32_t)__builtin_amdgcn_readlane((int)T.tzl, j);
            const int ny = __builtin_amdgcn_readlane(T.tny, j);
            const uint32_t b = (uint32_t)__builtin_ctz(xl), sx = tile_slot(xl);
            const uint32_t l0 = ((tid >> b) << (b + 1)) | (tid & ((1u << b) - 1)), s0 = tile_slot(l0);
            const bool im = ny & 1;
            double s = 0.0;
#pragma unroll
            for (uint32_t r = 0; r < (uint32_t)kTilePerLane / 2; ++r) {
                const uint32_t ir = r << 8;  // pair number tid | ir; a cleared bit goes in linearly over xor
                const uint32_t lr = ((ir >> b) << (b + 1)) | (ir & ((1u << b) - 1));
                const uint32_t at = s0 ^ tile_slot(lr);
                const double2 u = tile[at], v = tile[at ^ sx];
                const double w = im ? u.x * v.y - u.y * v.x : u.x * v.x + u.y * v.y;
                s = __builtin_fma((__popc(zl & lr) & 1) ? -1.0 : 1.0, w, s);
            }
            const bool neg = (ny == 1 || ny == 2) != (bool)(__popc(zl & (l0 ^ xl)) & 1);
            tile_push(T, j, neg ? -2.0 * s : 2.0 * s, lane);
        }
        for (; j & 3; ++j)
            tile_push(T, j, 0.0, lane);
        add_exact(sum0, rest0, T.acc0);
        add_exact(sum1, rest1, T.acc1);
        add_exact(sum2, rest2, T.acc2);
        add_exact(sum3, rest3, T.acc3);
    }
    __syncthreads();  // the tile's LDS now holds the rows' sums
    double2 *wsum = reinterpret_cast<double2 *>(tile);
    double2 *row = wsum + (tid >> 4) * kTileTerms + (tid & 15u);
    row[0] = make_double2(sum0, rest0);
    row[16] = make_double2(sum1, rest1);
    row[32] = make_double2(sum2, rest2);
    row[48] = make_double2(sum3, rest3);
    __syncthreads();
    if ((int)tid < nt) {
        double2 w[kTileThreads / 16];
#pragma unroll
        for (int q = 0; q < kTileThreads / 16; ++q)
            w[q] = wsum[q * kTileTerms + tid];
#pragma unroll
        for (int h = 1; h < kTileThreads / 16; h <<= 1)
#pragma unroll
            for (int q = 0; q < kTileThreads / 16; q += 2 * h) {
                w[q].y += w[q + h].y;
                add_exact(w[q].x, w[q].y, w[q + h].x);
            }
        partials[(size_t)P.t[tid].slot * kMaxPartials + blockIdx.x] = with_rest(w[0].x, w[0].y);
    }
}

// Every term's sum of its partials, one workgroup per term (plan order,
// each in the fixed order of block_sum_array).
__global__ __launch_bounds__(kRedThreads) void k_expect_sums(const int32_t *__restrict__ nblk,
                                                             const double *__restrict__ partials,
                                                             double *__restrict__ sums) {
    __shared__ double red[kRedThreads / 64];
    const int j = blockIdx.x;
    const double s = block_sum_array(partials + (size_t)j * kMaxPartials, nblk[j], red);
    if (threadIdx.x == 0)
        sums[j] = s;
}

// Per-term values in the caller's order, and the coefficient-weighted total
// summed in plan order by one lane.
__global__ __launch_bounds__(64) void k_expect_final(const DTerm *__restrict__ terms, int nterms,
                                                     const double *__restrict__ sums, double *__restrict__ out_total,
                                                     double *__restrict__ out_terms) {
    if (out_terms)
        for (int j = threadIdx.x; j < nterms; j += blockDim.x)
            out_terms[terms[j].idx] = sums[j];
    if (threadIdx.x == 0 && out_total) {
        double total = 0.0;
        for (int j = 0; j < nterms; ++j)
            total += terms[j].coef * sums[j];
        out_total[0] = total;
    }
}

// Both for few terms, whose table comes as a kernel argument: one workgroup, a
// wavefront per term (its partials in index order by lanes).  Small states
// spend their time in launches and copies: with the tables copied to the device
// and two kernels a call at 8 to 20 qubits took 72 to 79 us, now 31 to 40; one
// at 26 qubits 861 and 839.
constexpr int kFewTerms = SV_EXPECT_NOALLOC_MAX_TERMS, kFewThreads = 1024;
struct FewTerms {
    int32_t nterms, nblk[kFewTerms], idx[kFewTerms];
    double coef[kFewTerms];
};
__global__ __launch_bounds__(kFewThreads) void k_expect_few(const FewTerms t, const double *__restrict__ partials,
                                                            double *__restrict__ out_total,
                                                            double *__restrict__ out_terms) {
    __shared__ double sums[kFewTerms];
    const int lane = threadIdx.x & 63;
    for (int j = threadIdx.x >> 6; j < t.nterms; j += kFewThreads / 64) {
        // What the additions round off is kept beside the sum.  (The partials of
        // a term may be all of one sign in a lane and cancel between lanes: plain
        // sums left up to twice the error of the partials themselves.)
        double v = 0.0, e = 0.0;
#pragma unroll 8
        for (int i = lane; i < t.nblk[j]; i += 64)
            add_exact(v, e, partials[(size_t)j * kMaxPartials + i]);
#pragma unroll
        for (int h = 1; h < 64; h <<= 1) {
            e += __shfl_xor(e, h);
            add_exact(v, e, __shfl_xor(v, h));
        }
        v = with_rest(v, e);
        if (lane == 0) {
            sums[j] = v;
            if (out_terms)
                out_terms[t.idx[j]] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && out_total) {
        double total = 0.0;
        for (int j = 0; j < t.nterms; ++j)
            total += t.coef[j] * sums[j];
        out_total[0] = total;
    }
}

// out_k = sum_groups sum_terms coef i^ny (-1)^{z.(k^X)} psi_{k^X}; partials
// of Re conj(psi_k) out_k per workgroup.  47 terms (25 x masks) on 2^24
// complex128 amplitudes: 766 us when every sign was a 64-bit parity and both
// parts of the factor were summed, 597 now; the partner loads bound it.
template <typename R, typename I>
__global__ __launch_bounds__(kRedThreads) void k_apply_paulis(const cplx_t<R> *__restrict__ psi,
                                                              cplx_t<R> *__restrict__ out, uint64_t N,
                                                              const DGroup *__restrict__ groups, int ngroups,
                                                              const DTerm *__restrict__ terms,
                                                              double *__restrict__ partials) {
    __shared__ double red[kRedThreads / 64];
    double lp = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * kRedThreads;
    for (uint64_t k = (uint64_t)blockIdx.x * kRedThreads + threadIdx.x; k < N; k += stride) {
        double ar = 0.0, ai = 0.0;
        for (int g = 0; g < ngroups; ++g) {
            const DGroup G = groups[g];
            const uint64_t kx = k ^ G.x;
            const cplx_t<R> v = psi[kx];
            double cr = 0.0, ci = 0.0;  // sum over the group's terms of coef i^ny (-1)^{z.kx}
            for (int j = G.first; j < G.first + G.count; ++j) {
                const DTerm T = terms[j];
                add_term<I>(T, kx, cr, ci);
            }
            ar += cr * (double)v.x - ci * (double)v.y;
            ai += cr * (double)v.y + ci * (double)v.x;
        }
        cplx_t<R> o;
        o.x = (R)ar;
        o.y = (R)ai;
        out[k] = o;
        const cplx_t<R> p = psi[k];
        lp += (double)p.x * ar + (double)p.y * ai;
    }
    const double s = block_sum(lp, red);
    if (threadIdx.x == 0 && partials)
        partials[blockIdx.x] = s;
}

int launch_apply_paulis(int dtype, const void *psi, void *out, int n, const PauliDevice &d, hipStream_t st,
                        unsigned *grid) {
    const uint64_t N = 1ull << n;
    const unsigned g = reduce_grid(N);
    auto go = [&](auto fn, auto *in, auto *to) {
        hipLaunchKernelGGL(fn, dim3(g), dim3(kRedThreads), 0, st, in, to, N, d.groups, d.ngroups, d.terms, d.partials);
    };
    if (dtype == SV_C128)
        n <= 32 ? go(k_apply_paulis<double, uint32_t>, (const double2 *)psi, (double2 *)out)
                : go(k_apply_paulis<double, uint64_t>, (const double2 *)psi, (double2 *)out);
    else
        n <= 32 ? go(k_apply_paulis<float, uint32_t>, (const float2 *)psi, (float2 *)out)
                : go(k_apply_paulis<float, uint64_t>, (const float2 *)psi, (float2 *)out);
    SV_LAUNCH_CHECK();
    if (grid)
        *grid = g;
    return SV_OK;
}


// The passes of one expectation call: tile passes for the terms whose x
// mask fits a tile set, one pass per group for the rest, and every plan
// term's partial count (the grid of the pass that evaluates it).
struct ExpectPlan {
    PauliPlan pp;
    std::vector<TilePass> tiles;
    std::vector<DGroup> rest;
    std::vector<int32_t> nblk;
    unsigned tile_grid = 0;
};

// mask's bits on the tile's qubits (0..L-1 and himask) as tile-local bits,
// and its other bits.
static void tile_split(uint64_t mask, int L, uint64_t himask, uint32_t *local, uint64_t *outside) {
    const uint64_t lowm = (1ull << L) - 1;
    uint32_t l = (uint32_t)(mask & lowm);
    int q = 0;
    for (uint64_t h = himask; h; h &= h - 1, ++q)
        if (mask & h & (~h + 1ull))
            l |= 1u << (L + q);
    *local = l;
    *outside = mask & ~lowm & ~himask;
}

static int make_expect_plan(int n, int dtype, const sv_pauli_t *terms, int nterms, ExpectPlan *e) {
    SV_TRY(make_pauli_plan(n, terms, nterms, &e->pp));
    const PauliPlan &pp = e->pp;
    e->tiles.clear();
    e->rest.clear();
    e->nblk.assign(pp.terms.size(), 0);
    const int low = dtype == SV_C128 ? CplxAmps<double>::kLow
                    : dtype == SV_C64 ? CplxAmps<float>::kLow
                    : dtype == SV_CQ16 ? Q16Amps::kLow
                                       : Q32Amps::kLow;
    const int m = std::min(n, kTileBits), L = std::min(m, low), nh = m - L;
    const uint64_t lowm = (1ull << L) - 1;
    DeviceInfo di;
    const uint64_t cus = device_info(&di) == SV_OK ? (uint64_t)di.num_cus : 256;
    e->tile_grid = (unsigned)std::min<uint64_t>({1ull << (n - m), 2 * cus, (uint64_t)kMaxPartials});
    // tile sets (qubits above L), first fit; the first is qubits L..m-1
    std::vector<uint64_t> sets{((1ull << m) - 1) & ~lowm};
    std::vector<std::vector<int>> members(1);
    for (int gi = 0; gi < (int)pp.groups.size(); ++gi) {
        const DGroup &g = pp.groups[gi];
        const uint64_t h = g.x & ~lowm;
        int at = -1;
        for (size_t k = 0; k < sets.size() && at < 0; ++k)
            if (popcount64(sets[k] | h) <= nh)
                at = (int)k;
        if (at < 0 && popcount64(h) <= nh) {
            sets.push_back(0);
            members.emplace_back();
            at = (int)sets.size() - 1;
        }
        if (at < 0) {  // too many qubits above L for one tile
            e->rest.push_back(g);
            for (int j = g.first; j < g.first + g.count; ++j)
                e->nblk[j] = (int32_t)reduce_grid(g.x == 0 ? (1ull << n) : (1ull << (n - 1)));
            continue;
        }
        sets[at] |= h;
        members[at].push_back(gi);
    }
    for (size_t k = 0; k < sets.size(); ++k) {
        if (members[k].empty())
            continue;
        uint64_t set = sets[k];
        for (int q = L; q < n && popcount64(set) < nh; ++q)  // fill up with the lowest unused qubits
            set |= 1ull << q;
        TilePass P;
        memset(&P, 0, sizeof(P));
        P.m = m;
        P.L = L;
        P.nfree = n - m;
        P.himask = set;
        P.frmask = ((n >= 64) ? ~0ull : ((1ull << n) - 1)) & ~lowm & ~set;
        for (int gi : members[k]) {
            const DGroup &g = pp.groups[gi];
            for (int j = g.first; j < g.first + g.count; ++j) {
                if (P.nt == kTileTerms) {
                    e->tiles.push_back(P);
                    P.nt = 0;
                }
                TTerm &T = P.t[P.nt++];
                uint64_t xo = 0, zh = 0;
                tile_split(g.x, L, P.himask, &T.xl, &xo);
                tile_split(pp.terms[j].z, L, P.himask, &T.zl, &zh);
                if (xo)
                    return fail(SV_EINVAL, "internal: x mask 0x%llx outside its tile set", (unsigned long long)g.x);
                T.zh = zh;
                T.ny = pp.terms[j].ny;
                T.slot = j;
                e->nblk[j] = (int32_t)e->tile_grid;
            }
        }
        if (P.nt)
            e->tiles.push_back(P);
    }
    for (TilePass &P : e->tiles) {
        // place of a term in the pass's order: 0..15 diagonal, 16.. register
        // groups and masks, 37 the others
        auto place = [](const TTerm &t) {
            if (t.xl == 0)
                return (int)(t.zl >> 8);
            for (int p = 0; p < 3; ++p)
                for (int k = 0; k < 7; ++k)
                    if (t.xl == (uint32_t)kRegMasks[k] << (8 - 4 * p))
                        return 16 + 7 * p + k;
            return 37;
        };
        std::stable_sort(P.t, P.t + P.nt, [&](const TTerm &a, const TTerm &b) { return place(a) < place(b); });
        for (int j = 0; j < P.nt; ++j)
            for (int at = place(P.t[j]); at < 37; ++at)
                P.end[at] = j + 1;
    }
    return SV_OK;
}

// f(amps) with the state's amplitude source.
template <typename F> static void with_amps(const sv_state_t *s, F &&f) {
    const char *base = static_cast<const char *>(s->data);
    const int8_t *scales = reinterpret_cast<const int8_t *>(base + (((size_t)1 << s->n) * amp_bytes(s->dtype)));
    switch (s->dtype) {
    case SV_C128:
        f(CplxAmps<double>{(const double2 *)base});
        break;
    case SV_C64:
        f(CplxAmps<float>{(const float2 *)base});
        break;
    case SV_CQ16:
        f(Q16Amps{(const uint32_t *)base, scales});
        break;
    default:
        f(Q32Amps{(const uint2 *)base, scales});
        break;
    }
}

// The passes: every plan term's partial sums, plan.nblk[j] of them at
// partials[j * kMaxPartials].
static int expect_passes(const sv_state_t *s, const ExpectPlan &plan, double *partials, hipStream_t st) {
    const int n = s->n;
    for (const TilePass &P : plan.tiles) {
        with_amps(s, [&](auto amps) {
            using A = decltype(amps);
            hipLaunchKernelGGL((k_expect_tile<A>), dim3(plan.tile_grid), dim3(kTileThreads), 0, st, amps, P,
                               partials);
        });
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return fail(SV_EHIP, "expectation launch failed: %s", hipGetErrorString(e));
    }
    for (const DGroup &g : plan.rest) {
        const uint64_t count = g.x == 0 ? (1ull << n) : (1ull << (n - 1));
        const unsigned grid = reduce_grid(count);
        const uint32_t b = g.x ? (uint32_t)__builtin_ctzll(g.x) : 0;
        GroupTerms t;
        memset(&t, 0, sizeof(t));
        for (int j = 0; j < g.count; ++j) {
            t.z[j] = plan.pp.terms[g.first + j].z;
            t.ny[j] = plan.pp.terms[g.first + j].ny;
        }
        with_amps(s, [&](auto amps) {
            using A = decltype(amps);
            hipLaunchKernelGGL((k_expect_group<A>), dim3(grid), dim3(kRedThreads), 0, st, amps, count, g.x, b, t,
                               g.first, g.count, partials);
        });
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return fail(SV_EHIP, "expectation launch failed: %s", hipGetErrorString(e));
    }
    return SV_OK;
}

// Passes and sums for at most kFewTerms terms.
static int expect_few(const sv_state_t *s, const ExpectPlan &plan, double *partials, double *out_total,
                      double *out_terms, hipStream_t st) {
    SV_TRY(expect_passes(s, plan, partials, st));
    FewTerms t;
    memset(&t, 0, sizeof(t));
    t.nterms = (int32_t)plan.pp.terms.size();
    for (int j = 0; j < t.nterms; ++j) {
        t.nblk[j] = plan.nblk[j];
        t.idx[j] = plan.pp.terms[j].idx;
        t.coef[j] = plan.pp.terms[j].coef;
    }
    hipLaunchKernelGGL(k_expect_few, dim3(1), dim3(kFewThreads), 0, st, t, partials, out_total, out_terms);
    SV_LAUNCH_CHECK();
    return SV_OK;
}

static int expect_impl(const sv_state_t *s, const sv_pauli_t *terms, int nterms, double *out_total,
                       double *out_terms, hipStream_t st) {
    SV_TRY(validate_state(s, true));
    ExpectPlan plan;
    SV_TRY(make_expect_plan(s->n, s->dtype, terms, nterms, &plan));
    const size_t nt = plan.pp.terms.size();
    auto alloc = [&](void **p, size_t bytes) -> int {
        hipError_t e = hipMallocAsync(p, bytes, st);
        if (e == hipSuccess)
            return SV_OK;
        (void)hipGetLastError();
        *p = nullptr;
        return fail(SV_ENOMEM, "device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    };
    if (nt <= (size_t)kFewTerms) {
        double *partials = nullptr;
        SV_TRY(alloc((void **)&partials, nt * kMaxPartials * sizeof(double)));
        const int r = expect_few(s, plan, partials, out_total, out_terms, st);
        (void)hipFreeAsync(partials, st);
        return r;
    }
    PauliDevice d;
    SV_TRY(pauli_upload(plan.pp, nt * (kMaxPartials + 1), st, &d));
    int32_t *nblk = nullptr;
    int r = alloc((void **)&nblk, nt * sizeof(int32_t));
    if (r == SV_OK) {
        hipError_t e = hipMemcpyAsync(nblk, plan.nblk.data(), nt * sizeof(int32_t), hipMemcpyHostToDevice, st);
        if (e != hipSuccess)
            r = fail(SV_EHIP, "copy failed: %s", hipGetErrorString(e));
    }
    if (r == SV_OK)
        r = expect_passes(s, plan, d.partials, st);
    if (r == SV_OK) {
        double *sums = d.partials + nt * kMaxPartials;
        hipLaunchKernelGGL(k_expect_sums, dim3((unsigned)nt), dim3(kRedThreads), 0, st, nblk, d.partials, sums);
        hipLaunchKernelGGL(k_expect_final, dim3(1), dim3(64), 0, st, d.terms, (int)nt, sums, out_total, out_terms);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            r = fail(SV_EHIP, "expectation launch failed: %s", hipGetErrorString(e));
    }
    if (nblk)
        (void)hipFreeAsync(nblk, st);
    pauli_release(&d, st);
    return r;
}

// ---------------------------------------------------------------------------
// Allocation-free expectation.  The partial sums live in one file-scope
// device array.  Host code never passes the array's name to a kernel: its
// device address is looked up once per device with hipGetSymbolAddress and
// kept.  The term tables travel as kernel arguments (no host-to-device copy),
// and every partial a call reads is written by that call first, so nothing
// needs clearing.  Every call on one device shares the array: calls that
// overlap on one device race.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[(size_t)kFewTerms * kMaxPartials * sizeof(double)];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices];

// Device address of the scratch array on the current device (looked up on
// the first call per device).
static int scratch_address(double **out) {
    int dev = 0;
    SV_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(SV_ENOTSUP, "device %d beyond the %d devices the scratch table holds", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(SV_EHIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<double *>(g_scratch_ptr[dev]);
    return SV_OK;
}

static int expect_noalloc_impl(const sv_state_t *s, const sv_pauli_t *terms, int nterms, double *out_total,
                               hipStream_t st) {
    SV_TRY(validate_state(s, true));
    if (nterms > kFewTerms)
        return fail(SV_EINVAL, "nterms %d exceeds the allocation-free limit of %d terms", nterms, kFewTerms);
    ExpectPlan plan;
    SV_TRY(make_expect_plan(s->n, s->dtype, terms, nterms, &plan));
    double *partials = nullptr;
    SV_TRY(scratch_address(&partials));
    return expect_few(s, plan, partials, out_total, nullptr, st);
}

} // namespace sv

using namespace sv;

extern "C" {

int sv_expect(const sv_state_t *s, const sv_pauli_t *terms, int nterms, double *out_dev, sv_stream_t st) {
    clear_error();
    if (!out_dev)
        return fail(SV_EINVAL, "out_dev is NULL");
    return expect_impl(s, terms, nterms, out_dev, nullptr, (hipStream_t)st);
}

int sv_expect_noalloc(const sv_state_t *s, const sv_pauli_t *terms, int nterms, double *out_dev, sv_stream_t st) {
    clear_error();
    if (!out_dev)
        return fail(SV_EINVAL, "out_dev is NULL");
    return expect_noalloc_impl(s, terms, nterms, out_dev, (hipStream_t)st);
}

int sv_expect_terms(const sv_state_t *s, const sv_pauli_t *terms, int nterms, double *out_dev, sv_stream_t st) {
    clear_error();
    if (!out_dev)
        return fail(SV_EINVAL, "out_dev is NULL");
    return expect_impl(s, terms, nterms, nullptr, out_dev, (hipStream_t)st);
}

int sv_apply_pauli_sum(const sv_state_t *in, const sv_state_t *out, const sv_pauli_t *terms, int nterms,
                       sv_stream_t st) {
    clear_error();
    SV_TRY(validate_state(in));
    SV_TRY(validate_state(out));
    if (in->n != out->n || in->dtype != out->dtype)
        return fail(SV_EINVAL, "states differ in size or dtype");
    if (in->data == out->data)
        return fail(SV_EINVAL, "in and out must not alias");
    PauliPlan plan;
    SV_TRY(make_pauli_plan(in->n, terms, nterms, &plan));
    PauliDevice d;
    SV_TRY(pauli_upload(plan, 0, (hipStream_t)st, &d));
    const int r = launch_apply_paulis(in->dtype, in->data, out->data, in->n, d, (hipStream_t)st, nullptr);
    pauli_release(&d, (hipStream_t)st);
    return r;
}

} // extern "C"
