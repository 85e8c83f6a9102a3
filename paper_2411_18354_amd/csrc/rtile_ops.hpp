// The gate operations of the register tile pass (rtile.hpp) on a lane's
// amplitudes, as one block of instructions per call.
//
// Written as instructions because the amplitudes have to stay where they are:
// 64 registers live through every branch of an interpreter loop leave the
// compiler's allocator copying and spilling at each operation (measured: 130
// to 800 spilled registers of 128), while operands tied to the block cannot
// move.  The block jumps by operation code to one of its variants (a kind and
// a register bit), which updates the pairs, or registers, of its mask under
// the lanes' condition.
//
// The rounding of each update is that of apply_pair (gate_math.hpp), products
// with an entry known to be zero left out (with finite amplitudes they change
// nothing; an infinite one stays infinite where 0 times it would be NaN).
#pragma once

#include "gate_math.hpp"

namespace sv {

// One step of a pair (x, y): operands are named x<i>, y<i> (real and
// imaginary part of register i); t0 .. t3 are scratch; ar .. di the matrix.
#define RT_N(c, i) "%[" #c #i "]"
#define RT_STEP_REAL(SZ, i, j)                                                                                     \
    "v_mul_" SZ " %[t0], %[br], " RT_N(x, j) "\n"                                                                  \
    "v_mul_" SZ " %[t1], %[br], " RT_N(y, j) "\n"                                                                  \
    "v_mul_" SZ " " RT_N(x, j) ", %[dr], " RT_N(x, j) "\n"                                                         \
    "v_mul_" SZ " " RT_N(y, j) ", %[dr], " RT_N(y, j) "\n"                                                         \
    "v_fma_" SZ " " RT_N(x, j) ", %[cr], " RT_N(x, i) ", " RT_N(x, j) "\n"                                         \
    "v_fma_" SZ " " RT_N(y, j) ", %[cr], " RT_N(y, i) ", " RT_N(y, j) "\n"                                         \
    "v_fma_" SZ " " RT_N(x, i) ", %[ar], " RT_N(x, i) ", %[t0]\n"                                                  \
    "v_fma_" SZ " " RT_N(y, i) ", %[ar], " RT_N(y, i) ", %[t1]\n"
#define RT_STEP_CROSS(SZ, i, j)                                                                                    \
    "v_mul_" SZ " %[t0], %[bi], " RT_N(y, j) "\n"                                                                  \
    "v_mul_" SZ " %[t1], %[bi], " RT_N(x, j) "\n"                                                                  \
    "v_mul_" SZ " " RT_N(x, j) ", %[dr], " RT_N(x, j) "\n"                                                         \
    "v_mul_" SZ " " RT_N(y, j) ", %[dr], " RT_N(y, j) "\n"                                                         \
    "v_fma_" SZ " " RT_N(x, j) ", -%[ci], " RT_N(y, i) ", " RT_N(x, j) "\n"                                        \
    "v_fma_" SZ " " RT_N(y, j) ", %[ci], " RT_N(x, i) ", " RT_N(y, j) "\n"                                         \
    "v_fma_" SZ " " RT_N(x, i) ", %[ar], " RT_N(x, i) ", -%[t0]\n"                                                 \
    "v_fma_" SZ " " RT_N(y, i) ", %[ar], " RT_N(y, i) ", %[t1]\n"
#define RT_STEP_GEN(SZ, i, j)                                                                                      \
    "v_mul_" SZ " %[t0], %[bi], " RT_N(y, j) "\n"                                                                  \
    "v_mul_" SZ " %[t1], %[bi], " RT_N(x, j) "\n"                                                                  \
    "v_mul_" SZ " %[t2], %[di], " RT_N(y, j) "\n"                                                                  \
    "v_mul_" SZ " %[t3], %[di], " RT_N(x, j) "\n"                                                                  \
    "v_fma_" SZ " %[t0], %[br], " RT_N(x, j) ", -%[t0]\n"                                                          \
    "v_fma_" SZ " %[t1], %[br], " RT_N(y, j) ", %[t1]\n"                                                           \
    "v_fma_" SZ " " RT_N(x, j) ", %[dr], " RT_N(x, j) ", -%[t2]\n"                                                 \
    "v_fma_" SZ " " RT_N(y, j) ", %[dr], " RT_N(y, j) ", %[t3]\n"                                                  \
    "v_fma_" SZ " %[t0], -%[ai], " RT_N(y, i) ", %[t0]\n"                                                          \
    "v_fma_" SZ " %[t1], %[ai], " RT_N(x, i) ", %[t1]\n"                                                           \
    "v_fma_" SZ " " RT_N(x, j) ", -%[ci], " RT_N(y, i) ", " RT_N(x, j) "\n"                                        \
    "v_fma_" SZ " " RT_N(y, j) ", %[ci], " RT_N(x, i) ", " RT_N(y, j) "\n"                                         \
    "v_fma_" SZ " " RT_N(x, j) ", %[cr], " RT_N(x, i) ", " RT_N(x, j) "\n"                                         \
    "v_fma_" SZ " " RT_N(y, j) ", %[cr], " RT_N(y, i) ", " RT_N(y, j) "\n"                                         \
    "v_fma_" SZ " " RT_N(x, i) ", %[ar], " RT_N(x, i) ", %[t0]\n"                                                  \
    "v_fma_" SZ " " RT_N(y, i) ", %[ar], " RT_N(y, i) ", %[t1]\n"
#define RT_STEP_SWAP_f64(i, j)                                                                                     \
    "v_mov_b64 %[t0], " RT_N(x, i) "\n"                                                                            \
    "v_mov_b64 %[t1], " RT_N(y, i) "\n"                                                                            \
    "v_mov_b64 " RT_N(x, i) ", " RT_N(x, j) "\n"                                                                   \
    "v_mov_b64 " RT_N(y, i) ", " RT_N(y, j) "\n"                                                                   \
    "v_mov_b64 " RT_N(x, j) ", %[t0]\n"                                                                            \
    "v_mov_b64 " RT_N(y, j) ", %[t1]\n"
#define RT_STEP_SWAP_f32(i, j)                                                                                     \
    "v_swap_b32 " RT_N(x, i) ", " RT_N(x, j) "\n"                                                                  \
    "v_swap_b32 " RT_N(y, i) ", " RT_N(y, j) "\n"
// one register times a factor
#define RT_STEP_MUL(SZ, i, fr, fi)                                                                                 \
    "v_mul_" SZ " %[t0], %[" #fi "], " RT_N(y, i) "\n"                                                             \
    "v_mul_" SZ " %[t1], %[" #fi "], " RT_N(x, i) "\n"                                                             \
    "v_fma_" SZ " " RT_N(x, i) ", %[" #fr "], " RT_N(x, i) ", -%[t0]\n"                                            \
    "v_fma_" SZ " " RT_N(y, i) ", %[" #fr "], " RT_N(y, i) ", %[t1]\n"

// one register times its own factor, read from the table at byte address ta
// (two components of SB bytes each)
#define RT_STEP_TAB(SZ, RD, i, off0, off1)                                                                         \
    RD " %[t2], %[ta] offset:" #off0 "\n" RD " %[t3], %[ta] offset:" #off1 "\n"                                    \
    "s_waitcnt lgkmcnt(0)\n"                                                                                       \
    "v_mul_" SZ " %[t0], %[t3], " RT_N(y, i) "\n"                                                                  \
    "v_mul_" SZ " %[t1], %[t3], " RT_N(x, i) "\n"                                                                  \
    "v_fma_" SZ " " RT_N(x, i) ", %[t2], " RT_N(x, i) ", -%[t0]\n"                                                 \
    "v_fma_" SZ " " RT_N(y, i) ", %[t2], " RT_N(y, i) ", %[t1]\n"

// Gradient terms of a reverse sweep, where registers i, j are psi and I, J the
// same amplitudes of lambda: sums over pairs (or registers) into a0 .. a3; the
// term is (a0 + a1) - (a2 + a3).
#define RT_DOT_f64(a, p, q) "v_fma_f64 %[" #a "], " p ", " q ", %[" #a "]\n"
// Re(conj(lambda_1) psi_0) - Re(conj(lambda_0) psi_1)
#define RT_STEP_GY(D, i, j, I, J)                                                                                  \
    D(a0, RT_N(x, J), RT_N(x, i)) D(a1, RT_N(y, J), RT_N(y, i)) D(a2, RT_N(x, I), RT_N(x, j))                      \
    D(a3, RT_N(y, I), RT_N(y, j))
// Im(conj(lambda_0) psi_1) + Im(conj(lambda_1) psi_0)
#define RT_STEP_GX(D, i, j, I, J)                                                                                  \
    D(a0, RT_N(x, I), RT_N(y, j)) D(a1, RT_N(x, J), RT_N(y, i)) D(a2, RT_N(y, I), RT_N(x, j))                      \
    D(a3, RT_N(y, J), RT_N(x, i))
// Im(conj(lambda) psi), added for the registers of pm, subtracted for pm2
#define RT_STEP_GD(D, i, I) D(a0, RT_N(x, I), RT_N(y, i)) D(a2, RT_N(y, I), RT_N(x, i))
#define RT_STEP_GE(D, i, I) D(a3, RT_N(x, I), RT_N(y, i)) D(a1, RT_N(y, I), RT_N(x, i))

#define RT_REAL_f64(i, j) RT_STEP_REAL("f64", i, j)
#define RT_REAL_f32(i, j) RT_STEP_REAL("f32", i, j)
#define RT_CROSS_f64(i, j) RT_STEP_CROSS("f64", i, j)
#define RT_CROSS_f32(i, j) RT_STEP_CROSS("f32", i, j)
#define RT_GEN_f64(i, j) RT_STEP_GEN("f64", i, j)
#define RT_GEN_f32(i, j) RT_STEP_GEN("f32", i, j)
#define RT_SWAP_f64(i, j) RT_STEP_SWAP_f64(i, j)
#define RT_SWAP_f32(i, j) RT_STEP_SWAP_f32(i, j)
#define RT_MUL_f64(i) RT_STEP_MUL("f64", i, fr, fi)
#define RT_MUL_f32(i) RT_STEP_MUL("f32", i, t2, t3)

// Step of pair p = (i, j), skipped where the mask's bit is clear.
#define RT_PAIR(OP, V, p, i, j)                                                                                    \
    "s_bitcmp1_b32 %[pm], " #p "\n"                                                                                \
    "s_cbranch_scc0 .Lrt_" V "_" #p "_%=\n" OP(i, j) ".Lrt_" V "_" #p "_%=:\n"
// the same where every pair is meant: no test per pair (a test and branch
// cost a wavefront about 30 cycles beside the 32 of a real pair's update)
#define RT_FULL(OP, V, p, i, j) OP(i, j)
#define RT_REG(OP, i)                                                                                              \
    "s_bitcmp1_b32 %[pm], " #i "\n"                                                                                \
    "s_cbranch_scc0 .Lrt_mul_" #i "_%=\n" OP(i) ".Lrt_mul_" #i "_%=:\n"

// The pairs of register bit T among 8 registers, in pair order.
#define RT_PAIRS3_0(P, F, V) P(F, V, 0, 0, 1) P(F, V, 1, 2, 3) P(F, V, 2, 4, 5) P(F, V, 3, 6, 7)
#define RT_PAIRS3_1(P, F, V) P(F, V, 0, 0, 2) P(F, V, 1, 1, 3) P(F, V, 2, 4, 6) P(F, V, 3, 5, 7)
#define RT_PAIRS3_2(P, F, V) P(F, V, 0, 0, 4) P(F, V, 1, 1, 5) P(F, V, 2, 2, 6) P(F, V, 3, 3, 7)
// among 16
#define RT_PAIRS4_0(P, F, V)                                                                                          \
    P(F, V, 0, 0, 1) P(F, V, 1, 2, 3) P(F, V, 2, 4, 5) P(F, V, 3, 6, 7)                    \
    P(F, V, 4, 8, 9) P(F, V, 5, 10, 11) P(F, V, 6, 12, 13) P(F, V, 7, 14, 15)
#define RT_PAIRS4_1(P, F, V)                                                                                          \
    P(F, V, 0, 0, 2) P(F, V, 1, 1, 3) P(F, V, 2, 4, 6) P(F, V, 3, 5, 7)                    \
    P(F, V, 4, 8, 10) P(F, V, 5, 9, 11) P(F, V, 6, 12, 14) P(F, V, 7, 13, 15)
#define RT_PAIRS4_2(P, F, V)                                                                                          \
    P(F, V, 0, 0, 4) P(F, V, 1, 1, 5) P(F, V, 2, 2, 6) P(F, V, 3, 3, 7)                    \
    P(F, V, 4, 8, 12) P(F, V, 5, 9, 13) P(F, V, 6, 10, 14) P(F, V, 7, 11, 15)
#define RT_PAIRS4_3(P, F, V)                                                                                          \
    P(F, V, 0, 0, 8) P(F, V, 1, 1, 9) P(F, V, 2, 2, 10) P(F, V, 3, 3, 11)                  \
    P(F, V, 4, 4, 12) P(F, V, 5, 5, 13) P(F, V, 6, 6, 14) P(F, V, 7, 7, 15)
// and among 32
#define RT_PAIRS5_0(P, F, V)                                                                                          \
    RT_PAIRS4_0(P, F, V)                                                                                              \
    P(F, V, 8, 16, 17) P(F, V, 9, 18, 19) P(F, V, 10, 20, 21) P(F, V, 11, 22, 23)          \
    P(F, V, 12, 24, 25) P(F, V, 13, 26, 27) P(F, V, 14, 28, 29) P(F, V, 15, 30, 31)
#define RT_PAIRS5_1(P, F, V)                                                                                          \
    RT_PAIRS4_1(P, F, V)                                                                                              \
    P(F, V, 8, 16, 18) P(F, V, 9, 17, 19) P(F, V, 10, 20, 22) P(F, V, 11, 21, 23)          \
    P(F, V, 12, 24, 26) P(F, V, 13, 25, 27) P(F, V, 14, 28, 30) P(F, V, 15, 29, 31)
#define RT_PAIRS5_2(P, F, V)                                                                                          \
    RT_PAIRS4_2(P, F, V)                                                                                              \
    P(F, V, 8, 16, 20) P(F, V, 9, 17, 21) P(F, V, 10, 18, 22) P(F, V, 11, 19, 23)          \
    P(F, V, 12, 24, 28) P(F, V, 13, 25, 29) P(F, V, 14, 26, 30) P(F, V, 15, 27, 31)
#define RT_PAIRS5_3(P, F, V)                                                                                          \
    RT_PAIRS4_3(P, F, V)                                                                                              \
    P(F, V, 8, 16, 24) P(F, V, 9, 17, 25) P(F, V, 10, 18, 26) P(F, V, 11, 19, 27)          \
    P(F, V, 12, 20, 28) P(F, V, 13, 21, 29) P(F, V, 14, 22, 30) P(F, V, 15, 23, 31)
#define RT_PAIRS5_4(P, F, V)                                                                                          \
    P(F, V, 0, 0, 16) P(F, V, 1, 1, 17) P(F, V, 2, 2, 18) P(F, V, 3, 3, 19)                \
    P(F, V, 4, 4, 20) P(F, V, 5, 5, 21) P(F, V, 6, 6, 22) P(F, V, 7, 7, 23)                \
    P(F, V, 8, 8, 24) P(F, V, 9, 9, 25) P(F, V, 10, 10, 26) P(F, V, 11, 11, 27)            \
    P(F, V, 12, 12, 28) P(F, V, 13, 13, 29) P(F, V, 14, 14, 30) P(F, V, 15, 15, 31)
#define RT_REGS3(F)                                                                                                \
    RT_REG(F, 0) RT_REG(F, 1) RT_REG(F, 2) RT_REG(F, 3) RT_REG(F, 4) RT_REG(F, 5) RT_REG(F, 6) RT_REG(F, 7)
#define RT_REGS4(F)                                                                                                \
    RT_REGS3(F)                                                                                                    \
    RT_REG(F, 8) RT_REG(F, 9) RT_REG(F, 10) RT_REG(F, 11) RT_REG(F, 12) RT_REG(F, 13) RT_REG(F, 14) RT_REG(F, 15)
#define RT_REGS5(F)                                                                                                \
    RT_REGS4(F)                                                                                                    \
    RT_REG(F, 16) RT_REG(F, 17) RT_REG(F, 18) RT_REG(F, 19) RT_REG(F, 20) RT_REG(F, 21) RT_REG(F, 22)              \
    RT_REG(F, 23) RT_REG(F, 24) RT_REG(F, 25) RT_REG(F, 26) RT_REG(F, 27) RT_REG(F, 28) RT_REG(F, 29)              \
    RT_REG(F, 30) RT_REG(F, 31)

#define RT_QUAD(S, D, V, p, i, j, I, J)                                                                            \
    "s_bitcmp1_b32 %[pm], " #p "\n"                                                                                \
    "s_cbranch_scc0 .Lrt_" V "_" #p "_%=\n" S(D, i, j, I, J) ".Lrt_" V "_" #p "_%=:\n"
#define RT_BOTH(D, i, I)                                                                                           \
    "s_bitcmp1_b32 %[pm], " #i "\n"                                                                                \
    "s_cbranch_scc0 .Lrt_gd_" #i "_%=\n" RT_STEP_GD(D, i, I) ".Lrt_gd_" #i "_%=:\n"                                \
    "s_bitcmp1_b32 %[pm2], " #i "\n"                                                                               \
    "s_cbranch_scc0 .Lrt_ge_" #i "_%=\n" RT_STEP_GE(D, i, I) ".Lrt_ge_" #i "_%=:\n"
// the pairs of register bit T among 8 registers of each state
#define RT_QUADS4_0(S, D, V)                                                                                       \
    RT_QUAD(S, D, V, 0, 0, 1, 8, 9) RT_QUAD(S, D, V, 1, 2, 3, 10, 11) RT_QUAD(S, D, V, 2, 4, 5, 12, 13)            \
    RT_QUAD(S, D, V, 3, 6, 7, 14, 15)
#define RT_QUADS4_1(S, D, V)                                                                                       \
    RT_QUAD(S, D, V, 0, 0, 2, 8, 10) RT_QUAD(S, D, V, 1, 1, 3, 9, 11) RT_QUAD(S, D, V, 2, 4, 6, 12, 14)            \
    RT_QUAD(S, D, V, 3, 5, 7, 13, 15)
#define RT_QUADS4_2(S, D, V)                                                                                       \
    RT_QUAD(S, D, V, 0, 0, 4, 8, 12) RT_QUAD(S, D, V, 1, 1, 5, 9, 13) RT_QUAD(S, D, V, 2, 2, 6, 10, 14)            \
    RT_QUAD(S, D, V, 3, 3, 7, 11, 15)
#define RT_BOTHS4(D)                                                                                               \
    RT_BOTH(D, 0, 8) RT_BOTH(D, 1, 9) RT_BOTH(D, 2, 10) RT_BOTH(D, 3, 11) RT_BOTH(D, 4, 12) RT_BOTH(D, 5, 13)      \
    RT_BOTH(D, 6, 14) RT_BOTH(D, 7, 15)

// The registers in Gray-code order, S a step and F(b) the flip of register bit
// b between two; R: the same order backwards.
#define RT_GRAY3(S, F) S(0) F(0) S(1) F(1) S(3) F(0) S(2) F(2) S(6) F(0) S(7) F(1) S(5) F(0) S(4)
#define RT_GRAY3R(S, F) S(4) F(0) S(5) F(1) S(7) F(0) S(6) F(2) S(2) F(0) S(3) F(1) S(1) F(0) S(0)
#define RT_GRAY4(S, F)                                                                                             \
    S(0) F(0) S(1) F(1) S(3) F(0) S(2) F(2) S(6) F(0) S(7) F(1) S(5) F(0) S(4) F(3)                                \
    S(12) F(0) S(13) F(1) S(15) F(0) S(14) F(2) S(10) F(0) S(11) F(1) S(9) F(0) S(8)
#define RT_GRAY4R(S, F)                                                                                            \
    S(8) F(0) S(9) F(1) S(11) F(0) S(10) F(2) S(14) F(0) S(15) F(1) S(13) F(0) S(12) F(3)                          \
    S(4) F(0) S(5) F(1) S(7) F(0) S(6) F(2) S(2) F(0) S(3) F(1) S(1) F(0) S(0)
#define RT_GRAY5(S, F)                                                                                             \
    RT_GRAY4(S, F) F(4)                                                                                            \
    S(24) F(0) S(25) F(1) S(27) F(0) S(26) F(2) S(30) F(0) S(31) F(1) S(29) F(0) S(28) F(3)                        \
    S(20) F(0) S(21) F(1) S(23) F(0) S(22) F(2) S(18) F(0) S(19) F(1) S(17) F(0) S(16)
#define RT_GRAY5R(S, F)                                                                                            \
    S(16) F(0) S(17) F(1) S(19) F(0) S(18) F(2) S(22) F(0) S(23) F(1) S(21) F(0) S(20) F(3)                        \
    S(28) F(0) S(29) F(1) S(31) F(0) S(30) F(2) S(26) F(0) S(27) F(1) S(25) F(0) S(24) F(4)                        \
    RT_GRAY4R(S, F)
// Exchange: one component written in the old layout, read in the new one, the
// lane's slot stepping through the registers by xor; the second component
// walks back, so both slots end where they began.
#define RT_FW(b) "v_xor_b32 %[sa], %[w" #b "], %[sa]\n"
#define RT_FD(b) "v_xor_b32 %[na], %[d" #b "], %[na]\n"
#define RT_WX_f64(i) "ds_write_b64 %[sa], " RT_N(x, i) "\n"
#define RT_WY_f64(i) "ds_write_b64 %[sa], " RT_N(y, i) "\n"
#define RT_RX_f64(i) "ds_read_b64 " RT_N(x, i) ", %[na]\n"
#define RT_RY_f64(i) "ds_read_b64 " RT_N(y, i) ", %[na]\n"
#define RT_WX_f32(i) "ds_write_b32 %[sa], " RT_N(x, i) "\n"
#define RT_WY_f32(i) "ds_write_b32 %[sa], " RT_N(y, i) "\n"
#define RT_RX_f32(i) "ds_read_b32 " RT_N(x, i) ", %[na]\n"
#define RT_RY_f32(i) "ds_read_b32 " RT_N(y, i) ", %[na]\n"
#define RT_MEET "s_waitcnt lgkmcnt(0)\ns_barrier\n"
#define RT_EXCH(G, GR, SZ)                                                                                         \
    RT_MEET G(RT_WX_##SZ, RT_FW) RT_MEET G(RT_RX_##SZ, RT_FD) RT_MEET GR(RT_WY_##SZ, RT_FW)                        \
    RT_MEET GR(RT_RY_##SZ, RT_FD) "s_waitcnt lgkmcnt(0)\n"

#define RT_TABLED_f64(i, o0, o1) RT_STEP_TAB("f64", "ds_read_b64", i, o0, o1)
#define RT_TABLE3_f64                                                                                              \
    RT_TABLED_f64(0, 0, 8) RT_TABLED_f64(1, 16, 24) RT_TABLED_f64(2, 32, 40) RT_TABLED_f64(3, 48, 56)                          \
    RT_TABLED_f64(4, 64, 72) RT_TABLED_f64(5, 80, 88) RT_TABLED_f64(6, 96, 104) RT_TABLED_f64(7, 112, 120)
#define RT_TABLE4_f64                                                                                              \
    RT_TABLE3_f64                                                                                                  \
    RT_TABLED_f64(8, 128, 136) RT_TABLED_f64(9, 144, 152) RT_TABLED_f64(10, 160, 168) RT_TABLED_f64(11, 176, 184)              \
    RT_TABLED_f64(12, 192, 200) RT_TABLED_f64(13, 208, 216) RT_TABLED_f64(14, 224, 232) RT_TABLED_f64(15, 240, 248)
// A block of diagonal gates on complex64 registers.  A register's factor is
// formed in double precision and rounded once, so a block costs an amplitude
// the rounding of one factor and one product, however many phases it sums:
// the factor of the lane (g, then h and g in turn), which follows the
// registers in Gray-code order, one product with the factor (u<b>) of the
// register bit that flips (U: it is set, V: cleared), times the register's own
// from the table.  The product is rounded to single precision and multiplies
// the register.
#define RT_PHASES4(T, U, V)                                                                                            \
    T(g, h, 0) U(g, h, 0) T(h, g, 1) U(h, g, 1) T(g, h, 3) V(g, h, 0) T(h, g, 2) U(h, g, 2) T(g, h, 6) U(g, h, 0)      \
    T(h, g, 7) V(h, g, 1) T(g, h, 5) V(g, h, 0) T(h, g, 4) U(h, g, 3) T(g, h, 12) U(g, h, 0) T(h, g, 13) U(h, g, 1)    \
    T(g, h, 15) V(g, h, 0) T(h, g, 14) V(h, g, 2) T(g, h, 10) U(g, h, 0) T(h, g, 11) V(h, g, 1) T(g, h, 9)             \
    V(g, h, 0) T(h, g, 8)
#define RT_PHASES5(T, U, V)                                                                                            \
    T(g, h, 0) U(g, h, 0) T(h, g, 1) U(h, g, 1) T(g, h, 3) V(g, h, 0) T(h, g, 2) U(h, g, 2) T(g, h, 6) U(g, h, 0)      \
    T(h, g, 7) V(h, g, 1) T(g, h, 5) V(g, h, 0) T(h, g, 4) U(h, g, 3) T(g, h, 12) U(g, h, 0) T(h, g, 13) U(h, g, 1)    \
    T(g, h, 15) V(g, h, 0) T(h, g, 14) V(h, g, 2) T(g, h, 10) U(g, h, 0) T(h, g, 11) V(h, g, 1) T(g, h, 9)             \
    V(g, h, 0) T(h, g, 8) U(h, g, 4) T(g, h, 24) U(g, h, 0) T(h, g, 25) U(h, g, 1) T(g, h, 27) V(g, h, 0)              \
    T(h, g, 26) U(h, g, 2) T(g, h, 30) U(g, h, 0) T(h, g, 31) V(h, g, 1) T(g, h, 29) V(g, h, 0) T(h, g, 28)            \
    V(h, g, 3) T(g, h, 20) U(g, h, 0) T(h, g, 21) U(h, g, 1) T(g, h, 23) V(g, h, 0) T(h, g, 22) V(h, g, 2)             \
    T(g, h, 18) U(g, h, 0) T(h, g, 19) V(h, g, 1) T(g, h, 17) V(g, h, 0) T(h, g, 16)
#define RT_PH_APPLY(p, i)                                                                                              \
    "v_cvt_f32_f64 %[t2], %[" #p "r]\n"                                                                                \
    "v_cvt_f32_f64 %[t3], %[" #p "i]\n" RT_MUL_f32(i)
#define RT_PH_TABLED(g, h, i)                                                                                          \
    "ds_read_b64 %[qr], %[ta] offset:16*" #i "\n"                                                                      \
    "ds_read_b64 %[qi], %[ta] offset:16*" #i "+8\n"                                                                    \
    "s_waitcnt lgkmcnt(0)\n"                                                                                           \
    "v_mul_f64 %[" #h "r], %[" #g "i], %[qi]\n"                                                                        \
    "v_mul_f64 %[" #h "i], %[" #g "i], %[qr]\n"                                                                        \
    "v_fma_f64 %[qr], %[" #g "r], %[qr], -%[" #h "r]\n"                                                                \
    "v_fma_f64 %[qi], %[" #g "r], %[qi], %[" #h "i]\n" RT_PH_APPLY(q, i)
#define RT_PH_LANE(g_, h_, i) RT_PH_TABLED(g, h, i)
#define RT_PH_PLAIN(g, h, i) RT_PH_APPLY(g, i)
#define RT_PH_UP(g, h, b)                                                                                              \
    "v_mul_f64 %[" #h "r], %[" #g "i], %[ui" #b "]\n"                                                                  \
    "v_mul_f64 %[" #h "i], %[" #g "i], %[ur" #b "]\n"                                                                  \
    "v_fma_f64 %[" #h "r], %[" #g "r], %[ur" #b "], -%[" #h "r]\n"                                                     \
    "v_fma_f64 %[" #h "i], %[" #g "r], %[ui" #b "], %[" #h "i]\n"
#define RT_PH_DOWN(g, h, b)                                                                                            \
    "v_mul_f64 %[" #h "r], %[" #g "i], %[ui" #b "]\n"                                                                  \
    "v_mul_f64 %[" #h "i], %[" #g "r], %[ui" #b "]\n"                                                                  \
    "v_fma_f64 %[" #h "r], %[" #g "r], %[ur" #b "], %[" #h "r]\n"                                                      \
    "v_fma_f64 %[" #h "i], %[" #g "i], %[ur" #b "], -%[" #h "i]\n"
#define RT_PH_STAY(g, h, b)
// Registers of a list times u<b> and the table's factor.
#define RT_PH_BIT(b, i)                                                                                                \
    "ds_read_b64 %[qr], %[ta] offset:16*" #i "\n"                                                                      \
    "ds_read_b64 %[qi], %[ta] offset:16*" #i "+8\n"                                                                    \
    "s_waitcnt lgkmcnt(0)\n"                                                                                           \
    "v_mul_f64 %[hr], %[ui" #b "], %[qi]\n"                                                                            \
    "v_mul_f64 %[hi], %[ui" #b "], %[qr]\n"                                                                            \
    "v_fma_f64 %[qr], %[ur" #b "], %[qr], -%[hr]\n"                                                                    \
    "v_fma_f64 %[qi], %[ur" #b "], %[qi], %[hi]\n" RT_PH_APPLY(q, i)
// the second registers of the pairs of bit b
#define RT_PH_SECOND(b, V, p, i, j) RT_PH_BIT(b, j)
#define RT_PH_BITS4                                                                                                    \
    RT_AT("po0") RT_PAIRS4_0(RT_PH_SECOND, 0, "") RT_END RT_AT("po1") RT_PAIRS4_1(RT_PH_SECOND, 1, "") RT_END          \
    RT_AT("po2") RT_PAIRS4_2(RT_PH_SECOND, 2, "") RT_END RT_AT("po3") RT_PAIRS4_3(RT_PH_SECOND, 3, "") RT_END
#define RT_PH_BITS5                                                                                                    \
    RT_AT("po0") RT_PAIRS5_0(RT_PH_SECOND, 0, "") RT_END RT_AT("po1") RT_PAIRS5_1(RT_PH_SECOND, 1, "") RT_END          \
    RT_AT("po2") RT_PAIRS5_2(RT_PH_SECOND, 2, "") RT_END RT_AT("po3") RT_PAIRS5_3(RT_PH_SECOND, 3, "") RT_END          \
    RT_AT("po4") RT_PAIRS5_4(RT_PH_SECOND, 4, "") RT_END
// lane's factor and table; register bits too; those without a table; one
// register bit and table
#define RT_ENTRIES_f32(B) RT_GO("pg") RT_GO("pn") RT_ENTRIES##B("po")
#define RT_TAB_f32(B) RT_PHASES##B(RT_PH_LANE, RT_PH_STAY, RT_PH_STAY)
#define RT_MORE_f32(B)                                                                                                 \
    RT_AT("pg") RT_PHASES##B(RT_PH_TABLED, RT_PH_UP, RT_PH_DOWN) RT_END                                                \
    RT_AT("pn") RT_PHASES##B(RT_PH_PLAIN, RT_PH_UP, RT_PH_DOWN) RT_END RT_PH_BITS##B
#define RT_FACTOR_f32 "v_cvt_f32_f64 %[t2], %[gr]\nv_cvt_f32_f64 %[t3], %[gi]\n"
#define RT_FACTOR_f64
#define RT_ENTRIES_f64(B)
#define RT_TAB_f64(B) RT_TABLE##B##_f64
#define RT_MORE_f64(B)

// The lanes' condition, then a jump into the branch table that follows, whose
// entry k (4 k bytes into it) is the branch to a variant; %[jo] = rt_jump(k)
// counts from behind s_getpc, past the three instructions before the table.
#define RT_DISPATCH                                                                                                \
    "s_mov_b64 %[sv], exec\n"                                                                                      \
    "s_and_b64 exec, exec, %[lm]\n"                                                                                \
    "s_cbranch_execz .Lrt_end_%=\n"                                                                                \
    "s_getpc_b64 vcc\n"                                                                                            \
    "s_add_u32 vcc_lo, vcc_lo, %[jo]\n"                                                                            \
    "s_addc_u32 vcc_hi, vcc_hi, 0\n"                                                                               \
    "s_setpc_b64 vcc\n"
#define RT_GO(V) "s_branch .Lrt_" V "_%=\n"
#define RT_AT(V) ".Lrt_" V "_%=:\n"
#define RT_END "s_branch .Lrt_end_%=\n"
#define RT_NONE "s_branch .Lrt_end_%=\n"
// entries of one kind: register bits 0 .. 7 (those there are)
#define RT_ENTRIES3(K) RT_GO(K "0") RT_GO(K "1") RT_GO(K "2") RT_NONE RT_NONE RT_NONE RT_NONE RT_NONE
#define RT_ENTRIES4(K) RT_GO(K "0") RT_GO(K "1") RT_GO(K "2") RT_GO(K "3") RT_NONE RT_NONE RT_NONE RT_NONE
#define RT_ENTRIES5(K) RT_GO(K "0") RT_GO(K "1") RT_GO(K "2") RT_GO(K "3") RT_GO(K "4") RT_NONE RT_NONE RT_NONE
#define RT_KIND3(P, OP, K)                                                                                         \
    RT_AT(K "0") RT_PAIRS3_0(P, OP, K "0") RT_END RT_AT(K "1") RT_PAIRS3_1(P, OP, K "1") RT_END                    \
    RT_AT(K "2") RT_PAIRS3_2(P, OP, K "2") RT_END
#define RT_KIND4(P, OP, K)                                                                                         \
    RT_AT(K "0") RT_PAIRS4_0(P, OP, K "0") RT_END RT_AT(K "1") RT_PAIRS4_1(P, OP, K "1") RT_END                    \
    RT_AT(K "2") RT_PAIRS4_2(P, OP, K "2") RT_END RT_AT(K "3") RT_PAIRS4_3(P, OP, K "3") RT_END
#define RT_KIND5(P, OP, K)                                                                                         \
    RT_AT(K "0") RT_PAIRS5_0(P, OP, K "0") RT_END RT_AT(K "1") RT_PAIRS5_1(P, OP, K "1") RT_END                    \
    RT_AT(K "2") RT_PAIRS5_2(P, OP, K "2") RT_END RT_AT(K "3") RT_PAIRS5_3(P, OP, K "3") RT_END                    \
    RT_AT(K "4") RT_PAIRS5_4(P, OP, K "4") RT_END
// every variant: entry kind * 8 + register bit of the pair kinds, again with
// every pair from kRtEntryFull on, then the rest (RT_ENTRIES_f32: complex64's own)
#define RT_HEAD(B)                                                                                                 \
    RT_DISPATCH RT_ENTRIES##B("r") RT_ENTRIES##B("c") RT_ENTRIES##B("g") RT_ENTRIES##B("s")                        \
    RT_ENTRIES##B("rf") RT_ENTRIES##B("cf") RT_ENTRIES##B("gf") RT_ENTRIES##B("sf") RT_GO("mul") RT_GO("tab") RT_GO("ex")
#define RT_BODY(B, SZ)                                                                                             \
    RT_KIND##B(RT_PAIR, RT_REAL_##SZ, "r")                                                                         \
    RT_KIND##B(RT_PAIR, RT_CROSS_##SZ, "c")                                                                        \
    RT_KIND##B(RT_PAIR, RT_GEN_##SZ, "g")                                                                          \
    RT_KIND##B(RT_PAIR, RT_SWAP_##SZ, "s")                                                                         \
    RT_KIND##B(RT_FULL, RT_REAL_##SZ, "rf")                                                                        \
    RT_KIND##B(RT_FULL, RT_CROSS_##SZ, "cf")                                                                       \
    RT_KIND##B(RT_FULL, RT_GEN_##SZ, "gf")                                                                         \
    RT_KIND##B(RT_FULL, RT_SWAP_##SZ, "sf")                                                                        \
    RT_AT("tab") RT_TAB_##SZ(B) RT_END RT_AT("ex") RT_EXCH(RT_GRAY##B, RT_GRAY##B##R, SZ) RT_END
#define RT_TAIL(B, SZ)                                                                                             \
    RT_AT("mul") RT_FACTOR_##SZ RT_REGS##B(RT_MUL_##SZ) RT_AT("end") "s_mov_b64 exec, %[sv]\n"
#define RT_BLOCK(B, SZ) RT_HEAD(B) RT_ENTRIES_##SZ(B) RT_BODY(B, SZ) RT_MORE_##SZ(B) RT_TAIL(B, SZ)
// the same with the gradient terms
#define RT_BLOCK_GRAD_f64                                                                                          \
    RT_HEAD(4) RT_GO("gd") RT_NONE RT_NONE RT_NONE RT_NONE                                                         \
    RT_GO("gy0") RT_GO("gy1") RT_GO("gy2") RT_NONE RT_NONE RT_NONE RT_NONE RT_NONE                                 \
    RT_GO("gx0") RT_GO("gx1") RT_GO("gx2") RT_NONE RT_NONE RT_NONE RT_NONE RT_NONE                                 \
    RT_BODY(4, f64)                                                                                                \
    RT_AT("gy0") RT_QUADS4_0(RT_STEP_GY, RT_DOT_f64, "gy0") RT_END                                                 \
    RT_AT("gy1") RT_QUADS4_1(RT_STEP_GY, RT_DOT_f64, "gy1") RT_END                                                 \
    RT_AT("gy2") RT_QUADS4_2(RT_STEP_GY, RT_DOT_f64, "gy2") RT_END                                                 \
    RT_AT("gx0") RT_QUADS4_0(RT_STEP_GX, RT_DOT_f64, "gx0") RT_END                                                 \
    RT_AT("gx1") RT_QUADS4_1(RT_STEP_GX, RT_DOT_f64, "gx1") RT_END                                                 \
    RT_AT("gx2") RT_QUADS4_2(RT_STEP_GX, RT_DOT_f64, "gx2") RT_END                                                 \
    RT_AT("gd") RT_BOTHS4(RT_DOT_f64) RT_END RT_TAIL(4, f64)

#define RT_AMP(i) [x##i] "+v"(v.x[i]), [y##i] "+v"(v.y[i])
#define RT_AMPS8                                                                                                   \
    RT_AMP(0), RT_AMP(1), RT_AMP(2), RT_AMP(3), RT_AMP(4), RT_AMP(5), RT_AMP(6), RT_AMP(7)
#define RT_AMPS16                                                                                                  \
    RT_AMP(0), RT_AMP(1), RT_AMP(2), RT_AMP(3), RT_AMP(4), RT_AMP(5), RT_AMP(6), RT_AMP(7), RT_AMP(8), RT_AMP(9),  \
        RT_AMP(10), RT_AMP(11), RT_AMP(12), RT_AMP(13), RT_AMP(14), RT_AMP(15)
#define RT_AMPS32                                                                                                  \
    RT_AMPS16, RT_AMP(16), RT_AMP(17), RT_AMP(18), RT_AMP(19), RT_AMP(20), RT_AMP(21), RT_AMP(22), RT_AMP(23),     \
        RT_AMP(24), RT_AMP(25), RT_AMP(26), RT_AMP(27), RT_AMP(28), RT_AMP(29), RT_AMP(30), RT_AMP(31)

#define RT_OPERANDS                                                                                                \
    [ar] "s"(m.ar), [ai] "s"(m.ai), [br] "s"(m.br), [bi] "s"(m.bi), [cr] "s"(m.cr), [ci] "s"(m.ci), [dr] "s"(m.dr), \
        [di] "s"(m.di), [pm] "s"(w[1]), [lm] "s"(lanes), [jo] "s"(w[5]),                                           \
        [ta] "v"(table), [w0] "s"(w[2]), [w1] "s"(w[3]), [w2] "s"(w[4]), [w3] "s"(w[6]), [d0] "s"(w[8]),           \
        [d1] "s"(w[9]), [d2] "s"(w[10]), [d3] "s"(w[11])
#define RT_FACTOR_IN [fr] "v"(fr), [fi] "v"(fi)
#define RT_SCRATCH                                                                                                 \
    [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [sv] "=&s"(save), [sa] "+v"(slot),             \
        [na] "+v"(next)

// A lane's amplitudes, components apart.
template <typename R, int NB> struct RtRegs {
    R x[1 << NB], y[1 << NB];
};

// Factors of a block of diagonal gates (kRtBlock): the lane's, and the one an
// amplitude takes with each register bit that is set.
template <int NB> struct RtPhases {
    double gr, gi, ur[NB], ui[NB];
};

constexpr uint32_t kRtEntryFull = 32, kRtEntryMul = 64, kRtEntryTab = 65, kRtEntryExch = 66;
constexpr uint32_t kRtEntryGradD = 67, kRtEntryGradY = 72, kRtEntryGradX = 80;  // reverse sweep
constexpr uint32_t kRtEntryBits = 67, kRtEntryBitsOnly = 68, kRtEntryOneBit = 69;  // complex64, kRtBlock
constexpr uint32_t rt_jump(uint32_t entry) { return 4 * entry + 12; }

// One operation in the lanes of `lanes` (uniform).  w: the operation's first
// 16 words: w[1] the pairs or registers, w[5] rt_jump(entry); an exchange has
// the register terms of the old layout in w[2], w[3], w[4], w[6], w[7] and of
// the new one in w[8] .. w[12].  m: the matrix; fr, fi: the lane's factor
// (entry kRtEntryMul); table: byte address in LDS (kRtEntryTab); ph: factors
// (kRtBlock); slot, next:
// the lane's byte address in the exchange buffer in the old and new layout.
// All lanes of the workgroup call together, with every load of LDS done.
__device__ __forceinline__ void rt_apply(RtRegs<double, 4> &v, const uint32_t (&w)[16], const Mat2<double> &m,
                                         double fr, double fi, uint64_t lanes, uint32_t table, uint32_t &slot,
                                         uint32_t &next) {
    double t0, t1, t2, t3;
    uint64_t save;
    asm volatile(RT_BLOCK(4, f64) : RT_AMPS16, RT_SCRATCH : RT_OPERANDS, RT_FACTOR_IN : "scc", "vcc", "memory");
}
#define RT_PHASE_OUT                                                                                                   \
    [gr] "+v"(ph.gr), [gi] "+v"(ph.gi), [hr] "=&v"(hr), [hi] "=&v"(hi), [qr] "=&v"(qr), [qi] "=&v"(qi)
#define RT_UNIT(b) [ur##b] "v"(ph.ur[b]), [ui##b] "v"(ph.ui[b])
#define RT_PHASE_IN RT_UNIT(0), RT_UNIT(1), RT_UNIT(2), RT_UNIT(3)
__device__ __forceinline__ void rt_apply(RtRegs<float, 5> &v, const uint32_t (&w)[16], const Mat2<float> &m,
                                         uint64_t lanes, uint32_t table, uint32_t &slot, uint32_t &next,
                                         RtPhases<5> &ph) {
    float t0, t1, t2, t3;
    double hr, hi, qr, qi;
    uint64_t save;
    asm volatile(RT_BLOCK(5, f32)
                 : RT_AMPS32, RT_SCRATCH, RT_PHASE_OUT
                 : RT_OPERANDS, RT_PHASE_IN, RT_UNIT(4), [w4] "s"(w[7]), [d4] "s"(w[12])
                 : "scc", "vcc", "memory");
}

// with half as many amplitudes per lane
__device__ __forceinline__ void rt_apply(RtRegs<double, 3> &v, const uint32_t (&w)[16], const Mat2<double> &m,
                                         double fr, double fi, uint64_t lanes, uint32_t table, uint32_t &slot,
                                         uint32_t &next) {
    double t0, t1, t2, t3;
    uint64_t save;
    asm volatile(RT_BLOCK(3, f64) : RT_AMPS8, RT_SCRATCH : RT_OPERANDS, RT_FACTOR_IN : "scc", "vcc", "memory");
}
__device__ __forceinline__ void rt_apply(RtRegs<float, 4> &v, const uint32_t (&w)[16], const Mat2<float> &m,
                                         uint64_t lanes, uint32_t table, uint32_t &slot, uint32_t &next,
                                         RtPhases<4> &ph) {
    float t0, t1, t2, t3;
    double hr, hi, qr, qi;
    uint64_t save;
    asm volatile(RT_BLOCK(4, f32)
                 : RT_AMPS16, RT_SCRATCH, RT_PHASE_OUT
                 : RT_OPERANDS, RT_PHASE_IN
                 : "scc", "vcc", "memory");
}

// The same on a lane's amplitudes of psi (registers with the top bit 0) and
// lambda (1), with the gradient entries: g accumulates a0 .. a3.  w[12]: the
// registers kRtEntryGradD subtracts.
#define RT_GRAD_OUT [a0] "+v"(g[0]), [a1] "+v"(g[1]), [a2] "+v"(g[2]), [a3] "+v"(g[3])
__device__ __forceinline__ void rt_apply_grad(RtRegs<double, 4> &v, const uint32_t (&w)[16], const Mat2<double> &m,
                                              double fr, double fi, uint64_t lanes, uint32_t table, uint32_t &slot,
                                              uint32_t &next, double (&g)[4]) {
    double t0, t1, t2, t3;
    uint64_t save;
    asm volatile(RT_BLOCK_GRAD_f64
                 : RT_AMPS16, RT_SCRATCH, RT_GRAD_OUT
                 : RT_OPERANDS, RT_FACTOR_IN, [pm2] "s"(w[12])
                 : "scc", "vcc", "memory");
}

} // namespace sv
