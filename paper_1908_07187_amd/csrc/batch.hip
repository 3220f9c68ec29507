// Batched execution: many circuits of uneven qubit counts in one persistent
// launch, and the stage kernel of the simulator's LDS-tile mode.
//
// Each circuit ("job") is compiled on the host into compact device records:
// builtin gates as rotations, in coefficients of the state's precision, their
// controls as predicates, up to two classical conditions, measurements with
// their pre-drawn uniform.  Gates are
// packed into passes: a pass names four slots (positions of the state, see
// stage_records.h) and carries the gates whose dense targets are among them
// (diagonal and phase gates may act on any qubits).  One persistent grid runs
// all jobs: every workgroup takes the next job from a device counter (largest
// jobs first).  The job's amplitudes stay in registers for its whole circuit,
// 16 per thread: in a pass they are the 2^4 combinations of its slots, so its
// gates need no other thread's; between passes they change hands through an
// LDS buffer, one component at a time.  A 12-qubit, 360-gate circuit costs one
// HBM write instead of 360 sweeps and 360 launches.  Every workgroup leaves
// the loop once the counter passes the job count.
//
// What bounds it is the vector unit: a real one-qubit gate on a chunk of 2^12
// amplitudes is 32 FP64 instructions per wave.  2048 12-qubit circuits of
// 360 gates: 1180 us with the amplitudes in LDS and one pass per three qubits,
// 420 us like this.  What the rest of the design is for:
// - amplitudes in registers and half the LDS: four workgroups per CU (two
//   with the whole state in LDS, whose load, gate and store phases left the
//   vector unit idle half the time);
// - records by scalar loads (see RecWords);
// - the gate loop in assembly: a jump per gate into code for its kind and
//   slot, where compiled switches moved the 32 to 64 amplitude registers
//   around at every join.
//
// Larger jobs (above 13 qubits complex128, 14 complex64; up to 24) run in the
// same launch with their state in global memory.  The host splits such a job
// into stages: runs of gates, reordered only where they commute, whose qubits
// fit one chunk (12 qubits complex128, 13 complex64), and measurements between
// them.  A stage's chunks (the
// amplitudes that share the values of the qubits outside the stage) are
// independent, so any free workgroup claims a run of them: it gathers each
// into registers, runs the stage's items on it exactly as for a small job, and
// scatters it back; the workgroup that completes a stage's last chunk opens
// the next stage.  A stage costs one read and one write of the state
// whatever its gate count; a measurement is two stages of its own, sums and
// scaling.  Workgroups take staged chunks first and small
// jobs when no chunk is free, and leave once every staged job has finished
// and the small-job counter has passed the job count.
//
// The simulator's LDS-tile mode (k_stage) runs one stage of a single state
// per launch with the same chunk code.
//
// Measurement inside a job uses the same rule as the per-gate path (FP64
// sums, outcome 0 iff u < P0, renormalise by 1/sqrt(p_outcome)), reduced in a
// fixed order that depends only on the job, so a job's result does not depend
// on which other jobs share the launch.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <numeric>
#include <string>
#include <utility>
#include <vector>

#include "qk_internal.h"
#include "stage_records.h"

using namespace qk;

namespace {

struct BJob {
  uint64_t state_off;   // amplitudes
  uint32_t rec;         // the job's header record
  int32_t n, ncbits;
  uint32_t cbit_off;
  uint32_t st_begin, nst;   // staged jobs: their stages in the launch's stage table
};

constexpr int kMaxJobCbits = 256;
constexpr int kMaxWaves = 16;             // waves of a workgroup at most

template <typename R> struct EVb;
template <> struct EVb<float> { typedef float T __attribute__((ext_vector_type(2))); };
template <> struct EVb<double> { typedef double T __attribute__((ext_vector_type(2))); };

__device__ __forceinline__ uint32_t rfl(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// Records are read through the constant address space, that is by scalar
// loads: from a plain pointer the compiler loads them by vector loads (the
// kernels store to memory that it cannot tell apart), which wait behind the
// amplitudes' loads and stores, three times per pass, and take registers
// that the amplitudes then spilled from.  A stage of 48 gates on 28 qubits
// complex128: 5.2 ms by vector loads, 3.05 ms like this.  (The records are
// written before the launch and by no kernel.)
typedef const __attribute__((address_space(4))) uint32_t* RecWords;
__device__ __forceinline__ RecWords rec_words(const uint32_t* recs, uint32_t rec) {
  return (RecWords)(uintptr_t)(recs + (size_t)rec * kRecWords);
}
template <typename R>
__device__ __forceinline__ R rec_real(RecWords w, int e) {
  return ((const __attribute__((address_space(4))) R*)w)[e];
}

__device__ __forceinline__ double bwave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ uint32_t ins0(uint32_t p, uint32_t q) { return ((p >> q) << (q + 1)) | (p & ((1u << q) - 1)); }

// The place (in bytes) of position p in an LDS buffer of one component per
// position.  A pass whose slots include the lowest positions gives
// consecutive lanes groups 16 (or more) positions apart, all in the same
// banks; XOR-ing the next bits into the place within a 128-byte row (4 bits
// for doubles, 5 for floats) spreads them, and keeps contiguous runs
// contiguous within each row.  A bijection on [0, 2^n), and linear over XOR.
template <typename R>
__device__ __forceinline__ uint32_t place(uint32_t i) {
  constexpr uint32_t b = sizeof(R) == 8 ? 4 : 5, m = (1u << b) - 1;
  return (i ^ ((i >> b) & m)) * (uint32_t)sizeof(R);
}

// The places of a thread's 16 members: member r is at sb ^ (the v_j of its bits).
struct Places {
  uint32_t sb, v0, v1, v2, v3;
  __device__ __forceinline__ uint32_t at(int r) const {
    return sb ^ ((r & 1 ? v0 : 0u) ^ (r & 2 ? v1 : 0u) ^ (r & 4 ? v2 : 0u) ^ (r & 8 ? v3 : 0u));
  }
};

// The value of a functional (in, out) at position p of the chunk c.
__device__ __forceinline__ uint32_t lane_bit(uint32_t in, uint32_t out, uint32_t p, uint32_t c) {
  return (uint32_t)(__popc(in & p) + __popc(out & c)) & 1u;
}

// The gate loop of a pass, in assembly: plain gates on the thread's 16
// amplitudes a0..a15 + i b0..b15, updated in place, from record p on; it
// leaves p at the first record with another op (the one that ends the pass
// among them).
//
// A gate rotates 16 pairs of real registers (x, y).  It is written as x += A y,
// y += B x, which needs no temporaries: 32 instructions, where the four
// products of each pair with a 2x2 matrix are 64 (a stage of 12 passes of 4 H
// and 8 RZZ on 28 qubits, complex128: 7.5 ms with those, 5.5 ms like this;
// complex64 4.5 and 3.5 ms).  What is left over are
// scales of the registers, which the host keeps track of and which one
// multiplication per register takes out when the pass ends.  Angles past 45
// degrees, where the second sum would cancel, come as what they are short of 90
// (see stage_records.h).  The lane factor is a double in complex64 too, and
// phases of up to 45 degrees take three steps (gate_turn): with a factor of
// floats, products for the larger angles and for all phases, a QFT on 25 qubits
// was 8.8e-7 off, 4.4e-7 like this, 28 qubits and 8 layers 6.2e-7, 5.7e-7 like this
// (15.8 and 14.9 ms).
//
// What a compiled loop added to the gates cost as much again: a tree of
// compares and taken branches for each gate, results moved back into the
// amplitudes' registers, a wait for each record.  Here each record holds the
// place of its gate's code, and is read while the gate before it runs; that
// gate works out the jump before it ends.
//
// The records come by scalar loads: the next one into s40..s51 while this one's
// coefficients c0..c3 stay in s56..s63; s80:81 is the address of the gates'
// code, s82:83 the next gate's, s84:85 the record that is read, s89 the chunk's
// outside bits.
#define QK_FETCH "s_load_dwordx4 s[40:43], s[84:85], 0x0\n\ts_load_dwordx8 s[44:51], s[84:85], 0x10\n\t"
#define QK_BEGIN                                                                                         \
  "s_mov_b64 s[56:57], s[44:45]\n\ts_mov_b64 s[58:59], s[46:47]\n\ts_mov_b64 s[60:61], s[48:49]\n\t"        \
  "s_mov_b64 s[62:63], s[50:51]\n\ts_add_u32 s84, s84, 48\n\ts_addc_u32 s85, s85, 0\n\t" QK_FETCH
// Reads one word of each of the 15 lines after the first record's, so that the
// records of the pass, and often the next one's header, come from the scalar
// cache: a record is used once per chunk, and with a miss for each a pass was
// bound by their latency (2048 12-qubit circuits of 360 gates, complex128: 525
// us without this, 420 us with it; 21 qubits, 820 gates: 611 and 514 us).
// The values go to s88, which nothing reads.
#define QK_TOUCH1(O) "s_load_dword s88, s[84:85], " #O "\n\t"
#define QK_TOUCH                                                                                         \
  QK_TOUCH1(0x40) QK_TOUCH1(0x80) QK_TOUCH1(0xc0) QK_TOUCH1(0x100) QK_TOUCH1(0x140) QK_TOUCH1(0x180)       \
  QK_TOUCH1(0x1c0) QK_TOUCH1(0x200) QK_TOUCH1(0x240) QK_TOUCH1(0x280) QK_TOUCH1(0x2c0) QK_TOUCH1(0x300)    \
  QK_TOUCH1(0x340) QK_TOUCH1(0x380) QK_TOUCH1(0x3c0)
#define QK_NEXT "s_waitcnt lgkmcnt(0)\n\ts_add_u32 s82, s80, s40\n\ts_addc_u32 s83, s81, 0\n\t"
#define QK_JUMP "s_setpc_b64 s[82:83]\n\t"
#define QK_C0_f64 "s[56:57]"
#define QK_C1_f64 "s[58:59]"
#define QK_C2_f64 "s[60:61]"
#define QK_C3_f64 "s[62:63]"
#define QK_C0_f32 "s56"
#define QK_C1_f32 "s57"
#define QK_C2_f32 "s58"
#define QK_C3_f32 "s59"
// D += C S
#define QK_ADD(W, C, S, D) "v_fma_" #W " %[" #D "], " C ", %[" #S "], %[" #D "]\n\t"
// The two steps on the pair of members (P, Q): a real gate turns (a_P, a_Q) and
// (b_P, b_Q), an imaginary one (a_P, b_Q) by c0, c1 and (b_P, a_Q) by c2, c3.
#define QK_REALX(W, P, Q) QK_ADD(W, QK_C0_##W, a##Q, a##P) QK_ADD(W, QK_C0_##W, b##Q, b##P)
#define QK_REALY(W, P, Q) QK_ADD(W, QK_C1_##W, a##P, a##Q) QK_ADD(W, QK_C1_##W, b##P, b##Q)
#define QK_IMAGX(W, P, Q) QK_ADD(W, QK_C0_##W, b##Q, a##P) QK_ADD(W, QK_C2_##W, a##Q, b##P)
#define QK_IMAGY(W, P, Q) QK_ADD(W, QK_C1_##W, a##P, b##Q) QK_ADD(W, QK_C3_##W, b##P, a##Q)
// The pairs of each slot (with the next gate's place worked out before the last two, in a gate's last step).
#define QK_SLOT0(ONE, W, NEXT) ONE(W, 0, 1) ONE(W, 2, 3) ONE(W, 4, 5) ONE(W, 6, 7) ONE(W, 8, 9) ONE(W, 10, 11) NEXT ONE(W, 12, 13) ONE(W, 14, 15)
#define QK_SLOT1(ONE, W, NEXT) ONE(W, 0, 2) ONE(W, 1, 3) ONE(W, 4, 6) ONE(W, 5, 7) ONE(W, 8, 10) ONE(W, 9, 11) NEXT ONE(W, 12, 14) ONE(W, 13, 15)
#define QK_SLOT2(ONE, W, NEXT) ONE(W, 0, 4) ONE(W, 1, 5) ONE(W, 2, 6) ONE(W, 3, 7) ONE(W, 8, 12) ONE(W, 9, 13) NEXT ONE(W, 10, 14) ONE(W, 11, 15)
#define QK_SLOT3(ONE, W, NEXT) ONE(W, 0, 8) ONE(W, 1, 9) ONE(W, 2, 10) ONE(W, 3, 11) ONE(W, 4, 12) ONE(W, 5, 13) NEXT ONE(W, 6, 14) ONE(W, 7, 15)
// re and im of a member turn by s and t0, or by their opposites.
#define QK_SIGNX(W, G, R) "v_fma_" #W " %[a" #R "], " G "%[s], %[b" #R "], %[a" #R "]\n\t"
#define QK_SIGNY(W, G, R) "v_fma_" #W " %[b" #R "], " G "%[t0], %[a" #R "], %[b" #R "]\n\t"
#define QK_SIGN16(ONE, W, NEXT, A, B, C, D, E, F, G, H, I, J, K, L, M, N, O, P)                                    \
  ONE(W, "", A) ONE(W, "", B) ONE(W, "", C) ONE(W, "", D) ONE(W, "", E) ONE(W, "", F) ONE(W, "", G) ONE(W, "", H)  \
  ONE(W, "-", I) ONE(W, "-", J) ONE(W, "-", K) ONE(W, "-", L) NEXT                                                 \
  ONE(W, "-", M) ONE(W, "-", N) ONE(W, "-", O) ONE(W, "-", P)
#define QK_SIGNM(ONE, W, NEXT, ...) QK_SIGN16(ONE, W, NEXT, __VA_ARGS__)
// The members by the parity of (r & m): eight with 0, eight with 1.
#define QK_MEMBERS1 0, 2, 4, 6, 8, 10, 12, 14, 1, 3, 5, 7, 9, 11, 13, 15
#define QK_MEMBERS2 0, 1, 4, 5, 8, 9, 12, 13, 2, 3, 6, 7, 10, 11, 14, 15
#define QK_MEMBERS3 0, 3, 4, 7, 8, 11, 12, 15, 1, 2, 5, 6, 9, 10, 13, 14
#define QK_MEMBERS4 0, 1, 2, 3, 8, 9, 10, 11, 4, 5, 6, 7, 12, 13, 14, 15
#define QK_MEMBERS5 0, 2, 5, 7, 8, 10, 13, 15, 1, 3, 4, 6, 9, 11, 12, 14
#define QK_MEMBERS6 0, 1, 6, 7, 8, 9, 14, 15, 2, 3, 4, 5, 10, 11, 12, 13
#define QK_MEMBERS7 0, 3, 5, 6, 8, 11, 13, 14, 1, 2, 4, 7, 9, 10, 12, 15
#define QK_MEMBERS8 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15
#define QK_MEMBERS9 0, 2, 4, 6, 9, 11, 13, 15, 1, 3, 5, 7, 8, 10, 12, 14
#define QK_MEMBERS10 0, 1, 4, 5, 10, 11, 14, 15, 2, 3, 6, 7, 8, 9, 12, 13
#define QK_MEMBERS11 0, 3, 4, 7, 9, 10, 13, 14, 1, 2, 5, 6, 8, 11, 12, 15
#define QK_MEMBERS12 0, 1, 2, 3, 12, 13, 14, 15, 4, 5, 6, 7, 8, 9, 10, 11
#define QK_MEMBERS13 0, 2, 5, 7, 9, 11, 12, 14, 1, 3, 4, 6, 8, 10, 13, 15
#define QK_MEMBERS14 0, 1, 6, 7, 10, 11, 12, 13, 2, 3, 4, 5, 8, 9, 14, 15
#define QK_MEMBERS15 0, 3, 5, 6, 9, 10, 12, 15, 1, 2, 4, 7, 8, 11, 13, 14
// The parity of the lane functional in bit 0 of v (other bits: garbage), from
// the record's words before the next record replaces them.
#define QK_LANE_BIT                                                                                      \
  "s_lshr_b32 s86, s41, 16\n\ts_and_b32 s87, s42, s89\n\ts_bcnt1_i32_b32 s87, s87\n\t"                     \
  "v_and_b32 %[v], s86, %[bs]\n\tv_bcnt_u32_b32 %[v], %[v], s87\n\t"
// s = c0 and t0 = c1, both negated where it is 1.
#define QK_LANE_SIGN_f64                                                                                 \
  "v_bfe_i32 %[v], %[v], 0, 1\n\tv_lshl_or_b32 %[v], %[v], 1, 1\n\tv_cvt_f64_i32 %[t0], %[v]\n\t"         \
  "v_mul_f64 %[s], s[56:57], %[t0]\n\tv_mul_f64 %[t0], s[58:59], %[t0]\n\t"
#define QK_LANE_SIGN_f32                                                                                 \
  "v_lshlrev_b32 %[v], 31, %[v]\n\tv_xor_b32 %[s], s56, %[v]\n\tv_xor_b32 %[t0], s57, %[v]\n\t"
// One gate's code, kGateBytes long.
#define QK_GATE(N, ...) "LQKg" #N "%=:\n\t" __VA_ARGS__ QK_JUMP ".org LQKg" #N "%=+512\n"
#define QK_REAL(N, S, W) QK_GATE(N, QK_BEGIN QK_SLOT##S(QK_REALX, W, ) QK_SLOT##S(QK_REALY, W, QK_NEXT))
#define QK_IMAG(N, S, W) QK_GATE(N, QK_BEGIN QK_SLOT##S(QK_IMAGX, W, ) QK_SLOT##S(QK_IMAGY, W, QK_NEXT))
#define QK_SIGN(N, M, W)                                                                                 \
  QK_GATE(N, QK_LANE_BIT QK_BEGIN QK_LANE_SIGN_##W QK_SIGNM(QK_SIGNX, W, , QK_MEMBERS##M)                  \
          QK_SIGNM(QK_SIGNY, W, QK_NEXT, QK_MEMBERS##M))
// The lane factor fr + i fi times c0 - i c1 (or c0 + i c1), in doubles.
#define QK_LANE_FACTOR(T, U)                                                                             \
  "v_bfe_i32 %[v], %[v], 0, 1\n\tv_lshl_or_b32 %[v], %[v], 1, 1\n\tv_cvt_f64_i32 %[" #T "], %[v]\n\t"     \
  "v_mul_f64 %[" #T "], s[58:59], %[" #T "]\n\tv_mul_f64 %[" #U "], %[" #T "], %[fr]\n\t"                  \
  "v_mul_f64 %[fr], s[56:57], %[fr]\n\tv_fma_f64 %[fr], %[" #T "], %[fi], %[fr]\n\t"                     \
  "v_fma_f64 %[fi], s[56:57], %[fi], -%[" #U "]\n\t"
#define QK_GATE_LOOP(W)                                                                                  \
  asm volatile(                                                                                          \
      "s_mov_b64 s[84:85], %[p]\n\t" QK_FETCH "s_mov_b32 s89, %[cc]\n\ts_getpc_b64 s[80:81]\n"             \
      "LQKpc%=:\n\t"                                                                                     \
      "s_add_u32 s80, s80, LQKg0%=-LQKpc%=\n\ts_addc_u32 s81, s81, 0\n\t" QK_NEXT QK_TOUCH QK_JUMP         \
      QK_REAL(0, 0, W) QK_REAL(1, 1, W) QK_REAL(2, 2, W) QK_REAL(3, 3, W)                                \
      QK_IMAG(4, 0, W) QK_IMAG(5, 1, W) QK_IMAG(6, 2, W) QK_IMAG(7, 3, W)                                \
      QK_GATE(8, QK_LANE_BIT QK_BEGIN QK_LANE_FACTOR(d0, d1) QK_NEXT)                                    \
      QK_SIGN(9, 1, W) QK_SIGN(10, 2, W) QK_SIGN(11, 3, W) QK_SIGN(12, 4, W)                             \
      QK_SIGN(13, 5, W) QK_SIGN(14, 6, W) QK_SIGN(15, 7, W) QK_SIGN(16, 8, W)                            \
      QK_SIGN(17, 9, W) QK_SIGN(18, 10, W) QK_SIGN(19, 11, W) QK_SIGN(20, 12, W)                         \
      QK_SIGN(21, 13, W) QK_SIGN(22, 14, W) QK_SIGN(23, 15, W)                                           \
      "s_waitcnt lgkmcnt(0)\n\ts_mov_b64 %[p], s[84:85]"   /* RG_OTHER */                                                        \
      : [a0] "+v"(xr[0]), [a1] "+v"(xr[1]), [a2] "+v"(xr[2]), [a3] "+v"(xr[3]), [a4] "+v"(xr[4]),        \
        [a5] "+v"(xr[5]), [a6] "+v"(xr[6]), [a7] "+v"(xr[7]), [a8] "+v"(xr[8]), [a9] "+v"(xr[9]),        \
        [a10] "+v"(xr[10]), [a11] "+v"(xr[11]), [a12] "+v"(xr[12]), [a13] "+v"(xr[13]),                  \
        [a14] "+v"(xr[14]), [a15] "+v"(xr[15]), [b0] "+v"(xi[0]), [b1] "+v"(xi[1]), [b2] "+v"(xi[2]),    \
        [b3] "+v"(xi[3]), [b4] "+v"(xi[4]), [b5] "+v"(xi[5]), [b6] "+v"(xi[6]), [b7] "+v"(xi[7]),        \
        [b8] "+v"(xi[8]), [b9] "+v"(xi[9]), [b10] "+v"(xi[10]), [b11] "+v"(xi[11]),                      \
        [b12] "+v"(xi[12]), [b13] "+v"(xi[13]), [b14] "+v"(xi[14]), [b15] "+v"(xi[15]),                  \
        [fr] "+v"(fr), [fi] "+v"(fi), [p] "+s"(p), [t0] "=&v"(t0), [s] "=&v"(s), [d0] "=&v"(d0),         \
        [d1] "=&v"(d1), [v] "=&v"(vt)                                                                    \
      : [cc] "s"(c), [bs] "v"(base)                                                                      \
      : "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s56", "s57", "s58", \
        "s59", "s60", "s61", "s62", "s63", "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "scc")
static_assert(kGateBytes == 512 && kRecWords * 4 == 48 && RG_SIGN == 8 && RG_OTHER == 24, "the gate loop's layout");

template <typename R>
__device__ __forceinline__ void gate_loop(R (&xr)[kMembers], R (&xi)[kMembers], double& fr, double& fi, RecWords& p,
                                          uint32_t c, uint32_t base) {
  R t0, s;
  double d0, d1;
  uint32_t vt;
  if constexpr (sizeof(R) == 8) QK_GATE_LOOP(f64);
  else QK_GATE_LOOP(f32);
}

// fr + i fi times c + i s on lanes that act, in place (compiled, its copies of
// the factor push complex64's amplitudes out of the registers).
__device__ __forceinline__ void lane_factor(double& fr, double& fi, double c, double s, bool act) {
  double d;
  uint64_t exec = __builtin_amdgcn_ballot_w64(act), save;
  asm volatile(
      "s_and_saveexec_b64 %[e], %[m]\n\tv_mul_f64 %[d], %[s], %[fr]\n\tv_mul_f64 %[fr], %[c], %[fr]\n\t"
      "v_fma_f64 %[fr], -%[s], %[fi], %[fr]\n\tv_fma_f64 %[fi], %[c], %[fi], %[d]\n\ts_mov_b64 exec, %[e]"
      : [fr] "+v"(fr), [fi] "+v"(fi), [d] "=&v"(d), [e] "=&s"(save)
      : [c] "s"(c), [s] "s"(s), [m] "s"(exec)
      : "scc");
}

// Masked gates and phases (other ops), compiled.
template <typename R>
__device__ __forceinline__ void gate_real(R& pr, R& pi, R& qr, R& qi, const R* u) {
  const R t0 = u[0] * pr, t1 = u[0] * pi, t2 = u[2] * pr, t3 = u[2] * pi;
  pr = u[1] * qr + t0;
  pi = u[1] * qi + t1;
  qr = u[3] * qr + t2;
  qi = u[3] * qi + t3;
}
template <typename R>
__device__ __forceinline__ void gate_imag(R& pr, R& pi, R& qr, R& qi, const R* u) {
  const R t0 = u[0] * pr, t1 = u[0] * pi, t2 = u[2] * pr, t3 = u[2] * pi;
  pr = t0 - u[1] * qi;
  pi = u[1] * qr + t1;
  qi = u[3] * qi + t2;
  qr = u[3] * qr - t3;
}
template <typename R>
__device__ __forceinline__ void gate_factor(R& re, R& im, R c, R s) {
  const R t0 = c * re, t1 = s * re;
  re = t0 - s * im;
  im = c * im + t1;
}

// The same for a phase of up to 45 degrees in three steps, a = -tan(phi/2), b =
// sin phi: 3 roundings for 4 and no norm of c + i s, 3 operations for 4.  (In
// assembly: compiled, its results were copied at the branches' joins, which took
// 16 registers and spilled.)
template <typename R>
__device__ __forceinline__ void gate_turn(R& re, R& im, R a, R b) {
  if constexpr (sizeof(R) == 8)
    asm("v_fma_f64 %0, %2, %1, %0\n\tv_fma_f64 %1, %3, %0, %1\n\tv_fma_f64 %0, %2, %1, %0" : "+v"(re), "+v"(im) : "v"(a), "v"(b));
  else
    asm("v_fma_f32 %0, %2, %1, %0\n\tv_fma_f32 %1, %3, %0, %1\n\tv_fma_f32 %0, %2, %1, %0" : "+v"(re), "+v"(im) : "v"(a), "v"(b));
}

// re + i im, held at scales 1 and lambda, times c + i s: s1 = s lambda, s2 = s / lambda.
template <typename R>
__device__ __forceinline__ void gate_phase(R& re, R& im, R c, R s1, R s2) {
  const R t0 = c * re, t1 = s2 * re;
  re = t0 - s1 * im;
  im = c * im + t1;
}

// Expanded in the kernel body on the kernel's own register arrays with
// constant indices: passing an array to a function (by reference) made the
// compiler keep part of it in scratch memory.
// Pairs in the record's member mask (uniform) where the lane's mask has them;
// the others keep their values (chosen by selects: a branch per pair would copy
// its results; multiplied by the identity's entries instead, a value that is
// not finite would reach the other one of its pair).
#define QK_PAIRS_M(S, FN)                                                               \
  do {                                                                                  \
    _Pragma("unroll") for (int r = 0; r < kMembers; ++r)                                \
      if (!(r & (1 << (S)))) {                                                          \
        const bool on = ((mm & memb) >> r) & 1u;                                        \
        R pr = xr[r], pi = xi[r], qr = xr[r | (1 << (S))], qi = xi[r | (1 << (S))];       \
        FN(pr, pi, qr, qi, u);                                                          \
        xr[r] = on ? pr : xr[r];                                                        \
        xi[r] = on ? pi : xi[r];                                                        \
        xr[r | (1 << (S))] = on ? qr : xr[r | (1 << (S))];                              \
        xi[r | (1 << (S))] = on ? qi : xi[r | (1 << (S))];                              \
      }                                                                                 \
  } while (0)
#define QK_FLIP_M(S)                                                                    \
  do {                                                                                  \
    _Pragma("unroll") for (int r = 0; r < kMembers; ++r)                                \
      if (!(r & (1 << (S)))) {                                                          \
        const bool on = ((mm & memb) >> r) & 1u;                                        \
        const R pr = xr[r], pi = xi[r], qr = xr[r | (1 << (S))], qi = xi[r | (1 << (S))]; \
        xr[r] = on ? u[0] * qr : pr;                                                    \
        xi[r] = on ? u[0] * qi : pi;                                                    \
        xr[r | (1 << (S))] = on ? u[0] * pr : qr;                                       \
        xi[r | (1 << (S))] = on ? u[0] * pi : qi;                                       \
      }                                                                                 \
  } while (0)
// Staged states: qubits of the chunk a stage works on.
template <typename R> constexpr int stage_qubits() { return sizeof(R) == 8 ? 12 : 13; }
// Threads of a batch workgroup at most: one group of 16 amplitudes each of
// the largest state kept on chip (13 qubits complex128, 14 complex64).
template <typename R> constexpr int max_block() { return sizeof(R) == 8 ? 512 : 1024; }
// Waves per SIMD of the stage kernel: four workgroups per CU, 32 KiB of LDS
// each.  Loading the next chunk ahead takes the registers of one of them and
// is slower (28 qubits, 7 stages: 22.7 against 21.4 ms complex128, 14.8
// against 13.9 complex64).
template <typename R> constexpr int stage_waves() { return sizeof(R) == 8 ? 4 : 8; }

// Sums s0, s1 over the workgroup in a fixed order (wave, then the waves in
// order); thread 0 has the sums.
__device__ __forceinline__ void sum_waves(double& s0, double& s1, double (*red)[kMaxWaves]) {
  const uint32_t tid = threadIdx.x;
  s0 = bwave_sum(s0);
  s1 = bwave_sum(s1);
  if ((tid & 63u) == 0) {
    red[0][tid >> 6] = s0;
    red[1][tid >> 6] = s1;
  }
  __syncthreads();
  if (tid == 0) {
    double q0 = 0, q1 = 0;
    for (int k = 0; k < (int)(blockDim.x / 64); ++k) {
      q0 += red[0][k];
      q1 += red[1][k];
    }
    s0 = q0;
    s1 = q1;
  }
}

// Sums s0, s1 over the workgroup and decides the outcome: 0 iff u < P0.  meas[0] = 1/sqrt(p) of the
// outcome (0 if its probability is 0), meas[1] = the outcome; cbit (>= 0)
// receives it unless its probability is 0.
__device__ __forceinline__ void meas_decide(double s0, double s1, double u, int cbit, uint8_t* cb,
                                            double (*red)[kMaxWaves], double* meas) {
  sum_waves(s0, s1, red);
  if (threadIdx.x == 0) {
    const double q0 = s0, q1 = s1;
    const double P0 = q0 / (q0 + q1);
    const int oc = (u < P0) ? 0 : 1;
    const double po = oc ? q1 : q0;
    meas[0] = po > 0 ? 1.0 / sqrt(po) : 0.0;
    meas[1] = (double)oc;
    if (cbit >= 0 && po > 0) cb[cbit] = (uint8_t)oc;
  }
  __syncthreads();
}

// Accesses to a staged job's state: written through this XCD's L2, and read past
// it (sc1, as agent-scope atomics), so that a chunk needs no agent-scope acquire
// and release around it.  Those invalidate and write back the whole L2, the
// other workgroups' lines and records too (96 circuits of 8-20 qubits,
// complex64: 2834 us with them, 2736 us like this).
//
// So the order between workgroups rests on gfx950's rules and not on the
// language's, whose relaxed atomics alone promise none: a store with sc1 counts
// as complete (vmcnt) once it is written through, every wave waits for its own
// (stores_done) before the barrier behind which the chunks count as done, and
// a load with sc1, issued after a claim has returned the stage, is served past
// this XCD's caches.
typedef uint32_t Words2 __attribute__((ext_vector_type(2)));
typedef uint32_t Words4 __attribute__((ext_vector_type(4)));
constexpr int kThrough = 16;               // cache policy sc1
constexpr int kRawBuffer = 0x00027000;     // resource word 3 of a raw buffer of dwords
template <typename C>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t state_buffer(C* st, uint32_t dim) {
  const uint64_t a = (uint64_t)(uintptr_t)st;
  const uint64_t u = (uint64_t)rfl((uint32_t)a) | ((uint64_t)rfl((uint32_t)(a >> 32)) << 32);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)u, 0, (int)(rfl(dim) * (uint32_t)sizeof(C)), kRawBuffer);
}
__device__ __forceinline__ void store_through(__amdgpu_buffer_rsrc_t b, uint32_t i, EVb<float>::T x) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(Words2, x), b, (int)(i * 8), 0, kThrough);
}
__device__ __forceinline__ void store_through(__amdgpu_buffer_rsrc_t b, uint32_t i, EVb<double>::T x) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(Words4, x), b, (int)(i * 16), 0, kThrough);
}
__device__ __forceinline__ void load_through(__amdgpu_buffer_rsrc_t b, uint32_t i, EVb<float>::T& x) {
  x = __builtin_bit_cast(EVb<float>::T, __builtin_amdgcn_raw_buffer_load_b64(b, (int)(i * 8), 0, kThrough));
}
__device__ __forceinline__ void load_through(__amdgpu_buffer_rsrc_t b, uint32_t i, EVb<double>::T& x) {
  x = __builtin_bit_cast(EVb<double>::T, __builtin_amdgcn_raw_buffer_load_b128(b, (int)(i * 16), 0, kThrough));
}
__device__ __forceinline__ double load_through(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Measurement of the qubit mask qb over a staged job's state in global memory,
// as two stages of at most kMeasParts chunks of 2^mq amplitudes in order: the
// first leaves each chunk's FP64 sums, the second adds them, decides, scales
// the outcome's half by 1/sqrt(p) and zeroes the other.  All sums in a fixed
// order: strided over the threads that a stage's chunk takes, whatever the
// workgroup's size, then by chunk.  A zero-probability outcome leaves the
// state and the cbit as they are.
//
// Bound by memory, on many workgroups; one workgroup per measurement reads and
// writes its state alone (96 circuits of 8-20 qubits, complex64, a third of them
// measured: 2944 us that way, 2834 us like this).
constexpr int kMeasParts = 256;
constexpr int kMeasLoads = 8;   // amplitudes in flight per thread
template <typename R> constexpr uint32_t meas_threads() { return 1u << (stage_qubits<R>() - kPassSlots); }
__device__ __forceinline__ int meas_qubits(int n, int lq) { return max(lq, n - 8); }   // (2^8 = kMeasParts)

template <typename R>
__device__ __forceinline__ void meas_sums(__amdgpu_buffer_rsrc_t st, uint32_t first, uint32_t count, uint32_t qb,
                                          double (*red)[kMaxWaves], double* part) {
  using C = typename EVb<R>::T;
  constexpr uint32_t nt = meas_threads<R>();   // <= the workgroup's threads
  const uint32_t tid = threadIdx.x;
  double s0 = 0, s1 = 0;
  if (tid < nt)
    for (uint32_t i0 = first + tid; i0 < first + count; i0 += kMeasLoads * nt) {
      C x[kMeasLoads];
#pragma unroll
      for (int k = 0; k < kMeasLoads; ++k) load_through(st, i0 + k * nt, x[k]);
#pragma unroll
      for (int k = 0; k < kMeasLoads; ++k) {
        const double pr = (double)x[k].x * (double)x[k].x + (double)x[k].y * (double)x[k].y;
        if ((i0 + k * nt) & qb) s1 += pr; else s0 += pr;
      }
    }
  sum_waves(s0, s1, red);
  if (tid == 0) {   // for other XCDs, as the state
    __hip_atomic_store(&part[0], s0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&part[1], s1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();   // red[] is written again by the next chunk
}

template <typename R>
__device__ __forceinline__ void meas_scale(__amdgpu_buffer_rsrc_t st, uint32_t first, uint32_t count,
                                           uint32_t qb, R scale, bool oc) {
  using C = typename EVb<R>::T;
  constexpr uint32_t nt = meas_threads<R>();
  const uint32_t tid = threadIdx.x;
  if (tid < nt)
    for (uint32_t i0 = first + tid; i0 < first + count; i0 += kMeasLoads * nt) {
      C x[kMeasLoads];
#pragma unroll
      for (int k = 0; k < kMeasLoads; ++k) load_through(st, i0 + k * nt, x[k]);
#pragma unroll
      for (int k = 0; k < kMeasLoads; ++k) {
        const bool keep = (((i0 + k * nt) & qb) != 0) == oc;
        x[k].x = keep ? x[k].x * scale : (R)0;
        x[k].y = keep ? x[k].y * scale : (R)0;
        store_through(st, i0 + k * nt, x[k]);
      }
    }
}

// Bits of v deposited, lowest first, at the set bits of mask.
__device__ __forceinline__ uint32_t deposit(uint32_t v, uint32_t mask) {
  uint32_t out = 0;
  for (uint32_t m = mask; m; m &= m - 1, v >>= 1)
    if (v & 1u) out |= m & (~m + 1u);
  return out;
}

// The amplitudes of a chunk of 2^L (of a stage, or a whole small job) with
// header words h: thread t's member k is local index t + (k << TB), TB = L -
// 4 (0 below four qubits: one thread, members past the state unused); the
// thread's bits on the lowest TB qubits, k on the others (the same for every
// thread).  base and index(k) give its amplitude index, cmask where the chunk
// number goes, out_places its LDS places once the stage's items have run.
struct ChunkMap {
  uint32_t base, cmask, tpart;
  uint32_t kq0, kq1, kq2, kq3;   // amplitude-index bit of each bit of k
  bool live;                     // the thread has amplitudes

  __device__ __forceinline__ ChunkMap(RecWords h, int L, uint32_t dim, uint32_t tid) {
    const int TB = L > kPassSlots ? L - kPassSlots : 0;
    live = tid < (1u << TB);
    auto qubit_bit = [&](int j) { return 1u << ((h[4 + (j >> 2)] >> (8 * (j & 3))) & 0xffu); };
    RecWords raw = h + kRecWords;
    uint32_t smask = 0;
    base = tpart = 0;
    for (int j = 0; j < TB; ++j) {
      const uint32_t b = qubit_bit(j), on = 0u - ((tid >> j) & 1u);
      smask |= b;
      base |= b & on;
      tpart ^= raw[j] & on;
    }
    kq0 = qubit_bit(TB);
    kq1 = qubit_bit(TB + 1);
    kq2 = qubit_bit(TB + 2);
    kq3 = qubit_bit(TB + 3);
    cmask = (dim - 1) & ~(smask | kq0 | kq1 | kq2 | kq3);
  }
  __device__ __forceinline__ uint32_t index(int k) const {
    return (k & 1 ? kq0 : 0u) | (k & 2 ? kq1 : 0u) | (k & 4 ? kq2 : 0u) | (k & 8 ? kq3 : 0u);
  }
  // Keeps the compiler from holding 16 addresses from the loads to the stores.
  __device__ __forceinline__ void opaque() { asm volatile("" : "+s"(kq0), "+s"(kq1), "+s"(kq2), "+s"(kq3)); }
  __device__ __forceinline__ Places out_places(RecWords h, int L, uint32_t c) const {
    const int TB = L > kPassSlots ? L - kPassSlots : 0;
    RecWords raw = h + kRecWords;
    Places p{tpart, raw[TB], raw[TB + 1], raw[TB + 2], raw[TB + 3]};
    if (!h[2])   // the frame has constants
      for (int j = 0; j < L; ++j)
        if (__popc(raw[16 + j] & c) & 1) p.sb ^= raw[j];
    return p;
  }
};

// Moves the amplitudes of a chunk between threads: written at `from`, read
// back at `to`, the real parts through the LDS buffer first, then the
// imaginary parts (both at once would take 64 KiB: two workgroups per CU
// instead of four).
template <typename R>
__device__ __forceinline__ void exchange(unsigned char* lds, R (&xr)[kMembers], R (&xi)[kMembers], Places from, Places to,
                                         bool live) {
  __syncthreads();   // the buffer's last readers
  if (live) {
#pragma unroll
    for (int r = 0; r < kMembers; ++r) *reinterpret_cast<R*>(lds + from.at(r)) = xr[r];
  }
  __syncthreads();
  if (live) {
#pragma unroll
    for (int r = 0; r < kMembers; ++r) xr[r] = *reinterpret_cast<const R*>(lds + to.at(r));
  }
  // the places are worked out again rather than held in 32 registers
  asm volatile("" : "+v"(from.sb), "+v"(to.sb));
  __syncthreads();
  if (live) {
#pragma unroll
    for (int r = 0; r < kMembers; ++r) *reinterpret_cast<R*>(lds + from.at(r)) = xi[r];
  }
  __syncthreads();
  if (live) {
#pragma unroll
    for (int r = 0; r < kMembers; ++r) xi[r] = *reinterpret_cast<const R*>(lds + to.at(r));
  }
}

// The registers' scales, 16 of the real parts and 16 of the imaginary ones.
template <typename R> constexpr int kScaleRecords = sizeof(R) == 8 ? 6 : 3;
template <typename R>
__device__ __forceinline__ void take_scales(R (&xr)[kMembers], R (&xi)[kMembers], RecWords w) {
#pragma unroll
  for (int r = 0; r < kMembers; ++r) {
    xr[r] *= rec_real<R>(w, r);
    xi[r] *= rec_real<R>(w, kMembers + r);
  }
}

// The items of a chunk (header words h, L qubits) on the amplitudes in
// registers, which start and end as the chunk map has them.  c: the chunk's
// outside bits with the constant.
template <typename R>
__device__ __forceinline__ void run_chunk(unsigned char* lds, R (&xr)[kMembers], R (&xi)[kMembers], const ChunkMap& cm,
                                          RecWords h, int L, uint32_t c, uint8_t* cb, double (*red)[kMaxWaves],
                                          double* meas) {
  const uint32_t tid = threadIdx.x;
  const int TB = L > kPassSlots ? L - kPassSlots : 0;
  const bool wave_live = rfl(tid & ~63u) < (1u << TB);   // whole waves run the gates: their control flow is uniform
  RecWords rec = h + kHeadRecords * kRecWords;
  const RecWords rec_end = rec + h[1] * kRecWords;
  uint32_t base = tid;
  Places cur{place<R>(tid), place<R>(1u << TB), place<R>(2u << TB), place<R>(4u << TB), place<R>(8u << TB)};
  while (rec != rec_end) {
    const uint32_t head = rec[0];
    if ((head & 0xffu) == RK_MEAS) {
      const uint32_t on = lane_bit(rec[1], rec[2], base, c), members = rec[6];
      double s[2] = {0, 0};
      if (cm.live) {
#pragma unroll
        for (int r = 0; r < kMembers; ++r) {
          const double pr = (double)xr[r] * (double)xr[r] + (double)xi[r] * (double)xi[r];
          if ((members >> r) & 1u) s[1] += pr; else s[0] += pr;
        }
      }
      const uint64_t ulo = rec[4], uhi = rec[5];
      meas_decide(on ? s[1] : s[0], on ? s[0] : s[1], __longlong_as_double((long long)(ulo | (uhi << 32))), (int)rec[3],
                  cb, red, meas);
      const R scale = (R)meas[0];
      if (meas[0] != 0.0) {
        const uint32_t keep = (meas[1] != 0.0) != (on != 0) ? members : ~members;
#pragma unroll
        for (int r = 0; r < kMembers; ++r) {
          const bool k = (keep >> r) & 1u;
          xr[r] = k ? xr[r] * scale : (R)0;
          xi[r] = k ? xi[r] * scale : (R)0;
        }
      }
      __syncthreads();   // red[] and meas[] are written again by the next measurement
      rec += kRecWords;
      continue;
    }
    // ---- a pass: the threads' members become the groups of its slots
    const uint32_t pv = rec[1];
    base = ins0(ins0(ins0(ins0(tid, pv & 0xff), (pv >> 8) & 0xff), (pv >> 16) & 0xff), pv >> 24);
    Places to{place<R>(base), rec[8], rec[9], rec[10], rec[11]};
    if (head & 0xf00u) {   // member 0 is where every slot has value 0
      const uint32_t r01 = rec[2], r23 = rec[3];
      if (head & 0x100u) to.sb ^= (0u - lane_bit(r01 & 0xffffu, rec[4], base, c)) & to.v0;
      if (head & 0x200u) to.sb ^= (0u - lane_bit(r01 >> 16, rec[5], base, c)) & to.v1;
      if (head & 0x400u) to.sb ^= (0u - lane_bit(r23 & 0xffffu, rec[6], base, c)) & to.v2;
      if (head & 0x800u) to.sb ^= (0u - lane_bit(r23 >> 16, rec[7], base, c)) & to.v3;
    }
    exchange<R>(lds, xr, xi, cur, to, cm.live);
    cur = to;
    RecWords p = rec + kRecWords;
    rec = p + (head >> 16) * kRecWords;
    const RecWords scales = rec - kScaleRecords<R> * kRecWords;   // (where the pass has them)
    const RecWords end = (head & 0x2000u ? scales : rec) - kRecWords;   // the record that ends the pass
    if (!wave_live) continue;
    uint32_t mm = 0xffffu;   // the lane's member mask (narrowed by RG_PRED for the next gate)
    double fr = 1, fi = 0;   // the lane factor: gates that act alike on all members
    for (;;) {
      gate_loop<R>(xr, xi, fr, fi, p, rfl(c), base);
      if (p == end) break;
      const RecWords gc = p;
      p += kRecWords;
      const uint32_t w1 = gc[1], om = gc[2], oh = gc[3];
      const uint32_t op = oh >> 24, memb = w1 & 0xffffu, ncond = (oh >> 18) & 3u;
      if (ncond) {
        if (rfl(cb[oh & 0xff]) != ((oh >> 16) & 1u) || (ncond > 1 && rfl(cb[(oh >> 8) & 0xff]) != ((oh >> 17) & 1u))) {
          mm = 0xffffu;
          continue;
        }
      }
      if (op == RG_SCALE) {
        take_scales<R>(xr, xi, p);
        p += kScaleRecords<R> * kRecWords;
        continue;
      }
      R u[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e] = rec_real<R>(gc + 4, e);
      if (op >= RG_PHASE) {
        const uint32_t on = lane_bit(w1 >> 16, om, base, c);
        if (op == RG_PRED) {
          const uint32_t mw = gc[4];
          mm &= on ? mw : mw >> 16;
          continue;
        }
        const bool act = mm != 0 && (!(oh & kOwnPredicate) || on), turn = (oh & kThreeSteps) != 0;
        if (op == RG_LANE_Z) {
          lane_factor(fr, fi, rec_real<double>(gc + 4, 0), rec_real<double>(gc + 4, 1), act);
        } else if (op == RG_PHASE) {
          if (turn) {
            const R a = act ? u[0] : (R)0, b = act ? u[1] : (R)0;
#pragma unroll
            for (int r = 0; r < kMembers; ++r)
              if ((memb >> r) & 1u) gate_turn<R>(xr[r], xi[r], a, b);
          } else {
            const R zr = act ? u[0] : (R)1, zi = act ? u[1] : (R)0, zj = act ? u[2] : (R)0;
#pragma unroll
            for (int r = 0; r < kMembers; ++r)
              if ((memb >> r) & 1u) gate_phase<R>(xr[r], xi[r], zr, zi, zj);
          }
        } else if (turn) {
#pragma unroll
          for (int r = 0; r < kMembers; ++r)
            if ((memb >> r) & 1u) {
              const bool here = (mm >> r) & 1u;
              gate_turn<R>(xr[r], xi[r], here ? u[0] : (R)0, here ? u[1] : (R)0);
            }
        } else {
#pragma unroll
          for (int r = 0; r < kMembers; ++r)
            if ((memb >> r) & 1u) {
              const bool here = (mm >> r) & 1u;
              gate_phase<R>(xr[r], xi[r], here ? u[0] : (R)1, here ? u[1] : (R)0, here ? u[2] : (R)0);
            }
        }
      } else {
        switch (op) {
          case RG_REAL_M: QK_PAIRS_M(0, gate_real); break;
          case RG_REAL_M + 1: QK_PAIRS_M(1, gate_real); break;
          case RG_REAL_M + 2: QK_PAIRS_M(2, gate_real); break;
          case RG_REAL_M + 3: QK_PAIRS_M(3, gate_real); break;
          case RG_IMAG_M: QK_PAIRS_M(0, gate_imag); break;
          case RG_IMAG_M + 1: QK_PAIRS_M(1, gate_imag); break;
          case RG_IMAG_M + 2: QK_PAIRS_M(2, gate_imag); break;
          case RG_IMAG_M + 3: QK_PAIRS_M(3, gate_imag); break;
          case RG_FLIP_M: QK_FLIP_M(0); break;
          case RG_FLIP_M + 1: QK_FLIP_M(1); break;
          case RG_FLIP_M + 2: QK_FLIP_M(2); break;
          case RG_FLIP_M + 3: QK_FLIP_M(3); break;
        }
      }
      mm = 0xffffu;
    }
    if (head & 0x2000u) take_scales<R>(xr, xi, scales);
    if (head & 0x1000u) {
#pragma unroll
      for (int r = 0; r < kMembers; ++r) gate_factor<R>(xr[r], xi[r], (R)fr, (R)fi);
    }
  }
  exchange<R>(lds, xr, xi, cur, cm.out_places(h, L, c), cm.live);
}

// Scheduling state of a batch launch.  Staged jobs: per job a 64-bit word
// (current stage << 32 | chunks claimed in it; the stage count once the job has
// finished) and the chunks completed in the current stage.  sched[0]: every
// staged job below it has finished (a scan hint); sched[1]: small jobs taken;
// sched[2]: set when a workgroup found no work for stall_ticks of the wall
// clock, 10 s (the host reports it); sched[3]: stages completed so far.
//
// What bounds many workgroups here is the memory behind these words: several
// hundred atomics on one line keep a channel busy, and every access to a state
// that falls on that channel waits (with all workgroups claiming from the oldest
// job, and the jobs' words side by side, loading a chunk of 64 KiB took 20 us
// instead of 5).  So each job has a line of its own, each workgroup starts its
// search at another job, and one that finds nothing looks again only when
// sched[3] has changed (or after kIdlePolls looks at it).  96 circuits of 8-20
// qubits, complex64: 2736 us without these, 2052 us with them and the cbits in
// pinned memory.
struct BStage {
  uint32_t rec;       // record of the stage header or measurement
  uint32_t nchunks;   // chunks of the stage
  uint32_t kind;      // StageKind
};
enum StageKind { ST_GATES = 0, ST_SUMS = 1, ST_SCALE = 2 };
struct alignas(128) JobCtl {
  unsigned long long word;
  unsigned done;
};
constexpr int kIdlePolls = 32;                           // about 50 us
constexpr uint32_t kScanWindow = 128;                   // staged jobs a workgroup looks at for a free chunk

__device__ __forceinline__ unsigned ld_acq(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_acq64(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until this wave's stores and atomics have completed, and keeps the
// compiler from moving memory operations across.
__device__ __forceinline__ void stores_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
  asm volatile("" ::: "memory");
}

template <typename R>
__global__ __launch_bounds__(max_block<R>(), 4) void k_batch(
    const BJob* __restrict__ jobs, int njobs, int nstaged, const BStage* __restrict__ stages, JobCtl* ctl,
    unsigned* sched, const uint32_t* __restrict__ opw, typename EVb<R>::T* __restrict__ states,
    uint8_t* __restrict__ cbits, uint8_t* __restrict__ host_cbits, double* __restrict__ parts, unsigned long long stall_ticks, uint32_t run_max) {
  using C = typename EVb<R>::T;
  constexpr int LQ = stage_qubits<R>();
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ uint8_t cb[kMaxJobCbits];
  __shared__ double red[2][kMaxWaves];
  __shared__ double meas[2];
  __shared__ int task[5];
  const uint32_t tid = threadIdx.x, bd = rfl(blockDim.x);
  const int lane = tid & 63, w = tid >> 6;
  const uint32_t rot = (blockIdx.x * 37u) & 63u;   // where its search starts
  unsigned long long idle_since = 0;
  uint32_t seen = 0;   // sched[3] before the last search
  bool idle = false, moved = false;   // which found nothing; which moved the hint on
  for (;;) {
    // ---- find work (wave 0): a free chunk of a staged job, 64 jobs (the
    // oldest first) looked at per load round; else the next small job; else
    // wait for the stages in flight, or leave once every staged job has finished
    if (w == 0) {
      int job = -1, stage = 0, chunk = 0, count = 1, status = 0;   // status 0: work, 1: wait, 2: leave
      uint32_t done = rfl(ld_acq(&sched[3]));
      if (idle)
        for (int k = 0; k < kIdlePolls && done == seen; ++k) {
          __builtin_amdgcn_s_sleep(64);
          done = rfl(ld_acq(&sched[3]));
        }
      seen = done;
      moved = false;
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane(ld_acq(&sched[0]));
      for (uint32_t b0 = lo; job < 0 && b0 < (uint32_t)nstaged && b0 < lo + kScanWindow; b0 += 64) {
        const uint32_t j = b0 + lane;
        bool fin = true, avail = false;
        if (j < (uint32_t)nstaged) {
          const BJob& jb = jobs[j];
          const unsigned long long wd = ld_acq64(&ctl[j].word);
          const uint32_t s0 = (uint32_t)(wd >> 32);
          fin = s0 >= jb.nst;
          avail = !fin && (uint32_t)wd < stages[jb.st_begin + s0].nchunks;
        }
        const unsigned long long fm = __ballot(fin);
        if (b0 == lo && (fm & 1ull)) {   // a finished prefix: move the hint past it
          moved = true;
          const uint32_t np = ~fm == 0 ? 64u : (uint32_t)__builtin_ctzll(~fm);
          if (lane == 0) atomicMax(&sched[0], b0 + np);
        }
        unsigned long long av = __ballot(avail);
        while (av) {
          const unsigned long long rv = rot ? (av >> rot) | (av << (64 - rot)) : av;
          const int l = (int)((__builtin_ctzll(rv) + rot) & 63u);
          int got = 0, s2 = 0, c2 = 0, cnt = 0;
          if (lane == l) {
            // a run of chunks per claim: fewer atomics on the job's line
            const BJob& jb = jobs[j];
            const uint32_t nck = stages[jb.st_begin + (uint32_t)(ld_acq64(&ctl[j].word) >> 32) % jb.nst].nchunks;
            const uint32_t want = min(run_max, max(1u, nck >> 4));
            const unsigned long long old = atomicAdd(&ctl[j].word, (unsigned long long)want);
            s2 = (int)(old >> 32);
            c2 = (int)(uint32_t)old;
            if ((uint32_t)s2 < jb.nst) {
              const uint32_t n2 = stages[jb.st_begin + s2].nchunks;
              got = (uint32_t)c2 < n2;
              cnt = got ? (int)min(want, n2 - (uint32_t)c2) : 0;
            }
          }
          if (__ballot(got)) {
            job = (int)(b0 + l);
            stage = __shfl(s2, l, 64);
            chunk = __shfl(c2, l, 64);
            count = __shfl(cnt, l, 64);
            break;
          }
          av &= ~(1ull << l);
        }
      }
      if (lane == 0) {
        if (job < 0 && ld_acq(&sched[1]) < (unsigned)(njobs - nstaged)) {
          const unsigned q = atomicAdd(&sched[1], 1u);
          if (q < (unsigned)(njobs - nstaged)) job = nstaged + (int)q;
        }
        if (job < 0) {
          if (ld_acq(&sched[0]) >= (unsigned)nstaged) {
            status = 2;
          } else {
            const unsigned long long t = wall_clock64();
            if (idle_since == 0) idle_since = t;
            if (t - idle_since > stall_ticks) {
              atomicOr(&sched[2], 1u);
              status = 2;
            } else {
              status = 1;
            }
          }
        } else {
          idle_since = 0;
        }
        task[0] = job;
        task[1] = stage;
        task[2] = chunk;
        task[3] = status;
        task[4] = count;
      }
    }
    __syncthreads();
    const int job = __builtin_amdgcn_readfirstlane(task[0]);
    const uint32_t stage = (uint32_t)__builtin_amdgcn_readfirstlane(task[1]);
    const uint32_t chunk = (uint32_t)__builtin_amdgcn_readfirstlane(task[2]);
    const int status = __builtin_amdgcn_readfirstlane(task[3]);
    const uint32_t count = (uint32_t)__builtin_amdgcn_readfirstlane(task[4]);
    __syncthreads();   // task[] is rewritten by the next search
    if (status == 2) break;
    idle = status == 1 && !moved;
    if (status == 1) continue;
    const BJob jb = jobs[job];
    const uint32_t dim = 1u << jb.n;
    C* gst = states + jb.state_off;
    const __amdgpu_buffer_rsrc_t gbuf = state_buffer(gst, dim);
    // a small job (its whole state one chunk), or a run of chunks of a stage
    // of a staged job.  The latter's reads go past the caches (load_through),
    // after the claim and the barrier above, so every chunk of the earlier
    // stages, written through by any workgroup, is visible.
    const bool small = job >= nstaged;
    BStage bs{jb.rec, 1u, ST_GATES};
    if (!small) bs = stages[jb.st_begin + stage];
    for (int c = tid; c < jb.ncbits; c += bd) cb[c] = small ? (uint8_t)0 : __hip_atomic_load(&cbits[jb.cbit_off + c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const RecWords h = rec_words(opw, rfl(bs.rec));
    if (bs.kind != ST_GATES) {
      const uint32_t mq = (uint32_t)meas_qubits(jb.n, LQ), nparts = 1u << (jb.n - mq), qb = h[1];
      double* part = parts + (size_t)job * 2 * kMeasParts;
      if (bs.kind == ST_SUMS) {
        for (uint32_t ch = chunk; ch < chunk + count; ++ch)
          meas_sums<R>(gbuf, ch << mq, 1u << mq, qb, red, part + 2 * ch);
      } else {
        const uint64_t ulo = h[4], uhi = h[5];
        const double u = __longlong_as_double((long long)(ulo | (uhi << 32)));
        const int cbit = (int)h[3];
        const bool on = tid < nparts;
        meas_decide(on ? load_through(&part[2 * tid]) : 0.0, on ? load_through(&part[2 * tid + 1]) : 0.0, u, cbit, cb, red, meas);
        if (meas[0] != 0.0)
          meas_scale<R>(gbuf, chunk << mq, count << mq, qb, (R)meas[0], meas[1] != 0.0);
        if (tid == 0 && chunk == 0 && cbit >= 0)
          __hip_atomic_store(&cbits[jb.cbit_off + cbit], cb[cbit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    } else {
      const int L = small ? jb.n : LQ;
      ChunkMap cm(h, L, dim, tid);
#pragma unroll 1
      for (uint32_t ch = chunk; ch < chunk + count; ++ch) {
        const uint32_t cpart = small ? 0u : deposit(ch, cm.cmask), g0 = cm.base | cpart;
        R xr[kMembers], xi[kMembers];
#pragma unroll
        for (int k = 0; k < kMembers; ++k) {   // small jobs, and a staged job's first stage, start from |0...0>
          xr[k] = (k == 0 && g0 == 0) ? (R)1 : (R)0;
          xi[k] = 0;
        }
        if (!small && stage != 0 && cm.live) {
#pragma unroll
          for (int k = 0; k < kMembers; ++k) {
            C x;
            load_through(gbuf, g0 | cm.index(k), x);
            xr[k] = x.x;
            xi[k] = x.y;
          }
        }
        run_chunk<R>(lds, xr, xi, cm, h, L, cpart | kOneBit, cb, red, meas);
        cm.opaque();
#pragma unroll
        for (int k = 0; k < kMembers; ++k) {
          C x;
          x.x = xr[k];
          x.y = xi[k];
          if (cm.live && (L >= kPassSlots || k < (1 << L))) store_through(gbuf, g0 | cm.index(k), x);
        }
      }
    }
    __syncthreads();   // cb[] is read by all threads below and set again for the next task
    if (small) {
      for (int c = tid; c < jb.ncbits; c += bd) {
        cbits[jb.cbit_off + c] = cb[c];
        if (host_cbits) host_cbits[jb.cbit_off + c] = cb[c];
      }
      __syncthreads();
      continue;
    }
    // Every wave's stores have completed, written through (see store_through),
    // before the barrier, and so before the chunks count as done; the
    // workgroup that completes a stage opens the next one.
    stores_done();
    __syncthreads();
    if (tid == 0) {
      const unsigned d = atomicAdd(&ctl[job].done, count) + count;
      if (d == bs.nchunks) {
        atomicExch(&ctl[job].done, 0u);
        stores_done();
        if (stage + 1 == jb.nst && host_cbits)
          for (int c = 0; c < jb.ncbits; ++c)
            host_cbits[jb.cbit_off + c] =
                __hip_atomic_load(&cbits[jb.cbit_off + c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicExch(&ctl[job].word, (unsigned long long)(stage + 1) << 32);
        stores_done();
        atomicAdd(&sched[3], 1u);
      }
    }
  }
}

// Clears a launch's scheduling state and every cbit (a staged job's cbits
// are read by each of its chunks; the host's copy too, so that a launch that
// ended early leaves no outcomes of the one before).  A kernel rather than a
// memset so that a captured batch launch replays correctly.
__global__ void k_batch_reset(JobCtl* ctl, int nctl, unsigned* sched, uint8_t* cbits, uint8_t* host_cbits, uint32_t ncbits) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
  for (uint32_t k = i; k < (uint32_t)nctl; k += stride) {
    ctl[k].word = 0;
    ctl[k].done = 0;
  }
  for (uint32_t k = i; k < ncbits; k += stride) {
    cbits[k] = 0;
    if (host_cbits) host_cbits[k] = 0;
  }
  if (i < 4) sched[i] = 0;
}

// The chunk that the i-th position of the stage kernel's chunk loop takes:
// i with its low 3 bits rotated to the top.  Workgroups go to the 8 XCDs in
// turn (workgroup b to XCD b mod 8) and the grid is a multiple of 8, so XCD
// x takes the chunks [x R, (x + 1) R), R = nchunks / 8, and the workgroups
// of one XCD hold consecutive chunks at any time: chunks that differ only
// in the lowest qubits outside the stage share 128-byte lines where the
// stage's runs are shorter (complex64: 2^3 amplitudes are 64 bytes), and then
// meet in that XCD's L2.
__device__ __forceinline__ uint32_t xcd_chunk(uint32_t i, uint32_t nchunks) {
  return nchunks >= 8 ? ((i & 7u) * (nchunks >> 3)) | (i >> 3) : i;
}

// One stage of a simulator's held-back gates (the LDS-tile mode): every
// chunk of the state, a chunk per workgroup at a time.  The stage's header
// is record hrec of opw; the gates' cbit conditions read cbits.
template <typename R>
__global__ __launch_bounds__(1 << (stage_qubits<R>() - kPassSlots), stage_waves<R>()) void k_stage(
    typename EVb<R>::T* __restrict__ psi, int n, const uint32_t* __restrict__ opw, uint32_t hrec,
    const uint8_t* __restrict__ cbits, int ncbits) {
  using C = typename EVb<R>::T;
  constexpr int LQ = stage_qubits<R>(), BD = 1 << (LQ - kPassSlots);
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ uint8_t cb[kMaxJobCbits];
  const uint32_t tid = threadIdx.x, dim = 1u << n;
  for (int i = tid; i < ncbits && i < kMaxJobCbits; i += BD) cb[i] = cbits[i];
  __syncthreads();
  const RecWords h = rec_words(opw, hrec);
  ChunkMap cm(h, LQ, dim, tid);
  const uint32_t nchunks = dim >> LQ;
  for (uint32_t i = blockIdx.x; i < nchunks; i += gridDim.x) {
    const uint32_t cpart = deposit(xcd_chunk(i, nchunks), cm.cmask);
    C* p = psi + (cm.base | cpart);
    R xr[kMembers], xi[kMembers];
#pragma unroll
    for (int k = 0; k < kMembers; ++k) {
      const C x = p[cm.index(k)];
      xr[k] = x.x;
      xi[k] = x.y;
    }
    run_chunk<R>(lds, xr, xi, cm, h, LQ, cpart | kOneBit, cb, nullptr, nullptr);
    cm.opaque();
#pragma unroll
    for (int k = 0; k < kMembers; ++k) {
      C x;
      x.x = xr[k];
      x.y = xi[k];
      p[cm.index(k)] = x;
    }
  }
}

struct HostJob {
  int n, ncbits;
  bool staged = false;    // state in global memory, run by stages
  std::vector<uint32_t> rec;     // records (stage_records.h), ready to upload
  std::vector<uint32_t> heads;   // staged: the record index of each stage or measurement
  uint64_t state_off = 0;
  uint32_t cbit_off = 0;
};

std::string g_batch_error;

}  // namespace

struct qk_batch_s {
  qk_dtype dtype = QK_C128;
  bool c64 = false;
  qk_allocator alloc{};
  bool has_alloc = false;
  hipStream_t stream = nullptr;
  std::vector<HostJob> jobs;
  std::vector<PlanOp> plan;       // of the job being added; as the records, kept for the next one
  std::vector<uint32_t> rec;
  void* d_states = nullptr;
  size_t states_bytes = 0;
  void* d_cbits = nullptr;
  size_t cbits_bytes = 0;
  std::vector<std::pair<uint8_t*, size_t>> h_cbits;   // the same in pinned host memory, written by the kernel at each
                                                      // job's end: the last block, and outgrown ones (grow_mirror)
  uint8_t* mirror = nullptr;   // that block, for the current jobs, or nullptr (reads then copy from the device)
  bool cbit_reads = false, async_reads = false;   // how this batch's results have been read
  void* d_ops = nullptr;
  size_t ops_bytes = 0;
  void* d_jobs = nullptr;
  size_t jobs_bytes = 0;
  void* d_stages = nullptr;   // stage table of the staged jobs
  size_t stages_bytes = 0;
  void* d_ctl = nullptr;      // per staged job scheduling state
  size_t ctl_bytes = 0;
  void* d_parts = nullptr;    // sums of a staged job's measurement, kMeasParts pairs each
  size_t parts_bytes = 0;
  void* d_sched = nullptr;    // scan hint, small-job counter, stall flag, stages completed
  size_t sched_bytes = 0;
  size_t nstaged = 0;
  size_t ncbits_total = 0;
  uint32_t run_max = 1;       // longest run of chunks one claim takes
  bool ran = false;
  bool uploaded = false;   // the device job table and ops match `jobs` (a rerun only relaunches)
  size_t njobs_dev = 0;
  size_t shm = 0;
  unsigned grid = 0, block = 64;
  std::string err;
};

namespace {

qk_status bfail(qk_batch b, qk_status st, const std::string& m) {
  if (b) b->err = m;
  else g_batch_error = m;
  return st;
}

void* balloc(qk_batch b, size_t bytes) {
  if (bytes == 0) bytes = 256;
  if (b->has_alloc) return b->alloc.alloc(bytes, (void*)b->stream, b->alloc.ctx);
  void* p = nullptr;
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return p;
}

void bfree(qk_batch b, void*& p, size_t& bytes) {
  if (!p) return;
  if (b->has_alloc) b->alloc.free(p, bytes, (void*)b->stream, b->alloc.ctx);
  else (void)hipFree(p);
  p = nullptr;
  bytes = 0;
}

qk_status bensure(qk_batch b, void*& p, size_t& cur, size_t need, const char* what) {
  if (p && cur >= need) return QK_OK;
  bfree(b, p, cur);
  p = balloc(b, need);
  if (!p) return bfail(b, QK_E_OOM, std::string("device allocation failed: ") + what);
  cur = need;
  return QK_OK;
}

// Calls of this thread that a stream capture of any thread forbids (pinned
// memory's) neither fail in one nor end it.
class CaptureAllowed {
 public:
  CaptureAllowed() { on_ = hipThreadExchangeStreamCaptureMode(&mode_) == hipSuccess; }
  ~CaptureAllowed() {
    if (on_) (void)hipThreadExchangeStreamCaptureMode(&mode_);
  }

 private:
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
  bool on_;
};

// Pinned blocks for cbits, kept for the life of the process and shared by every
// batch: one that is made, run once and read would pay for pinning its own
// and, as that waits for the device, for unpinning.  A block is given back once
// its batch's stream has drained.
constexpr size_t kMirrorBytes = 64 << 10, kMirrorPoolMax = 16;
std::mutex g_mirror_mu;
std::vector<uint8_t*> g_mirror_free;

uint8_t* mirror_take(size_t bytes) {
  if (bytes == kMirrorBytes) {
    std::lock_guard<std::mutex> lk(g_mirror_mu);
    if (!g_mirror_free.empty()) {
      uint8_t* p = g_mirror_free.back();
      g_mirror_free.pop_back();
      return p;
    }
  }
  CaptureAllowed allowed;
  void* p = nullptr;
  if (hipHostMalloc(&p, bytes, hipHostMallocDefault) == hipSuccess) return (uint8_t*)p;
  (void)hipGetLastError();
  return nullptr;
}

void mirror_give(uint8_t* p, size_t bytes) {
  if (bytes == kMirrorBytes) {
    std::lock_guard<std::mutex> lk(g_mirror_mu);
    if (g_mirror_free.size() < kMirrorPoolMax) {
      g_mirror_free.push_back(p);
      return;
    }
  }
  CaptureAllowed allowed;
  (void)hipHostFree(p);
}

// The blocks of a batch grow by doubling, and an outgrown one is kept until the
// batch goes (together they are smaller than the last), so that a batch filled
// again and again allocates a few times and never waits: a launch may still
// write the old one.
void grow_mirror(qk_batch b, size_t need) {
  const size_t have = b->h_cbits.empty() ? 0 : b->h_cbits.back().second;
  if (need <= have) return;
  const size_t bytes = std::max<size_t>({need, 2 * have, kMirrorBytes});
  if (uint8_t* p = mirror_take(bytes)) b->h_cbits.emplace_back(p, bytes);
}

// Jobs up to these sizes keep their whole state on chip; larger ones, up to
// kMaxStagedQubits, keep it in global memory and run by stages of
// stage_qubits() qubits.  (Staged as well, 1024 jobs of the largest size here
// take 3.3 ms in complex64 and 2.8 ms in complex128, against 1.0 and 0.6 ms.)
int max_lds_qubits(bool c64) { return c64 ? 14 : 13; }
constexpr int kMaxStagedQubits = 24;

}  // namespace

extern "C" {

qk_status qk_batch_create(qk_dtype dtype, const qk_allocator* alloc, void* hip_stream, qk_batch* out) {
  if (!out) return bfail(nullptr, QK_E_ARG, "out is NULL");
  *out = nullptr;
  if (dtype != QK_C64 && dtype != QK_C128) return bfail(nullptr, QK_E_ARG, "dtype must be QK_C64 or QK_C128");
  if (alloc && (!alloc->alloc || !alloc->free)) return bfail(nullptr, QK_E_ARG, "allocator needs alloc and free");
  qk_batch b = new qk_batch_s;
  b->dtype = dtype;
  b->c64 = dtype == QK_C64;
  if (alloc) {
    b->alloc = *alloc;
    b->has_alloc = true;
  }
  b->stream = (hipStream_t)hip_stream;
  *out = b;
  return QK_OK;
}

qk_status qk_batch_destroy(qk_batch b) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (b->d_states || b->d_ops) (void)hipStreamSynchronize(b->stream);
  bfree(b, b->d_states, b->states_bytes);
  bfree(b, b->d_cbits, b->cbits_bytes);
  bfree(b, b->d_ops, b->ops_bytes);
  bfree(b, b->d_jobs, b->jobs_bytes);
  bfree(b, b->d_stages, b->stages_bytes);
  bfree(b, b->d_ctl, b->ctl_bytes);
  bfree(b, b->d_sched, b->sched_bytes);
  bfree(b, b->d_parts, b->parts_bytes);
  for (const auto& m : b->h_cbits) mirror_give(m.first, m.second);
  delete b;
  return QK_OK;
}

const char* qk_batch_last_error(qk_batch b) { return b ? b->err.c_str() : g_batch_error.c_str(); }

qk_status qk_batch_add(qk_batch b, int32_t n, int32_t ncbits, const qk_op* ops, int32_t nops, int32_t* job) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (n < 1 || n > kMaxStagedQubits)
    return bfail(b, QK_E_ARG, "qubit count outside the batched range (1.." + std::to_string(kMaxStagedQubits) + ")");
  if (ncbits < 0 || ncbits > kMaxJobCbits) return bfail(b, QK_E_ARG, "cbit count outside 0..256");
  if (nops < 0 || (nops > 0 && !ops)) return bfail(b, QK_E_ARG, "bad op array");
  HostJob hj;
  hj.n = n;
  hj.ncbits = ncbits;
  b->plan.clear();
  for (int i = 0; i < nops; ++i) {
    std::string err;
    const qk_status st = expand_op(ops[i], n, ncbits, b->plan, err);
    if (st) return bfail(b, st, "op " + std::to_string(i) + ": " + err);
  }
  hj.staged = n > max_lds_qubits(b->c64);
  b->rec.clear();
  if (hj.staged) build_stages(n, stage_chunk_qubits(b->c64), b->c64, b->plan, true, b->rec, hj.heads);
  else build_job(n, b->c64, b->plan, b->rec);
  hj.rec = b->rec;   // (grown in the job's own vector, they cost a fifth of compiling it)
  b->jobs.push_back(std::move(hj));
  if (job) *job = (int32_t)b->jobs.size() - 1;
  b->ran = false;
  b->uploaded = false;
  return QK_OK;
}

}  // extern "C"

template <typename R>
static void launch_batch_t(qk_batch b) {
  hipLaunchKernelGGL(k_batch_reset, dim3(64), dim3(256), 0, b->stream, (JobCtl*)b->d_ctl, (int)b->nstaged,
                     (unsigned*)b->d_sched, (uint8_t*)b->d_cbits, b->mirror, (uint32_t)b->ncbits_total);
  static unsigned long long stall = 0;   // 10 s of the device wall clock
  if (!stall) {
    int khz = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
      khz = 100000;
    stall = 10000ull * (unsigned long long)khz;
  }
  hipLaunchKernelGGL(k_batch<R>, dim3(b->grid), dim3(b->block), b->shm, b->stream, (const BJob*)b->d_jobs,
                     (int)b->njobs_dev, (int)b->nstaged, (const BStage*)b->d_stages, (JobCtl*)b->d_ctl,
                     (unsigned*)b->d_sched, (const uint32_t*)b->d_ops, (typename EVb<R>::T*)b->d_states,
                     (uint8_t*)b->d_cbits, b->mirror, (double*)b->d_parts, stall, b->run_max);
}

static void launch_batch(qk_batch b) {
  if (b->c64) launch_batch_t<float>(b);
  else launch_batch_t<double>(b);
}

extern "C" {

qk_status qk_batch_run(qk_batch b) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (b->jobs.empty()) return QK_OK;
  if (b->uploaded) {   // same jobs as the last run: only the scheduling state is reset
    launch_batch(b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch launch: ") + hipGetErrorString(e));
    b->ran = true;
    return QK_OK;
  }
  const size_t amp = b->c64 ? 8 : 16;
  const int lq = b->c64 ? stage_qubits<float>() : stage_qubits<double>();
  // layout: states and cbits in job order; the device table lists the staged
  // jobs first, then the small ones, each part largest first
  uint64_t soff = 0;
  uint32_t coff = 0, ooff = 0;
  int nmax = 0;   // largest job that is one chunk, or the stage chunk when larger
  for (auto& j : b->jobs) {
    j.state_off = soff;
    j.cbit_off = coff;
    soff += 1ull << j.n;
    coff += (uint32_t)j.ncbits;
    nmax = std::max(nmax, j.staged ? lq : j.n);
  }
  std::vector<int> order(b->jobs.size());
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
    const auto& a = b->jobs[x];
    const auto& c = b->jobs[y];
    if (a.staged != c.staged) return a.staged;
    return ((uint64_t)a.rec.size() << a.n) > ((uint64_t)c.rec.size() << c.n);
  });
  std::vector<uint32_t> all_ops;
  std::vector<BJob> table;
  std::vector<BStage> stab;
  size_t nstaged = 0, words = (size_t)kPadRecords * kRecWords;
  for (const auto& j : b->jobs) words += j.rec.size();
  all_ops.reserve(words);
  bool measured = false;   // staged jobs with measurements
  for (int id : order) {
    const auto& j = b->jobs[id];
    BJob t{};
    t.state_off = j.state_off;
    t.rec = ooff;
    all_ops.insert(all_ops.end(), j.rec.begin(), j.rec.end());
    t.n = j.n;
    t.ncbits = j.ncbits;
    t.cbit_off = j.cbit_off;
    if (j.staged) {
      ++nstaged;
      t.st_begin = (uint32_t)stab.size();
      for (uint32_t r : j.heads) {
        const uint32_t nchunks = 1u << (j.n - lq);
        if ((j.rec[(size_t)r * kRecWords] & 0xff) == RK_MEAS) {
          measured = true;
          for (uint32_t kind : {ST_SUMS, ST_SCALE})
            stab.push_back({ooff + r, std::min<uint32_t>(nchunks, kMeasParts), kind});
        } else {
          stab.push_back({ooff + r, nchunks, ST_GATES});
        }
      }
      t.nst = (uint32_t)stab.size() - t.st_begin;
    }
    ooff += (uint32_t)(j.rec.size() / kRecWords);
    table.push_back(t);
  }
  all_ops.resize(words);   // a gate reads the record after it
  qk_status st;
  if ((st = bensure(b, b->d_states, b->states_bytes, soff * amp, "batch states"))) return st;
  if ((st = bensure(b, b->d_cbits, b->cbits_bytes, std::max<size_t>(coff, 1), "batch cbits"))) return st;
  // a batch whose results are read by qk_batch_read_async alone needs no copy of the cbits
  const bool wanted = coff && (b->cbit_reads || !b->async_reads);
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  (void)hipStreamIsCapturing(b->stream, &cap);
  if (wanted && cap == hipStreamCaptureStatusNone) grow_mirror(b, coff);
  b->mirror = wanted && !b->h_cbits.empty() && b->h_cbits.back().second >= coff ? b->h_cbits.back().first : nullptr;
  if ((st = bensure(b, b->d_ops, b->ops_bytes, all_ops.size() * sizeof(uint32_t), "batch ops"))) return st;
  if ((st = bensure(b, b->d_jobs, b->jobs_bytes, table.size() * sizeof(BJob), "batch job table"))) return st;
  if ((st = bensure(b, b->d_stages, b->stages_bytes, std::max<size_t>(stab.size(), 1) * sizeof(BStage), "batch stages")))
    return st;
  if ((st = bensure(b, b->d_ctl, b->ctl_bytes, std::max<size_t>(nstaged, 1) * sizeof(JobCtl), "batch scheduling")))
    return st;
  if (measured && (st = bensure(b, b->d_parts, b->parts_bytes, nstaged * 2 * kMeasParts * sizeof(double), "batch sums")))
    return st;
  if ((st = bensure(b, b->d_sched, b->sched_bytes, 4 * sizeof(unsigned), "batch scheduling"))) return st;
  hipError_t e = hipMemcpyAsync(b->d_ops, all_ops.data(), all_ops.size() * sizeof(uint32_t), hipMemcpyHostToDevice, b->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(b->d_jobs, table.data(), table.size() * sizeof(BJob), hipMemcpyHostToDevice, b->stream);
  if (e == hipSuccess && !stab.empty())
    e = hipMemcpyAsync(b->d_stages, stab.data(), stab.size() * sizeof(BStage), hipMemcpyHostToDevice, b->stream);
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch upload: ") + hipGetErrorString(e));
  // one component of the largest state or chunk (one group of a pass at
  // least) in LDS, and a thread for each of its groups
  nmax = std::max(nmax, kPassSlots);
  const size_t shm = (amp / 2) << nmax;
  b->block = 1u << std::max(6, nmax - kPassSlots);
  int ncu = 256, dev = 0, per_cu = 1;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  const void* fn = b->c64 ? (const void*)k_batch<float> : (const void*)k_batch<double>;
  (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, (int)b->block, shm) != hipSuccess || per_cu < 1) per_cu = 1;
  // staged jobs spread their chunks over every workgroup that fits; small
  // jobs need at most one workgroup each
  const size_t want = nstaged ? (size_t)ncu * per_cu : std::min<size_t>(table.size(), (size_t)ncu * per_cu);
  b->shm = shm;
  b->grid = (unsigned)std::max<size_t>(1, want);
  b->njobs_dev = table.size();
  b->nstaged = nstaged;
  b->ncbits_total = coff;
  // Runs of chunks per claim save atomics on the jobs' lines when the staged
  // work is plentiful (about two claims per workgroup per round of stages),
  // and shrink to single chunks when a few jobs must spread over the grid.  96
  // circuits of 8-20 qubits: 3.55 ms by single chunks, 2.20 ms like this
  // (complex128), 2.23 and 1.92 ms (complex64).
  uint64_t chunks = 0;
  for (const BJob& t : table)
    if (t.nst) chunks += 1ull << (t.n - lq);
  b->run_max = (uint32_t)std::min<uint64_t>(16, std::max<uint64_t>(1, chunks / (2ull * b->grid)));
  launch_batch(b);
  e = hipGetLastError();
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch launch: ") + hipGetErrorString(e));
  b->ran = true;
  b->uploaded = true;
  return QK_OK;
}

qk_status qk_batch_sync(qk_batch b) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  hipError_t e = hipStreamSynchronize(b->stream);
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch: ") + hipGetErrorString(e));
  if (b->ran && b->nstaged && b->d_sched) {
    unsigned flags[4] = {0, 0, 0, 0};
    e = hipMemcpy(flags, b->d_sched, sizeof(flags), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch: ") + hipGetErrorString(e));
    if (flags[2]) return bfail(b, QK_E_HIP, "batch: a workgroup found no work for 10 s while stages were open (scheduler stall)");
  }
  return QK_OK;
}

qk_status qk_batch_get_state(qk_batch b, int32_t job, void* host_out, size_t bytes) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (job < 0 || job >= (int)b->jobs.size()) return bfail(b, QK_E_ARG, "job index out of range");
  if (!b->ran) return bfail(b, QK_E_STATE, "batch has not run since the job was added");
  const size_t amp = b->c64 ? 8 : 16;
  const auto& j = b->jobs[job];
  const size_t need = ((size_t)1 << j.n) * amp;
  if (!host_out || bytes != need) return bfail(b, QK_E_ARG, "buffer size must be 2^n * amplitude size");
  hipError_t e = hipMemcpyAsync(host_out, (char*)b->d_states + j.state_off * amp, need, hipMemcpyDeviceToHost, b->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch readback: ") + hipGetErrorString(e));
  return QK_OK;
}

qk_status qk_batch_read_cbits(qk_batch b, int32_t job, uint8_t* out, int32_t n) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (job < 0 || job >= (int)b->jobs.size()) return bfail(b, QK_E_ARG, "job index out of range");
  if (!b->ran) return bfail(b, QK_E_STATE, "batch has not run since the job was added");
  const auto& j = b->jobs[job];
  if (n < 0 || n > j.ncbits || (n > 0 && !out)) return bfail(b, QK_E_ARG, "bad cbit count");
  b->cbit_reads = true;
  hipError_t e = hipSuccess;
  if (n > 0 && !b->mirror)
    e = hipMemcpyAsync(out, (char*)b->d_cbits + j.cbit_off, (size_t)n, hipMemcpyDeviceToHost, b->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch readback: ") + hipGetErrorString(e));
  if (n > 0 && b->mirror) std::memcpy(out, b->mirror + j.cbit_off, (size_t)n);
  return QK_OK;
}

qk_status qk_batch_state_ptr(qk_batch b, int32_t job, void** dev_ptr, size_t* bytes) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (job < 0 || job >= (int)b->jobs.size()) return bfail(b, QK_E_ARG, "job index out of range");
  if (!b->ran) return bfail(b, QK_E_STATE, "batch has not run since the job was added");
  const size_t amp = b->c64 ? 8 : 16;
  const auto& j = b->jobs[job];
  if (dev_ptr) *dev_ptr = (char*)b->d_states + j.state_off * amp;
  if (bytes) *bytes = ((size_t)1 << j.n) * amp;
  return QK_OK;
}

qk_status qk_batch_layout(qk_batch b, int32_t job, size_t* state_offset, size_t* state_bytes, size_t* cbit_offset) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (job < 0 || job >= (int)b->jobs.size()) return bfail(b, QK_E_ARG, "job index out of range");
  uint64_t soff = 0, coff = 0;   // the layout qk_batch_run uses: states and cbits in job order
  for (int32_t i = 0; i < job; ++i) {
    soff += 1ull << b->jobs[i].n;
    coff += (uint64_t)b->jobs[i].ncbits;
  }
  const size_t amp = b->c64 ? 8 : 16;
  if (state_offset) *state_offset = soff * amp;
  if (state_bytes) *state_bytes = ((size_t)1 << b->jobs[job].n) * amp;
  if (cbit_offset) *cbit_offset = coff;
  return QK_OK;
}

qk_status qk_batch_read_async(qk_batch b, void* host_states, size_t state_bytes, uint8_t* host_cbits,
                              size_t cbit_bytes) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  if (!b->ran || !b->uploaded) return bfail(b, QK_E_STATE, "batch has not run since the last job was added");
  b->async_reads = true;
  uint64_t samps = 0, cbytes = 0;
  for (const auto& j : b->jobs) {
    samps += 1ull << j.n;
    cbytes += (uint64_t)j.ncbits;
  }
  const size_t need = samps * (b->c64 ? 8 : 16);
  if (!host_states || state_bytes < need) return bfail(b, QK_E_ARG, "state buffer smaller than the batch's states");
  if (cbytes && (!host_cbits || cbit_bytes < cbytes)) return bfail(b, QK_E_ARG, "cbit buffer smaller than the batch's cbits");
  hipError_t e = hipMemcpyAsync(host_states, b->d_states, need, hipMemcpyDeviceToHost, b->stream);
  if (e == hipSuccess && cbytes) e = hipMemcpyAsync(host_cbits, b->d_cbits, cbytes, hipMemcpyDeviceToHost, b->stream);
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch asynchronous read: ") + hipGetErrorString(e));
  return QK_OK;
}

qk_status qk_batch_clear(qk_batch b) {
  if (!b) return bfail(nullptr, QK_E_ARG, "batch is NULL");
  b->jobs.clear();
  b->ran = false;
  b->uploaded = false;
  return QK_OK;
}

qk_status qk_batch_num_jobs(qk_batch b, int32_t* n) {
  if (!b || !n) return bfail(b, QK_E_ARG, "NULL argument");
  *n = (int32_t)b->jobs.size();
  return QK_OK;
}

}  // extern "C"

// ---- the simulator's LDS-tile mode ---------------------------------------------

namespace qk {

int stage_chunk_qubits(bool c64) { return c64 ? stage_qubits<float>() : stage_qubits<double>(); }

qk_status stage_plan(bool c64, int n, int ncbits, const std::vector<qk_op>& ops, std::vector<uint32_t>& recs,
                     std::vector<uint32_t>& headers, std::string& err) {
  std::vector<PlanOp> plan;
  plan.reserve(ops.size() + 8);
  for (size_t i = 0; i < ops.size(); ++i) {
    qk_status st = QK_OK;
    if (ops[i].kind == QK_OP_MEASURE) {
      err = "measurements are not staged";
      st = QK_E_ARG;
    } else {
      st = expand_op(ops[i], n, std::min(ncbits, kMaxJobCbits), plan, err);
    }
    if (st) {
      err = "op " + std::to_string(i) + ": " + err;
      return st;
    }
  }
  headers.clear();
  recs.clear();
  build_stages(n, stage_chunk_qubits(c64), c64, plan, false, recs, headers);
  recs.resize(recs.size() + (size_t)kPadRecords * kRecWords, 0u);   // a gate reads the record after it
  return QK_OK;
}

template <typename R>
static void launch_stage_t(void* psi, int n, const void* d_recs, uint32_t hrec, const uint8_t* d_cbits, int ncbits,
                           hipStream_t stream) {
  constexpr int LQ = stage_qubits<R>(), BD = 1 << (LQ - kPassSlots);
  const size_t shm = sizeof(R) << LQ;   // one component of a chunk: 32 KiB
  static unsigned resident = 0;         // workgroups that run at a time
  if (!resident) {
    int ncu = 256, dev = 0, per_cu = 1;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)k_stage<R>, BD, shm) != hipSuccess || per_cu < 1)
      per_cu = 1;
    resident = (unsigned)(ncu * per_cu);
  }
  const uint32_t nchunks = 1u << (n - LQ);
  hipLaunchKernelGGL(k_stage<R>, dim3(std::min<uint32_t>(nchunks, resident)), dim3(BD), shm, stream,
                     (typename EVb<R>::T*)psi, n, (const uint32_t*)d_recs, hrec, d_cbits, ncbits);
}

void launch_stage(bool c64, void* psi, int n, const void* d_recs, uint32_t hrec, const uint8_t* d_cbits, int ncbits,
                  hipStream_t stream) {
  if (c64) launch_stage_t<float>(psi, n, d_recs, hrec, d_cbits, ncbits, stream);
  else launch_stage_t<double>(psi, n, d_recs, hrec, d_cbits, ncbits, stream);
}

}  // namespace qk
