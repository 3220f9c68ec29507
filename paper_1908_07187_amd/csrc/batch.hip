// Batched execution: many circuits of uneven qubit counts in one persistent
// launch, and the stage kernel of the simulator's LDS-tile mode.
//
// Each circuit ("job") is compiled on the host (stages.cpp) into compact
// device records (stage_records.h): passes over four slot qubits, and
// measurements.  Bit flips, CNOTs and swaps cost nothing there: they change
// what the LDS positions stand for.  One persistent grid runs all jobs: every
// workgroup takes the next job from a device counter (largest jobs first),
// builds |0...0> in LDS and runs the job's items one after another, a barrier
// after each.  In a pass every thread loads the 16 amplitudes of its group
// (the combinations of the pass's slots) from LDS, applies the pass's gates
// in registers and stores them back, so a pass costs one LDS round trip
// whatever its gate count; one-qubit gates act on the slots, diagonal and
// phase gates on any qubits.  A job's state stays in LDS for its whole
// circuit, so a 12-qubit, 360-gate circuit costs one HBM write instead of 360
// sweeps and 360 launches.  Every workgroup leaves the loop once the counter
// passes the job count.
//
// Jobs too large for LDS (above 13 qubits complex128, 14 complex64; up to
// 24) run in the same launch with their state in global memory.  The host
// splits such a job into stages: runs of gates, reordered only where they
// commute, whose targets fit one LDS chunk (12 qubits complex128, 13
// complex64; controls and the qubits of diagonal gates may lie outside: for a
// chunk they are constants), and measurements between them.  A stage's chunks (the
// amplitudes that share the values of the qubits outside the stage) are
// independent, so any free workgroup claims a run of them: it gathers each
// into LDS, runs the stage's items on it exactly as for a small job, and
// scatters it back; the workgroup that completes a stage's last chunk opens
// the next stage.  A stage costs one read and one write of the state
// whatever its gate count; a measurement runs over the state in global
// memory on one workgroup.  Workgroups take staged chunks first and small
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
#include <numeric>
#include <string>
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

constexpr int kBatchThreads = 256;        // threads of a batch workgroup at most (the stage kernel's complex128 form too)
constexpr int kMaxJobCbits = 256;
constexpr int kMaxWaves = 8;
// Items per thread whose LDS reads are issued together in a measurement.
constexpr int kBU = 2;

typedef uint32_t QkU4 __attribute__((ext_vector_type(4)));

template <typename R> struct EVb;
template <> struct EVb<float> { typedef float T __attribute__((ext_vector_type(2))); };
template <> struct EVb<double> { typedef double T __attribute__((ext_vector_type(2))); };

__device__ __forceinline__ uint32_t rfl(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

__device__ __forceinline__ double bwave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// An item's records (at most kItemWords dwords) are read from global memory
// one item ahead, lane l of wave 0 holding dwords l, 64 + l, ...; it copies
// them into one of two LDS buffers before the barrier
// that ends the current item, and the next item reads its fields from there
// as broadcast LDS loads (all lanes read the same address).
struct ItemRegs {
  uint32_t w[kItemWords / 64];
};

__device__ __forceinline__ ItemRegs load_item(const uint32_t* __restrict__ opw, uint32_t rec, int lane) {
  const uint32_t* p = opw + (size_t)rec * kRecWords;
  ItemRegs it;
#pragma unroll
  for (int j = 0; j < kItemWords / 64; ++j) it.w[j] = p[64 * j + lane];
  return it;
}

__device__ __forceinline__ void stage_item(uint32_t* buf, const ItemRegs& it, int lane) {
#pragma unroll
  for (int j = 0; j < kItemWords / 64; ++j) buf[64 * j + lane] = it.w[j];
}

__device__ __forceinline__ double ldbl(const uint32_t* buf, int d) {
  const uint64_t lo = buf[d], hi = buf[d + 1];
  return __longlong_as_double((long long)(lo | (hi << 32)));
}

__device__ __forceinline__ uint32_t ins0(uint32_t p, uint32_t q) { return ((p >> q) << (q + 1)) | (p & ((1u << q) - 1)); }

// LDS: the real parts of all positions, then the imaginary parts, `plane`
// bytes further on.  (As pairs of components, 16 bytes per amplitude, the
// registers of a read or written pair had to be neighbours, and the compiler
// copied all 32 components of a group between the registers that the gates
// use and those that the LDS accesses use.)  The place of position p within
// a plane: a pass whose slots include the lowest positions gives consecutive
// lanes groups 16 (or more) amplitudes apart, all in the same banks; XOR-ing
// the next bits into the place within a 128-byte row (4 bits for doubles, 5
// for floats) spreads them, and keeps contiguous runs contiguous within each
// row.  A bijection on [0, 2^n), and linear over XOR.
template <typename R>
__device__ __forceinline__ uint32_t place(uint32_t i) {
  constexpr uint32_t b = sizeof(R) == 8 ? 4 : 5, m = (1u << b) - 1;
  return (i ^ ((i >> b) & m)) * (uint32_t)sizeof(R);
}

// A state in LDS.  PLANE: the plane distance in bytes where it is a constant
// that fits an LDS instruction's offset field, else 0 (`plane` holds it).
template <typename R, int PLANE>
struct LdsState {
  using C = typename EVb<R>::T;
  unsigned char* p;
  uint32_t plane;
  static __device__ __forceinline__ uint32_t at(uint32_t i) { return place<R>(i); }
  __device__ __forceinline__ R* re(uint32_t at) const { return reinterpret_cast<R*>(p + at); }
  __device__ __forceinline__ R* im(uint32_t at) const {
    return reinterpret_cast<R*>(p + at + (PLANE ? (uint32_t)PLANE : plane));
  }
  __device__ __forceinline__ C get(uint32_t at) const {
    C x;
    x.x = *re(at);
    x.y = *im(at);
    return x;
  }
  __device__ __forceinline__ void put(uint32_t at, C x) const {
    *re(at) = x.x;
    *im(at) = x.y;
  }
};

// A state in global memory, for a measurement.
template <typename R>
struct GlobalState {
  using C = typename EVb<R>::T;
  C* p;
  static __device__ __forceinline__ uint32_t at(uint32_t i) { return i; }
  __device__ __forceinline__ C get(uint32_t i) const { return p[i]; }
  __device__ __forceinline__ void put(uint32_t i, C x) const { p[i] = x; }
};

// The value of a functional (in, out) at position p of the chunk c.
__device__ __forceinline__ uint32_t lane_bit(uint32_t in, uint32_t out, uint32_t p, uint32_t c) {
  return (uint32_t)(__popc(in & p) + __popc(out & c)) & 1u;
}

// The gate loop of a pass, in assembly: plain gates on the thread's 16
// amplitudes a0..a15 + i b0..b15, updated in place, from the record at LDS
// address `at` on; it leaves the address of the first record with another op
// (the one that ends the pass among them).  A gate is 64 arithmetic
// instructions; what a compiled loop added to them cost as much again: a tree
// of compares and taken branches for each gate, results moved back into the
// amplitudes' registers, a wait for each record.  Here each record holds the
// place of its gate's code, and is read while the gate before it runs; that
// gate works out the jump before it ends.
//
// Coefficients c0..c3 (the next record's: n0..n3), h0..h2 the next record's
// first dwords, s80:81 the address of the gates' code, s82:83 the next
// gate's, s89 = the chunk's outside bits.
#define QK_FETCH(LD, O0, O1, O2, O3)                                                                     \
  "ds_read_b32 %[h0], %[ad]\n\tds_read_b32 %[h1], %[ad] offset:4\n\tds_read_b32 %[h2], %[ad] offset:8\n\t" \
  LD " %[n0], %[ad] offset:" O0 "\n\t" LD " %[n1], %[ad] offset:" O1 "\n\t"                                \
  LD " %[n2], %[ad] offset:" O2 "\n\t" LD " %[n3], %[ad] offset:" O3 "\n\t"
#define QK_BEGIN(MOV, FETCH)                                                                             \
  MOV " %[c0], %[n0]\n\t" MOV " %[c1], %[n1]\n\t" MOV " %[c2], %[n2]\n\t" MOV " %[c3], %[n3]\n\t"          \
  "v_add_u32 %[ad], 48, %[ad]\n\t" FETCH
#define QK_NEXT                                                                                          \
  "s_waitcnt lgkmcnt(0)\n\tv_readfirstlane_b32 s84, %[h0]\n\ts_add_u32 s82, s80, s84\n\ts_addc_u32 s83, s81, 0\n\t"
#define QK_JUMP "s_setpc_b64 s[82:83]\n\t"
// [[a, b], [c, d]] and [[a, i b], [i c, d]] on the pair (P, Q): every product
// with P goes to a temporary, and the sums take the operands' registers.
#define QK_REAL1(W, P, Q)                                                                                \
  "v_mul_" W " %[t0], %[c0], %[a" #P "]\n\tv_mul_" W " %[t1], %[c0], %[b" #P "]\n\t"                       \
  "v_mul_" W " %[t2], %[c2], %[a" #P "]\n\tv_mul_" W " %[t3], %[c2], %[b" #P "]\n\t"                       \
  "v_fma_" W " %[a" #P "], %[c1], %[a" #Q "], %[t0]\n\tv_fma_" W " %[b" #P "], %[c1], %[b" #Q "], %[t1]\n\t" \
  "v_fma_" W " %[a" #Q "], %[c3], %[a" #Q "], %[t2]\n\tv_fma_" W " %[b" #Q "], %[c3], %[b" #Q "], %[t3]\n\t"
#define QK_IMAG1(W, P, Q)                                                                                \
  "v_mul_" W " %[t0], %[c0], %[a" #P "]\n\tv_mul_" W " %[t1], %[c0], %[b" #P "]\n\t"                       \
  "v_mul_" W " %[t2], %[c2], %[a" #P "]\n\tv_mul_" W " %[t3], %[c2], %[b" #P "]\n\t"                       \
  "v_fma_" W " %[a" #P "], -%[c1], %[b" #Q "], %[t0]\n\tv_fma_" W " %[b" #P "], %[c1], %[a" #Q "], %[t1]\n\t" \
  "v_fma_" W " %[b" #Q "], %[c3], %[b" #Q "], %[t2]\n\tv_fma_" W " %[a" #Q "], %[c3], %[a" #Q "], -%[t3]\n\t"
// The pairs of each slot.
#define QK_SLOT0(ONE, W) ONE(W, 0, 1) ONE(W, 2, 3) ONE(W, 4, 5) ONE(W, 6, 7) ONE(W, 8, 9) ONE(W, 10, 11) QK_NEXT ONE(W, 12, 13) ONE(W, 14, 15)
#define QK_SLOT1(ONE, W) ONE(W, 0, 2) ONE(W, 1, 3) ONE(W, 4, 6) ONE(W, 5, 7) ONE(W, 8, 10) ONE(W, 9, 11) QK_NEXT ONE(W, 12, 14) ONE(W, 13, 15)
#define QK_SLOT2(ONE, W) ONE(W, 0, 4) ONE(W, 1, 5) ONE(W, 2, 6) ONE(W, 3, 7) ONE(W, 8, 12) ONE(W, 9, 13) QK_NEXT ONE(W, 10, 14) ONE(W, 11, 15)
#define QK_SLOT3(ONE, W) ONE(W, 0, 8) ONE(W, 1, 9) ONE(W, 2, 10) ONE(W, 3, 11) ONE(W, 4, 12) ONE(W, 5, 13) QK_NEXT ONE(W, 6, 14) ONE(W, 7, 15)
// Two amplitudes times c0 - i c1 (A "", B "-") or c0 + i c1 (A "-", B "").
#define QK_FACTOR2(W, A, B, P, Q)                                                                        \
  "v_mul_" W " %[t0], %[c0], %[a" #P "]\n\tv_mul_" W " %[t1], %[c1], %[a" #P "]\n\t"                       \
  "v_mul_" W " %[t2], %[c0], %[a" #Q "]\n\tv_mul_" W " %[t3], %[c1], %[a" #Q "]\n\t"                       \
  "v_fma_" W " %[a" #P "], " A "%[c1], %[b" #P "], %[t0]\n\tv_fma_" W " %[b" #P "], %[c0], %[b" #P "], " B "%[t1]\n\t" \
  "v_fma_" W " %[a" #Q "], " A "%[c1], %[b" #Q "], %[t2]\n\tv_fma_" W " %[b" #Q "], %[c0], %[b" #Q "], " B "%[t3]\n\t"
#define QK_SIGN16(W, A, B, C, D, E, F, G, H, I, J, K, L, M, N, O, P)                                     \
  QK_FACTOR2(W, "", "-", A, B) QK_FACTOR2(W, "", "-", C, D) QK_FACTOR2(W, "", "-", E, F)                 \
  QK_FACTOR2(W, "", "-", G, H) QK_FACTOR2(W, "-", "", I, J) QK_FACTOR2(W, "-", "", K, L)                 \
  QK_NEXT QK_FACTOR2(W, "-", "", M, N) QK_FACTOR2(W, "-", "", O, P)
#define QK_SIGNM(W, ...) QK_SIGN16(W, __VA_ARGS__)
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
// The parity of the lane functional in bit 0 of v (other bits: garbage).
#define QK_LANE_WORDS "v_readfirstlane_b32 s85, %[h1]\n\tv_readfirstlane_b32 s86, %[h2]\n\t"
#define QK_LANE_BIT                                                                                      \
  "s_lshr_b32 s85, s85, 16\n\ts_and_b32 s87, s86, s89\n\ts_bcnt1_i32_b32 s87, s87\n\t"                     \
  "v_and_b32 %[v], s85, %[bs]\n\tv_bcnt_u32_b32 %[v], %[v], s87\n\t"
// c1 negated where it is 1.
#define QK_LANE_SIGN_f64                                                                                 \
  QK_LANE_BIT "v_bfe_i32 %[v], %[v], 0, 1\n\tv_lshl_or_b32 %[v], %[v], 1, 1\n\t"                           \
  "v_cvt_f64_i32 %[t0], %[v]\n\tv_mul_f64 %[c1], %[t0], %[c1]\n\t"
#define QK_LANE_SIGN_f32 QK_LANE_BIT "v_lshlrev_b32 %[v], 31, %[v]\n\tv_xor_b32 %[c1], %[v], %[c1]\n\t"
// One gate's code, kGateBytes long.
#define QK_GATE(N, ...) "LQKg" #N "%=:\n\t" __VA_ARGS__ QK_JUMP ".org LQKg" #N "%=+768\n"
#define QK_REAL(N, S, W, BEGIN) QK_GATE(N, BEGIN QK_SLOT##S(QK_REAL1, W))
#define QK_IMAG(N, S, W, BEGIN) QK_GATE(N, BEGIN QK_SLOT##S(QK_IMAG1, W))
#define QK_SIGN(N, M, W, SIGN, BEGIN) QK_GATE(N, QK_LANE_WORDS BEGIN SIGN QK_SIGNM(W, QK_MEMBERS##M))
#define QK_GATE_LOOP(W, SIGN, BEGIN, FETCH)                                                              \
  asm volatile(                                                                                          \
      "s_mov_b32 s89, %[cc]\n\tv_mov_b32 %[ad], %[at]\n\t" FETCH                                          \
      "s_getpc_b64 s[80:81]\n"                                                                           \
      "LQKpc%=:\n\t"                                                                                     \
      "s_add_u32 s80, s80, LQKg0%=-LQKpc%=\n\ts_addc_u32 s81, s81, 0\n\t" QK_NEXT QK_JUMP                  \
      QK_REAL(0, 0, W, BEGIN) QK_REAL(1, 1, W, BEGIN) QK_REAL(2, 2, W, BEGIN) QK_REAL(3, 3, W, BEGIN)    \
      QK_IMAG(4, 0, W, BEGIN) QK_IMAG(5, 1, W, BEGIN) QK_IMAG(6, 2, W, BEGIN) QK_IMAG(7, 3, W, BEGIN)    \
      QK_GATE(8, QK_LANE_WORDS BEGIN SIGN                                                                \
              "v_mul_" W " %[t0], %[c0], %[fr]\n\tv_mul_" W " %[t1], %[c1], %[fr]\n\t"                     \
              "v_fma_" W " %[fr], %[c1], %[fi], %[t0]\n\tv_fma_" W " %[fi], %[c0], %[fi], -%[t1]\n\t" QK_NEXT) \
      QK_SIGN(9, 1, W, SIGN, BEGIN) QK_SIGN(10, 2, W, SIGN, BEGIN) QK_SIGN(11, 3, W, SIGN, BEGIN)        \
      QK_SIGN(12, 4, W, SIGN, BEGIN) QK_SIGN(13, 5, W, SIGN, BEGIN) QK_SIGN(14, 6, W, SIGN, BEGIN)       \
      QK_SIGN(15, 7, W, SIGN, BEGIN) QK_SIGN(16, 8, W, SIGN, BEGIN) QK_SIGN(17, 9, W, SIGN, BEGIN)       \
      QK_SIGN(18, 10, W, SIGN, BEGIN) QK_SIGN(19, 11, W, SIGN, BEGIN) QK_SIGN(20, 12, W, SIGN, BEGIN)    \
      QK_SIGN(21, 13, W, SIGN, BEGIN) QK_SIGN(22, 14, W, SIGN, BEGIN) QK_SIGN(23, 15, W, SIGN, BEGIN)    \
      "v_readfirstlane_b32 %[at], %[ad]"   /* RG_OTHER */                                                \
      : [a0] "+v"(xr[0]), [a1] "+v"(xr[1]), [a2] "+v"(xr[2]), [a3] "+v"(xr[3]), [a4] "+v"(xr[4]),        \
        [a5] "+v"(xr[5]), [a6] "+v"(xr[6]), [a7] "+v"(xr[7]), [a8] "+v"(xr[8]), [a9] "+v"(xr[9]),        \
        [a10] "+v"(xr[10]), [a11] "+v"(xr[11]), [a12] "+v"(xr[12]), [a13] "+v"(xr[13]),                  \
        [a14] "+v"(xr[14]), [a15] "+v"(xr[15]), [b0] "+v"(xi[0]), [b1] "+v"(xi[1]), [b2] "+v"(xi[2]),    \
        [b3] "+v"(xi[3]), [b4] "+v"(xi[4]), [b5] "+v"(xi[5]), [b6] "+v"(xi[6]), [b7] "+v"(xi[7]),        \
        [b8] "+v"(xi[8]), [b9] "+v"(xi[9]), [b10] "+v"(xi[10]), [b11] "+v"(xi[11]),                      \
        [b12] "+v"(xi[12]), [b13] "+v"(xi[13]), [b14] "+v"(xi[14]), [b15] "+v"(xi[15]),                  \
        [fr] "+v"(fr), [fi] "+v"(fi), [at] "+s"(at), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2),     \
        [t3] "=&v"(t3), [c0] "=&v"(c0), [c1] "=&v"(c1), [c2] "=&v"(c2), [c3] "=&v"(c3), [n0] "=&v"(n0),  \
        [n1] "=&v"(n1), [n2] "=&v"(n2), [n3] "=&v"(n3), [h0] "=&v"(h0), [h1] "=&v"(h1), [h2] "=&v"(h2),  \
        [ad] "=&v"(ad), [v] "=&v"(vt)                                                                    \
      : [cc] "s"(c), [bs] "v"(base)                                                                      \
      : "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s89", "scc", "memory")
static_assert(kGateBytes == 768 && kRecWords * 4 == 48 && RG_SIGN == 8 && RG_OTHER == 24, "the gate loop's layout");

template <typename R>
__device__ __forceinline__ void gate_loop(R (&xr)[kMembers], R (&xi)[kMembers], R& fr, R& fi, uint32_t& at, uint32_t c,
                                          uint32_t base) {
  R t0, t1, t2, t3, c0, c1, c2, c3, n0, n1, n2, n3;
  uint32_t h0, h1, h2, ad, vt;
  if constexpr (sizeof(R) == 8)
    QK_GATE_LOOP("f64", QK_LANE_SIGN_f64, QK_BEGIN("v_mov_b64", QK_FETCH("ds_read_b64", "16", "24", "32", "40")),
                 QK_FETCH("ds_read_b64", "16", "24", "32", "40"));
  else
    QK_GATE_LOOP("f32", QK_LANE_SIGN_f32, QK_BEGIN("v_mov_b32", QK_FETCH("ds_read_b32", "16", "20", "24", "28")),
                 QK_FETCH("ds_read_b32", "16", "20", "24", "28"));
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

// Expanded in the kernel body on the kernel's own register arrays with
// constant indices: passing an array to a function (by reference) made the
// compiler keep part of it in scratch memory.
// Pairs in the record's member mask (uniform) where the lane's mask has them;
// elsewhere the identity's entries (a branch per pair would copy its results).
#define QK_PAIRS_M(S, FN)                                                               \
  do {                                                                                  \
    _Pragma("unroll") for (int r = 0; r < kMembers; ++r)                                \
      if (!(r & (1 << (S)))) {                                                          \
        const bool on = ((mm & memb) >> r) & 1u;                                        \
        const R um[4] = {on ? u[0] : (R)1, on ? u[1] : (R)0, on ? u[2] : (R)0, on ? u[3] : (R)1}; \
        FN(xr[r], xi[r], xr[r | (1 << (S))], xi[r | (1 << (S))], um);                   \
      }                                                                                 \
  } while (0)
#define QK_FLIP_M(S)                                                                    \
  do {                                                                                  \
    _Pragma("unroll") for (int r = 0; r < kMembers; ++r)                                \
      if (!(r & (1 << (S)))) {                                                          \
        const bool on = ((mm & memb) >> r) & 1u;                                        \
        const R pr = xr[r], pi = xi[r], qr = xr[r | (1 << (S))], qi = xi[r | (1 << (S))]; \
        xr[r] = on ? qr : pr;                                                           \
        xi[r] = on ? qi : pi;                                                           \
        xr[r | (1 << (S))] = on ? pr : qr;                                              \
        xi[r | (1 << (S))] = on ? pi : qi;                                              \
      }                                                                                 \
  } while (0)
// Waves per SIMD to keep resident.  A thread holds the 16 amplitudes of its
// group, and the stage kernel 16 more of its next chunk (128 registers
// together for complex128, 64 for complex64).
template <typename R> constexpr int lds_waves_per_simd() { return sizeof(R) == 8 ? 2 : 4; }

// Staged states: qubits of the LDS chunk (64 KiB) a stage works on.
template <typename R> constexpr int stage_qubits() { return sizeof(R) == 8 ? 12 : 13; }
// Threads of the stage kernel: one group of 16 amplitudes each.
template <typename R> constexpr int stage_threads() { return 1 << (stage_qubits<R>() - kPassSlots); }
// Records of a stage kept in LDS beside its chunk by the stage kernel (10 KiB:
// 213 records; two workgroups of 64 + 10 KiB and their static arrays fit a
// compute unit).
constexpr uint32_t kStageLdsWords = 2560;

// Measurement over a state of dim amplitudes, in LDS (positions, read
// through the swizzle) or in global memory, of the functional (in, out): FP64
// sums of |x|^2 by outcome in a fixed order (strided over nt threads, which
// depends on the state's size alone, then wave, then the waves in order),
// outcome 0 iff u < P0, the outcome's half scaled by 1/sqrt(p), the other
// half zeroed; cbit (>= 0) receives the outcome.  A zero-probability outcome
// leaves the state and the cbit as they are.
template <typename R, typename S>
__device__ __forceinline__ void meas_run(S st, uint32_t bd, uint32_t dim, uint32_t in, uint32_t flip, double u,
                                         int cbit, uint8_t* cb, double (*red)[kMaxWaves], double* meas) {
  using C = typename EVb<R>::T;
  const uint32_t tid = threadIdx.x;
  const uint32_t nt = min((uint32_t)kBatchThreads, max(1u, dim >> kPassSlots));   // <= bd
  const int lane = tid & 63, w = tid >> 6;
  auto one = [&](uint32_t i) { return ((uint32_t)__popc(i & in) & 1u) != flip; };
  double s0 = 0, s1 = 0;
  for (uint32_t i0 = tid < nt ? tid : dim; i0 < dim; i0 += kBU * nt) {
    C x[kBU];
#pragma unroll
    for (int k = 0; k < kBU; ++k)
      if (i0 + k * nt < dim) x[k] = st.get(st.at(i0 + k * nt));
#pragma unroll
    for (int k = 0; k < kBU; ++k) {
      const uint32_t i = i0 + k * nt;
      if (i < dim) {
        const double pr = (double)x[k].x * (double)x[k].x + (double)x[k].y * (double)x[k].y;
        if (one(i)) s1 += pr; else s0 += pr;
      }
    }
  }
  s0 = bwave_sum(s0);
  s1 = bwave_sum(s1);
  if (lane == 0) {
    red[0][w] = s0;
    red[1][w] = s1;
  }
  __syncthreads();
  if (tid == 0) {
    double q0 = 0, q1 = 0;
    for (int k = 0; k < (int)(bd / 64); ++k) {
      q0 += red[0][k];
      q1 += red[1][k];
    }
    const double P0 = q0 / (q0 + q1);
    const int oc = (u < P0) ? 0 : 1;
    const double po = oc ? q1 : q0;
    meas[0] = po > 0 ? 1.0 / sqrt(po) : 0.0;
    meas[1] = (double)oc;
    if (cbit >= 0 && po > 0) cb[cbit] = (uint8_t)oc;
  }
  __syncthreads();
  const double sc = meas[0];
  const bool oc = meas[1] != 0.0;
  if (sc != 0.0) {
    const R scale = (R)sc;
    for (uint32_t i0 = tid; i0 < dim; i0 += kBU * bd) {
      C x[kBU];
#pragma unroll
      for (int k = 0; k < kBU; ++k)
        if (i0 + k * bd < dim) x[k] = st.get(st.at(i0 + k * bd));
#pragma unroll
      for (int k = 0; k < kBU; ++k) {
        const uint32_t i = i0 + k * bd;
        if (i < dim) {
          C v = x[k];
          if (one(i) == oc) {
            v.x *= scale;
            v.y *= scale;
          } else {
            v.x = 0;
            v.y = 0;
          }
          st.put(st.at(i), v);
        }
      }
    }
  }
}

// One pass over the LDS state: each thread loads a group's 16 members, runs
// the pass's gate records on them in registers and stores them back.  `cur`
// is the pass header in LDS, head its first dword, c the chunk's outside bits
// with the constant.
template <typename R, int PLANE>
__device__ __forceinline__ void run_pass(LdsState<R, PLANE> st, uint32_t bd, uint32_t dim, const uint32_t* cur, uint32_t head,
                                         const uint8_t* cb, uint32_t c) {
  using C = typename EVb<R>::T;
  const uint32_t tid = threadIdx.x;
  const int nrec = (int)(head >> 16);
  const uint32_t hw = cur[min(tid & 63u, (uint32_t)kRecWords - 1)];   // the header, a dword per lane
  auto word = [&](int i) { return (uint32_t)__builtin_amdgcn_readlane((int)hw, i); };
  const uint32_t pv = word(1), p0 = pv & 0xff, p1 = (pv >> 8) & 0xff, p2 = (pv >> 16) & 0xff, p3 = pv >> 24;
  const uint32_t v0 = word(8), v1 = word(9), v2 = word(10), v3 = word(11);
  const uint32_t ngroups = dim >= (uint32_t)kMembers ? dim >> kPassSlots : 1u;
  // Whole waves run the gates (lanes past the last group on group 0's
  // amplitudes, which they do not store), so that their control flow is
  // uniform.
  for (uint32_t gw = rfl(tid & ~63u); gw < ngroups; gw += bd) {
    const bool live = gw + (tid & 63u) < ngroups;
    const uint32_t g = live ? gw + (tid & 63u) : 0u;
    const uint32_t base = ins0(ins0(ins0(ins0(g, p0), p1), p2), p3);
    uint32_t sb = place<R>(base);
    if (head & 0xf00u) {   // member 0 is where every slot has value 0
      const uint32_t r01 = word(2), r23 = word(3);
      if (head & 0x100u) sb ^= (0u - lane_bit(r01 & 0xffffu, word(4), base, c)) & v0;
      if (head & 0x200u) sb ^= (0u - lane_bit(r01 >> 16, word(5), base, c)) & v1;
      if (head & 0x400u) sb ^= (0u - lane_bit(r23 & 0xffffu, word(6), base, c)) & v2;
      if (head & 0x800u) sb ^= (0u - lane_bit(r23 >> 16, word(7), base, c)) & v3;
    }
    auto member = [&](int r) {
      return sb ^ ((r & 1 ? v0 : 0u) ^ (r & 2 ? v1 : 0u) ^ (r & 4 ? v2 : 0u) ^ (r & 8 ? v3 : 0u));
    };
    R xr[kMembers], xi[kMembers];
#pragma unroll
    for (int r = 0; r < kMembers; ++r) {
      xr[r] = *st.re(member(r));
      xi[r] = *st.im(member(r));
    }
    uint32_t mm = 0xffffu;   // the lane's member mask (narrowed by RG_PRED for the next gate)
    R fr = 1, fi = 0;        // the lane factor: gates that act alike on all members
    uint32_t at = rfl((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint32_t*)(cur + kRecWords));
    const uint32_t end = at + (uint32_t)(nrec - 1) * (kRecWords * 4);   // the record that ends the pass
    for (;;) {
      at = rfl(at);
      gate_loop<R>(xr, xi, fr, fi, at, rfl(c), base);
      if (at == end) break;
      const auto* gc = (const __attribute__((address_space(3))) uint32_t*)(uintptr_t)at;
      at += kRecWords * 4;
      const uint32_t w1 = rfl(gc[1]), om = rfl(gc[2]), oh = rfl(gc[3]);
      const uint32_t op = oh >> 24, memb = w1 & 0xffffu, ncond = (oh >> 18) & 3u;
      if (ncond) {
        if (rfl(cb[oh & 0xff]) != ((oh >> 16) & 1u) || (ncond > 1 && rfl(cb[(oh >> 8) & 0xff]) != ((oh >> 17) & 1u))) {
          mm = 0xffffu;
          continue;
        }
      }
      R u[4];
      const auto* gu = (const __attribute__((address_space(3))) R*)(gc + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e] = gu[e];
      if (op >= RG_PHASE) {
        const uint32_t on = lane_bit(w1 >> 16, om, base, c);
        if (op == RG_PRED) {
          const uint32_t mw = rfl(gc[4]);
          mm &= on ? mw : mw >> 16;
          continue;
        }
        const bool act = mm != 0 && (!(oh & kOwnPredicate) || on);
        const R zr = act ? u[0] : (R)1, zi = act ? u[1] : (R)0;
        if (op == RG_LANE_Z) {
          gate_factor<R>(fr, fi, zr, zi);
        } else if (op == RG_PHASE) {
#pragma unroll
          for (int r = 0; r < kMembers; ++r)
            if ((memb >> r) & 1u) gate_factor<R>(xr[r], xi[r], zr, zi);
        } else {
#pragma unroll
          for (int r = 0; r < kMembers; ++r)
            if ((memb >> r) & 1u) {
              const bool here = (mm >> r) & 1u;
              gate_factor<R>(xr[r], xi[r], here ? u[0] : (R)1, here ? u[1] : (R)0);
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
    if (head & 0x1000u) {
#pragma unroll
      for (int r = 0; r < kMembers; ++r) gate_factor<R>(xr[r], xi[r], fr, fi);
    }
    asm volatile("" : "+v"(sb));   // the places are worked out again rather than held in 16 registers
    if (live) {
#pragma unroll
      for (int r = 0; r < kMembers; ++r) {
        *st.re(member(r)) = xr[r];
        *st.im(member(r)) = xi[r];
      }
    }
  }
}

// Runs item records [rec, end) over a state of dim amplitudes in LDS with bd
// threads (a constant or a value read once: read from the dispatch packet in
// the pass loop, the load's wait was one for every outstanding access, the
// prefetched amplitudes' among them); every item ends with a barrier.  With lrec the records of the whole range lie in
// LDS there; otherwise the first item's records sit in items[0], staged
// before a barrier, and each next item is loaded while the current one runs
// (AHEAD), or after it (the stage kernel, for the rare stage whose records
// exceed its LDS: the registers go to the prefetched amplitudes).
// after_first is called after the first item.
template <typename R, int PLANE, bool AHEAD, typename F>
__device__ __forceinline__ void run_items(LdsState<R, PLANE> st, uint32_t bd, uint32_t dim, uint32_t rec, uint32_t end,
                                          const uint32_t* __restrict__ opw, uint32_t c, uint8_t* cb,
                                          uint32_t (*items)[kItemWords], double (*red)[kMaxWaves], double* meas,
                                          const uint32_t* lrec, F after_first) {
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const uint32_t* cur = lrec ? lrec : items[0];
  const uint32_t begin = rec;
  int buf = 0;
  while (rec < end) {
    const uint32_t head = rfl(cur[0]);
    const bool pass = (head & 0xffu) == RK_PASS;
    const uint32_t next = rec + 1 + (pass ? head >> 16 : 0u);
    ItemRegs nxt;
    if (AHEAD && !lrec && w == 0) nxt = load_item(opw, next, lane);   // the record array ends with padding
    if (pass) {
      run_pass<R, PLANE>(st, bd, dim, cur, head, cb, c);
    } else {
      const uint32_t flip = (uint32_t)__popc(rfl(cur[2]) & c) & 1u;
      meas_run<R>(st, bd, dim, rfl(cur[1]), flip, ldbl(cur, 4), (int)cur[3], cb, red, meas);
    }
    // the next item's records into the other buffer (its last readers
    // finished before the barrier that ended the previous item)
    if (!AHEAD && !lrec && w == 0) nxt = load_item(opw, next, lane);
    if (!lrec && w == 0) stage_item(items[buf ^ 1], nxt, lane);
    __syncthreads();
    buf ^= 1;
    cur = lrec ? cur + (size_t)(next - rec) * kRecWords : items[buf];
    if (rec == begin) after_first();
    rec = next;
  }
}

// Bits of v deposited, lowest first, at the set bits of mask.
__device__ __forceinline__ uint32_t deposit(uint32_t v, uint32_t mask) {
  uint32_t out = 0;
  for (uint32_t m = mask; m; m &= m - 1, v >>= 1)
    if (v & 1u) out |= m & (~m + 1u);
  return out;
}

// The chunk layout of a stage whose header is record rec (words h), for a
// workgroup of 2^TB threads: its item range, the qubits outside it (cmask:
// where the chunk number goes), and how local index tid + (k << TB) maps to
// the amplitude index (the thread's bits on the stage's lowest TB qubits, k
// on the others, the same for every thread) and to its LDS place.
template <int LQ, int TB>
struct ChunkMap {
  static constexpr int KB = LQ - TB, PT = 1 << KB;
  const uint32_t* raw;
  uint32_t it_begin, it_end, cmask, base, tpart;
  uint32_t kq[KB], kv[KB];   // bit j of k: its amplitude-index bit, its LDS byte offset
  bool plain;

  __device__ __forceinline__ ChunkMap(const uint32_t* h, uint32_t rec, uint32_t dim, uint32_t tid) {
    it_begin = rec + kHeadRecords;
    it_end = it_begin + rfl(h[1]);
    plain = rfl(h[2]) != 0;
    raw = h + kRecWords;
    uint32_t smask = 0;
    base = 0;
    tpart = 0;
#pragma unroll
    for (int j = 0; j < LQ; ++j) {
      const uint32_t b = 1u << ((rfl(h[4 + j / 4]) >> (8 * (j & 3))) & 0xffu), v = rfl(raw[j]);
      smask |= b;
      if (j < TB) {
        if ((tid >> j) & 1u) {
          base |= b;
          tpart ^= v;
        }
      } else {
        kq[j - TB] = b;
        kv[j - TB] = v;
      }
    }
    cmask = (dim - 1) & ~smask;
  }
  __device__ __forceinline__ uint32_t index(int k) const {
    uint32_t o = 0;
#pragma unroll
    for (int j = 0; j < KB; ++j)
      if ((k >> j) & 1) o |= kq[j];
    return o;
  }
  __device__ __forceinline__ uint32_t place(int k) const {
    uint32_t o = 0;
#pragma unroll
    for (int j = 0; j < KB; ++j)
      if ((k >> j) & 1) o ^= kv[j];
    return o;
  }
  // Keeps the compiler from holding every index(k) and place(k) in registers
  // while the passes run.
  __device__ __forceinline__ void opaque() {
#pragma unroll
    for (int j = 0; j < KB; ++j) asm volatile("" : "+s"(kq[j]), "+s"(kv[j]));
  }
  // The place of the chunk's amplitude 0, where the frame has constants.
  __device__ __forceinline__ uint32_t origin(uint32_t c) const {
    uint32_t o = 0;
    if (!plain) {
      for (int j = 0; j < LQ; ++j)
        if (__popc(rfl(raw[16 + j]) & c) & 1) o ^= rfl(raw[j]);
    }
    return o;
  }
};

// A staged batch job's chunk: gathered from the state into LDS (or, with
// zero, made |0...0>'s slice) and scattered back.
template <typename R, int PLANE>
__device__ __forceinline__ void chunk_in(LdsState<R, PLANE> st, const typename EVb<R>::T* gst,
                                         const ChunkMap<stage_qubits<R>(), 8>& cm, uint32_t cpart, bool zero) {
  using C = typename EVb<R>::T;
  constexpr int PT = ChunkMap<stage_qubits<R>(), 8>::PT;
#pragma unroll
  for (int k0 = 0; k0 < PT; k0 += 16) {   // 16 loads in flight per thread
    C x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const uint32_t g = cm.base | cm.index(k0 + k) | cpart;
      if (zero) {
        x[k].x = g == 0 ? (R)1 : (R)0;
        x[k].y = 0;
      } else {
        x[k] = gst[g];
      }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) st.put(place<R>(threadIdx.x + (uint32_t)(k0 + k) * 256u), x[k]);
  }
}
template <typename R, int PLANE>
__device__ __forceinline__ void chunk_out(LdsState<R, PLANE> st, typename EVb<R>::T* gst,
                                          const ChunkMap<stage_qubits<R>(), 8>& cm, uint32_t cpart) {
  constexpr int PT = ChunkMap<stage_qubits<R>(), 8>::PT;
  const uint32_t org = cm.origin(cpart | kOneBit) ^ cm.tpart;
#pragma unroll
  for (int k = 0; k < PT; ++k)
    gst[cm.base | cm.index(k) | cpart] = st.get(org ^ cm.place(k));
}

// A small job in LDS: |0...0> before its items, written out after them
// (h: its header).
template <typename R, int PLANE>
__device__ __forceinline__ void job_in(LdsState<R, PLANE> st, uint32_t bd, uint32_t dim) {
  for (uint32_t i = threadIdx.x; i < dim; i += bd) {
    typename EVb<R>::T z;
    z.x = (i == 0) ? (R)1 : (R)0;
    z.y = 0;
    st.put(place<R>(i), z);
  }
}
template <typename R, int PLANE>
__device__ __forceinline__ void job_out(LdsState<R, PLANE> st, uint32_t bd, typename EVb<R>::T* gst, const uint32_t* h, int n) {
  const uint32_t tid = threadIdx.x, dim = 1u << n, tb = 31u - (uint32_t)__builtin_clz(bd);
  const uint32_t* raw = h + kRecWords;
  uint32_t at = 0;   // the LDS place of amplitude i
  for (int j = 0; j < n; ++j) {
    const uint32_t v = rfl(raw[j]);
    if (rfl(raw[16 + j]) >> 31) at ^= v;
    if ((uint32_t)j < tb && ((tid >> j) & 1u)) at ^= v;
  }
  for (uint32_t i = tid, k = bd; i < dim; i += bd, k += bd) {
    gst[i] = st.get(at);
    if (k < dim)   // the bits above the thread's own that change: the same for the whole workgroup
      for (uint32_t ch = k ^ (k - bd); ch; ch &= ch - 1) at ^= rfl(raw[__builtin_ctz(ch)]);
  }
}

// Scheduling state of a batch launch.  Staged jobs: per job a 64-bit word
// (current stage << 32 | chunks claimed in it), the chunks completed in the
// current stage and a finished flag.  sched[0]: every staged job below it has
// finished (a scan hint); sched[1]: small jobs taken; sched[2]: set when a
// workgroup found no work for stall_ticks of the wall clock, 10 s (the host
// reports it).
struct BStage {
  uint32_t rec;       // record of the stage header or measurement
  uint32_t nchunks;   // chunks of the stage (1 for a measurement)
};
struct JobCtl {
  unsigned long long word;
  unsigned int done;
  unsigned int finished;
};
constexpr uint32_t kScanWindow = 128;                   // staged jobs a workgroup looks at for a free chunk

__device__ __forceinline__ unsigned ld_acq(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_acq64(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename R, int PLANE>
__global__ __launch_bounds__(kBatchThreads, sizeof(R) == 8 ? 3 : 4) void k_batch(
    const BJob* __restrict__ jobs, int njobs, int nstaged, const BStage* __restrict__ stages, JobCtl* ctl,
    unsigned* sched, const uint32_t* __restrict__ opw, typename EVb<R>::T* __restrict__ states,
    uint8_t* __restrict__ cbits, unsigned long long stall_ticks, uint32_t run_max, uint32_t plane) {
  using C = typename EVb<R>::T;
  constexpr int LQ = stage_qubits<R>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const LdsState<R, PLANE> st{smem_raw, plane};
  __shared__ uint8_t cb[kMaxJobCbits];
  __shared__ double red[2][kMaxWaves];
  __shared__ double meas[2];
  __shared__ int task[5];
  __shared__ __align__(16) uint32_t items[2][kItemWords];
  const uint32_t tid = threadIdx.x, bd = rfl(blockDim.x);
  const int lane = tid & 63, w = tid >> 6;
  unsigned long long idle_since = 0;
  for (;;) {
    // ---- find work (wave 0): a free chunk of a staged job, oldest first,
    // 64 jobs looked at per load round; else the next small job; else wait
    // for the stages in flight, or leave once every staged job has finished
    if (w == 0) {
      int job = -1, stage = 0, chunk = 0, count = 1, status = 0;   // status 0: work, 1: wait, 2: leave
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane(ld_acq(&sched[0]));
      for (uint32_t b0 = lo; job < 0 && b0 < (uint32_t)nstaged && b0 < lo + kScanWindow; b0 += 64) {
        const uint32_t j = b0 + lane;
        bool fin = true, avail = false;
        if (j < (uint32_t)nstaged) {
          fin = ld_acq(&ctl[j].finished) != 0;
          if (!fin) {
            const BJob& jb = jobs[j];
            const unsigned long long wd = ld_acq64(&ctl[j].word);
            const uint32_t s0 = (uint32_t)(wd >> 32);
            avail = s0 < jb.nst && (uint32_t)wd < stages[jb.st_begin + s0].nchunks;
          }
        }
        const unsigned long long fm = __ballot(fin);
        if (b0 == lo && (fm & 1ull)) {   // a finished prefix: move the hint past it
          const uint32_t np = ~fm == 0 ? 64u : (uint32_t)__builtin_ctzll(~fm);
          if (lane == 0) atomicMax(&sched[0], b0 + np);
        }
        unsigned long long av = __ballot(avail);
        while (av) {
          const int l = __builtin_ctzll(av);
          int got = 0, s2 = 0, c2 = 0, cnt = 0;
          if (lane == l) {
            // a run of chunks per claim: fewer claims and fences on large stages
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
          av &= av - 1;
        }
      }
      if (job >= 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // pairs with the release that opened the stage
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
    if (status == 1) {
      __builtin_amdgcn_s_sleep(8);
      continue;
    }
    const BJob jb = jobs[job];
    const uint32_t dim = 1u << jb.n;
    C* gst = states + jb.state_off;
    // a small job (its whole state one chunk), or a run of chunks of a stage
    // (or a measurement) of a staged job.  For the latter wave 0 acquired
    // after its claim (the invalidation covers this compute unit's caches),
    // and the barrier above orders every wave after it, so every chunk of
    // the earlier stages, written by any workgroup, is visible.
    const bool small = job >= nstaged;
    BStage bs{jb.rec, 1u};
    if (!small) bs = stages[jb.st_begin + stage];
    for (int c = tid; c < jb.ncbits; c += bd) cb[c] = small ? (uint8_t)0 : cbits[jb.cbit_off + c];
    __syncthreads();
    const uint32_t* h = opw + (size_t)bs.rec * kRecWords;
    if ((rfl(h[0]) & 0xff) == RK_MEAS) {
      const uint64_t ulo = rfl(h[4]), uhi = rfl(h[5]);
      const double u = __longlong_as_double((long long)(ulo | (uhi << 32)));
      const int cbit = (int)rfl(h[3]);
      meas_run<R>(GlobalState<R>{gst}, bd, dim, rfl(h[1]), 0u, u, cbit, cb, red, meas);
      if (tid == 0 && cbit >= 0) cbits[jb.cbit_off + cbit] = cb[cbit];
    } else {
      const uint32_t it0 = bs.rec + kHeadRecords, it1 = it0 + rfl(h[1]);
#pragma unroll 1
      for (uint32_t ch = chunk; ch < chunk + count; ++ch) {
        uint32_t cpart = 0;
        if (w == 0) stage_item(items[0], load_item(opw, it0, lane), lane);
        if (small) {
          job_in<R, PLANE>(st, bd, dim);
        } else {   // the first stage starts from |0...0>
          const ChunkMap<LQ, 8> cm(h, bs.rec, dim, tid);
          cpart = deposit(ch, cm.cmask);
          chunk_in<R, PLANE>(st, gst, cm, cpart, stage == 0);
        }
        __syncthreads();
        run_items<R, PLANE, true>(st, bd, small ? dim : 1u << LQ, it0, it1, opw, cpart | kOneBit, cb, items, red, meas, nullptr, [] {});
        if (small) job_out<R, PLANE>(st, bd, gst, h, jb.n);
        else chunk_out<R, PLANE>(st, gst, ChunkMap<LQ, 8>(h, bs.rec, dim, tid), cpart);
        __syncthreads();   // the next chunk's gather overwrites LDS
      }
    }
    if (small) {
      for (int c = tid; c < jb.ncbits; c += bd) cbits[jb.cbit_off + c] = cb[c];
      __syncthreads();
      continue;
    }
    // Release: every wave's stores have completed (waitcnt) before the
    // barrier, then one agent-scope release (the write-back of this XCD's
    // L2) before the chunks count as done; the workgroup that completes a
    // stage opens the next one.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");   // the whole workgroup's stores, through the barrier
      const unsigned d = atomicAdd(&ctl[job].done, count) + count;
      if (d == bs.nchunks) {
        atomicExch(&ctl[job].done, 0u);
        __threadfence();
        if (stage + 1 == jb.nst) atomicExch(&ctl[job].finished, 1u);
        __threadfence();
        atomicExch(&ctl[job].word, (unsigned long long)(stage + 1) << 32);
      }
    }
  }
}

// Clears a launch's scheduling state and every cbit (a staged job's cbits
// are read by each of its chunks).  A kernel rather than a memset so that a
// captured batch launch replays correctly.
__global__ void k_batch_reset(JobCtl* ctl, int nctl, unsigned* sched, uint8_t* cbits, uint32_t ncbits) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
  for (uint32_t k = i; k < (uint32_t)nctl; k += stride) {
    ctl[k].word = 0;
    ctl[k].done = 0;
    ctl[k].finished = 0;
  }
  for (uint32_t k = i; k < ncbits; k += stride) cbits[k] = 0;
  if (i < 4) sched[i] = 0;
}

// The chunk that the i-th position of the stage kernel's chunk loop takes:
// i with its low 3 bits rotated to the top.  Workgroups go to the 8 XCDs in
// turn (workgroup b to XCD b mod 8) and the grid is a multiple of 8, so XCD
// x takes the chunks [x R, (x + 1) R), R = nchunks / 8, and the workgroups
// of one XCD hold consecutive chunks at any time: chunks that differ only
// in the lowest qubits outside the stage share cache lines when the stage
// leaves out some of qubits 0..2, and then meet in that XCD's L2.
__device__ __forceinline__ uint32_t xcd_chunk(uint32_t i, uint32_t nchunks) {
  return nchunks >= 8 ? ((i & 7u) * (nchunks >> 3)) | (i >> 3) : i;
}

// s_waitcnt operand: vmcnt 0, the other counters not waited for.
constexpr int kWaitLoads = 0x0f70;

// One stage of a simulator's held-back gates (the LDS-tile mode): every
// chunk of the state, a chunk per workgroup at a time.  The stage's header
// is record hrec of opw; the gates' cbit conditions read cbits.  The next
// chunk's amplitudes are loaded into registers while the current chunk's
// passes run.
template <typename R>
__global__ __launch_bounds__(stage_threads<R>(), lds_waves_per_simd<R>()) void k_stage(
    typename EVb<R>::T* __restrict__ psi, int n, const uint32_t* __restrict__ opw, uint32_t hrec,
    const uint8_t* __restrict__ cbits, int ncbits) {
  using C = typename EVb<R>::T;
  constexpr int LQ = stage_qubits<R>(), TB = LQ - kPassSlots, PT = 1 << kPassSlots, BD = stage_threads<R>();
  constexpr int PLANE = (int)sizeof(R) << LQ;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const LdsState<R, PLANE> st{smem_raw, 0u};
  __shared__ uint8_t cb[kMaxJobCbits];
  __shared__ double red[2][kMaxWaves];
  __shared__ double meas[2];
  __shared__ __align__(16) uint32_t items[2][kItemWords];
  const uint32_t tid = threadIdx.x, dim = 1u << n;
  const int lane = tid & 63, w = tid >> 6;
  for (int i = tid; i < ncbits && i < kMaxJobCbits; i += BD) cb[i] = cbits[i];
  ChunkMap<LQ, TB> cm(opw + (size_t)hrec * kRecWords, hrec, dim, tid);
  const uint32_t nchunks = dim >> LQ;
  const uint32_t nwords = (cm.it_end - cm.it_begin) * kRecWords;
  // the stage's records once into LDS beside the chunk, for all of this
  // workgroup's chunks, where they fit
  const bool lds_recs = nwords + kRecWords <= kStageLdsWords;   // (gates read one header past the last)
  uint32_t* lrec = reinterpret_cast<uint32_t*>(smem_raw + (sizeof(C) << LQ));
  if (lds_recs)
    for (uint32_t i = tid; i < nwords; i += BD) lrec[i] = opw[(size_t)cm.it_begin * kRecWords + i];
  C pre[PT];
  uint32_t i = blockIdx.x;
  if (i < nchunks) {
    const C* p = psi + (cm.base | deposit(xcd_chunk(i, nchunks), cm.cmask));
#pragma unroll
    for (int k = 0; k < PT; ++k) pre[k] = p[cm.index(k)];
  }
  __builtin_amdgcn_s_waitcnt(kWaitLoads);
  for (; i < nchunks; i += gridDim.x) {
    const uint32_t cpart = deposit(xcd_chunk(i, nchunks), cm.cmask), c = cpart | kOneBit;
    uint32_t t = tid;   // (kept from being turned into places held across the passes)
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int k = 0; k < PT; ++k) st.put(place<R>(t + (uint32_t)k * BD), pre[k]);
    if (!lds_recs && w == 0) stage_item(items[0], load_item(opw, cm.it_begin, lane), lane);
    __syncthreads();
    // The next chunk's loads are issued after the first pass: issued at once,
    // they stood in line behind this workgroup's stores of the chunk before,
    // and the waves with them (about 7000 cycles).
    const uint32_t inext = i + gridDim.x;
    auto prefetch = [&]() {
      cm.opaque();
      if (inext < nchunks) {
        const C* p = psi + (cm.base | deposit(xcd_chunk(inext, nchunks), cm.cmask));
#pragma unroll
        for (int k = 0; k < PT; ++k) pre[k] = p[cm.index(k)];
      }
    };
    if (cm.it_begin == cm.it_end) prefetch();   // (a stage of bit flips alone has no passes)
    run_items<R, PLANE, false>(st, (uint32_t)BD, 1u << LQ, cm.it_begin, cm.it_end, opw, c, cb, items, red, meas,
                               lds_recs ? lrec : nullptr, prefetch);
    cm.opaque();
    // The next chunk's loads, which had all passes to arrive, are waited for
    // here: waited for after the stores below (both count down one counter,
    // in order), the wait was for the stores as well.
    __builtin_amdgcn_s_waitcnt(kWaitLoads);
    const uint32_t org = cm.origin(c) ^ cm.tpart;
    C* p = psi + (cm.base | cpart);
#pragma unroll
    for (int k = 0; k < PT; ++k) p[cm.index(k)] = st.get(org ^ cm.place(k));
    __syncthreads();   // the next chunk's amplitudes overwrite LDS
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
  void* d_states = nullptr;
  size_t states_bytes = 0;
  void* d_cbits = nullptr;
  size_t cbits_bytes = 0;
  void* d_ops = nullptr;
  size_t ops_bytes = 0;
  void* d_jobs = nullptr;
  size_t jobs_bytes = 0;
  void* d_stages = nullptr;   // stage table of the staged jobs
  size_t stages_bytes = 0;
  void* d_ctl = nullptr;      // per staged job scheduling state
  size_t ctl_bytes = 0;
  void* d_sched = nullptr;    // scan hint, small-job counter, stall flag
  size_t sched_bytes = 0;
  size_t nstaged = 0;
  size_t ncbits_total = 0;
  uint32_t run_max = 1;       // longest run of chunks one claim takes
  bool ran = false;
  bool uploaded = false;   // the device job table and ops match `jobs` (a rerun only relaunches)
  size_t njobs_dev = 0;
  size_t shm = 0;
  unsigned grid = 0, block = kBatchThreads;
  uint32_t plane = 0;         // LDS bytes between the real and the imaginary parts
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

// Jobs up to these sizes keep their whole state in LDS; larger ones, up to
// kMaxStagedQubits, keep it in global memory and run by stages of
// stage_qubits() qubits through LDS.
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
  std::vector<PlanOp> plan;
  plan.reserve((size_t)nops + 8);
  for (int i = 0; i < nops; ++i) {
    std::string err;
    const qk_status st = expand_op(ops[i], n, ncbits, plan, err);
    if (st) return bfail(b, st, "op " + std::to_string(i) + ": " + err);
  }
  hj.staged = n > max_lds_qubits(b->c64);
  if (hj.staged) build_stages(n, stage_chunk_qubits(b->c64), b->c64, plan, true, hj.rec, hj.heads);
  else build_job(n, b->c64, plan, hj.rec);
  b->jobs.push_back(std::move(hj));
  if (job) *job = (int32_t)b->jobs.size() - 1;
  b->ran = false;
  b->uploaded = false;
  return QK_OK;
}

}  // extern "C"

// The plane distances that k_batch is compiled for: small states, a staged
// chunk's (32 KiB), and any (0: read from the launch's argument).
constexpr int kSmallPlane = 4096, kChunkPlane = 32768;

template <typename R, int PLANE>
static void launch_batch_p(qk_batch b) {
  hipLaunchKernelGGL(k_batch_reset, dim3(64), dim3(256), 0, b->stream, (JobCtl*)b->d_ctl, (int)b->nstaged,
                     (unsigned*)b->d_sched, (uint8_t*)b->d_cbits, (uint32_t)b->ncbits_total);
  static unsigned long long stall = 0;   // 10 s of the device wall clock
  if (!stall) {
    int khz = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
      khz = 100000;
    stall = 10000ull * (unsigned long long)khz;
  }
  hipLaunchKernelGGL((k_batch<R, PLANE>), dim3(b->grid), dim3(b->block), b->shm, b->stream, (const BJob*)b->d_jobs,
                     (int)b->njobs_dev, (int)b->nstaged, (const BStage*)b->d_stages, (JobCtl*)b->d_ctl,
                     (unsigned*)b->d_sched, (const uint32_t*)b->d_ops, (typename EVb<R>::T*)b->d_states,
                     (uint8_t*)b->d_cbits, stall, b->run_max, b->plane);
}

template <typename R>
static void launch_batch_t(qk_batch b) {
  if (b->plane == (uint32_t)kSmallPlane) launch_batch_p<R, kSmallPlane>(b);
  else if (b->plane == (uint32_t)kChunkPlane) launch_batch_p<R, kChunkPlane>(b);
  else launch_batch_p<R, 0>(b);
}

static void launch_batch(qk_batch b) {
  if (b->c64) launch_batch_t<float>(b);
  else launch_batch_t<double>(b);
}

template <typename R>
static const void* batch_kernel(uint32_t plane) {
  return plane == (uint32_t)kSmallPlane ? (const void*)k_batch<R, kSmallPlane>
       : plane == (uint32_t)kChunkPlane ? (const void*)k_batch<R, kChunkPlane>
                                        : (const void*)k_batch<R, 0>;
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
  int nmax = 0;   // largest job kept in LDS, or the stage chunk when larger
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
  size_t nstaged = 0;
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
      for (uint32_t r : j.heads)
        stab.push_back({ooff + r, (j.rec[(size_t)r * kRecWords] & 0xff) == RK_MEAS ? 1u : 1u << (j.n - lq)});
      t.nst = (uint32_t)stab.size() - t.st_begin;
    }
    ooff += (uint32_t)(j.rec.size() / kRecWords);
    table.push_back(t);
  }
  all_ops.resize(all_ops.size() + (size_t)kPadRecords * kRecWords);   // padding: the kernel reads the next item before knowing its size
  qk_status st;
  if ((st = bensure(b, b->d_states, b->states_bytes, soff * amp, "batch states"))) return st;
  if ((st = bensure(b, b->d_cbits, b->cbits_bytes, std::max<size_t>(coff, 1), "batch cbits"))) return st;
  if ((st = bensure(b, b->d_ops, b->ops_bytes, all_ops.size() * sizeof(uint32_t), "batch ops"))) return st;
  if ((st = bensure(b, b->d_jobs, b->jobs_bytes, table.size() * sizeof(BJob), "batch job table"))) return st;
  if ((st = bensure(b, b->d_stages, b->stages_bytes, std::max<size_t>(stab.size(), 1) * sizeof(BStage), "batch stages")))
    return st;
  if ((st = bensure(b, b->d_ctl, b->ctl_bytes, std::max<size_t>(nstaged, 1) * sizeof(JobCtl), "batch scheduling")))
    return st;
  if ((st = bensure(b, b->d_sched, b->sched_bytes, 4 * sizeof(unsigned), "batch scheduling"))) return st;
  hipError_t e = hipMemcpyAsync(b->d_ops, all_ops.data(), all_ops.size() * sizeof(uint32_t), hipMemcpyHostToDevice, b->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(b->d_jobs, table.data(), table.size() * sizeof(BJob), hipMemcpyHostToDevice, b->stream);
  if (e == hipSuccess && !stab.empty())
    e = hipMemcpyAsync(b->d_stages, stab.data(), stab.size() * sizeof(BStage), hipMemcpyHostToDevice, b->stream);
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch upload: ") + hipGetErrorString(e));
  // the real parts of the largest state (one group of a pass at least), the
  // imaginary parts after them or at the next distance the kernel is compiled for
  const uint32_t part = (uint32_t)(amp / 2) << std::max(nmax, kPassSlots);
  b->plane = part <= (uint32_t)kSmallPlane ? kSmallPlane : part <= (uint32_t)kChunkPlane ? kChunkPlane : part;
  const size_t shm = (size_t)b->plane + part;
  // one group of 16 amplitudes per thread, from one wave to the 256 threads
  // that staged chunks take
  const int bits = std::max(6, std::min(8, nmax - kPassSlots));
  b->block = nstaged ? kBatchThreads : 1u << bits;
  int ncu = 256, dev = 0, per_cu = 1;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  const void* fn = b->c64 ? batch_kernel<float>(b->plane) : batch_kernel<double>(b->plane);
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
  // Runs of chunks per claim amortise the claim's fences when the staged
  // work is plentiful (about two claims per workgroup per round of stages),
  // and shrink to single chunks when a few jobs must spread over the grid.
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
  hipError_t e = hipSuccess;
  if (n > 0) e = hipMemcpyAsync(out, (char*)b->d_cbits + j.cbit_off, (size_t)n, hipMemcpyDeviceToHost, b->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
  if (e != hipSuccess) return bfail(b, QK_E_HIP, std::string("batch readback: ") + hipGetErrorString(e));
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
  recs.resize(recs.size() + (size_t)kPadRecords * kRecWords, 0u);   // the item prefetch reads past a stage's last record
  return QK_OK;
}

template <typename R>
static void launch_stage_t(void* psi, int n, const void* d_recs, uint32_t hrec, const uint8_t* d_cbits, int ncbits,
                           hipStream_t stream) {
  static int ncu = 0;
  if (!ncu) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      ncu = 256;
    (void)hipFuncSetAttribute((const void*)k_stage<R>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
  }
  const size_t shm = (sizeof(typename EVb<R>::T) << stage_qubits<R>()) + kStageLdsWords * 4;   // 64 + 12 KiB
  const uint32_t nchunks = 1u << (n - stage_qubits<R>());
  const unsigned grid = (unsigned)std::min<uint32_t>(nchunks, (uint32_t)ncu * 2);   // two 64 KiB chunks per CU
  hipLaunchKernelGGL(k_stage<R>, dim3(grid), dim3(stage_threads<R>()), shm, stream, (typename EVb<R>::T*)psi, n,
                     (const uint32_t*)d_recs, hrec, d_cbits, ncbits);
}

void launch_stage(bool c64, void* psi, int n, const void* d_recs, uint32_t hrec, const uint8_t* d_cbits, int ncbits,
                  hipStream_t stream) {
  if (c64) launch_stage_t<float>(psi, n, d_recs, hrec, d_cbits, ncbits, stream);
  else launch_stage_t<double>(psi, n, d_recs, hrec, d_cbits, ncbits, stream);
}

}  // namespace qk
