// Device records of the LDS circuits (batch jobs and stages): written by the
// host compiler (stages.cpp), run by the pass interpreter (batch.hip).
//
// The interpreter works on a chunk of 2^L amplitudes, one per position p of L
// bits.  Bit flips, CNOTs and swaps move nothing: they only change what a
// position stands for.  The value of qubit q at position p of a chunk is the
// parity of (in & p) xor the parity of (out & c), its "functional" (in, out),
// where c holds the chunk's amplitude-index bits outside the stage and, in
// bit 31, the constant 1.  A qubit of the stage starts as its own position
// bit, a qubit outside it as its own bit of c; a CNOT adds the control's
// functional to the target's, a bit flip adds the constant.
//
// A pass takes K = 4 slot qubits t_0..t_3, each with the position vector v_j
// along which only t_j's value changes, so that a thread holds the 16
// members of one group (base + the 2^4 combinations of the v_j) in
// registers; member r has value bit j of r at t_j.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "qk.h"

namespace qk {

constexpr int kRecWords = 12;                  // dwords of a record (48 bytes: 16-byte aligned reads)
constexpr int kPassSlots = 4;                  // slot qubits of a pass
constexpr int kMembers = 1 << kPassSlots;
constexpr int kPassGates = 40;                 // gate records that a pass takes at most (up to two more for the lane
                                               // factor, and one that ends them, follow)
constexpr int kHeadRecords = 4;                // records of a stage or job header
constexpr int kPadRecords = 24;                // zero records after the last item: a gate reads ahead, up to 1 KiB
constexpr int kMapBits = 14;                   // the largest chunk: 2^14 amplitudes
// Lowest qubits that every stage holds: its chunks are made of runs of 128 bytes
// (complex128; complex64: 64, two of which meet in an L2, see xcd_chunk).  With
// 4, complex64: 28 qubits, 8 layers 14.9 -> 14.4 ms, 30 qubits, 3 layers 28.6 ->
// 27.3 ms, but a qubit less for gates: 23 qubits, 20 layers 18 -> 21 stages, 0.95 ->
// 1.02 ms; complex128: 28 qubits 11 -> 13 stages, 24.0 -> 25.8 ms.
constexpr int kStageLowQubits = 3;
// From this many qubits the planner weighs each stage qubit by look-ahead: 28
// qubits, 8 layers, complex128 15 -> 11 stages, 31.1 -> 24.0 ms.  Below, it saves less
// on the device (20 qubits, 20 layers 508 -> 442 us, 14 qubits 203 -> 202 us)
// and makes planning a quarter longer (0.26 -> 0.33 ms at 20 qubits), which a
// batch's job pays when it is added.
constexpr int kStageLookQubits = 24;
constexpr uint32_t kOneBit = 1u << 31;         // the constant 1 of an `out` mask

// Item kinds (dword 0, low byte).
//   RK_STAGE: header of a stage or of a small job, kHeadRecords records:
//     dword 0 kind | L << 8, dword 1 the number of item records that follow,
//     dword 2 is 1 when positions are amplitudes in order (no map), dwords
//     4..7 the stage's qubits ascending (a byte each); in the other three
//     records (36 dwords) dwords 0..13: the LDS byte offset of local
//     amplitude-index bit j (position vector, swizzled), dwords 16..29: the
//     `out` mask whose parity in a chunk adds that offset once more.
//   RK_MEAS: measurement, in the layout of the pass before it (at first: the
//     four highest positions as slots): dword 1 `in`, dword 2 `out` mask of
//     the qubit's lane part, dword 3 the cbit or -1, dwords 4, 5 the uniform
//     (a double), dword 6 the members where its slot part is 1.  In a staged
//     job's list (on the state in global memory) dword 1 is the qubit's mask.
//   RK_PASS: kind | adjust << 8 | factor << 12 | scales << 13 | records << 16; dword 1: the
//     four pivot positions ascending (a byte each): a group's base has zeros
//     there; dwords 2, 3: the slots' `in` masks (16 bits each) off the
//     pivots, dwords 4..7 their `out` masks: where slot j's value at the base
//     is 1 (bit j of `adjust`: it can be) v_j is added; dwords 8..11: v_j as
//     swizzled LDS byte offsets.  factor: the pass has gates for the lane
//     factor.  scales: its last records (after the one that ends the gates) are
//     the scales that its gates leave on the registers: 16 reals for the real
//     parts, 16 for the imaginary ones.
enum RecKind { RK_PASS = 1, RK_MEAS = 2, RK_STAGE = 3 };

// Gate records of a pass: dword 0 the gate's place in the interpreter's code
// (kGateBytes times its op, at most RG_OTHER), dword 1 member mask | `in` <<
// 16, dword 2 `out` (the lane functional of the op), dword 3 op << 24 | own
// predicate << 20 | conditions << 18 | cv1 << 17 | cv0 << 16 | cb1 << 8 | cb0,
// dwords 4.. coefficients in the state's precision (the lane factor's: doubles).  The ops below RG_OTHER
// have no conditions and no masks.  The last gate record of a pass is RG_OTHER
// with nothing else.
//
// A rotation of the pair (x, y) by phi, at most 45 degrees, is done in place as
// x += A y, y += B x, which leaves x at the scale cos(phi) and y at 1/cos(phi) (A =
// -tan phi, B = sin phi cos phi).  A gate that turns further is one that does not
// after a quarter turn, which costs nothing: it exchanges what x and y stand for
// (a bit flip of the qubit in the frame) or turns signs, and a factor i or -i of
// the whole state goes to the lane factor.  The host keeps the scales: g
// lambda^[imaginary part] prod_j mu_j^[bit j of the member] is the true value of
// a register that holds 1.
enum RecGate {
  RG_REAL = 0,       // + slot: A, B on (re, re) and (im, im)
  RG_IMAG = 4,       // + slot: A, B on (re, im), A', B' on (im, re)
  RG_SIGN = 8,       // + m: A, B on (re, im) of each member, opposite where the parity of (r & m) xor the lane functional
                     // is 1; m = 0: the lane factor (a double in either precision), which multiplies all members when
                     // the pass ends, takes c - i s (opposite s likewise; c, s are doubles)
  RG_OTHER = 24,
  RG_REAL_M = 24,    // + slot: a real 2x2 matrix on the members of the mask and of the lane's member mask
  RG_IMAG_M = 28,    // + slot: [[a, i b], [i c, d]], masked likewise
  RG_FLIP_M = 32,    // + slot: pair exchange, with the sign of its coefficient (1 or -1), masked likewise
  RG_PHASE = 36,     // members of the mask times c + i s, on lanes whose predicates hold: c, s lambda, s / lambda, or
                     // (kThreeSteps) up to 45 degrees re += A im, im += B re, re += A im: A = -tan(phi/2) lambda, B =
                     // sin phi / lambda
  RG_PHASE_M = 37,   // members of the mask and of the lane's member mask likewise
  RG_PRED = 38,      // narrows the lane's member mask for the next gate: dword 4 = members where the functional is 1 |
                     // members where it is 0 << 16
  RG_LANE_Z = 39,    // lane factor times z (doubles) where the predicates hold
  RG_SCALE = 40,     // the registers times the scales in the records that follow (as after a pass)
};
constexpr uint32_t kGateBytes = 512;           // code bytes of one plain gate
constexpr uint32_t kOwnPredicate = 1u << 20;   // RG_PHASE, RG_LANE_Z: only where the lane functional is 1
constexpr uint32_t kThreeSteps = 1u << 21;     // RG_PHASE, RG_PHASE_M: see there

// A circuit operation as the planner and the packer see it.
enum PType { PT_MAPX = 0, PT_MAPSWAP, PT_REAL, PT_IMAG, PT_FLIP, PT_SIGN, PT_PHASE, PT_MEAS };
struct PlanOp {
  uint8_t type = 0;
  int8_t t = 0, t2 = 0;          // target qubit (PT_MAPSWAP: both; PT_MEAS: the qubit)
  int8_t ncond = 0;
  uint32_t ctl = 0;              // control qubits (PT_MAPX: at most one)
  uint32_t xf = 0;               // PT_SIGN: the qubits whose parity is the sign; PT_PHASE: an extra condition, the
  int32_t xv = 1;                // parity of these qubits equal to xv
  uint32_t need = 0;             // qubits that must be inside the stage
  uint32_t dmask = 0, xmask = 0, nmask = 0;   // qubits used as controls or diagonally, as bit flips, otherwise
  uint32_t conds = 0;
  int32_t cbit = -1;
  double c[4] = {0, 0, 0, 0};
};

// Appends the operations of one builtin gate or measurement record.
qk_status expand_op(const qk_op& o, int n, int ncbits, std::vector<PlanOp>& out, std::string& err);
// Records of a job that is one chunk (n qubits): header, then items.
void build_job(int n, bool c64, const std::vector<PlanOp>& ops, std::vector<uint32_t>& rec);
// Records of a state in global memory, by stages of L qubits; heads[i] = the
// record index of stage or measurement i.  With `job` the list starts with a
// stage (whose chunks are made |0...0>).
void build_stages(int n, int L, bool c64, const std::vector<PlanOp>& ops, bool job, std::vector<uint32_t>& rec,
                  std::vector<uint32_t>& heads);

}  // namespace qk
