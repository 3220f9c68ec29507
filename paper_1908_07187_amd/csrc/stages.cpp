// Host compiler of the LDS circuits: builtin gates to plan operations, the
// stage planner, and the pass packer that writes the interpreter's records.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "qk_internal.h"
#include "stage_records.h"

namespace qk {

namespace {

qk_status cfail(std::string& err, qk_status st, const std::string& m) {
  err = m;
  return st;
}

inline uint32_t bit(int q) { return 1u << q; }
inline uint32_t parity(uint32_t v) { return (uint32_t)__builtin_parity(v); }

// The place of position i in LDS (place() in batch.hip), in bytes.
inline uint32_t place_bytes(uint32_t i, bool c64) {
  const uint32_t b = c64 ? 5 : 4, m = (1u << b) - 1;
  return (i ^ ((i >> b) & m)) * (c64 ? 4u : 8u);
}

// ---- what every qubit of the circuit stands for at a position -----------------
struct Frame {
  uint32_t in[32], out[32];   // the qubit's functional
  uint32_t v[32];             // the position vector along which only this qubit changes (stage qubits)
};

// Which ops may pass which: ops commute when on every qubit they share both
// act diagonally or both by bit flips.
struct Roles {
  uint32_t d = 0, x = 0, n = 0;
  bool passes(const PlanOp& o) const {
    return ((o.dmask & (x | n)) | (o.xmask & (d | n)) | (o.nmask & (d | x | n))) == 0;
  }
  void add(const PlanOp& o) {
    d |= o.dmask;
    x |= o.xmask;
    n |= o.nmask;
  }
  // The qubits on which no op passes.
  uint32_t blocked() const { return n | (d & x); }
};

// What gates past 45 degrees leave for the last pass of a circuit (its stages
// share it): the state is (-i)^quarter and a Z on each qubit of z times what the
// registers hold.
struct Left {
  uint32_t z = 0;
  int quarter = 0;
};

// ---- the pass packer ---------------------------------------------------------------
// Writes the items of a list of operations (in an order that is valid to
// apply) on the local qubits of one stage or job.  A pass starts at the first
// unplaced operation and takes every later one (kWindow looked at) that
// commutes with those it passes and fits: bit flips, CNOTs and swaps change
// the frame and cost nothing; a one-qubit gate needs its qubit as a slot,
// with the position vector and (up to the constant) the functional that the
// qubit had when the pass began; diagonal and phase gates act on any qubits,
// inside the stage or outside.
class Packer {
 public:
  Packer(int L, bool c64, std::vector<uint32_t>& rec, Left& left) : L_(L), c64_(c64), rec_(rec), left_(left) {
    for (int j = 0; j < kPassSlots; ++j) {   // the threads' amplitudes at first: the four highest positions
      v_[j] = in_[j] = bit(std::max(L, kPassSlots) - kPassSlots + j);
      out_[j] = 0;
    }
  }

  void run(const PlanOp* ops, size_t n, Frame& f, uint32_t local, bool final) {
    std::vector<char> used(n, 0);
    size_t first = 0;
    Taken taken[kPassGates];   // (each has a record at least)
    int count = 0;
    uint32_t qubits = 0;   // all that the ops act on
    for (size_t i = 0; i < n; ++i) qubits |= ops[i].dmask | ops[i].xmask | ops[i].nmask;
    while (first < n) {
      if (used[first]) {
        ++first;
        continue;
      }
      if (ops[first].type == PT_MEAS) {
        measure(ops[first], f);
        used[first++] = 1;
        continue;
      }
      const Frame f0 = f;
      Roles skipped;
      int slots[kPassSlots], ns = 0, records = 0, seen = 0;
      count = 0;
      for (size_t i = first; i < n && seen < kWindow && records < kPassGates; ++i) {
        if (used[i]) continue;
        if (skipped.blocked() == qubits) break;
        const PlanOp& o = ops[i];
        if (o.type == PT_MEAS) break;
        ++seen;
        bool ok = skipped.passes(o);
        if (ok) ok = take(o, f, f0, slots, ns, records, taken, count);
        if (ok) used[i] = 1;
        else skipped.add(o);
      }
      if (!count) continue;
      size_t next = first;   // the next op that a pass is for
      while (next < n && (used[next] || ops[next].type <= PT_MAPSWAP || ops[next].type == PT_MEAS)) ++next;
      close(f0, f, slots, ns, taken, count, local, final && next == n);
    }
    int slots[kPassSlots];
    if (final && (left_.z || (left_.quarter & 3))) close(f, f, slots, 0, nullptr, 0, local, true);   // (flips came after)
  }

 private:
  static constexpr int kWindow = 96;
  struct Fun { uint32_t in, out; };
  struct Taken {
    const PlanOp* o;
    double m[4];     // its coefficients as applied (see Left)
    int nfun;
    Fun fun[6];      // controls' functionals (value 1 wanted), the xf functional last
    int8_t want_xf;  // PT_PHASE: index of the xf functional or -1
    bool flip;       // the target's orientation is turned round
  };

  static Fun functional(const Frame& f, uint32_t qubits) {
    Fun r{0, 0};
    for (uint32_t m = qubits; m; m &= m - 1) {
      const int q = __builtin_ctz(m);
      r.in ^= f.in[q];
      r.out ^= f.out[q];
    }
    return r;
  }

  bool take(const PlanOp& o, Frame& f, const Frame& f0, int* slots, int& ns, int& records, Taken* taken, int& count) {
    if (o.type == PT_MAPX) {
      if (o.ctl) {
        const int c = __builtin_ctz(o.ctl);
        f.in[o.t] ^= f.in[c];
        f.out[o.t] ^= f.out[c];
        f.v[c] ^= f.v[o.t];   // (an outside control has no vector; its entry is unused)
        if (left_.z & bit(o.t)) left_.z ^= bit(c);
      } else {
        f.out[o.t] ^= kOneBit;
        if (left_.z & bit(o.t)) left_.quarter += 2;
      }
      return true;
    }
    if (o.type == PT_MAPSWAP) {
      if (((left_.z >> o.t) ^ (left_.z >> o.t2)) & 1u) left_.z ^= bit(o.t) | bit(o.t2);
      std::swap(f.in[o.t], f.in[o.t2]);
      std::swap(f.out[o.t], f.out[o.t2]);
      std::swap(f.v[o.t], f.v[o.t2]);
      return true;
    }
    Taken& k = taken[count];
    k.o = &o;
    k.nfun = 0;
    k.want_xf = -1;
    k.flip = false;
    std::copy(o.c, o.c + 4, k.m);
    const bool dense = o.type == PT_REAL || o.type == PT_IMAG;
    const int need = 1 + __builtin_popcount(o.ctl) + (o.type == PT_PHASE && o.xf ? 1 : 0);
    if (records + need > kPassGates) return false;
    if (dense || o.type == PT_FLIP) {
      const int t = o.t;
      if (f.v[t] != f0.v[t] || f.in[t] != f0.in[t] || ((f.out[t] ^ f0.out[t]) & ~kOneBit)) return false;
      k.flip = (f.out[t] ^ f0.out[t]) != 0;
      int s = 0;
      while (s < ns && slots[s] != t) ++s;
      if (s == ns) {
        if (ns == kPassSlots) return false;
        slots[ns++] = t;
      }
    }
    for (uint32_t m = o.ctl; m; m &= m - 1) k.fun[k.nfun++] = functional(f, m & (~m + 1));
    if (o.type == PT_SIGN) k.fun[k.nfun++] = functional(f, o.xf);
    if (o.type == PT_PHASE && o.xf) {
      k.want_xf = (int8_t)k.nfun;
      k.fun[k.nfun++] = functional(f, o.xf);
    }
    if (o.type == PT_FLIP) k.m[0] = left_.z & bit(o.t) ? -1.0 : 1.0;   // U Z = Z (Z U Z)
    if (dense && (left_.z & bit(o.t))) {
      k.m[1] = -k.m[1];
      k.m[2] = -k.m[2];
    }
    if (dense && k.flip) {
      std::swap(k.m[0], k.m[3]);
      std::swap(k.m[1], k.m[2]);
    }
    if (o.type == PT_SIGN && past45(k.m[0], k.m[1])) {   // c -+ i s = (-i) (+-1) (s +- i c): -i, and Z on each qubit
      std::swap(k.m[0], k.m[1]);
      k.m[1] = -k.m[1];
      left_.z ^= o.xf;
      ++left_.quarter;
    } else if (dense && o.ctl == 0 && o.ncond == 0 && past45(k.m[0], k.m[2])) {   // the rows exchanged
      std::swap(k.m[0], k.m[2]);
      std::swap(k.m[1], k.m[3]);
      if (o.type == PT_IMAG) {   // [[i c, d], [a, i b]] = i [[c, -i d], [-i a, b]]
        k.m[1] = -k.m[1];
        k.m[2] = -k.m[2];
        left_.quarter += 3;
      }
      f.out[o.t] ^= kOneBit;
    }
    records += need;
    ++count;
    return true;
  }

  static bool past45(double c, double s) { return std::fabs(s) > std::fabs(c) * (1 + 1e-12); }

  uint32_t* push() {
    rec_.resize(rec_.size() + kRecWords, 0u);
    return rec_.data() + rec_.size() - kRecWords;
  }

  // A gate record's op, conditions and own predicate.
  static void op_words(uint32_t* w, uint32_t op, const PlanOp& o, uint32_t flags) {
    const uint32_t c = o.conds;   // cb0 | cv0 << 8 | cb1 << 16 | cv1 << 24
    w[0] = std::min<uint32_t>(op, RG_OTHER) * kGateBytes;
    w[3] = (op << 24) | flags | ((uint32_t)o.ncond << 18) | ((c >> 24) & 1u) << 17 | ((c >> 8) & 1u) << 16 |
           ((c >> 16) & 0xffu) << 8 | (c & 0xffu);
  }

  void coef(uint32_t* w, int i, double x) const {
    if (c64_) {
      const float y = (float)x;
      std::memcpy(w + 4 + i, &y, 4);
    } else {
      std::memcpy(w + 4 + 2 * i, &x, 8);
    }
  }

  // A record of the lane factor: times c - i s, or c + i s where the functional is 1 (see RG_SIGN).
  void lane_factor(const Fun& f, double c, double s, bool& factor) {
    uint32_t* w = push();
    w[1] = ((1u << kMembers) - 1) | (f.in << 16);
    w[2] = f.out;
    op_words(w, RG_SIGN, PlanOp(), 0);
    std::memcpy(w + 4, &c, 8);
    std::memcpy(w + 6, &s, 8);
    factor = true;
  }

  void measure(const PlanOp& o, const Frame& f) {
    Fun lane{f.in[o.t], f.out[o.t]};
    uint32_t alpha = 0, members = 0;
    for (int j = 0; j < kPassSlots; ++j)
      if (parity(f.in[o.t] & v_[j])) {
        alpha |= bit(j);
        lane.in ^= in_[j];
        lane.out ^= out_[j];
      }
    for (int r = 0; r < kMembers; ++r) members |= parity((uint32_t)r & alpha) << r;
    uint32_t* w = push();
    w[0] = RK_MEAS;
    w[1] = lane.in;
    w[2] = lane.out;
    w[3] = (uint32_t)o.cbit;
    std::memcpy(w + 4, &o.c[0], 8);
    w[6] = members;
  }

  // The records of one gate.
  void gate(const Taken& k, int slot, const uint32_t* v, const uint32_t* in, const uint32_t* out, bool& factor) {
    const PlanOp& o = *k.o;
    const uint32_t all = (1u << kMembers) - 1;
    // every functional as slot bits (alpha) and a part that is the same for
    // all members of a group
    uint32_t alpha[6];
    Fun lane[6];
    for (int i = 0; i < k.nfun; ++i) {
      alpha[i] = 0;
      lane[i] = k.fun[i];
      for (int j = 0; j < kPassSlots; ++j)
        if (parity(k.fun[i].in & v[j])) {
          alpha[i] |= bit(j);
          lane[i].in ^= in[j];
          lane[i].out ^= out[j];
        }
    }
    if (o.type == PT_SIGN) {
      if (!alpha[0]) {
        lane_factor(lane[0], k.m[0], k.m[1], factor);
        return;
      }
      uint32_t* w = push();
      w[1] = all | (lane[0].in << 16);
      w[2] = lane[0].out;
      const double m[4] = {k.m[0], k.m[1], -k.m[1], k.m[0]};
      rotation(w, RG_SIGN + alpha[0], o, m, sc_.lambda, 1.0);
      return;
    }
    // predicates: a static member mask, lane predicates, mixed ones
    uint32_t memb = all;
    struct Pred { Fun f; uint32_t on, off; } pr[6];
    int np = 0;
    bool mixed = false;
    for (int i = 0; i < k.nfun; ++i) {
      const uint32_t want = i == k.want_xf ? (uint32_t)o.xv : 1u;
      uint32_t on = 0, off = 0;   // members that satisfy it where the lane part is 1 / 0
      for (int r = 0; r < kMembers; ++r) {
        const uint32_t pb = parity((uint32_t)r & alpha[i]);
        if ((pb ^ 1u) == want) on |= bit(r);
        if (pb == want) off |= bit(r);
      }
      if (lane[i].in == 0 && (lane[i].out & ~kOneBit) == 0) {
        memb &= lane[i].out ? on : off;
      } else if (alpha[i] == 0) {
        Fun g = lane[i];
        if (!want) g.out ^= kOneBit;
        pr[np++] = {g, all, 0};
      } else {
        pr[np++] = {lane[i], on, off};
        mixed = true;
      }
    }
    const bool phase = o.type == PT_PHASE;
    const bool plain = k.nfun == 0 && o.ncond == 0;
    if (!phase && !plain && (o.type == PT_FLIP ? sc_.mu[slot] != 1.0 : o.type == PT_IMAG && sc_.lambda != 1.0)) {
      op_words(push(), RG_SCALE, PlanOp(), 0);
      put_scales();
    }
    const int own = phase && !mixed && np > 0 ? np - 1 : np;   // the last lane predicate goes into the gate's record
    for (int i = 0; i < own; ++i) {
      uint32_t* w = push();
      op_words(w, RG_PRED, PlanOp(), 0);
      w[1] = pr[i].f.in << 16;
      w[2] = pr[i].f.out;
      w[4] = pr[i].on | (pr[i].off << 16);
    }
    uint32_t* w = push();
    w[1] = memb;
    if (phase) {
      const bool lz = !mixed && memb == all;
      op_words(w, mixed ? RG_PHASE_M : lz ? RG_LANE_Z : RG_PHASE, o, own < np ? kOwnPredicate : 0u);
      if (own < np) {
        w[1] |= pr[own].f.in << 16;
        w[2] = pr[own].f.out;
      }
      const double c = k.m[0], s = k.m[1];
      if (lz) {
        std::memcpy(w + 4, &c, 8);
        std::memcpy(w + 6, &s, 8);
        factor = true;
      } else if (c > 0 && !past45(c, s)) {
        w[3] |= kThreeSteps;
        coef(w, 0, -s / (1 + c) * sc_.lambda);
        coef(w, 1, s / sc_.lambda);
      } else {
        coef(w, 0, c);
        coef(w, 1, s * sc_.lambda);
        coef(w, 2, s / sc_.lambda);
      }
      return;
    }
    const double* m = k.m;
    if (plain && o.type == PT_REAL) {
      rotation(w, RG_REAL + slot, o, m, sc_.mu[slot], 1.0);
    } else if (plain && o.type == PT_IMAG) {   // on (re, im); the opposite angle on (im, re)
      const double x[4] = {m[0], -m[1], m[2], m[3]};
      rotation(w, RG_IMAG + slot, o, x, sc_.mu[slot], sc_.lambda);
    } else {
      const double mu = sc_.mu[slot];   // (1 for a flip)
      op_words(w, (uint32_t)((o.type == PT_FLIP ? RG_FLIP_M : o.type == PT_REAL ? RG_REAL_M : RG_IMAG_M) + slot), o, 0);
      coef(w, 0, m[0]);
      coef(w, 1, m[1] * mu);
      coef(w, 2, m[2] / mu);
      coef(w, 3, m[3]);
    }
  }

  // A plain gate of at most 45 degrees, given as the orthogonal matrix m on
  // pairs (x, y) with y at the scale mu relative to x's (for RG_IMAG: mu lambda,
  // and mu / lambda for the pairs that turn by the opposite angle), as a
  // rotation: the sign of a reflection goes to y's scale, that of angles past 90
  // degrees to g.  Tangents are taken from the rounded A, so that the scales fit
  // what the steps do.
  void rotation(uint32_t* w, int op, const PlanOp& o, const double* m, double& mu, double lambda) {
    double a = m[0], c = m[2];
    if (m[0] * m[3] - m[1] * m[2] < 0) mu = -mu;
    if (a < 0) {
      a = -a;
      c = -c;
      sc_.g = -sc_.g;
    }
    const bool imag = op >= RG_IMAG && op < RG_SIGN;
    op_words(w, (uint32_t)op, o, 0);
    const double t = c / a;   // tan phi
    double t2 = 1;
    for (int e = 0; e < (imag ? 2 : 1); ++e) {
      const double rel = e ? mu / lambda : mu * lambda, sign = e ? -1 : 1;
      const double A = rounded(-sign * t * rel), ta = -sign * A / rel;
      coef(w, 2 * e, A);
      coef(w, 2 * e + 1, sign * (ta / (1 + ta * ta)) / rel);
      t2 *= 1 + ta * ta;
    }
    if (imag) t2 = std::sqrt(t2);
    sc_.g /= std::sqrt(t2);
    mu *= t2;
  }

  double rounded(double x) const { return c64_ ? (double)(float)x : x; }

  // The scales of the registers, which are 1 after that.  What rounding them
  // changes of the norm is made good by the next ones.
  bool scaled() const {
    bool one = sc_.g == 1.0 && sc_.lambda == 1.0;
    for (int j = 0; j < kPassSlots; ++j) one = one && sc_.mu[j] == 1.0;
    return !one;
  }
  void put_scales() {
    const int words = c64_ ? 1 : 2;
    const size_t at = rec_.size();
    rec_.resize(at + (c64_ ? 3 : 6) * kRecWords, 0u);
    double scale[2 * kMembers] = {sc_.g};
    scale[kMembers] = sc_.g * sc_.lambda;
    for (int j = 0; j < kPassSlots; ++j)
      for (int r = 0; r < 1 << j; ++r) {
        scale[r | 1 << j] = scale[r] * sc_.mu[j];
        scale[kMembers | r | 1 << j] = scale[kMembers | r] * sc_.mu[j];
      }
    double off = 0;
    for (int i = 0; i < 2 * kMembers; ++i) {
      const double x = scale[i];
      const double y = x * (1 - drift_);
      if (c64_) {
        const float r = (float)y;
        std::memcpy(rec_.data() + at + i * words, &r, 4);
        off += (double)r / x - 1;
      } else {
        std::memcpy(rec_.data() + at + i * words, &y, 8);
      }
    }
    drift_ += off / (2 * kMembers);
    sc_ = Scales();
  }

  void close(const Frame& f0, const Frame& f, int* slots, int ns, const Taken* taken, int count, uint32_t local,
             bool last) {
    // fill the slots with unused qubits, the highest first; below four
    // qubits with positions L, L + 1, ... (LDS padding, which no gate names)
    uint32_t v[kPassSlots], in[kPassSlots], out[kPassSlots];
    for (int j = 0; j < ns; ++j) {
      v[j] = f0.v[slots[j]];
      in[j] = f0.in[slots[j]];
      out[j] = f0.out[slots[j]];
    }
    int n = ns;
    uint32_t left = local;
    for (int j = 0; j < ns; ++j) left &= ~bit(slots[j]);
    while (left && n < kPassSlots) {
      const int q = 31 - __builtin_clz(left);
      left ^= bit(q);
      v[n] = f0.v[q];
      in[n] = f0.in[q];
      out[n++] = f0.out[q];
    }
    for (int p = L_; n < kPassSlots; ++p, ++n) {
      v[n] = in[n] = bit(p);
      out[n] = 0;
    }
    for (int j = 0; j < kPassSlots; ++j) {
      v_[j] = v[j];
      in_[j] = in[j];
      out_[j] = out[j];
    }
    // pivots of the span of the v_j
    uint32_t piv[kPassSlots], red[kPassSlots], pmask = 0;
    for (int j = 0; j < kPassSlots; ++j) {
      uint32_t x = v[j];
      for (int i = 0; i < j; ++i)
        if (x & bit((int)piv[i])) x ^= red[i];
      piv[j] = 31u - (uint32_t)__builtin_clz(x);
      red[j] = x;
      for (int i = 0; i < j; ++i)
        if (red[i] & bit((int)piv[j])) red[i] ^= x;
      pmask |= bit((int)piv[j]);
    }
    std::sort(piv, piv + kPassSlots);
    const size_t head = rec_.size();
    push();
    bool factor = false;
    for (int i = 0; i < count; ++i) {
      const Taken& k = taken[i];
      const int slot = (int)(std::find(slots, slots + ns, (int)k.o->t) - slots);   // (of a one-qubit gate)
      gate(k, slot, v, in, out, factor);
    }
    // what gates past 45 degrees left: signs, after the last pass, and a factor i
    // of the whole state, where the pass has a lane factor anyway or is the last
    Fun sign{0, 0};
    if (last) {
      sign = functional(f, left_.z);
      left_.z = 0;
      uint32_t in0 = sign.in;
      for (int j = 0; j < kPassSlots; ++j)
        if (parity(in0 & v[j])) {
          sc_.mu[j] = -sc_.mu[j];
          sign.in ^= in[j];
          sign.out ^= out[j];
        }
      if (sign.in || (sign.out & ~kOneBit)) {
        lane_factor(sign, 0.0, 1.0, factor);
        left_.quarter += 3;
      } else if (sign.out) {
        left_.quarter += 2;
      }
    }
    if ((left_.quarter & 1) && (factor || last)) {
      lane_factor(Fun{0, 0}, 0.0, 1.0, factor);
      left_.quarter += 3;
    }
    if (left_.quarter & 2) sc_.g = -sc_.g;
    left_.quarter &= 1;
    op_words(push(), RG_OTHER, PlanOp(), 0);   // ends the pass
    const bool scales = scaled();
    if (scales) put_scales();
    uint32_t* h = rec_.data() + head;
    uint32_t adjust = 0;
    for (int j = 0; j < kPassSlots; ++j) {
      const uint32_t row = in[j] & ~pmask;
      if (row || out[j]) adjust |= bit(j);
      h[2 + j / 2] |= row << (16 * (j & 1));
      h[4 + j] = out[j];
      h[8 + j] = place_bytes(v[j], c64_);
      h[1] |= piv[j] << (8 * j);
    }
    const uint32_t ngates = (uint32_t)((rec_.size() - head) / kRecWords) - 1;
    h[0] = RK_PASS | (adjust << 8) | (factor ? 1u << 12 : 0u) | (scales ? 1u << 13 : 0u) | (ngates << 16);
  }

  // The true value of a register that holds 1 is g, times lambda for an
  // imaginary part, times mu_j where bit j of its member is 1.
  struct Scales {
    double g = 1, lambda = 1, mu[kPassSlots] = {1, 1, 1, 1};
  };

  int L_;
  bool c64_;
  std::vector<uint32_t>& rec_;
  Scales sc_;
  double drift_ = 0;   // relative norm that rounded scales added
  Left& left_;
  uint32_t v_[kPassSlots], in_[kPassSlots], out_[kPassSlots];   // the slots of the last pass
};

// One stage or job: header, items, and the map from amplitudes back to
// positions.  local: its qubits; final: the circuit ends with it.
void build_items(int L, bool c64, uint32_t local, const PlanOp* ops, size_t n, int nq,
                 std::vector<uint32_t>& rec, Left& left, bool final) {
  const size_t head = rec.size();
  rec.resize(head + (size_t)kHeadRecords * kRecWords, 0u);
  Frame f;
  for (int q = 0; q < nq; ++q) {
    f.in[q] = 0;
    f.out[q] = bit(q);
    f.v[q] = 0;
  }
  int count = 0;
  for (uint32_t m = local; m; m &= m - 1) {
    const int q = __builtin_ctz(m);
    f.in[q] = f.v[q] = bit(count++);
    f.out[q] = 0;
  }
  Packer(L, c64, rec, left).run(ops, n, f, local, final);
  uint32_t* h = rec.data() + head;
  h[0] = RK_STAGE | ((uint32_t)L << 8);
  h[1] = (uint32_t)((rec.size() - head) / kRecWords) - kHeadRecords;
  // amplitude i sits at position sum_j (i_j + const_j) v_j
  bool plain = true;
  uint32_t* raw = h + kRecWords;
  uint8_t* bytes = reinterpret_cast<uint8_t*>(h + 4);
  int j = 0;
  for (uint32_t m = local; m; m &= m - 1, ++j) {
    const int q = __builtin_ctz(m);
    bytes[j] = (uint8_t)q;
    raw[j] = place_bytes(f.v[q], c64);
    raw[16 + j] = f.out[q];
    plain = plain && f.v[q] == bit(j) && f.out[q] == 0;
  }
  h[2] = plain ? 1u : 0u;
}

// ---- the stage planner --------------------------------------------------------------
// Operations are taken from a ready frontier: on each qubit the operations
// form runs of one role (all diagonal, or all bit flips, or one other), and an
// operation is ready when its run is the current one on each of its qubits.
class Planner {
 public:
  Planner(int n, const PlanOp* ops, size_t count) : ops_(ops), n_(count), pend_(count, 0), done_(count, 0) {
    for (int q = 0; q < n; ++q) runs_[q].clear();
    for (size_t i = 0; i < count; ++i) {
      add_role((int)i, ops[i].dmask, 0);
      add_role((int)i, ops[i].xmask, 1);
      add_role((int)i, ops[i].nmask, 2);
    }
    for (int q = 0; q < n; ++q) {
      cur_[q] = 0;
      rem_[q] = runs_[q].empty() ? 0 : (int)runs_[q][0].ops.size();
    }
    for (size_t i = 0; i < count; ++i)
      if (pend_[i] == 0) ready_.push_back((int)i);
  }

  bool empty() const { return ready_.empty(); }

  // The next stage on at most L qubits: starting from the qubits of S, takes
  // every ready operation inside, then the qubits that let the most further
  // operations in per qubit added (counted by taking them tentatively), or,
  // with look = false, those of the earliest ready operation.
  uint32_t stage(uint32_t S, int L, bool look, std::vector<int>& out) {
    for (;;) {
      closure(S, &out);
      uint32_t best = 0;
      double best_score = -1;
      int best_op = 0;
      uint32_t tried[64];
      int nt = 0;
      for (int r : ready_) {
        const uint32_t add = ops_[r].need & ~S;
        if (__builtin_popcount(S | add) > L) continue;
        if (!look) {
          if (!best || r < best_op) {
            best = add;
            best_op = r;
          }
          continue;
        }
        if (nt == 64 || std::find(tried, tried + nt, add) != tried + nt) continue;
        tried[nt++] = add;
        const double score = (double)closure(S | add, nullptr) / __builtin_popcount(add);
        if (score > best_score || (score == best_score && r < best_op)) {
          best = add;
          best_score = score;
          best_op = r;
        }
      }
      if (!best) return S;
      S |= best;
    }
  }

 private:
  struct Run {
    int role;
    std::vector<int> ops;
  };

  void add_role(int i, uint32_t mask, int role) {
    for (; mask; mask &= mask - 1) {
      auto& rq = runs_[__builtin_ctz(mask)];
      if (rq.empty() || role == 2 || rq.back().role != role) rq.push_back({role, {}});
      rq.back().ops.push_back(i);
      if (rq.size() > 1) ++pend_[i];
    }
  }

  // Marks an operation done; operations newly ready go to `fresh`.  Returns
  // the qubits on which it ended a run.
  uint32_t complete(int i, std::vector<int>& fresh) {
    uint32_t ended = 0;
    done_[i] = 1;
    for (uint32_t m = ops_[i].dmask | ops_[i].xmask | ops_[i].nmask; m; m &= m - 1) {
      const int q = __builtin_ctz(m);
      if (--rem_[q] > 0) continue;
      ended |= bit(q);
      if (++cur_[q] < (int)runs_[q].size()) {
        rem_[q] = (int)runs_[q][cur_[q]].ops.size();
        for (int j : runs_[q][cur_[q]].ops)
          if (--pend_[j] == 0) fresh.push_back(j);
      }
    }
    return ended;
  }

  void undo(int i, uint32_t ended) {
    done_[i] = 0;
    for (uint32_t m = ops_[i].dmask | ops_[i].xmask | ops_[i].nmask; m; m &= m - 1) {
      const int q = __builtin_ctz(m);
      if (ended & bit(q)) {
        if (cur_[q] < (int)runs_[q].size())
          for (int j : runs_[q][cur_[q]].ops) ++pend_[j];
        --cur_[q];
        rem_[q] = 0;
      }
      ++rem_[q];
    }
  }

  // Takes every ready operation whose qubits lie in S, and those that become
  // ready; with out == nullptr only counts them.
  size_t closure(uint32_t S, std::vector<int>* out) {
    log_.clear();
    ended_.clear();
    for (int r : ready_)
      if ((ops_[r].need & ~S) == 0) log_.push_back(r);
    for (size_t k = 0; k < log_.size(); ++k) {
      fresh_.clear();
      ended_.push_back(complete(log_[k], fresh_));
      for (int j : fresh_) {
        if ((ops_[j].need & ~S) == 0) log_.push_back(j);
        else if (out) ready_.push_back(j);
      }
    }
    if (out) {
      out->insert(out->end(), log_.begin(), log_.end());
      ready_.erase(std::remove_if(ready_.begin(), ready_.end(), [&](int r) { return done_[r] != 0; }), ready_.end());
    } else {
      for (size_t k = log_.size(); k-- > 0;) undo(log_[k], ended_[k]);
    }
    return log_.size();
  }

  const PlanOp* ops_;
  size_t n_;
  std::vector<int> pend_;
  std::vector<char> done_;
  std::vector<Run> runs_[32];
  int cur_[32], rem_[32];
  std::vector<int> ready_, log_, fresh_;
  std::vector<uint32_t> ended_;
};

}  // namespace

qk_status expand_op(const qk_op& o, int n, int ncbits, std::vector<PlanOp>& out, std::string& err) {
  if (o.n_conds < 0 || o.n_conds > 2) return cfail(err, QK_E_ARG, "at most 2 conditions");
  for (int c = 0; c < o.n_conds; ++c) {
    if (o.conds[c].cbit < 0 || o.conds[c].cbit >= ncbits) return cfail(err, QK_E_ARG, "condition cbit out of range");
    if (o.conds[c].value != 0 && o.conds[c].value != 1) return cfail(err, QK_E_ARG, "condition value must be 0 or 1");
  }
  PlanOp d;
  d.ncond = (int8_t)o.n_conds;
  if (o.n_conds > 0) d.conds = (uint32_t)o.conds[0].cbit | ((uint32_t)o.conds[0].value << 8);
  if (o.n_conds > 1) d.conds |= ((uint32_t)o.conds[1].cbit << 16) | ((uint32_t)o.conds[1].value << 24);
  if (o.kind == QK_OP_MEASURE) {
    if (o.qubit < 0 || o.qubit >= n) return cfail(err, QK_E_ARG, "qubit out of range");
    if (o.cbit < -1 || o.cbit >= ncbits) return cfail(err, QK_E_ARG, "cbit out of range");
    if (!(o.u >= 0.0 && o.u < 1.0)) return cfail(err, QK_E_ARG, "u must be in [0, 1)");
    if (o.n_conds) return cfail(err, QK_E_ARG, "measurements take no conditions");
    d.type = PT_MEAS;
    d.t = (int8_t)o.qubit;
    d.cbit = o.cbit;
    d.c[0] = o.u;
    out.push_back(d);
    return QK_OK;
  }
  if (o.kind != QK_OP_GATE) return cfail(err, QK_E_ARG, "unknown op kind");
  int arity = 0, np = 0;
  if (!builtin_info(o.gate, &arity, &np)) return cfail(err, QK_E_UNSUPPORTED, "batched circuits take builtin gates only");
  if (o.n_targets != arity) return cfail(err, QK_E_ARG, "target count does not match the gate");
  if (o.n_controls < 0 || o.n_controls > 4) return cfail(err, QK_E_ARG, "at most 4 controls");
  uint32_t seen = 0;
  for (int q = 0; q < o.n_targets + o.n_controls; ++q) {
    const int x = q < o.n_targets ? o.targets[q] : o.controls[q - o.n_targets];
    if (x < 0 || x >= n) return cfail(err, QK_E_ARG, "qubit index out of range");
    if (seen & bit(x)) return cfail(err, QK_E_ARG, "qubit used twice in one gate");
    seen |= bit(x);
  }
  for (int q = 0; q < o.n_controls; ++q) d.ctl |= bit(o.controls[q]);
  const int t = o.targets[0], t2 = arity > 1 ? o.targets[1] : 0;
  d.t = (int8_t)t;
  d.t2 = (int8_t)t2;
  // bit flips: at most one control and no condition only change the frame
  auto flip = [&](PlanOp x) {
    x.type = x.ncond == 0 && __builtin_popcount(x.ctl) <= 1 ? PT_MAPX : PT_FLIP;
    x.need = x.xmask = bit(x.t);
    x.dmask = x.ctl;
    out.push_back(x);
  };
  if (o.gate == QK_X) {
    flip(d);
    return QK_OK;
  }
  const BuiltinGate g = builtin_gate(o.gate, np ? o.param : 0.0);
  switch (g.cls) {
    case BG_DENSE1: {
      const cd* m = g.m;
      if (o.gate == QK_Y && d.ctl == 0 && d.ncond == 0) {   // X diag(i, -i)
        PlanOp s = d;
        s.type = PT_SIGN;
        s.xf = s.dmask = bit(t);
        s.c[0] = 0.0;
        s.c[1] = -1.0;
        out.push_back(s);
        flip(d);
        break;
      }
      // RX and Y have a real diagonal and imaginary off-diagonal entries, the
      // others are real (by name: with a parameter that is not finite the
      // entries are NaN in both parts)
      const bool real = o.gate != QK_RX && o.gate != QK_Y;
      for (int e = 0; e < 4; ++e)
        if (real && m[e].imag() != 0.0) return cfail(err, QK_E_UNSUPPORTED, "gate class not supported in batches");
      d.type = real ? PT_REAL : PT_IMAG;
      for (int e = 0; e < 4; ++e) d.c[e] = real || e == 0 || e == 3 ? m[e].real() : m[e].imag();
      d.need = bit(t);
      d.dmask = d.ctl;
      // RX is a function of X: it passes bit flips of its qubit
      if (!real && m[0] == m[3] && m[1] == m[2]) d.xmask = bit(t);
      else d.nmask = bit(t);
      out.push_back(d);
      break;
    }
    case BG_DIAG: {   // factors e^{-i phi}, e^{i phi} by the parity of the targets
      d.xf = bit(t) | (arity > 1 ? bit(t2) : 0u);
      d.dmask = d.xf | d.ctl;
      d.c[0] = g.m[1].real();
      d.c[1] = g.m[1].imag();
      if (d.ctl == 0 && d.ncond == 0) {
        d.type = PT_SIGN;
        out.push_back(d);
      } else {   // one factor on each half of the subspace
        d.type = PT_PHASE;
        d.xv = 1;
        out.push_back(d);
        d.xv = 0;
        d.c[1] = -d.c[1];
        out.push_back(d);
      }
      break;
    }
    case BG_PHASE:
      d.type = PT_PHASE;
      d.ctl |= bit(t) | (arity > 1 ? bit(t2) : 0u);
      d.dmask = d.ctl;
      d.c[0] = g.z.real();
      d.c[1] = g.z.imag();
      out.push_back(d);
      break;
    case BG_SWAP: {
      if (d.ctl == 0 && d.ncond == 0) {
        d.type = PT_MAPSWAP;
        d.need = d.nmask = bit(t) | bit(t2);
        out.push_back(d);
        break;
      }
      // CNOT(t2 -> t), flip of t2 controlled by t and the rest, CNOT(t2 -> t)
      PlanOp a;
      a.t = d.t;
      a.ctl = bit(t2);
      PlanOp b = d;
      b.t = d.t2;
      b.ctl = d.ctl | bit(t);
      flip(a);
      flip(b);
      flip(a);
      break;
    }
    default:
      return cfail(err, QK_E_UNSUPPORTED, "gate class not supported in batches");
  }
  return QK_OK;
}

void build_job(int n, bool c64, const std::vector<PlanOp>& ops, std::vector<uint32_t>& rec) {
  Left left;
  build_items(n, c64, (1u << n) - 1, ops.data(), ops.size(), n, rec, left, true);
}

void build_stages(int n, int L, bool c64, const std::vector<PlanOp>& ops, bool job, std::vector<uint32_t>& rec,
                  std::vector<uint32_t>& heads) {
  auto start = [&]() { heads.push_back((uint32_t)(rec.size() / kRecWords)); };
  const uint32_t low = (1u << kStageLowQubits) - 1;
  std::vector<PlanOp> local;
  std::vector<int> members;
  Left left;
  size_t end = ops.size();   // behind the last gate
  while (end > 0 && ops[end - 1].type == PT_MEAS) --end;
  auto emit = [&](uint32_t S, const PlanOp* base, bool final) {
    for (int q = 0; q < n && __builtin_popcount(S) < L; ++q) S |= bit(q);
    local.clear();
    for (int i : members) local.push_back(base[i]);
    start();
    build_items(L, c64, S, local.data(), local.size(), n, rec, left, final);
  };
  // the first stage of a job writes |0...0>: where the list is empty or
  // starts with a measurement, a stage without gates comes first
  if (job && (ops.empty() || ops[0].type == PT_MEAS)) emit(low, ops.data(), false);
  const bool look = n >= kStageLookQubits;
  size_t i0 = 0;
  while (i0 < ops.size()) {
    if (ops[i0].type == PT_MEAS) {
      start();
      rec.resize(rec.size() + kRecWords, 0u);
      uint32_t* w = rec.data() + rec.size() - kRecWords;
      w[0] = RK_MEAS;
      w[1] = bit(ops[i0].t);
      w[3] = (uint32_t)ops[i0].cbit;
      std::memcpy(w + 4, &ops[i0].c[0], 8);
      ++i0;
      continue;
    }
    size_t i1 = i0;
    while (i1 < ops.size() && ops[i1].type != PT_MEAS) ++i1;
    Planner plan(n, ops.data() + i0, i1 - i0);
    while (!plan.empty()) {
      members.clear();
      const uint32_t S = plan.stage(low, L, look, members);
      emit(S, ops.data() + i0, i1 == end && plan.empty());
    }
    i0 = i1;
  }
}

}  // namespace qk
