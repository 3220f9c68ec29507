// Random circuits through the host compiler of the LDS circuits (stages.cpp),
// its records run here as the interpreter runs them, in doubles, against a
// plain simulation: every builtin, controls, conditions, measurements, in one
// chunk of 1 to 13 qubits and in stages of 5 to 9.  Prints the largest
// difference; exits with 1 where one passes the bound given, a place in the
// buffer is taken twice or lies outside, or an outcome differs.
//   stage_records_emulator seed circuits bound
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "qk_internal.h"
#include "stage_records.h"

using namespace qk;

namespace qk {

struct Builtin {
  int arity, params;
};
const Builtin kGates[16] = {{0, 0}, {1, 0}, {1, 0}, {1, 0}, {1, 0}, {1, 0}, {1, 0}, {1, 0},
                            {1, 0}, {1, 1}, {1, 1}, {1, 1}, {1, 1}, {2, 1}, {2, 0}, {2, 1}};

bool builtin_info(int id, int* arity, int* nparams) {
  if (id < 1 || id > 15) return false;
  *arity = kGates[id].arity;
  *nparams = kGates[id].params;
  return true;
}

BuiltinGate builtin_gate(int id, double p) {
  const double c = std::cos(p / 2), s = std::sin(p / 2), r = std::sqrt(0.5);
  const cd i(0, 1), em = std::polar(1.0, -p / 2), ep = std::polar(1.0, p / 2);
  BuiltinGate g;
  auto set = [&](int cls, std::vector<cd> m) {
    g.cls = cls;
    g.nm = (int)m.size();
    std::copy(m.begin(), m.end(), g.m);
  };
  auto phase = [&](cd z) {
    g.cls = BG_PHASE;
    g.z = z;
  };
  switch (id) {
    case QK_H: set(BG_DENSE1, {r, r, r, -r}); break;
    case QK_X: set(BG_DENSE1, {0, 1, 1, 0}); break;
    case QK_Y: set(BG_DENSE1, {0, -i, i, 0}); break;
    case QK_RX: set(BG_DENSE1, {c, -i * s, -i * s, c}); break;
    case QK_RY: set(BG_DENSE1, {c, -s, s, c}); break;
    case QK_Z: phase(-1); break;
    case QK_S: phase(i); break;
    case QK_SDG: phase(-i); break;
    case QK_T: phase(std::polar(1.0, M_PI / 4)); break;
    case QK_TDG: phase(std::polar(1.0, -M_PI / 4)); break;
    case QK_PHASE:
    case QK_CPHASE: phase(std::polar(1.0, p)); break;
    case QK_RZ: set(BG_DIAG, {em, ep}); break;
    case QK_RZZ: set(BG_DIAG, {em, ep, ep, em}); break;
    case QK_SWAP: g.cls = BG_SWAP; break;
  }
  return g;
}

}  // namespace qk

namespace {

using State = std::vector<cd>;

[[noreturn]] void die(const char* what, long a = 0) {
  std::printf("%s (%ld)\n", what, a);
  std::exit(1);
}

uint32_t parity(uint32_t v) { return (uint32_t)__builtin_parity(v); }
uint32_t ins0(uint32_t p, uint32_t q) { return ((p >> q) << (q + 1)) | (p & ((1u << q) - 1)); }
uint32_t place(uint32_t i) { return (i ^ ((i >> 4) & 15)) * 8; }
double real_at(const uint32_t* w, int e) {
  double d;
  std::memcpy(&d, w + 2 * e, 8);
  return d;
}
uint32_t deposit(uint32_t v, uint32_t mask) {
  uint32_t out = 0;
  for (; mask; mask &= mask - 1, v >>= 1)
    if (v & 1u) out |= mask & (~mask + 1);
  return out;
}

// ---- plain simulation ---------------------------------------------------------------
void simulate(const std::vector<qk_op>& ops, State& st, std::vector<int>& cb) {
  for (const qk_op& o : ops) {
    if (o.kind == QK_OP_MEASURE) {
      double p[2] = {0, 0};
      for (size_t k = 0; k < st.size(); ++k) p[(k >> o.qubit) & 1] += std::norm(st[k]);
      const int oc = o.u < p[0] / (p[0] + p[1]) ? 0 : 1;
      for (size_t k = 0; k < st.size(); ++k) st[k] *= (int)((k >> o.qubit) & 1) == oc ? 1 / std::sqrt(p[oc]) : 0.0;
      if (o.cbit >= 0) cb[o.cbit] = oc;
      continue;
    }
    bool on = true;
    for (int c = 0; c < o.n_conds; ++c) on = on && cb[o.conds[c].cbit] == o.conds[c].value;
    if (!on) continue;
    const BuiltinGate g = builtin_gate(o.gate, o.param);
    const size_t a = (size_t)1 << o.targets[0], b = o.n_targets > 1 ? (size_t)1 << o.targets[1] : 0;
    size_t cm = 0;
    for (int c = 0; c < o.n_controls; ++c) cm |= (size_t)1 << o.controls[c];
    if (g.cls == BG_PHASE) cm |= a | b;
    for (size_t k = 0; k < st.size(); ++k) {
      if ((k & cm) != cm) continue;
      if (g.cls == BG_PHASE) st[k] *= g.z;
      else if (g.cls == BG_DIAG) st[k] *= g.m[(k & a ? 1 : 0) | (b && (k & b) ? 2 : 0)];
      else if (g.cls == BG_SWAP && (k & a) && !(k & b)) std::swap(st[k], st[k ^ a ^ b]);
      else if (g.cls == BG_DENSE1 && !(k & a)) {
        const cd x = st[k], y = st[k | a];
        st[k] = g.m[0] * x + g.m[1] * y;
        st[k | a] = g.m[2] * x + g.m[3] * y;
      }
    }
  }
}

// ---- the records -----------------------------------------------------------------------
struct Chunk {
  std::vector<cd> buf;   // by place
  uint32_t L, c;
  cd& at(uint32_t byte) {
    if (byte % 8 || byte / 8 >= buf.size()) die("outside the buffer", byte);
    return buf[byte / 8];
  }
};

// Places and bases of the groups in the layout of pass `lay` (nullptr: before the first).
template <typename F>
void groups(const Chunk& ch, const uint32_t* lay, F f) {
  const uint32_t tb = ch.L > 4 ? ch.L - 4 : 0;
  for (uint32_t g = 0; g < 1u << tb; ++g) {
    uint32_t base = g, v[4] = {place(1u << tb), place(2u << tb), place(4u << tb), place(8u << tb)}, sb;
    if (lay) {
      for (int j = 0; j < 4; ++j) {
        base = ins0(base, (lay[1] >> (8 * j)) & 0xff);
        v[j] = lay[8 + j];
      }
      sb = place(base);
      for (int j = 0; j < 4; ++j)
        if ((lay[0] >> (8 + j)) & 1)
          if (parity((lay[2 + j / 2] >> (16 * (j & 1))) & 0xffff & base) ^ parity(lay[4 + j] & ch.c)) sb ^= v[j];
    } else {
      sb = place(base);
    }
    uint32_t at[kMembers];
    for (int r = 0; r < kMembers; ++r) {
      at[r] = sb;
      for (int j = 0; j < 4; ++j)
        if ((r >> j) & 1) at[r] ^= v[j];
    }
    f(base, at);
  }
}

void run_pass(Chunk& ch, const uint32_t* w, const std::vector<int>& cb) {
  constexpr int kScales = 6;
  const bool scaled = w[0] & 0x2000;
  const int ng = (int)(w[0] >> 16) - (scaled ? kScales : 0);
  std::vector<char> seen(ch.buf.size(), 0);
  groups(ch, w, [&](uint32_t base, const uint32_t* at) {
    cd x[kMembers], factor = 1;
    for (int r = 0; r < kMembers; ++r) {
      x[r] = ch.at(at[r]);
      if (seen[at[r] / 8]++) die("a place taken twice", at[r]);
    }
    double* d = reinterpret_cast<double*>(x);   // re, im of member r: d[2 r], d[2 r + 1]
    uint32_t mm = 0xffff;
    for (int o = 1; o <= ng; ++o) {
      const uint32_t* h = w + o * kRecWords;
      const uint32_t op = h[3] >> 24, memb = h[1] & 0xffff, nc = (h[3] >> 18) & 3;
      const uint32_t lane = parity((h[1] >> 16) & base) ^ parity(h[2] & ch.c);
      auto u = [&](int e) { return real_at(h + 4, e); };
      if (h[0] != std::min<uint32_t>(op, RG_OTHER) * kGateBytes) die("a gate's place", op);
      if (o == ng) {
        if (op != RG_OTHER) die("a pass without its end", op);
        break;
      }
      if (nc > 0 && (cb[h[3] & 0xff] != (int)((h[3] >> 16) & 1) ||
                     (nc > 1 && cb[(h[3] >> 8) & 0xff] != (int)((h[3] >> 17) & 1)))) {
        mm = 0xffff;
        continue;
      }
      if (op == RG_PRED) {
        mm &= lane ? h[4] & 0xffff : h[4] >> 16;
        continue;
      }
      const bool act = mm != 0 && (!(h[3] & kOwnPredicate) || lane);
      if (op == RG_SCALE) {
        for (int r = 0; r < kMembers; ++r) {
          d[2 * r] *= real_at(h + kRecWords, r);
          d[2 * r + 1] *= real_at(h + kRecWords, kMembers + r);
        }
        o += kScales;
      } else if (op == RG_SIGN) {
        factor *= cd(u(0), lane ? u(1) : -u(1));
      } else if (op < RG_OTHER) {   // two steps
        for (int step = 0; step < 2; ++step)
          for (int r = 0; r < kMembers; ++r) {
            if (op >= RG_SIGN) {
              const double s = (parity((uint32_t)r & (op - RG_SIGN)) ^ lane) ? -1 : 1;
              if (step == 0) d[2 * r] += s * u(0) * d[2 * r + 1];
              else d[2 * r + 1] += s * u(1) * d[2 * r];
              continue;
            }
            const int q = r | 1 << (op & 3), im = op >= RG_IMAG;
            if (q == r) continue;
            if (step == 0) {
              d[2 * r] += u(0) * d[2 * q + im];
              d[2 * r + 1] += u(im ? 2 : 0) * d[2 * q + 1 - im];
            } else {
              d[2 * q + im] += u(1) * d[2 * r];
              d[2 * q + 1 - im] += u(im ? 3 : 1) * d[2 * r + 1];
            }
          }
      } else if (op == RG_LANE_Z) {
        if (act) factor *= cd(u(0), u(1));
      } else if (op == RG_PHASE || op == RG_PHASE_M) {
        for (int r = 0; r < kMembers; ++r) {
          if (op == RG_PHASE ? !act || !((memb >> r) & 1) : !((memb & mm) >> r & 1)) continue;
          double &re = d[2 * r], &im = d[2 * r + 1];
          if (h[3] & kThreeSteps) {
            re += u(0) * im;
            im += u(1) * re;
            re += u(0) * im;
          } else {
            const double t = re;
            re = u(0) * re - u(1) * im;
            im = u(0) * im + u(2) * t;
          }
        }
      } else {
        for (int r = 0; r < kMembers; ++r) {
          const int q = r | 1 << (op & 3);
          if (q == r || !((memb & mm) >> r & 1)) continue;
          const cd a = x[r], b = x[q], i(0, op >= RG_IMAG_M ? 1 : 0), one(1, 0), off = op >= RG_IMAG_M ? i : one;
          if (op >= RG_FLIP_M) {
            x[r] = u(0) * b;
            x[q] = u(0) * a;
          } else {
            x[r] = u(0) * a + off * u(1) * b;
            x[q] = off * u(2) * a + u(3) * b;
          }
        }
      }
      mm = 0xffff;
    }
    const uint32_t* sc = w + (1 + ng) * kRecWords;
    for (int r = 0; r < kMembers; ++r) {
      if (scaled) {
        d[2 * r] *= real_at(sc, r);
        d[2 * r + 1] *= real_at(sc, kMembers + r);
      }
      ch.at(at[r]) = w[0] & 0x1000 ? x[r] * factor : x[r];
    }
  });
}

// The items of a header on its chunk (amplitudes in order), in place.
void run_items(const uint32_t* h, State& amps, uint32_t outside, std::vector<int>& cb) {
  Chunk ch{std::vector<cd>(std::max<size_t>(16, amps.size())), (h[0] >> 8) & 0xff, outside | kOneBit};
  for (uint32_t i = 0; i < amps.size(); ++i) ch.at(place(i)) = amps[i];
  const uint32_t *w = h + kHeadRecords * kRecWords, *end = w + (size_t)h[1] * kRecWords, *lay = nullptr;
  while (w < end) {
    if ((w[0] & 0xff) == RK_PASS) {
      run_pass(ch, w, cb);
      lay = w;
      w += (size_t)(1 + (w[0] >> 16)) * kRecWords;
      continue;
    }
    double p[2] = {0, 0};
    auto value = [&](uint32_t base, int r) { return ((w[6] >> r) & 1) ^ parity(w[1] & base) ^ parity(w[2] & ch.c); };
    const uint32_t most = amps.size() < 16 ? (uint32_t)amps.size() : kMembers;   // members past the state are unused at first
    groups(ch, lay, [&](uint32_t base, const uint32_t* at) {
      for (uint32_t r = 0; r < (lay ? kMembers : most); ++r) p[value(base, (int)r)] += std::norm(ch.at(at[r]));
    });
    const int oc = real_at(w + 4, 0) < p[0] / (p[0] + p[1]) ? 0 : 1;
    groups(ch, lay, [&](uint32_t base, const uint32_t* at) {
      for (int r = 0; r < kMembers; ++r) ch.at(at[r]) *= (int)value(base, r) == oc ? 1 / std::sqrt(p[oc]) : 0.0;
    });
    if ((int32_t)w[3] >= 0) cb[w[3]] = oc;
    w += kRecWords;
  }
  const uint32_t* raw = h + kRecWords;
  for (uint32_t i = 0; i < amps.size(); ++i) {
    uint32_t at = 0;
    for (uint32_t j = 0; j < ch.L; ++j)
      if (((i >> j) & 1) ^ parity(raw[16 + j] & ch.c)) {
        at ^= raw[j];
        if (h[2] && !((i >> j) & 1)) die("a map that says it has no constants", (long)j);
      }
    amps[i] = ch.at(at);
  }
}

void run_stages(int n, int L, const std::vector<uint32_t>& rec, const std::vector<uint32_t>& heads, State& st,
                std::vector<int>& cb) {
  for (size_t k = 0; k < heads.size(); ++k) {
    const uint32_t* h = rec.data() + (size_t)heads[k] * kRecWords;
    if ((h[0] & 0xff) == RK_MEAS) {
      double p[2] = {0, 0};
      for (size_t i = 0; i < st.size(); ++i) p[(i & h[1]) != 0] += std::norm(st[i]);
      const int oc = real_at(h + 4, 0) < p[0] / (p[0] + p[1]) ? 0 : 1;
      for (size_t i = 0; i < st.size(); ++i) st[i] *= (int)((i & h[1]) != 0) == oc ? 1 / std::sqrt(p[oc]) : 0.0;
      if ((int32_t)h[3] >= 0) cb[h[3]] = oc;
      continue;
    }
    uint32_t in = 0;
    for (int j = 0; j < L; ++j) in |= 1u << ((h[4 + j / 4] >> (8 * (j % 4))) & 0xff);
    const uint32_t out = ((1u << n) - 1) & ~in;
    for (uint32_t ch = 0; ch < 1u << (n - L); ++ch) {
      const uint32_t c = deposit(ch, out);
      State amps((size_t)1 << L);
      for (uint32_t i = 0; i < amps.size(); ++i) amps[i] = k == 0 ? cd((c | i) == 0) : st[c | deposit(i, in)];
      run_items(h, amps, c, cb);
      for (uint32_t i = 0; i < amps.size(); ++i) st[c | deposit(i, in)] = amps[i];
    }
  }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc < 4) return 2;
  std::mt19937_64 rng(std::strtoull(argv[1], nullptr, 10));
  const double bound = std::atof(argv[3]);
  auto below = [&](int k) { return (int)(rng() % (uint64_t)k); };
  auto uniform = [&]() { return (double)(rng() >> 11) * 0x1p-53; };
  double worst = 0;
  for (int rep = 0; rep < std::atoi(argv[2]); ++rep) {
    const int n = 1 + below(13), count = below(120), style = below(3);   // style 1: rotations, H, CNOT and RZZ alone
    std::vector<qk_op> ops;
    while ((int)ops.size() < count) {
      qk_op o{};
      if (uniform() < 0.04) {
        o.kind = QK_OP_MEASURE;
        o.qubit = below(n);
        o.cbit = below(3) - 1;
        o.u = uniform();
        ops.push_back(o);
        continue;
      }
      const int layer[6] = {QK_H, QK_RX, QK_RY, QK_RZ, QK_X, QK_RZZ};
      o.kind = QK_OP_GATE;
      o.gate = style == 1 ? layer[below(6)] : 1 + below(15);
      o.n_targets = kGates[o.gate].arity;
      if (o.n_targets > n) continue;
      std::vector<int> q(n);
      for (int j = 0; j < n; ++j) q[j] = j;
      std::shuffle(q.begin(), q.end(), rng);
      const int room = std::min(4, n - o.n_targets);
      o.n_controls = style == 1 ? (o.gate == QK_X ? std::min(1, room) : 0) : uniform() < 0.4 ? below(room + 1) : 0;
      for (int j = 0; j < o.n_targets; ++j) o.targets[j] = q[j];
      for (int j = 0; j < o.n_controls; ++j) o.controls[j] = q[o.n_targets + j];
      if (style != 1 && uniform() < 0.15) {
        o.n_conds = 1 + below(2);
        for (int j = 0; j < o.n_conds; ++j) o.conds[j] = {below(2), below(2)};
      }
      o.param = 4 * M_PI * (uniform() - 0.5);
      ops.push_back(o);
    }
    std::vector<PlanOp> plan;
    std::string err;
    for (const qk_op& o : ops)
      if (expand_op(o, n, 2, plan, err)) die(err.c_str(), rep);
    State want((size_t)1 << n), got((size_t)1 << n);
    want[0] = got[0] = 1;
    std::vector<int> cw(2), cg(2);
    simulate(ops, want, cw);
    auto check = [&](const char* how) {
      double d = 0;
      for (size_t k = 0; k < want.size(); ++k) d = std::max(d, std::abs(want[k] - got[k]));
      worst = std::max(worst, d);
      if (!(d <= bound) || cw != cg) {
        std::printf("circuit %d, %d qubits, %s: %g\n", rep, n, how, d);
        std::exit(1);
      }
    };
    std::vector<uint32_t> rec, heads;
    build_job(n, false, plan, rec);
    run_items(rec.data(), got, 0, cg);
    check("one chunk");
    if (n < 5) continue;
    const int L = std::min(n, 5 + below(5));
    rec.clear();
    build_stages(n, L, false, plan, true, rec, heads);
    cg.assign(2, 0);
    run_stages(n, L, rec, heads, got, cg);
    check("stages");
  }
  std::printf("largest difference %g\n", worst);
  return 0;
}
