// Run-time specialisation of the step kernels: the firing tables of a program are turned into
// straight-line HIP source (one block of code per table entry, values in named variables) and
// compiled for the current GPU with hiprtc.  The generated sweep replaces the table interpreter
// inside the same step logic (step_device.h), so both produce identical results.  hiprtc is
// loaded lazily; without it, or with TDF_NO_JIT=1, the interpreter is used.
#include <dlfcn.h>
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "tdf_internal.h"

// headers of the device code as string literals, written by the build script
#include "embedded_headers.inc"

namespace tdf {

namespace {

// ---- the subset of the hiprtc API that is used, resolved with dlsym ------------------------------
typedef void* rtcProgram;
struct Rtc {
  int (*create)(rtcProgram*, const char*, const char*, int, const char* const*, const char* const*) = nullptr;
  int (*compile)(rtcProgram, int, const char* const*) = nullptr;
  int (*log_size)(rtcProgram, size_t*) = nullptr;
  int (*log)(rtcProgram, char*) = nullptr;
  int (*code_size)(rtcProgram, size_t*) = nullptr;
  int (*code)(rtcProgram, char*) = nullptr;
  int (*destroy)(rtcProgram*) = nullptr;
  bool ok = false;
};

Rtc& rtc() {
  static Rtc r;
  static std::once_flag once;
  std::call_once(once, [] {
    void* h = dlopen("libhiprtc.so.7", RTLD_NOW | RTLD_LOCAL);
    if (!h) h = dlopen("libhiprtc.so", RTLD_NOW | RTLD_LOCAL);
    if (!h) return;
    r.create = (decltype(r.create))dlsym(h, "hiprtcCreateProgram");
    r.compile = (decltype(r.compile))dlsym(h, "hiprtcCompileProgram");
    r.log_size = (decltype(r.log_size))dlsym(h, "hiprtcGetProgramLogSize");
    r.log = (decltype(r.log))dlsym(h, "hiprtcGetProgramLog");
    r.code_size = (decltype(r.code_size))dlsym(h, "hiprtcGetCodeSize");
    r.code = (decltype(r.code))dlsym(h, "hiprtcGetCode");
    r.destroy = (decltype(r.destroy))dlsym(h, "hiprtcDestroyProgram");
    r.ok = r.create && r.compile && r.log_size && r.log && r.code_size && r.code && r.destroy;
  });
  return r;
}

// ---- source generation ------------------------------------------------------------------------
struct Gen {
  std::ostringstream o;
  const DevProgram& P;
  explicit Gen(const DevProgram& p) : P(p) {}

  // value / present / dead expressions of source k of an entry
  static std::string val(const Instr& I, int k) {
    if (I.src[k] == SRC_IMM) return "(long long)" + std::to_string((unsigned long long)I.imm) + "ULL";
    return "v" + std::to_string(I.src[k]);
  }
  static std::string pre(const Instr& I, int k) { return I.src[k] == SRC_IMM ? "true" : "p" + std::to_string(I.src[k]); }
  static std::string ded(const Instr& I, int k) { return I.src[k] == SRC_IMM ? "false" : "d" + std::to_string(I.src[k]); }

  // One entry without tokens, in a block of its own for the lanes (lane: helpers ln_*, else sw_*).
  void entry(const Instr& I, bool lane) {
    const std::string D = std::to_string(I.dst), h = lane ? "ln_" : "sw_";
    if (lane) o << "        {\n";
    switch (I.op) {
      case D_IN:
        o << "          p" << D << " = on && ((x.present >> " << (int)I.aux << ") & 1); v" << D << " = x.sv[" << (int)I.aux
          << "]; live = p" << D << "; all_in = all_in && p" << D << ";\n";
        break;
      case D_RET: {
        std::string all_p = "true", any_d = "false";
        bool any_arg = false;
        for (int k = 0; k < 4; ++k) {
          if (I.src[k] == SRC_NONE) continue;
          any_arg = true;
          all_p += " && p" + std::to_string(I.src[k]);
          any_d += " || d" + std::to_string(I.src[k]);
        }
        o << "          const bool p = on && ((x.present >> " << (int)I.aux << ") & 1);\n";
        o << "          const bool is_dead = on && !p && " << (any_arg ? "true" : "false") << " && (" << all_p << ") && (" << any_d
          << ");\n";
        o << "          v" << D << " = x.sv[" << (int)I.aux << "]; p" << D << " = p || is_dead; d" << D << " = is_dead; live = p;\n";
        o << "          all_in = all_in && p" << D << ";\n";
        break;
      }
      case D_ADD: case D_SUB: case D_MUL: case D_EQ: case D_LT: {
        const std::string a = val(I, 0), b = val(I, 1);
        o << "          const bool p = on && " << pre(I, 0) << " && " << pre(I, 1) << "; const bool d = " << ded(I, 0) << " || "
          << ded(I, 1) << ";\n";
        if (I.op == D_ADD) o << "          v" << D << " = (long long)((unsigned long long)" << a << " + (unsigned long long)" << b << ");\n";
        if (I.op == D_SUB) o << "          v" << D << " = (long long)((unsigned long long)" << a << " - (unsigned long long)" << b << ");\n";
        if (I.op == D_MUL) o << "          v" << D << " = (long long)((unsigned long long)" << a << " * (unsigned long long)" << b << ");\n";
        if (I.op == D_EQ) o << "          v" << D << " = " << a << " == " << b << ";\n";
        if (I.op == D_LT) o << "          v" << D << " = " << a << " < " << b << ";\n";
        o << "          p" << D << " = p; d" << D << " = p && d; live = p && !d;\n";
        break;
      }
      case D_ID:
        o << "          v" << D << " = " << val(I, 0) << "; p" << D << " = on && " << pre(I, 0) << "; d" << D << " = p" << D << " && "
          << ded(I, 0) << "; live = p" << D << " && !d" << D << ";\n";
        break;
      case D_ISLEAF: case D_LEFT: case D_RIGHT: case D_TOKEN:
        o << "          const bool p = on && " << pre(I, 0) << "; bool d = " << ded(I, 0) << "; long long r = 0;\n";
        o << "          if (p && !d) r = " << h << "tree(x, " << val(I, 0) << ", " << (I.op - D_ISLEAF) << ", d);\n";
        o << "          v" << D << " = r; p" << D << " = p; d" << D << " = p && d; live = p && !d;\n";
        break;
      case D_CE_NODE:
        o << "          const bool p = on && " << pre(I, 0) << " && " << pre(I, 1) << "; bool d = " << ded(I, 0) << " || " << ded(I, 1)
          << ";\n";
        o << "          if (p && !d) " << h << "ce_node(x, " << val(I, 0) << ", " << val(I, 1) << ", d);\n";
        o << "          v" << D << " = " << val(I, 0) << "; p" << D << " = p; d" << D << " = p && d; live = p && !d;\n";
        break;
      case D_SWITCH: {
        const std::string D1 = std::to_string(I.dst + 1);
        o << "          const bool p = on && " << pre(I, 0) << " && " << pre(I, 1) << "; const bool d = " << ded(I, 0) << " || "
          << ded(I, 1) << "; const bool t = " << val(I, 0) << " != 0;\n";
        o << "          v" << D << " = " << val(I, 1) << "; p" << D << " = p; d" << D << " = p && (d || !t);\n";
        o << "          v" << D1 << " = " << val(I, 1) << "; p" << D1 << " = p; d" << D1 << " = p && (d || t);\n";
        o << "          live = p && !d;\n";
        break;
      }
      case D_MERGE: {
        o << "          bool any_live = false, all_p = true; long long r = 0;\n";
        for (int k = 0; k < 4; ++k) {
          if (I.src[k] == SRC_NONE) continue;
          o << "          if (" << pre(I, k) << " && !" << ded(I, k) << " && !any_live) { any_live = true; r = " << val(I, k) << "; }\n";
          o << "          all_p = all_p && " << pre(I, k) << ";\n";
        }
        o << "          const bool p = on && (any_live || all_p);\n";
        o << "          v" << D << " = r; p" << D << " = p; d" << D << " = p && !any_live; live = on && any_live;\n";
        break;
      }
      case D_EMBED:
        o << "          " << h << "embed(x, on, " << (int)I.aux << ", " << (lane ? "" : "x.sv[" + std::to_string(I.aux) + "], ") << pre(I, 0) << ", "
          << ded(I, 0) << ", " << val(I, 0) << ", v" << D << ", p" << D << ", live);\n";
        break;
      case D_CELL:
        o << "          " << h << "cell(x, on, " << (int)I.aux << ", " << (lane ? "" : "x.sv[" + std::to_string(I.aux) + "], ") << pre(I, 0) << ", "
          << ded(I, 0) << ", " << val(I, 0) << ", " << pre(I, 1) << ", " << ded(I, 1) << ", " << val(I, 1) << ", v" << D << ", p" << D
          << ", live);\n";
        break;
      case D_HEAD:
        o << "          " << h << "head(x, on, " << (int)I.aux << ", " << pre(I, 0) << ", " << ded(I, 0) << ", " << val(I, 0) << ", " << pre(I, 1)
          << ", " << ded(I, 1) << ", " << val(I, 1) << ", v" << D << ", p" << D << ", live);\n";
        break;
      default: break;
    }
    if (lane) o << "        }\n";
  }

  void function(int f) {
    const DevFn& fn = P.fn[f];
    o << "    {  // function " << f << "\n";
    o << "      const bool on = x.myfn == " << f << ";\n";
    o << "      if (__ballot(on) != 0) {\n";
    for (int v = 0; v < fn.n_values; ++v)
      o << "        long long v" << v << " = 0; bool p" << v << " = false, d" << v << " = false;\n";
    o << "        bool live = false, all_in = true;\n";
    for (int ip = 0; ip < fn.count; ++ip) {
      const Instr& I = P.instr[fn.first + ip];
      const std::string bit = "(1ull << " + std::to_string(ip) + ")";
      o << "        {  // entry " << ip << " op " << (int)I.op << "\n";
      switch (I.op) {
        case D_CALL:
          o << "          sw_emit(x, on && " << pre(I, 0) << " && !" << ded(I, 0) << " && !(x.fired & " << bit << "), "
            << (0x80000000u | I.aux | ((uint32_t)I.aux2 << 8)) << "u, " << val(I, 0) << ");\n";
          o << "          live = on && " << pre(I, 0) << " && !" << ded(I, 0) << ";\n";
          break;
        case D_NEXT:
          o << "          sw_emit(x, on && " << pre(I, 0) << " && !" << ded(I, 0) << " && !(x.fired & " << bit << "), "
            << (0xC0000000u | ((uint32_t)I.aux2 << 8)) << "u, " << val(I, 0) << ");\n";
          o << "          live = on && " << pre(I, 0) << " && !" << ded(I, 0) << ";\n";
          break;
        case D_OUT:
          o << "          const bool go = on && " << pre(I, 0) << " && !" << ded(I, 0) << " && !(x.fired & " << bit << ");\n";
          if (f == P.result_fn) o << "          sw_result(x, go, " << (int)I.aux << ", " << val(I, 0) << ");\n";
          else o << "          sw_emit(x, go, 0u, " << val(I, 0) << ");\n";
          o << "          live = on && " << pre(I, 0) << " && !" << ded(I, 0) << ";\n";
          break;
        default: entry(I, false); break;
      }
      o << "          if (live) x.fired |= " << bit << ";\n";
      o << "        }\n";
    }
    o << "        if (on) x.complete = all_in;\n";
    o << "      }\n    }\n";
  }

  // ---- the same tables for the depth-first lanes (lane_device.h) -------------------------------------
  // A lane's frame is in a state (function, calls opened), and a sweep ends
  // with the one thing the lane does next: a call all of whose arguments are live, the next iteration, the
  // return of a complete frame, or waiting.  What is present, and much of what is live, is known from the
  // state: the arguments of an opened call were live, so the Switches on their way went that side.  Every
  // reachable state gets code of its own with these facts folded in (fib's first sweep is a comparison,
  // its last one an addition); a lane whose sweep is a few instructions is what the machine's speed is.
  // Which opened calls are still outstanding is looked up in the frame: with a state for each such set tak has 32
  // and not 11 (and fib 12, not 6), of which a wave's lanes are in more at a time, each a turn of its own.
  // States beyond MAX_STATES (functions with many calls) run the generic code
  // of their function, which keeps the present and opened sets in registers.
  static constexpr int MAX_STATES = 24;
  struct State { int f; uint32_t mask; };
  std::vector<State> states;
  struct B {                      // a truth value: constant 0 / 1, or an expression
    int k;
    std::string e;
    bool has = false;             // in a loop's body: made of its predicates alone, `tt` is its truth table
    uint64_t tt = 0;
  };
  static B bc(bool v) { return B{v ? 1 : 0, v ? "true" : "false", true, v ? ~0ull : 0ull}; }
  static B bx(const std::string& e) { return B{2, e}; }
  // an expression with the table that its operands give it: one that is always or never true is a constant
  static B bt(const B& b, bool has, uint64_t tt) {
    if (!has) return b;
    return tt == 0 ? bc(false) : tt == ~0ull ? bc(true) : B{2, b.e, true, tt};
  }
  static B band(const B& a, const B& b) {
    if (a.k == 0 || b.k == 0) return bc(false);
    if (a.k == 1) return b;
    if (b.k == 1) return a;
    return bt(bx("(" + a.e + " && " + b.e + ")"), a.has && b.has, a.tt & b.tt);
  }
  static B bnot(const B& a) { return a.k == 2 ? bt(bx("!" + a.e), a.has, ~a.tt) : bc(!a.k); }
  static B bor(const B& a, const B& b) {
    if (a.k == 1 || b.k == 1) return bc(true);
    if (a.k == 0) return b;
    if (b.k == 0) return a;
    return bt(bx("(" + a.e + " || " + b.e + ")"), a.has && b.has, a.tt | b.tt);
  }
  // The predicates of a loop's body (loop_body below): value number and name; the table of the i-th.
  static constexpr int MAX_PREDICATES = 6;
  std::vector<std::pair<int, std::string>> predicates;
  bool loop_body = false;
  static uint64_t predicate_table(int i) {
    uint64_t t = 0;
    for (int r = 0; r < 64; ++r) t |= (uint64_t)((r >> i) & 1) << r;
    return t;
  }
  // `b` where `care` holds, as one predicate or its negation if it is one there
  B simplest(const B& b, const B& care) const {
    if (b.k != 2 || !b.has || !care.has) return b;
    if ((b.tt & care.tt) == care.tt) return bc(true);
    for (int i = 0; i < (int)predicates.size(); ++i) {
      const uint64_t t = predicate_table(i);
      if (((b.tt ^ t) & care.tt) == 0) return B{2, predicates[i].second, true, t};
      if (((b.tt ^ ~t) & care.tt) == 0) return B{2, "!" + predicates[i].second, true, ~t};
    }
    return b;
  }
  // What a state says about the values of its function.
  struct Facts {
    std::vector<int> live, truth;   // -1 unknown; live 1: present and not dead; truth of a predicate
    std::vector<int> def;           // instruction that makes the value
  };
  const Instr& at(int f, int ip) const { return P.instr[P.fn[f].first + ip]; }
  static bool has_value(uint8_t op) { return op != D_CALL && op != D_NEXT && op != D_OUT; }
  void mark_live(int f, Facts& F, int v) const {
    if (v >= SRC_NONE || F.live[v] == 1) return;
    F.live[v] = 1;
    const Instr& I = at(f, F.def[v]);
    switch (I.op) {
      case D_SWITCH:
        if (I.src[0] < SRC_NONE) F.truth[I.src[0]] = v == I.dst ? 1 : 0;
        mark_live(f, F, I.src[0]);
        mark_live(f, F, I.src[1]);
        break;
      case D_ADD: case D_SUB: case D_MUL: case D_EQ: case D_LT: case D_CE_NODE: case D_CELL: case D_HEAD:
        mark_live(f, F, I.src[0]);
        mark_live(f, F, I.src[1]);
        break;
      case D_ID: case D_ISLEAF: case D_LEFT: case D_RIGHT: case D_TOKEN: case D_EMBED:
        mark_live(f, F, I.src[0]);
        break;
      default: break;
    }
  }
  Facts facts(int f, uint32_t mask) const {
    Facts F;
    F.live.assign(MAX_VALUES + 2, -1);
    F.truth.assign(MAX_VALUES + 2, -1);
    F.def.assign(MAX_VALUES + 2, 0);
    for (int ip = 0; ip < P.fn[f].count; ++ip) {
      const Instr& I = at(f, ip);
      if (!has_value(I.op)) continue;
      F.def[I.dst] = ip;
      if (I.op == D_SWITCH) F.def[I.dst + 1] = ip;
    }
    for (int ip = 0; ip < P.fn[f].count; ++ip) {
      const Instr& I = at(f, ip);
      if (I.op == D_IN) F.live[I.dst] = 1;
      if (I.op == D_CALL && ((mask >> P.label_site[I.aux]) & 1)) mark_live(f, F, I.src[0]);
    }
    // forward: what is made of live values, and the side of a Switch that its known predicate names
    for (int ip = 0; ip < P.fn[f].count; ++ip) {
      const Instr& I = at(f, ip);
      auto lv = [&](int k) { return I.src[k] == SRC_IMM || (I.src[k] != SRC_NONE && F.live[I.src[k]] == 1); };
      switch (I.op) {
        case D_ADD: case D_SUB: case D_MUL: case D_EQ: case D_LT: if (lv(0) && lv(1)) F.live[I.dst] = 1; break;
        case D_ID: case D_ISLEAF: case D_LEFT: case D_RIGHT: case D_TOKEN: if (lv(0)) F.live[I.dst] = 1; break;
        case D_SWITCH:
          if (lv(1) && I.src[0] < SRC_NONE && F.truth[I.src[0]] >= 0) F.live[F.truth[I.src[0]] ? I.dst : I.dst + 1] = 1;
          break;
        default: break;
      }
    }
    return F;
  }
  struct Site { int label; std::vector<const Instr*> args; };   // label -1: the next iteration
  std::vector<Site> sites(int f) const {
    std::vector<Site> r;
    for (int ip = 0; ip < P.fn[f].count; ++ip) {
      const Instr& I = at(f, ip);
      if (I.op != D_CALL && I.op != D_NEXT) continue;
      const int label = I.op == D_CALL ? (int)I.aux : -1;
      size_t k = 0;
      while (k < r.size() && r[k].label != label) ++k;
      if (k == r.size()) r.push_back({label, {}});
      r[k].args.push_back(&I);
    }
    return r;
  }
  bool has_state(int f, uint32_t mask) const {
    for (const State& t : states)
      if (t.f == f && t.mask == mask) return true;
    return false;
  }
  // A state's number says what it is (LANE_ST in lane_device.h)
  static uint32_t state_code_of(int f, uint32_t mask, uint32_t out) { return (uint32_t)f | mask << 3 | out << 11; }
  // A value of the state's code: name, present, dead.
  struct Val { std::string v; B p, d; };
  // (the result of a call that was not opened is there only as a dead value: never live)
  static B live_of(const Val& a) { return a.p.k == 2 && a.p.e == a.d.e ? bc(false) : band(a.p, bnot(a.d)); }

  // A call that waits while another one runs: an argument that came from the forest is kept where its result
  // will be, so that it need not be read again.  That is sound for arguments that the first sweep decides (there, live or
  // dead, whatever the calls return): a call with such an argument that is live is ready in the first sweep, which ends
  // with it or with another call, and whoever calls keeps the arguments of the others.
  bool kept(int f, int v) {
    if (v >= SRC_NONE) return false;
    const uint8_t op = at(f, facts(f, 0).def[v]).op;
    return (op == D_LEFT || op == D_RIGHT || op == D_TOKEN) && decided(f, v);
  }
  // Whether the first sweep decides a value: it is there then, live or dead.
  bool decided(int f, int v) {
    std::vector<Val> V;
    B complete = bc(false);
    std::ostringstream sink;
    body(sink, State{f, 0}, "", "on", nullptr, V, complete, nullptr);
    return V[v].p.k == 1;
  }
  // The slot that holds value `v` in a state, or -1.
  int memo_slot(int f, uint32_t mask, int v) {
    if (mask == 0) return -1;
    for (const Site& t : sites(f))
      if (t.label >= 0 && !((mask >> P.label_site[t.label]) & 1) && t.args.size() == 1 && t.args[0]->src[0] == v)
        return kept(f, v) ? (int)P.label_ret_slot[t.label] : -1;
    return -1;
  }
  struct NodeAt {   // the node an inlined body looked at: index, suffix of its names, whether its entries were read
    std::string index, names;
    B loaded;
  };
  NodeAt node_at;
  // The entries of a state's code.  `q`: prefix of the names, `on`: which lanes, `ins`: the parameters of an
  // inlined callee (null: the lane's own frame).  Fills V and `complete`; clears *can where a callee cannot
  // be inlined.
  void body(std::ostringstream& c, const State& S, const std::string& q, const std::string& on, const std::vector<Val>* ins,
            std::vector<Val>& V, B& complete, bool* can) {
    body(c, S, q, on, ins, facts(S.f, S.mask), V, complete, can);
  }
  void body(std::ostringstream& c, const State& S, const std::string& q, const std::string& on, const std::vector<Val>* ins, const Facts& F,
            std::vector<Val>& V, B& complete, bool* can) {
    const int f = S.f;
    const DevFn& fn = P.fn[f];
    V.assign(MAX_VALUES + 2, Val{"0ll", bc(false), bc(false)});
    std::vector<int> alias(MAX_VALUES + 2, -1);   // the value it hands on
    std::map<int, B> node_loaded;   // by node: under which condition its entries have been read
    auto root = [&](int v) { while (v < SRC_NONE && alias[v] >= 0) v = alias[v]; return v; };
    auto src = [&](const Instr& I, int k) { return source(V, I, k); };
    auto name_b = [&](const std::string& nm, const B& b) { return named(c, q + nm, b); };
    auto put = [&](int dst, const std::string& expr, B p, B d) {
      const std::string D = std::to_string(dst);
      if (F.live[dst] == 1) { p = bc(true); d = bc(false); }
      c << "        const long long " << q << "v" << D << " = " << (expr.empty() ? "0" : expr) << ";\n";
      V[dst] = Val{q + "v" + D, name_b("p" + D, p), name_b("d" + D, band(p, d))};
    };
    complete = S.mask ? named(c, q + "back", bx("x.st < 2048u")) : bc(true);   // (nothing outstanding)
    for (int ip = 0; ip < fn.count; ++ip) {
      const Instr& I = at(f, ip);
      const std::string D = std::to_string(I.dst);
      switch (I.op) {
        case D_IN:
          if (ins) V[I.dst] = (*ins)[I.aux];
          else put(I.dst, "x.sv[" + std::to_string(I.aux) + "]", bc(true), bc(false));
          break;
        case D_RET: {
          const uint32_t bit = 1u << P.label_site[I.aux2];
          if (S.mask & bit) {
            c << "        const long long " << q << "v" << D << " = x.sv[" << (int)I.aux << "];\n";
            const B back = F.live[I.dst] == 1 ? bc(true) : name_b("p" + D, bx("!(x.st & " + std::to_string(bit << 11) + "u)"));
            V[I.dst] = Val{q + "v" + D, back, bc(false)};
          } else {
            B all_p = bc(true), any_d = bc(false), any_arg = bc(false);
            for (int k = 0; k < 4; ++k) {
              if (I.src[k] == SRC_NONE) continue;
              any_arg = bc(true);
              all_p = band(all_p, src(I, k).p);
              any_d = bor(any_d, src(I, k).d);
            }
            const B dead = name_b("r" + D, band(any_arg, band(all_p, any_d)));
            V[I.dst] = Val{"0ll", dead, dead};
            complete = band(complete, dead);
          }
          break;
        }
        case D_ADD: case D_SUB: case D_MUL: case D_EQ: case D_LT: {
          const Val a = src(I, 0), b = src(I, 1);
          std::string e;
          if (I.op == D_EQ || I.op == D_LT) e = "(" + a.v + (I.op == D_EQ ? " == " : " < ") + b.v + ")";
          else e = "(long long)((unsigned long long)" + a.v + (I.op == D_ADD ? " + " : I.op == D_SUB ? " - " : " * ") + "(unsigned long long)" + b.v + ")";
          put(I.dst, e, band(a.p, b.p), bor(a.d, b.d));
          break;
        }
        case D_ID: {
          const Val a = src(I, 0);
          if (I.src[0] < SRC_NONE) alias[I.dst] = I.src[0];
          put(I.dst, a.v, a.p, a.d);
          break;
        }
        case D_SWITCH: {
          const Val pr = src(I, 0), da = src(I, 1);
          const B p = name_b("q" + D, band(pr.p, da.p)), d = name_b("e" + D, bor(pr.d, da.d));
          const int known = I.src[0] < SRC_NONE ? F.truth[I.src[0]] : (I.imm != 0 ? 1 : 0);
          B t = bc(known > 0);
          if (known < 0) {
            const int r = I.src[0] < SRC_NONE ? root(I.src[0]) : -1;
            size_t k = 0;
            while (k < predicates.size() && predicates[k].first != r) ++k;
            if (!loop_body || r < 0 || k >= MAX_PREDICATES) {
              t = name_b("t" + D, bx("(" + pr.v + " != 0)"));
            } else {
              if (k == predicates.size()) predicates.push_back({r, name_b("t" + D, bx("(" + pr.v + " != 0)")).e});
              t = B{2, predicates[k].second, true, predicate_table((int)k)};
            }
          }
          if (I.src[1] < SRC_NONE) alias[I.dst] = alias[I.dst + 1] = I.src[1];
          put(I.dst, da.v, p, bor(d, bnot(t)));
          put(I.dst + 1, da.v, p, bor(d, t));
          break;
        }
        case D_MERGE: {
          B any_live = bc(false), all_p = bc(true);
          std::string e = "0ll";
          for (int k = 3; k >= 0; --k)
            if (I.src[k] != SRC_NONE) any_live = bor(live_of(src(I, k)), any_live);
          for (int k = 3; k >= 0; --k) {
            if (I.src[k] == SRC_NONE) continue;
            const Val a = src(I, k);
            B l = live_of(a);
            if (loop_body) {   // nobody looks at the value where it is dead, nor at this source where an earlier one is live
              B care = any_live;
              for (int j = 0; j < k; ++j)
                if (I.src[j] != SRC_NONE) care = band(care, bnot(live_of(src(I, j))));
              l = simplest(l, care);
            }
            all_p = band(a.p, all_p);
            if (l.k == 1) e = a.v;
            else if (l.k == 2) e = "(" + l.e + " ? " + a.v + " : " + e + ")";
          }
          const B al = name_b("m" + D, any_live);
          put(I.dst, e, bor(al, all_p), bnot(al));
          break;
        }
        case D_ISLEAF: case D_LEFT: case D_RIGHT: case D_TOKEN: {
          const Val a = src(I, 0);
          const B lv = live_of(a);
          const int r = I.src[0] < SRC_NONE ? root(I.src[0]) : 256 + ip;   // (an immediate: a node of its own)
          const std::string R = q + std::to_string(r);
          if (S.mask == 0) {   // first sweep: the node's entries in one round trip, index checked
            // (once for all accessors of the node, but each under its own condition: the first may be dead)
            const bool first = !node_loaded.count(r);
            B& loaded = node_loaded.emplace(r, bc(false)).first->second;
            if (first) c << "        int " << "nl" << R << " = x.pf_l, nr" << R << " = x.pf_r, nt" << R << " = x.pf_t;\n";
            const B load = loaded.k == 2 && loaded.e == lv.e ? bc(false) : band(lv, bnot(loaded));
            if (load.k) {
              c << "        if (" << on << " && " << load.e << (ins ? "" : " && (x.pf_v != " + a.v + " || " + a.v + " < 0)") << ") ln_node(x, " << a.v << ", nl" << R << ", nr" << R << ", nt" << R
                << ");\n";
              loaded = named(c, q + "n" + D, bor(loaded, lv));
              if (ins) node_at = NodeAt{a.v, R, loaded};
            }
            const char* which = I.op == D_RIGHT ? "nr" : I.op == D_TOKEN ? "nt" : "nl";
            put(I.dst, std::string("(long long)") + (I.op == D_ISLEAF ? "(nl" + R + " < 0)" : which + R), a.p, a.d);
          } else {
            // The node may be a value that a call has just returned, which nobody has looked at yet.  Where the first
            // sweep has, a bad index is known and this sweep's values do not count; only the read itself is checked,
            // so that the compiler can leave it out where nobody needs it.
            const int memo = memo_slot(f, S.mask, I.dst);
            std::string e = memo >= 0 ? "x.sv[" + std::to_string(memo) + "]" : lv.k == 0 ? "0ll" :
                            "(" + on + " && " + lv.e + " ? " + (decided(f, I.dst) ? "ln_entry_again" : "ln_entry") + "(x, " + a.v + ", " +
                            std::to_string(std::max<int>(I.op, D_LEFT) - D_ISLEAF) + ") : 0ll)";
            if (I.op == D_ISLEAF) e = F.truth[I.dst] >= 0 ? std::to_string(F.truth[I.dst]) + "ll" : "(" + e + " < 0)";
            put(I.dst, "(long long)" + e, a.p, a.d);
          }
          break;
        }
        case D_EMBED: case D_CELL: case D_HEAD: {
          const Val a = src(I, 0), b = I.op == D_EMBED ? Val{"0", bc(true), bc(false)} : src(I, 1);
          const B in = band(live_of(a), live_of(b));
          if (in.k == 0) {   // dead or absent now, so it was in every earlier state
            V[I.dst] = Val{"0ll", bc(false), bc(false)};
            break;
          }
          c << "        long long " << q << "v" << D << " = 0; bool " << q << "pp" << D << " = false, " << q << "ll" << D << " = false;\n";
          if (ins && I.op != D_EMBED) {   // (its place in the log would need a frame)
            *can = false;
            break;
          }
          if (ins) {   // an inlined callee has no stored values: its EMBED fires here and only here (see can_inline)
            c << "        ln_embed_now(x, " << on << " && " << in.e << ", " << a.v << ", " << q << "v" << D << ", " << q << "pp" << D << ");\n";
            V[I.dst] = Val{q + "v" + D, in.k == 1 ? bc(true) : in, bc(false)};
            break;
          }
          // fires when its inputs are live; a later state may find it fired already
          c << "        " << (I.op == D_EMBED ? "ln_embed" : I.op == D_CELL ? "ln_cell" : "ln_head") << "(x, " << on << ", " << (int)I.aux << ", "
            << a.p.e << ", " << a.d.e << ", " << a.v;
          if (I.op != D_EMBED) c << ", " << b.p.e << ", " << b.d.e << ", " << b.v;
          c << ", v" << D << ", pp" << D << ", ll" << D << ");\n";
          V[I.dst] = Val{"v" + D, in.k == 1 ? bc(true) : bx("pp" + D), bc(false)};
          break;
        }
        case D_CE_NODE: {
          const Val a = src(I, 0), b = src(I, 1);
          const B lv = band(live_of(a), live_of(b));
          if (lv.k != 0)
            c << "        if (" << on << " && " << lv.e << ") { bool dd = false; ln_ce_node(x, " << a.v << ", " << b.v << ", dd); }\n";
          put(I.dst, a.v, band(a.p, b.p), bor(a.d, b.d));
          break;
        }
        default: break;   // calls and the output: state_code
      }
    }
  }
  static B named(std::ostringstream& c, const std::string& nm, const B& b) {
    if (b.k != 2) return b;
    c << "        const bool " << nm << " = " << b.e << ";\n";
    return B{2, nm, b.has, b.tt};
  }
  static Val source(const std::vector<Val>& V, const Instr& I, int k) {
    if (I.src[k] == SRC_IMM) return Val{"(long long)" + std::to_string((unsigned long long)I.imm) + "ULL", bc(true), bc(false)};
    return V[I.src[k]];
  }
  const Instr& out_entry(int f) const {
    int k = 0;
    for (int ip = 0; ip < P.fn[f].count; ++ip)
      if (at(f, ip).op == D_OUT) k = ip;
    return at(f, k);
  }
  // Whether the first sweep of a callee is all there is to it: everything is there, nothing is left to call.
  B whole_callee(int f, const std::vector<Val>& W, const B& complete) const {
    B partly = bc(false);
    for (const Site& u : sites(f))
      for (const Instr* I : u.args) partly = bor(partly, live_of(source(W, *I, 0)));
    return band(band(complete, bnot(partly)), live_of(source(W, out_entry(f), 0)));
  }
  // A callee whose first sweep may be all there is (a base case) is tried in the caller's sweep: no frame
  // is pushed for it then.  Not where the body has operators with a stored value other than EMBED, and not where an
  // EMBED can fire although the callee turns out to need a frame, in which it would fire again.
  bool can_inline(int f) {
    if (f == P.result_fn) return false;
    for (int ip = 0; ip < P.fn[f].count; ++ip) {
      const Instr& I = at(f, ip);
      if (I.op == D_HEAD || I.op == D_NEXT) return false;
      if (I.op != D_EMBED) continue;
      Facts F = facts(f, 0);
      mark_live(f, F, I.dst);
      const std::vector<Val> ins(P.fn[f].n_params, Val{"0ll", bc(true), bc(false)});
      std::vector<Val> W;
      B complete = bc(false);
      bool can = true;
      std::ostringstream sink;
      body(sink, State{f, 0}, "", "on", &ins, F, W, complete, &can);
      if (whole_callee(f, W, complete).k != 1) return false;
    }
    return true;
  }
  // A loop graph without calls runs its iterations in the sweep (bounded; the iterations are tags like any).
  bool tight_loop(int f) const {
    bool next = false;
    for (int ip = 0; ip < P.fn[f].count; ++ip) {
      const uint8_t op = at(f, ip).op;
      if (op == D_CALL || op == D_EMBED || op == D_CELL || op == D_HEAD || op == D_CE_NODE || (op >= D_ISLEAF && op <= D_TOKEN)) return false;
      next = next || op == D_NEXT;
    }
    return next;
  }

  // Code of one state; `next` receives the sets of opened calls it can go to.  With emit false only `next`.
  void state_code(const State& S, std::vector<int>& next, bool emit) {
    const int f = S.f;
    std::ostringstream c;
    std::vector<Val> V;
    B complete = bc(false);
    const bool loop = tight_loop(f);
    body(c, S, "", "on", nullptr, V, complete, nullptr);
    auto src = [&](const Instr& I, int k) { return source(V, I, k); };
    // a frame's own next state, with what is outstanding as it is; a callee's first one
    auto state_name = [&](uint32_t m) {
      return S.mask ? "(x.st | " + std::to_string((m & ~S.mask) << 3) + "u)" : std::to_string(state_code_of(f, m, 0)) + "u";
    };
    auto first_state = [](int sf) { return std::to_string(state_code_of(sf, 0, 0)) + "u"; };
    // ---- what the lane does next
    const std::vector<Site> ss = sites(f);
    std::string chain, nx;
    B part = bc(false), taken = bc(false);
    std::string count = "0";
    int n_count = 0, n_chain = 0;
    // Calls that are ready, in table order.  Each is first tried in place; what is left over is called, the
    // first one now.  A call is tried in the first state it can be ready in only: it will not have changed.
    struct Ready { const Site* t; uint32_t bit; int callee, slot; std::string tag, args, done, value, node; B all; };
    std::vector<Ready> rs;
    std::vector<Val> V0;
    B c0 = bc(false);
    if (S.mask) {
      std::ostringstream sink;
      body(sink, State{f, 0}, "", "on", nullptr, V0, c0, nullptr);
    }
    for (const Site& t : ss) {
      const uint32_t bit = t.label >= 0 ? 1u << P.label_site[t.label] : 0u;
      if (S.mask & bit) continue;
      B all = bc(true), any = bc(false), before = bc(true);
      const int callee = t.label >= 0 ? P.label_callee[t.label] : f, np = P.fn[callee].n_params;
      for (const Instr* I : t.args) {
        const B l = live_of(src(*I, 0));
        all = band(all, l);
        any = bor(any, l);
        if (S.mask) before = band(before, live_of(source(V0, *I, 0)));
      }
      if ((int)t.args.size() != np) all = bc(false);
      const std::string tag = t.label >= 0 ? std::to_string(P.label_site[t.label]) : "n";
      all = named(c, "all" + tag, all);
      part = bor(part, band(any, bnot(all)));
      std::string args;
      for (const Instr* I : t.args) args += " x.arg[" + std::to_string((int)I->aux2) + "] = " + src(*I, 0).v + ";";
      args += " x.c_np = " + std::to_string(np) + "u;";
      if (t.label < 0) {
        if (loop && all.k) {
          nx = "if (" + all.e + ") {}   // on in the next sweep\n          else ";
        } else if (all.k) {
          nx = "if (" + all.e + ") { x.act = ACT_NEXT;" + args + " x.c_st = " + first_state(f) + "; }\n          else ";
        }
        continue;
      }
      if (all.k == 0) continue;
      Ready r{&t, bit, callee, (int)P.label_ret_slot[t.label], tag, args, "", "", "", all};
      const bool first_time = S.mask == 0 || before.k == 0;
      int inlined = 0;
      for (const Ready& o2 : rs) inlined += !o2.done.empty();
      if (first_time && inlined < 3 && can_inline(callee)) {
        const std::string q = "c" + tag + "_", con = "(on && " + all.e + ")";
        std::vector<Val> ins((size_t)np, Val{"0ll", bc(true), bc(false)}), W;
        for (const Instr* I : t.args) ins[I->aux2] = Val{src(*I, 0).v, bc(true), bc(false)};
        B complete0 = bc(false);
        std::ostringstream ic;
        bool can = true;
        node_at = NodeAt{"", "", bc(false)};
        body(ic, State{callee, 0}, q, con, &ins, W, complete0, &can);
        const Val ov = source(W, out_entry(callee), 0);
        const B done = whole_callee(callee, W, complete0);
        if (can && done.k != 0) {
          c << ic.str();
          r.done = named(c, "done" + tag, band(bx("(" + all.e + ")"), done)).e;
          r.value = ov.v;
          if (node_at.loaded.k)
            r.node = (node_at.loaded.k == 1 ? "" : " if (" + node_at.loaded.e + ") {") + std::string(" x.pf_v = ") + node_at.index + "; x.pf_l = nl" + node_at.names +
                     "; x.pf_r = nr" + node_at.names + "; x.pf_t = nt" + node_at.names + ";" + (node_at.loaded.k == 1 ? "" : " }");
        }
      }
      rs.push_back(r);
    }
    // Sets of calls done in place, each a state to go on from
    std::vector<uint32_t> sets(1, 0u);
    for (const Ready& r : rs)
      if (!r.done.empty())
        for (size_t k = 0, n = sets.size(); k < n; ++k) sets.push_back(sets[k] | r.bit);
    // the state once call `bit` (0: none) is back, by what was done in place (om: all calls opened)
    const bool in_place = sets.size() > 1;
    auto state_after = [&](uint32_t bit) {
      if (!in_place) return state_name(S.mask | bit);
      return "(x.st | " + (bit ? "(om | " + std::to_string(bit) + "u)" : std::string("om")) + " << 3)";
    };
    auto note = [&](uint32_t m) {
      if (m != S.mask) next.push_back((int)m);
    };
    std::string om = std::to_string(S.mask) + "u", put;
    for (const Ready& r : rs) {
      if (r.done.empty()) continue;
      om += " | (" + r.done + " ? " + std::to_string(r.bit) + "u : 0u)";
      put += "          if (" + r.done + ") { x.sv[" + std::to_string(r.slot) + "] = " + r.value + "; x.present |= " + std::to_string(1u << r.slot) +
             "u; ++x.n_tags; x.n_tokens += " + std::to_string(P.fn[r.callee].n_params + 1) + "u; }\n";
    }
    if (in_place) put += "          x.mx_depth = max(x.mx_depth, x.depth + (om != " + std::to_string(S.mask) + "u ? 1u : 0u));\n";
    for (uint32_t d : sets) note(S.mask | d);
    for (size_t k = 0; k < rs.size(); ++k) {
      const Ready& r = rs[k];
      count += " + (int)" + (r.done.empty() ? r.all.e : "(" + r.all.e + " && !" + r.done + ")");
      ++n_count;
      // could an earlier ready call always be there when this one is?  Then it is never the one chosen.
      bool never = taken.k == 1;
      for (const Ready& u : rs) {
        if (never || &u == &r) break;
        if (!u.done.empty()) continue;
        const Facts G = facts(f, S.mask | r.bit);
        bool sure = (int)u.t->args.size() == (int)P.fn[u.callee].n_params;
        for (const Instr* I : u.t->args) sure = sure && (I->src[0] >= SRC_NONE || (G.live[I->src[0]] == 1 && src(*I, 0).p.k == 1));
        never = sure;
      }
      if (never) continue;
      for (uint32_t d : sets)
        if (!(d & r.bit)) note(S.mask | r.bit | d);
      const std::string go = r.done.empty() ? r.all.e : "(" + r.all.e + " && !" + r.done + ")";
      std::string keep;   // arguments of calls that wait, kept in the place of their results
      for (const Ready& u : rs)
        if (&u != &r && u.t->args.size() == 1 && kept(f, u.t->args[0]->src[0]))
          keep += (u.done.empty() ? "" : " if (!" + u.done + ")") + std::string(" x.sv[") + std::to_string(u.slot) + "] = " + src(*u.t->args[0], 0).v + ";";
      chain += std::string(n_chain++ ? "          else " : "          ") + "if (" + go + ") { x.act = ACT_CALL; x.c_st = " + first_state(r.callee) + "; x.c_back = " +
               state_after(r.bit) + " | " + std::to_string((unsigned)r.slot << 20) + "u; x.c_label = " + std::to_string(r.t->label) + "u;" + r.args + r.node + keep + " }\n";
      taken = bor(taken, r.done.empty() ? r.all : bx(go));
    }
    if (in_place)
      chain += std::string(n_chain++ ? "          else " : "          ") + "if (om != " + std::to_string(S.mask) + "u) { x.st = " + state_after(0) + "; }\n";
    if (!emit) return;
    const Instr& oe = out_entry(f);
    const Val ov = src(oe, 0);
    const B ol = live_of(ov);
    c << "        if (on) {\n";
    if (n_count > 1) c << "          x.more = (" << count << ") > 1;\n";
    else c << "          x.more = false;\n";
    c << "          const uint32_t om = " << om << ";\n          (void)om;\n" << put;
    c << chain;
    c << "          " << (n_chain ? "else " : "");
    if (part.k) c << "if (" << part.e << ") x.act = " << (complete.k == 0 ? "ACT_WAIT" : "(" + complete.e + ") ? ACT_STUCK : ACT_WAIT") << ";\n          else ";
    if (complete.k != 1) c << "if (!" << complete.e << ") x.act = ACT_WAIT;\n          else ";
    c << nx;
    if (f == P.result_fn) {
      c << "{ ";
      if (ol.k) c << "if (" << ol.e << ") ln_result(x, " << (int)oe.aux << ", " << ov.v << "); ";
      c << "x.act = ACT_DONE; }\n";
    } else {
      if (ol.k) c << "if (" << ol.e << ") { x.act = ACT_RET; x.ret = " << ov.v << "; }\n          else ";
      c << "x.act = ACT_STUCK;\n";
    }
    c << "        }\n";
    const std::string code = std::to_string(state_code_of(f, S.mask, 0));
    o << "    {  // function " << f << ", opened " << S.mask << "\n";
    o << "      const bool on = x.run && (x.st & 2047u) == " << code << "u;\n      if (__ballot(on)) {\n";
    if (loop) iterations(f);
    o << c.str();
    if (unlisted) o << "        known = known || (on && (x.act != ACT_NONE || (x.st & 2047u) == " << code << "u));\n";
    o << "      }\n    }\n";
  }
  // The iterations of a sweep, before it looks at what the lane does next.  What bounds them is the instructions of one
  // iteration (a wave has its SIMD nearly to itself), so they are a straight run of arithmetic: every lane computes, one
  // that has left its loop keeps its variables, and the wave looks up every fourth time whether anybody goes on.  Which
  // entries are live is a function of the loop's predicates; with truth tables of up to six of them most of it comes out
  // constant, a Merge is one choice, and going on one predicate.  An iteration of subtractive gcd is 17 instructions; with
  // a way out of the loop in every iteration and the presence of every entry looked at it was 50 and 168 clocks, and
  // 65,536 pairs up to 1,024 took 136 us, not 96 (both with 64 iterations a sweep).
  void iterations(int f) {
    const int nv = P.fn[f].n_params;
    std::vector<Val> ins, V;
    for (int k = 0; k < nv; ++k) ins.push_back(Val{"u" + std::to_string(k), bc(true), bc(false)});
    B complete = bc(false), all = bc(true);
    bool can = true;
    std::ostringstream c;
    predicates.clear();
    loop_body = true;
    body(c, State{f, 0}, "i", "on", &ins, V, complete, &can);
    std::string next;
    int n_args = 0;
    for (const Site& t : sites(f))
      for (const Instr* I : t.args) {
        const Val a = source(V, *I, 0);
        all = band(all, live_of(a));
        ++n_args;
        next += "        const long long w" + std::to_string((int)I->aux2) + " = " + a.v + ";\n";
      }
    all = simplest(all, bc(true));
    loop_body = false;
    if (n_args != nv || all.k == 0) return;   // no iteration has a next one
    o << "        uint32_t n_it = 0;\n";
    for (int k = 0; k < nv; ++k) o << "        long long u" << k << " = x.sv[" << k << "];\n";
    o << "        const uint32_t share = __ballot(x.run && !on) ? LANE_LOOP_BESIDE : LANE_LOOP;\n";
    o << "        for (uint32_t k = 0; k < share / 4; ++k) {\n        bool any = false;\n#pragma unroll\n        for (int h = 0; h < 4; ++h) {\n"
      << c.str() << next << "        any = on && " << all.e << ";\n";
    for (int k = 0; k < nv; ++k) o << "        u" << k << " = any ? w" << k << " : u" << k << ";\n";
    o << "        n_it += any ? 1u : 0u;\n        }\n        if (__ballot(any) == 0) break;\n        }\n        if (on) {\n";
    for (int k = 0; k < nv; ++k) o << "          x.sv[" << k << "] = u" << k << ";\n";
    o << "          ln_loop(x, n_it, " << nv << "u);\n        }\n";
  }

  bool unlisted = false;   // whether there may be states without code of their own
  void find_states() {
    states.clear();
    for (int f = 0; f < P.n_fn; ++f) states.push_back({f, 0});
    unlisted = false;
    for (size_t k = 0; k < states.size(); ++k) {
      const State S = states[k];
      std::vector<int> nx;
      state_code(S, nx, false);
      for (int mask : nx) {
        if (has_state(S.f, (uint32_t)mask)) continue;
        if ((int)states.size() < MAX_STATES) states.push_back({S.f, (uint32_t)mask});
        else unlisted = true;
      }
    }
    // (a frame whose call was evaluated in place goes on in a later state, with more calls opened)
    std::sort(states.begin(), states.end(), [](const State& a, const State& b) { return a.f != b.f ? a.f < b.f : a.mask < b.mask; });
  }
  // The generic code of a function: present and opened sets from registers.
  void lane_function(int f) {
    const DevFn& fn = P.fn[f];
    o << "        case " << f << "u: {  // function " << f << ", generic\n";
    for (int v = 0; v < fn.n_values; ++v)
      o << "        long long v" << v << " = 0; bool p" << v << " = false, d" << v << " = false;\n";
    o << "        bool live = false, all_in = true;\n";
    std::vector<std::pair<int, std::vector<const Instr*>>> calls;   // by label, in table order; -1: the next iteration
    const Instr* out_entry = nullptr;
    for (int ip = 0; ip < fn.count; ++ip) {
      const Instr& I = P.instr[fn.first + ip];
      if (I.op == D_CALL || I.op == D_NEXT) {
        const int label = I.op == D_CALL ? (int)I.aux : -1;
        size_t k = 0;
        while (k < calls.size() && calls[k].first != label) ++k;
        if (k == calls.size()) calls.push_back({label, {}});
        calls[k].second.push_back(&I);
        continue;
      }
      if (I.op == D_OUT) {
        out_entry = &I;
        continue;
      }
      entry(I, true);
    }
    // calls: ready with every argument live; partly live is a case for the step machine
    int n_ready = 0;
    std::string chain, count = "0", part = "false", next;
    for (auto& c : calls) {
      std::string all = "true", any = "false";
      for (const Instr* I : c.second) {
        const std::string lv = "(" + pre(*I, 0) + " && !" + ded(*I, 0) + ")";
        all += " && " + lv;
        any += " || " + lv;
      }
      const int callee = c.first >= 0 ? P.label_callee[c.first] : f, np = P.fn[callee].n_params;
      const std::string id = c.first >= 0 ? std::to_string(P.label_site[c.first]) : "n";
      const std::string open = c.first >= 0 ? "!((s >> (3 + " + id + ")) & 1u) && " : "";
      o << "        const bool all" << id << " = on && " << open << "(" << all << ") && " << ((int)c.second.size() == np ? "true" : "false")
        << ";\n";
      o << "        const bool part" << id << " = on && " << open << "!all" << id << " && (" << any << ");\n";
      part += " || part" + id;
      std::string args;
      for (const Instr* I : c.second) args += " x.arg[" + std::to_string((int)I->aux2) + "] = " + val(*I, 0) + ";";
      args += " x.c_np = " + std::to_string(np) + "u;";
      if (c.first < 0) {
        next = "if (alln) { x.act = ACT_NEXT;" + args + " x.c_st = " + std::to_string(state_code_of(f, 0, 0)) + "u; }\n          else ";
        continue;
      }
      chain += std::string(n_ready++ ? "        else " : "        ") + "if (all" + id + ") { x.act = ACT_CALL; x.c_st = " +
               std::to_string(state_code_of(callee, 0, 0)) + "u; x.c_back = (s | 1u << (3 + " + id + ")) | " +
               std::to_string((unsigned)P.label_ret_slot[c.first] << 20) + "u; x.c_label = " + std::to_string(c.first) + "u;" + args + " }\n";
      count += " + (int)all" + id;
    }
    o << chain;
    if (n_ready) o << "        if (on) x.more = (" << count << ") > 1;\n";
    o << "        if (on && x.act == ACT_NONE) {\n";
    o << "          if (" << part << ") x.act = all_in ? ACT_STUCK : ACT_WAIT;\n";
    o << "          else if (!all_in) x.act = ACT_WAIT;\n          else ";
    o << next;
    const std::string olive = "(" + pre(*out_entry, 0) + " && !" + ded(*out_entry, 0) + ")";
    if (f == P.result_fn)
      o << "{ if (" << olive << ") ln_result(x, " << (int)out_entry->aux << ", " << val(*out_entry, 0) << "); x.act = ACT_DONE; }\n";
    else
      o << "if (" << olive << ") { x.act = ACT_RET; x.ret = " << val(*out_entry, 0) << "; }\n          else x.act = ACT_STUCK;\n";
    o << "        }\n";
    o << "        (void)live;\n      break; }\n";
  }

  // Place of call 0's result if call k's is k places further for all calls of the function, -1 if not, -2: no calls.
  int ret_base(int f) const {
    int base = -2;
    for (const Site& t : sites(f)) {
      if (t.label < 0) continue;
      const int b = (int)P.label_ret_slot[t.label] - (int)P.label_site[t.label];
      if (base == -2) base = b;
      else if (base != b) base = -1;
      if (b < 0) return -1;
    }
    return base;
  }
  std::string lane_source() {
    int ns = 1;
    for (int f = 0; f < P.n_fn; ++f) ns = std::max<int>(ns, P.fn[f].n_stored);
    find_states();
    o << "#include \"lane_device.h\"\n";
    o << "namespace tdf {\n";
    o << "struct GeneratedLanes {\n";
    o << "  static constexpr int kStored = " << ns << ";\n  static constexpr uint32_t kResultFn = " << P.result_fn << "u;\n";
    // Return_i of label i: the caller's stored value
    o << "  static __device__ __forceinline__ uint32_t ret_slot(uint32_t label) {\n    switch (label) {\n";
    for (int l = 0; l < P.n_labels; ++l) o << "      case " << l << ": return " << (int)P.label_ret_slot[l] << "u;\n";
    o << "      default: return 0u;\n    }\n  }\n";
    o << "  static constexpr bool kBranching = " << (lane_branching(P) ? "true" : "false") << ";\n";
    // stored values that the opened calls of a frame return into, and the calls whose value is not there yet: a
    // function's results have consecutive places, in the order of its calls, wherever the table puts them so
    o << "  static __device__ __forceinline__ uint32_t ret_bits(uint32_t fn, uint32_t opened) {\n    uint32_t r = 0;\n";
    for (int f = 0; f < P.n_fn; ++f) {
      const int base = ret_base(f);
      if (base >= 0) o << "    if (fn == " << f << "u) r = opened << " << base << ";\n";
      for (const Site& t : sites(f))
        if (base == -1 && t.label >= 0)
          o << "    if (fn == " << f << "u && ((opened >> " << (int)P.label_site[t.label] << ") & 1u)) r |= 1u << " << (int)P.label_ret_slot[t.label] << ";\n";
    }
    o << "    return r;\n  }\n";
    o << "  static __device__ __forceinline__ uint32_t outstanding(uint32_t fn, uint32_t opened, uint32_t present) {\n    uint32_t r = 0;\n";
    for (int f = 0; f < P.n_fn; ++f) {
      const int base = ret_base(f);
      if (base >= 0) o << "    if (fn == " << f << "u) r = opened & ~(present >> " << base << ");\n";
      for (const Site& t : sites(f))
        if (base == -1 && t.label >= 0)
          o << "    if (fn == " << f << "u && ((opened >> " << (int)P.label_site[t.label] << ") & 1u) && !((present >> "
            << (int)P.label_ret_slot[t.label] << ") & 1u)) r |= 1u << " << (int)P.label_site[t.label] << ";\n";
    }
    o << "    return r;\n  }\n";
    o << "  static __device__ __forceinline__ void sweep(LaneX& x) {\n";
    // One state after the other, those that some lane is in.  A lane whose call was evaluated in place is in a later state
    // then and comes up again.  A sweep is bound by the instructions of the states its lanes are in.  A loop that takes the
    // next lane's state and switches to its code, with a state for each set of outstanding calls, cost 20 copies of the
    // lane's registers a turn and a tree of branches: 1,950 clocks a sweep for fib, 2,800 for tak.  fib(30..32) takes 3,230 us
    // now, not 4,090; 256 of tak 1,695, not 2,360; fib(0..20) 165, not 189; eight small ones 70, not 77.
    if (unlisted) o << "    bool known = false;\n";
    for (const State& t : states) {
      std::vector<int> nx;
      state_code(t, nx, true);
    }
    if (unlisted) {
      o << "    unsigned long long todo = __ballot(x.run && !known);\n";
      o << "    while (todo) {\n";
      o << "      const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)x.st, __ffsll((long long)todo) - 1);\n";
      o << "      const bool on = ((todo >> lane_id()) & 1ull) && x.st == s;\n";
      o << "      switch (s & 7u) {\n";
      for (int f = 0; f < P.n_fn; ++f) lane_function(f);
      o << "        default: if (on) x.act = ACT_STUCK; break;\n      }\n";
      o << "      todo &= __ballot(!on);\n    }\n";
    }
    o << "  }\n};\n}  // namespace tdf\n";
    o << "extern \"C\" __global__ void __launch_bounds__(64, 2) tdf_generated_lanes(tdf::LaneArgs a) {\n";
    o << "  extern __shared__ __attribute__((aligned(16))) char lds[];\n";
    o << "  tdf::lanes_run<tdf::GeneratedLanes>(a, lds);\n}\n";
    return o.str();
  }

  std::string source() {
    o << "#include \"step_device.h\"\n";
    o << "namespace tdf {\n";
    o << "struct GeneratedSweep {\n";
    o << "  static constexpr bool kLdsValues = false;\n";
    o << "  static __device__ void run(LaneCtx& x, const DevProgram& P) {\n";
    o << "    (void)P;\n";
    for (int f = 0; f < P.n_fn; ++f) function(f);
    o << "  }\n};\n}  // namespace tdf\n";
    o << "extern \"C\" __global__ void __launch_bounds__(256) tdf_generated_step(tdf::Engine e, int max_steps, long long spin_ticks) {\n";
    o << "  extern __shared__ __attribute__((aligned(16))) char lds[];\n";
    o << "  __shared__ tdf::DevProgram P;\n  __shared__ uint32_t sh[4];\n";
    o << "  tdf::steps_grid<false, tdf::GeneratedSweep>(e, max_steps, spin_ticks, lds, &P, sh);\n}\n";
    o << "extern \"C\" __global__ void __launch_bounds__(tdf::GEN_LOCAL_BLOCK) tdf_generated_step_local(tdf::Engine e, int max_steps, long long spin_ticks) {\n";
    o << "  extern __shared__ __attribute__((aligned(16))) char lds[];\n";
    o << "  __shared__ tdf::DevProgram P;\n  __shared__ uint32_t sh[4];\n";
    o << "  tdf::steps_grid<true, tdf::GeneratedSweep>(e, max_steps, spin_ticks, lds, &P, sh);\n}\n";
    o << "extern \"C\" __global__ void __launch_bounds__(tdf::GEN_SMALL_BLOCK) tdf_generated_small(tdf::Engine e, int max_steps) {\n";
    o << "  extern __shared__ __attribute__((aligned(16))) char lds[];\n";
    o << "  __shared__ tdf::DevProgram P;\n  __shared__ tdf::Ctrl lc;\n";
    o << "  tdf::steps_small<tdf::GeneratedSweep>(e, max_steps, lds, &P, &lc);\n}\n";
    return o.str();
  }
};

// compiled code objects by firing-table contents: graphs with equal programs share the compile
struct CacheEntry {
  std::vector<char> code;
};
std::mutex g_cache_mutex;
std::map<std::string, CacheEntry> g_cache;

}  // namespace

// Code object of the generated kernels for `arch`, compiled once per (arch, firing tables).
static bool jit_code(const DevProgram& P, const std::string& arch, bool lanes, std::vector<char>& code, std::string& log) {
  for (int f = 0; f < P.n_fn; ++f)
    if (P.fn[f].n_stored > 8) {
      log = "a function keeps more than 8 stored values";
      return false;
    }
  const std::string key = arch + (lanes ? "\nlanes\n" : "\n") + std::string(reinterpret_cast<const char*>(&P), sizeof(DevProgram));
  {
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
      code = it->second.code;
      return true;
    }
  }
  Rtc& r = rtc();
  if (!r.ok) {
    log = "hiprtc is not available";
    return false;
  }
  Gen gen(P);
  const std::string src = lanes ? gen.lane_source() : gen.source();
  if (getenv("TDF_JIT_DUMP")) fprintf(stderr, "%s\n", src.c_str());
  rtcProgram prog = nullptr;
  if (r.create(&prog, src.c_str(), "tdf_generated.hip", kEmbeddedCount, kEmbeddedSources, kEmbeddedNames) != 0) {
    log = "hiprtcCreateProgram failed";
    return false;
  }
  const std::string arch_opt = "--offload-arch=" + arch;
  const char* opts[] = {arch_opt.c_str(), "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};
  const int rc = r.compile(prog, 7, opts);
  size_t ls = 0;
  r.log_size(prog, &ls);
  if (ls > 1) {
    log.resize(ls);
    r.log(prog, &log[0]);
  }
  if (rc != 0) {
    r.destroy(&prog);
    return false;
  }
  size_t cs = 0;
  r.code_size(prog, &cs);
  code.resize(cs);
  r.code(prog, code.data());
  r.destroy(&prog);
  std::lock_guard<std::mutex> lock(g_cache_mutex);
  g_cache[key].code = code;
  return true;
}

bool jit_compile(const DevProgram& P, JitKernels& out, std::string& log) {
  const char* off = getenv("TDF_NO_JIT");
  if (off && off[0] == '1') {
    log = "disabled by TDF_NO_JIT";
    return false;
  }
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
    log = "no device";
    return false;
  }
  std::vector<char> code;
  if (!jit_code(P, prop.gcnArchName, false, code, log)) return false;   // e.g. gfx950:sramecc+:xnack-
  hipModule_t mod = nullptr;
  if (hipModuleLoadData(&mod, code.data()) != hipSuccess) {
    log = "hipModuleLoadData failed";
    return false;
  }
  hipFunction_t f_step = nullptr, f_small = nullptr, f_local = nullptr;
  if (hipModuleGetFunction(&f_step, mod, "tdf_generated_step") != hipSuccess ||
      hipModuleGetFunction(&f_local, mod, "tdf_generated_step_local") != hipSuccess ||
      hipModuleGetFunction(&f_small, mod, "tdf_generated_small") != hipSuccess) {
    (void)hipModuleUnload(mod);
    log = "generated kernels not found in the module";
    return false;
  }
  out.module = mod;
  out.step = f_step;
  out.step_local = f_local;
  out.small = f_small;
  return true;
}

int lane_stored(const DevProgram& P) {
  int ns = 1;
  for (int f = 0; f < P.n_fn; ++f) ns = std::max<int>(ns, P.fn[f].n_stored);
  return ns;
}

bool lane_branching(const DevProgram& P) {
  for (int f = 0; f < P.n_fn; ++f)
    if (f != P.result_fn && P.fn[f].n_sites > 1) return true;
  return false;
}

bool jit_compile_lanes(const DevProgram& P, JitKernels& out, std::string& log) {
  const char* off = getenv("TDF_NO_JIT");
  if (off && off[0] == '1') {
    log = "disabled by TDF_NO_JIT";
    return false;
  }
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
    log = "no device";
    return false;
  }
  std::vector<char> code;
  if (!jit_code(P, prop.gcnArchName, true, code, log)) return false;
  hipModule_t mod = nullptr;
  hipFunction_t f = nullptr;
  if (hipModuleLoadData(&mod, code.data()) != hipSuccess) {
    log = "hipModuleLoadData failed";
    return false;
  }
  if (hipModuleGetFunction(&f, mod, "tdf_generated_lanes") != hipSuccess) {
    (void)hipModuleUnload(mod);
    log = "generated kernel not found in the module";
    return false;
  }
  out.lanes_module = mod;
  out.lanes = f;
  return true;
}

void jit_release(JitKernels& k) {
  if (k.lanes_module) (void)hipModuleUnload((hipModule_t)k.lanes_module);
  if (k.module) (void)hipModuleUnload((hipModule_t)k.module);
  k = JitKernels{};
}

}  // namespace tdf

extern "C" tdf_status tdf_graph_precompile(const tdf_graph* graph, const char* arch, size_t* code_bytes) {
  if (!graph || !arch || !arch[0]) {
    tdf::set_error("tdf_graph_precompile: graph and arch are required");
    return TDF_ERR_BAD_ARG;
  }
  std::vector<char> code, lanes;
  std::string log;
  if (!tdf::jit_code(graph->g.prog, arch, false, code, log) || !tdf::jit_code(graph->g.prog, arch, true, lanes, log)) {
    tdf::set_error("run-time compilation failed: " + log);
    return TDF_ERR_UNSUPPORTED;
  }
  if (code_bytes) *code_bytes = code.size() + lanes.size();
  return TDF_OK;
}
