// The tag machine of evaluations that keep no frames (statistics level 0): depth-first lanes.
//
// A lane owns one frame (= one call-context tag), sweeps its function body, and goes on with the
// first call whose arguments are all present: the caller's frame goes on the lane's own stack, the
// callee's frame takes its place in registers, and its Return pops the caller again.  Call_i, Return_i,
// Enter, Next and Exit are the paper's (Call_i <t,d> = <i:t,d>, Return_i <i:t,d> = <t,d>, ...); what
// differs from the step machine (step_device.h) is the order in which ready tags fire, which the
// dataflow semantics leaves open, and where a frame lives: in the lane, not in a table, as long as one
// lane has the tag and all tags below it.  A call whose arguments arrive one after the other is
// opened when the last one is there, and a function's output leaves when everything it started has
// come back (both orders give the same values and the same counts).
//
// Work is shared in two tiers.
//   Inside a wave (= one workgroup), through LDS: a lane gives the oldest frame of its stack that has a
//   ready call left, as a record that any lane of the wave can take as a task.  Records are finished by
//   whoever delivers the last awaited value (a join counter per record; nobody waits).  The frames below
//   the one given have nothing to share and wait for one value each: they stay a stack, in memory, and take one
//   record together, however many they are; who returns to it has that stack from then on.  Everything is
//   wave-synchronous: no barriers, a hand-over costs a few LDS round trips.
//   Between waves, through memory: a wave that has nothing takes a ticket of the global queue; a wave that
//   sees tickets outstanding sends calls (arguments and where to return to), and polls for the values that
//   come back.  Values are written before flags with a wait for the acknowledgement in between, all with
//   device-scope accesses, which are coherent between the dies; such a round trip is about a microsecond,
//   which is why the first tier does not use it.
// No wave waits for another one except for work or for a value it sent a call for; idle waves are sent
// home when the last instance is done, so nothing here assumes that workgroups are resident together.
//
// What bounds it: the instructions of a wave's sweeps, about 4 clocks each, vector, scalar and branch alike (a
// recursion without parallelism runs one lane, about 1.3 us a call there and back), and with many waves how evenly
// the calls spread over them.  A frame costs no memory traffic beyond the lane's stack, whose top is in LDS.
// Measured, whole evaluations in us, step machine -> lanes: fib(0..20) 606 -> 167; fib(30) + fib(31) + fib(32)
// 27600 -> 3270; tak over 256 instances 20500 -> 1700; 65536 gcd loops 7300 -> 84.
// The tag phase of tree networks: 4096 random trees of up to 64 leaves 1980 -> 600, 1500 small trees 366 -> 112, a chain
// of 512 leaves 4200 -> 1500.
//
// Conditions that this machine does not handle (a call some of whose arguments are dead, a function
// that completes without a value, more frames than there is room for, more tags than max_tags) set
// `status`; the host then runs the evaluation on the step machine, whose answer counts.  Up to max_tags the step machine
// would have had a record for every tag; whether the tags alive at once fit where there are more is its to say.  (The
// same limit ends a recursion without a base case; there is none on time while any wave works.)
#pragma once
#include "engine.h"

namespace tdf {

constexpr uint32_t LANE_NONE = 0xFFFFFFFFu;
constexpr uint32_t LANE_REMOTE = 0x80000000u;   // a caller in another wave: LANE_REMOTE | wave << 6 | reply
constexpr uint32_t LANE_STACK = 0x40000000u;    // a caller on a stack that nobody runs: LANE_STACK | record of the stack
// Global queue: state of a slot, and the round of tickets that it is in (a ticket's number without its place in the
// queue).  A slot is written only in the round of the ticket that it is written for, so a call that nobody has taken
// yet stays as it is, however many tickets have been dealt out since.
constexpr uint32_t LANE_EMPTY = 0u, LANE_PILL = 1u, LANE_TASK = 2u, LANE_LEFT = 3u;
__host__ __device__ constexpr uint32_t lane_slot(uint32_t ticket, uint32_t cap, uint32_t state) { return (ticket & ~(cap - 1u)) | state; }
__host__ __device__ constexpr bool lane_is_pill(uint32_t flag) { return (flag & 3u) == LANE_PILL; }
constexpr uint32_t LANE_WINDOW = 4;     // frames of a lane's stack that stay in LDS
constexpr uint32_t LANE_SEG = 16;       // frames of a segment of a lane's stack in memory
constexpr uint32_t LANE_SYNC = 4, LANE_SYNC_FULL = 8;   // sweeps between two looks at the other lanes; the latter while nearly all have work
constexpr uint32_t LANE_YOUNG = 12000;  // ticks (100 MHz) for which a run is young
constexpr uint32_t LANE_EARLY = 48;     // sweeps during which a wave gives work away although it has lanes without any
// idle lanes up to which a wave gives calls to other waves
constexpr uint32_t LANE_GIVE = 56;
// Iterations of a loop without calls in one sweep (multiples of four): where no lane of the wave has anything else to do, and
// beside others, which wait for the sweep's end.  A sweep costs as much as tens of iterations (of subtractive gcd, 80 clocks
// each): 65,536 gcds of pairs up to 1,024 take 102 us with 64 a sweep, 97 with 128 and 96 with 256.  A recursion whose 4,096 leaves
// are loops of 1 to 651 iterations takes 230 us with 64, 232 with 128, 250 with 256 and 230 with this; 64 of 256 such leaves 157,
// 162, 170 and 157; with loops of 1 to 4,096, of which few are long, 370, 337, 321 and 323.
constexpr uint32_t LANE_LOOP = 256, LANE_LOOP_BESIDE = 64;
constexpr uint32_t LANE_RECS = 96;      // records of a wave
constexpr uint32_t LANE_SCARCE = 8, LANE_FEW = 16;   // free records below which all frames below a given one take one; else the first so many take one each
constexpr uint32_t LANE_QUEUE = 128;    // tasks of a wave (at least LANE_RECS: a record is queued at most once)
constexpr uint32_t LANE_CHUNK = 128;    // log entries a wave reserves at once (at least a wave's lanes)
constexpr uint32_t LANE_LOG_HOLE = 0xFFFFFFFFu;

// State of a frame: function (3 bits) | opened calls (8) << 3 | those of them outstanding in other lanes (8) << 11.
__host__ __device__ constexpr uint32_t lane_state(uint32_t fn, uint32_t opened, uint32_t out) { return fn | opened << 3 | out << 11; }
__host__ __device__ constexpr uint32_t lane_fn(uint32_t st) { return st & 7u; }
__host__ __device__ constexpr uint32_t lane_opened(uint32_t st) { return (st >> 3) & 0xFFu; }

enum LaneAct : uint32_t { ACT_NONE = 0, ACT_CALL, ACT_RET, ACT_NEXT, ACT_DONE, ACT_WAIT, ACT_STUCK };

// 16-byte units of a segment: {segment below, segment above, -, -}, then LANE_SEG frames.
__host__ __device__ constexpr int lane_seg_units(int n_stored) { return 1 + (int)LANE_SEG * (1 + (n_stored + 1) / 2); }
// 16-byte chunks of a frame on a lane's stack, by the stored values of the program.
__host__ __device__ constexpr int lane_chunks(int n_stored) { return 1 + (n_stored + 1) / 2; }
__host__ __device__ constexpr size_t lane_lds_bytes(int n_stored) {
  return (size_t)LANE_WINDOW * lane_chunks(n_stored) * 64 * 16 + (size_t)LANE_RECS * (8 * n_stored + 7 * 4 + 4) + LANE_QUEUE * 4 + 64 * 4;
}

#if defined(__HIPCC__) || defined(__HIPCC_RTC__)

// A slot of the global queue: one call sent to another wave.
struct LaneMail {
  uint32_t flag, pad;            // lane_slot
  unsigned long long from;       // caller: LANE_REMOTE | wave << 6 | reply, | state << 32
  unsigned long long meta;       // label | depth << 32
  unsigned long long inst_np;    // instance | number of arguments << 32
  unsigned long long arg[8];
  unsigned long long fill[4];
};
static_assert(sizeof(LaneMail) == 128, "one line per slot");
struct LaneReply { unsigned long long value, flag; };   // flag 1: the value is there
// What has to be in place before the lanes start, by thread i of n.
__device__ inline void lane_init(const LaneArgs& a, uint32_t i, uint32_t n) {
  if (i == 0) {
    *a.ctl = LaneCtl{};
    a.ctl->log_used = a.walk_nodes ? a.walk_nodes : a.log_cap ? a.n_waves * LANE_CHUNK : 0u;
  }
  if (i < a.n_queues) a.queues[i] = LaneQueue{};
  if (a.walk_nodes) {   // nobody has visited a node
    for (uint32_t k = i; k < a.walk_nodes; k += n) a.log[k].z = LANE_LOG_HOLE;
    return;
  }
  for (uint32_t k = i; k < a.n_queues * a.queue_cap; k += n) a.mail[k].flag = lane_slot(0u, a.queue_cap, LANE_EMPTY);
  for (uint32_t k = i; k < a.n_waves * 64u; k += n) a.reply[k].flag = 0ull;
  if (a.row_node)
    for (uint32_t k = i; k < a.log_cap; k += n) a.row_node[k] = 0xFFFFFFFFu;
}

template <typename T> __device__ __forceinline__ T lane_ld(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ void lane_put(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ T lane_add(T* p, T v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over the lanes of a wave; every lane must call.
__device__ __forceinline__ uint32_t wave_usum(uint32_t v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// A lane: its frame, what the last sweep asks for, and its counts.
struct LaneX {
  const LaneArgs* a;
  long long sv[8];
  uint32_t st;              // state (lane_state)
  uint32_t present;         // stored values that are there
  uint32_t label, counter, depth;
  bool run;                 // the lane sweeps its frame
  uint32_t inst;
  // result of a sweep
  uint32_t act;
  uint32_t c_st, c_np, c_label;   // the new frame's state, number of arguments, label of the call
  uint32_t c_back;          // the caller's state once the call is back | the value's stored slot << 20
  long long arg[8];
  long long ret;
  bool more;                // further calls of the frame are ready
  // wave-uniform: the wave's part of the schedule log
  uint32_t log_next, log_end;
  // counts
  uint32_t n_tags, n_tokens, n_leaf, n_cell, mx_depth, mx_level;
  int bad;                  // a condition the host has to deal with
  // the tree node looked at last (the callee's, when a call was tried in place and then made): index and entries;
  // negative: none (no node has such an index: it is never taken for one)
  long long pf_v;
  int pf_l, pf_r, pf_t;
};

// ---- helpers of the generated sweeps ---------------------------------------------------------------
// forest accessors at node v: which = 0 isleaf, 1 left, 2 right, 3 token
__device__ __forceinline__ long long ln_tree(LaneX& x, long long v, int which, bool& dead) {
  const LaneArgs& a = *x.a;
  if (v < 0 || v >= a.n_tree_nodes || a.left == nullptr) {
    x.bad = TDF_ERR_BAD_ARG;
    dead = true;
    return 0;
  }
  const int32_t e = which == 2 ? a.right[v] : which == 3 ? a.token[v] : a.left[v];
  return which == 0 ? (long long)(e < 0) : (long long)e;
}
// the entry itself; 0 if there is no such node
__device__ __forceinline__ long long ln_entry(LaneX& x, long long v, int which) {
  bool dead = false;
  return ln_tree(x, v, which, dead);
}
// the same for a node that an earlier sweep has found bad if it is
__device__ __forceinline__ long long ln_entry_again(const LaneX& x, long long v, int which) {
  const LaneArgs& a = *x.a;
  if (v < 0 || v >= a.n_tree_nodes || a.left == nullptr) return 0;
  return which == 2 ? a.right[v] : which == 3 ? a.token[v] : a.left[v];
}
// a node's entries in one round trip; false: no such node
__device__ __forceinline__ bool ln_node(LaneX& x, long long v, int& l, int& r, int& t) {
  const LaneArgs& a = *x.a;
  if (v < 0 || v >= a.n_tree_nodes || a.left == nullptr) {
    x.bad = TDF_ERR_BAD_ARG;
    return false;
  }
  l = a.left[v];
  r = a.right[v];
  t = a.token[v];
  return true;
}
// positions in the schedule log for the lanes that take one; whole wave must call
__device__ __forceinline__ uint32_t ln_log(LaneX& x, bool take) {
  const unsigned long long m = __ballot(take);
  if (m == 0) return 0;
  const uint32_t n = (uint32_t)__popcll(m);
  if (x.log_next + n > x.log_end) {   // the wave's chunk is used up: what is left of it stays a hole
    const LaneArgs& a = *x.a;
    const uint32_t h = x.log_next + lane_id();
    if (h < x.log_end && h < a.log_cap) a.log[h].z = LANE_LOG_HOLE;
    uint32_t base = 0;
    if (lane_id() == 0) base = lane_add(&a.ctl->log_used, LANE_CHUNK);
    x.log_next = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    x.log_end = x.log_next + LANE_CHUNK;
  }
  const uint32_t pos = x.log_next + (uint32_t)__popcll(m & lanemask_lt());
  x.log_next += n;
  return pos;
}
// EMBED: one log entry {token, -, level 0, instance}; the value is named by its place in the log
__device__ __forceinline__ void ln_embed(LaneX& x, bool on, int slot, bool ap, bool ad, long long av, long long& v, bool& p, bool& live) {
  const bool had = on && ((x.present >> slot) & 1);
  const bool go = on && ap && !ad && !had;
  const bool ok = go && av >= 0 && av < (long long)x.a->vocab;
  if (go && !ok) x.bad = TDF_ERR_BAD_ARG;
  const uint32_t pos = ln_log(x, ok);
  long long r = x.sv[slot];
  if (ok) {
    if (pos < x.a->log_cap) x.a->log[pos] = make_uint4((uint32_t)av, 0u, 0u, x.inst);
    else x.bad = TDF_ERR_TABLE_FULL;
    r = (long long)pos;
    x.sv[slot] = r;
    x.present |= 1u << slot;
    ++x.n_leaf;
  }
  v = r;
  p = had || ok;
  live = p;
}
// the same for a callee that is tried in its caller's sweep
__device__ __forceinline__ void ln_embed_now(LaneX& x, bool go, long long av, long long& v, bool& p) {
  const bool ok = go && av >= 0 && av < (long long)x.a->vocab;
  if (go && !ok) x.bad = TDF_ERR_BAD_ARG;
  const uint32_t pos = ln_log(x, ok);
  if (ok) {
    if (pos < x.a->log_cap) x.a->log[pos] = make_uint4((uint32_t)av, 0u, 0u, x.inst);
    else x.bad = TDF_ERR_TABLE_FULL;
    ++x.n_leaf;
  }
  v = (long long)pos;
  p = ok;
}
// the iterations a loop graph has run in one sweep
__device__ __forceinline__ void ln_loop(LaneX& x, uint32_t n, uint32_t n_vars) {
  x.n_tags += n;
  x.n_tokens += n * n_vars;
  x.counter += n;
  if (x.counter > 0xFFFFFFu) x.bad = TDF_ERR_STEP_LIMIT;
  if (n) x.mx_depth = x.depth > x.mx_depth ? x.depth : x.mx_depth;
}
// RNN / LSTM cell: one log entry {left, right, level, instance}
__device__ __forceinline__ void ln_cell(LaneX& x, bool on, int slot, bool ap, bool ad, long long av, bool bp, bool bd, long long bv,
                                        long long& v, bool& p, bool& live) {
  const bool had = on && ((x.present >> slot) & 1);
  const bool go = on && ap && bp && !ad && !bd && !had;
  const uint32_t pos = ln_log(x, go);
  long long r = x.sv[slot];
  if (go) {
    const uint32_t la = (uint32_t)(av >> 32), lb = (uint32_t)(bv >> 32);
    const uint32_t lvl = 1 + (la > lb ? la : lb);
    if (pos < x.a->log_cap) x.a->log[pos] = make_uint4((uint32_t)av, (uint32_t)bv, lvl, x.inst);
    else x.bad = TDF_ERR_TABLE_FULL;
    r = (long long)pos | ((long long)lvl << 32);
    x.sv[slot] = r;
    x.present |= 1u << slot;
    x.mx_level = lvl > x.mx_level ? lvl : x.mx_level;
    ++x.n_cell;
  }
  v = r;
  p = had || go;
  live = p;
}
__device__ __forceinline__ void ln_ce_node(LaneX& x, long long row, long long v, bool& dead) {
  const LaneArgs& a = *x.a;
  if (v < 0 || v >= a.n_tree_nodes || a.row_node == nullptr) {
    x.bad = TDF_ERR_BAD_ARG;
    dead = true;
    return;
  }
  if ((uint32_t)row < a.log_cap) a.row_node[(uint32_t)row] = (uint32_t)v;
}
__device__ __forceinline__ void ln_head(LaneX& x, bool on, int slot, bool ap, bool ad, long long av, bool bp, bool bd, long long bv,
                                        long long& v, bool& p, bool& live) {
  const bool had = on && ((x.present >> slot) & 1);
  const bool go = on && ap && bp && !ad && !bd && !had;
  if (go) {
    x.a->head_row[x.inst] = (uint32_t)av;
    x.a->root_lvl[x.inst] = (uint32_t)(av >> 32);
    x.a->head_label[x.inst] = (uint32_t)bv;
    x.sv[slot] = x.inst;
    x.present |= 1u << slot;
  }
  v = (long long)x.inst;
  p = had || go;
  live = p;
}
__device__ __forceinline__ void ln_result(LaneX& x, int type, long long v) {
  if (type == T_INT) { if (x.a->out_i64) x.a->out_i64[x.inst] = v; }
  else if (type == T_VEC) {
    x.a->root_ref[x.inst] = (uint32_t)v;
    x.a->root_lvl[x.inst] = (uint32_t)(v >> 32);
  }
}

// Early on the lanes look at one another after every sweep instead of every fourth in two cases.  While a few lanes
// of the wave have all the work (8 recursions of 3 to 10 levels: 104 us, now 89; 1,000 of 3 to 12: 147 and 115;
// fib(0..20) 214 and 199; with as many lanes busy fib(0..20) takes 240), but not in a run that fills the GPU from a
// few roots, which pieces that small only chop up.  And in such a run at a wave's first sweeps, however many lanes are
// busy, while the run is young: fib(30..32) 4,090 us and 3,500, fib(30) 1,480 and 1,260, three of fib(28) 1,510 and 1,300.
// How much there is to do is not known then.  max_tags is only the room there is: with less than 1,024 tags for a wave
// the run is too small for this (fib(28), a million tags: 705 us, 775 in pieces), with more it may be all the same.
// What costs such a run most are the pieces that waves which join late make of pieces, so there is an end to it after
// 120 us: fib(28) with room for 16 times its tags 730 us.  (An end after 90 us takes back most of what the large runs gain:
// fib(30..32) 4,000.)  With many roots, where nobody joins late, that end is none: 256 of tak 2,030 us without it, 2,075 with
// none of this.  Where no function has two calls there is nothing to give.  And only for integer programs: a sweep of
// a tree program is several times as long, and pieces that small cost more than they bring (tag phase of 8 complete trees of
// 4,096 leaves 257 us, 188 without; of a random tree of 8,000 leaves with 63 small ones 531 and 390).
template <class Age>   // age(): ticks since the run began
__device__ __forceinline__ bool lane_spreads(uint32_t n_waves, uint32_t n_inst, uint32_t tags_at_once, uint32_t log_cap, uint32_t n_run,
                                             uint32_t iter, Age age) {
  if (log_cap) return false;
  const bool fills = n_waves >= 1024u, many = n_inst >= 16u;
  if (n_run < 32u && (!fills || many)) return iter < LANE_EARLY;
  return fills && tags_at_once >= 512u && iter < LANE_EARLY / 3 && (many || age() < LANE_YOUNG);
}

// ---- the machine ----------------------------------------------------------------------------------
// SW (generated): kStored (stored values per frame), kResultFn, kBranching (a function can have two calls
// under way at once), sweep(x), ret_bits(fn, opened) (stored values that the opened calls return into),
// outstanding(fn, opened, present) (opened calls whose value is not there), ret_slot(label).
template <class SW>
__device__ void lanes_run(const LaneArgs& a, char* lds) {
  constexpr int NS = SW::kStored, NC = lane_chunks(NS);
  uint4* const win = reinterpret_cast<uint4*>(lds);                       // [LANE_WINDOW][NC][64]
  // records: stored values, then one array per field; `po` = present values | opened calls << 24
  unsigned long long* const r_val = reinterpret_cast<unsigned long long*>(win + LANE_WINDOW * NC * 64);   // [NS][LANE_RECS]
  uint32_t* const r_parent = reinterpret_cast<uint32_t*>(r_val + NS * LANE_RECS);
  uint32_t* const r_meta = r_parent + LANE_RECS;      // label | function << 16 | nothing outstanding << 31
  uint32_t* const r_counter = r_meta + LANE_RECS;
  uint32_t* const r_depth = r_counter + LANE_RECS;
  uint32_t* const r_po = r_depth + LANE_RECS;
  uint32_t* const r_inst = r_po + LANE_RECS;
  uint32_t* const r_join = r_inst + LANE_RECS;        // calls outstanding, plus one for the lane or task that has the frame
  uint32_t* const lfree = r_join + LANE_RECS;         // [LANE_RECS] free record ids
  uint32_t* const lq = lfree + LANE_RECS;             // [LANE_QUEUE] tasks
  uint32_t* const sent = lq + LANE_QUEUE;             // [64] calls sent to other waves: record | slot << 16
  const uint32_t lane = threadIdx.x, wave = blockIdx.x;
  LaneReply* const reply = a.reply + (size_t)wave * 64 + lane;
  LaneCtl* const ctl = a.ctl;

  LaneX x;
  x.a = &a;
#pragma unroll
  for (int k = 0; k < 8; ++k) x.sv[k] = x.arg[k] = 0;
  x.st = x.present = x.label = x.counter = x.depth = x.inst = 0;
  x.c_st = x.c_np = x.c_label = x.c_back = 0;
  x.act = ACT_NONE;
  x.run = x.more = false;
  x.ret = 0;
  x.log_next = wave * LANE_CHUNK;   // (the first chunks of the log are dealt out)
  x.log_end = a.log_cap ? x.log_next + LANE_CHUNK : x.log_next;
  x.n_tags = x.n_tokens = x.n_leaf = x.n_cell = x.mx_depth = x.mx_level = 0;
  x.bad = 0;
  x.pf_v = -1;
  x.pf_l = x.pf_r = x.pf_t = 0;
  // The lane's stack: frames bs .. sp - 1 (the frame in registers is on top of them), of which those from lo
  // on lie in the LDS window and the others in a list of segments in memory: frame d in a segment whose
  // frames start at a multiple of LANE_SEG, `seg` the one of frame lo - 1, `seg_b` the one of frame bs.  `slack`
  // frames have a ready call left.  (The first frame of an empty stack has number 0: bs is reset then.)
  bool active = false;
  uint32_t sp = 0, bs = 0, lo = 0, slack = 0, seg = LANE_NONE, seg_b = LANE_NONE;
  uint32_t spare = LANE_NONE;             // segments the lane has and does not use (a list)
  // The bottom frame (frame bs, or the one in registers if the stack is empty): its record, if it has one, and
  // its caller: a record, a call from another wave, or none.
  uint32_t rec = LANE_NONE, parent = LANE_NONE;
  bool resumed = false;                   // the bottom frame has nothing outstanding in other lanes
  uint32_t mx_sp = 0;
  // wave-uniform
  const uint32_t t_begin = SW::kBranching ? (uint32_t)wall_clock64() : 0u;   // (all waves of a run are resident: they begin together)
  uint32_t n_told = 0;                    // tags reported
  uint32_t qh = 0, qt = 0, nfree = LANE_RECS, iter = 0, syncs = 0, ticket = 0, min_free = LANE_RECS;
  unsigned long long sent_mask = 0;       // replies awaited, by lane
  bool more_inst = true, stop = false, have_ticket = false;
  uint32_t n_own = 0, n_mine = 0, hungry = 0;   // instances of this wave that are not done; those taken since the last report
  // With every lane busy on work of its own a wave would have none to send a call to a wave without work: where
  // several waves share a recursion the last two lanes do that and nothing else.
  const unsigned long long exporter = a.n_waves > 1 && SW::kBranching ? 3ull << 62 : 0ull;
  for (uint32_t k = lane; k < LANE_RECS; k += 64) lfree[k] = k;

  auto seg_at = [&](uint32_t id) { return a.segs + (size_t)id * lane_seg_units(NS); };
  auto win_put = [&](uint32_t d, const uint4 (&c)[NC]) {
#pragma unroll
    for (int k = 0; k < NC; ++k) win[((d % LANE_WINDOW) * NC + k) * 64 + lane] = c[k];
  };
  auto win_get = [&](uint32_t d, uint4 (&c)[NC]) {
#pragma unroll
    for (int k = 0; k < NC; ++k) c[k] = win[((d % LANE_WINDOW) * NC + k) * 64 + lane];
  };
  auto mem_get = [&](uint32_t id, uint32_t d, uint4 (&c)[NC]) {
    const uint4* f = seg_at(id) + 1 + (d % LANE_SEG) * NC;
#pragma unroll
    for (int k = 0; k < NC; ++k) c[k] = f[k];
  };
  // a segment is empty: to the lane's list
  auto drop_seg = [&](uint32_t id) {
    seg_at(id)[0].x = spare;
    spare = id;
  };
  // LANE_NONE if there is none left: the caller then leaves everything as it is, and the run ends before anybody goes on
  auto new_seg = [&]() -> uint32_t {
    uint32_t id = spare;
    if (id != LANE_NONE) spare = seg_at(id)[0].x;
    else id = lane_add(&ctl->n_seg, 1u);
    if (id >= a.n_segs) {
      x.bad = TDF_ERR_TABLE_FULL;
      id = LANE_NONE;
    }
    return id;
  };
  // the window's oldest frame goes to memory
  auto evict = [&]() {
    if (lo % LANE_SEG == 0 || seg == LANE_NONE) {
      const uint32_t id = new_seg();
      if (id == LANE_NONE) {
        x.run = false;   // (the lane's stack is not whole any more)
        return;
      }
      seg_at(id)[0].x = seg;
      if (seg != LANE_NONE) seg_at(seg)[0].y = id;
      if (seg_b == LANE_NONE) seg_b = id;
      seg = id;
    }
    uint4 c[NC];
    win_get(lo, c);
    uint4* f = seg_at(seg) + 1 + (lo % LANE_SEG) * NC;
#pragma unroll
    for (int k = 0; k < NC; ++k) f[k] = c[k];
    ++lo;
  };
  // frame on the stack: {state | slot awaited << 20 | ready call left << 25 | label << 26, counter, depth, present} values
  auto pack = [&](uint4 (&c)[NC], uint32_t back_st, bool more) {
    c[0] = make_uint4(back_st | (more ? 1u << 25 : 0u) | (x.label << 26), x.counter, x.depth, x.present);
#pragma unroll
    for (int k = 1; k < NC; ++k) {
      const long long u = x.sv[2 * k - 2], v = 2 * k - 1 < NS ? x.sv[(2 * k - 1) & 7] : 0;
      c[k] = make_uint4((uint32_t)u, (uint32_t)(u >> 32), (uint32_t)v, (uint32_t)(v >> 32));
    }
  };
  auto unpack = [&](const uint4 (&c)[NC]) {
    x.st = c[0].x & 0xFFFFFu;
    x.label = c[0].x >> 26;
    x.counter = c[0].y;
    x.depth = c[0].z;
    x.present = c[0].w;
#pragma unroll
    for (int k = 1; k < NC; ++k) {
      x.sv[2 * k - 2] = (long long)((unsigned long long)c[k].x | ((unsigned long long)c[k].y << 32));
      if (2 * k - 1 < NS) x.sv[(2 * k - 1) & 7] = (long long)((unsigned long long)c[k].z | ((unsigned long long)c[k].w << 32));
    }
  };
  auto set_slot = [&](uint32_t slot, long long v) {
#pragma unroll
    for (int k = 0; k < NS; ++k)
      x.sv[k] = (uint32_t)k == slot ? v : x.sv[k];
    x.present |= 1u << slot;
  };
  // the stack's top frame becomes the lane's own, with the value that it waited for
  auto pop = [&](long long v) {
    --sp;
    uint4 c[NC];
    if (sp >= lo) {
      win_get(sp, c);
    } else {
      mem_get(seg, sp, c);
      lo = sp;
      if (sp % LANE_SEG == 0 || sp == bs) {   // that was the segment's last frame
        const uint32_t id = seg;
        seg = sp == bs ? LANE_NONE : seg_at(id)[0].x;
        if (sp == bs) seg_b = LANE_NONE;
        drop_seg(id);
      }
    }
    unpack(c);
    slack -= (c[0].x >> 25) & 1u;
    set_slot((c[0].x >> 20) & 31u, v);
  };
  // the frame of a record becomes the lane's own (bottom) frame
  auto load_rec = [&](bool on, uint32_t id) {
    if (on) {
#pragma unroll
      for (int k = 0; k < NS; ++k) x.sv[k] = (long long)r_val[k * LANE_RECS + id];
      parent = r_parent[id];
      const uint32_t m = r_meta[id], po = r_po[id], fn = (m >> 16) & 7u, opened = po >> 24;
      x.label = m & 0xFFFFu;
      x.counter = r_counter[id];
      x.depth = r_depth[id];
      x.present = po & 0xFFFFFFu;
      x.st = lane_state(fn, opened, SW::outstanding(fn, opened, x.present));
      x.inst = r_inst[id];
      rec = id;
      sp = bs = lo = slack = 0;
      resumed = (m >> 31) != 0;
      active = x.run = true;
    }
  };
  auto free_recs = [&](bool on, uint32_t id) {   // whole wave
    const unsigned long long m = __ballot(on);
    if (m == 0) return;
    if (on) lfree[nfree + (uint32_t)__popcll(m & lanemask_lt())] = id;
    nfree += (uint32_t)__popcll(m);
  };
  auto push_tasks = [&](bool on, uint32_t id) {  // whole wave
    const unsigned long long m = __ballot(on);
    if (m == 0) return;
    if (on) lq[(qt + (uint32_t)__popcll(m & lanemask_lt())) % LANE_QUEUE] = id;
    qt += (uint32_t)__popcll(m);
  };
  // Everything a frame has opened has come back: it is a task again.
  auto resume = [&](bool on, uint32_t id) {      // whole wave
    if (on) {
      r_join[id] = 1u;
      r_meta[id] |= 1u << 31;
    }
    push_tasks(on, id);
  };
  // A value for a record; true for the lane that delivers the last one awaited (it, or a task, goes on with the frame).
  auto deliver = [&](uint32_t id, uint32_t slot, long long v) -> bool {
    r_val[slot * LANE_RECS + id] = (unsigned long long)v;
    atomicOr(&r_po[id], 1u << slot);
    return atomicSub(&r_join[id], 1u) == 1u;
  };
  // Waves are spread over several queues, so that their tickets and polls do not meet on one line: a wave
  // waits at its own queue (wave % n_queues) and looks for waiting waves at one queue after the other.
  auto mail_slot = [&](uint32_t q, uint32_t t) { return a.mail + (size_t)q * a.queue_cap + (t & (a.queue_cap - 1)); };
  const uint32_t my_queue = wave % a.n_queues;
  uint32_t look = my_queue, send_queue = 0;   // the queue looked at next; the one `hungry` counts at
  // Pills for every wave: sent once, by the wave that saw the last instance finish or the first error.
  auto send_home = [&]() {
    if (lane < a.n_queues) {
      const uint32_t n = (a.n_waves - lane + a.n_queues - 1) / a.n_queues;   // waves of that queue
      const uint32_t t0 = lane_add(&a.queues[lane].tail, n);
      for (uint32_t k = 0; k < n; ++k) lane_put(&mail_slot(lane, t0 + k)->flag, lane_slot(t0 + k, a.queue_cap, LANE_PILL));
    }
  };
  auto given_up = [&]() { return (uint32_t)__builtin_amdgcn_readfirstlane((int)lane_ld(&ctl->status)); };
  auto raise_status = [&]() {   // whole wave
    const unsigned long long m = __ballot(x.bad != 0);
    if (m == 0) return;
    const int code = __shfl(x.bad, __ffsll((long long)m) - 1);
    uint32_t was = 1;
    if (lane == 0) {
      uint32_t expect = 0;
      was = __hip_atomic_compare_exchange_strong(&ctl->status, &expect, (uint32_t)(-code), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT) ? 0u : 1u;
    }
    if (__builtin_amdgcn_readfirstlane((int)was) == 0) send_home();
    stop = true;
  };
  // The wave's instances are done (they end in the wave they began in): counted per queue, then over the
  // queues; the last one sends everybody home.
  auto instances_done = [&]() {
    bool all = false;
    if (lane == 0) {
      const uint32_t n = (a.n_inst + a.n_queues - 1u - my_queue) / a.n_queues;
      all = lane_add(&a.queues[my_queue].inst_done, n_mine) + n_mine == n && lane_add(&ctl->queues_done, 1u) + 1u == min(a.n_queues, a.n_inst);
    }
    n_mine = 0;
    if (__ballot(all)) {
      send_home();
      stop = true;
    }
  };
  // values of calls that were sent to other waves; whole wave
  auto poll_replies = [&]() {
    const bool mine = ((sent_mask >> lane) & 1ull) != 0;
    const bool got = mine && lane_ld(&reply->flag) == 1ull;
    const unsigned long long m = __ballot(got);
    if (m == 0) return;
    bool last = false;
    uint32_t id = 0;
    if (got) {
      const long long v = (long long)lane_ld(&reply->value);
      lane_put(&reply->flag, 0ull);
      id = sent[lane] & 0xFFFFu;
      last = deliver(id, sent[lane] >> 16, v);
    }
    sent_mask &= ~m;
    resume(last, id);
  };

  // A call from another wave becomes a record and a task.  There is a free record: a wave takes a ticket only if it has
  // one, and keeps one back while it holds the ticket.  (Otherwise all records could wait for values from other waves, which
  // wait for the call that lies in this wave's slot.)
  auto spare_recs = [&]() { return nfree - (have_ticket ? 1u : 0u); };
  auto take_mail = [&](LaneMail* slot) {
    have_ticket = false;
    uint32_t id = 0;
    if (lane == 0) {
      id = lfree[nfree - 1];
      const unsigned long long w0 = lane_ld(&slot->from), w1 = lane_ld(&slot->meta), w2 = lane_ld(&slot->inst_np);
      unsigned long long v8[8];
#pragma unroll
      for (int k = 0; k < NS; ++k) v8[k] = lane_ld(&slot->arg[k]);
#pragma unroll
      for (int k = 0; k < NS; ++k) r_val[k * LANE_RECS + id] = v8[k];
      r_parent[id] = (uint32_t)w0;
      r_meta[id] = (uint32_t)w1 | (lane_fn((uint32_t)(w0 >> 32)) << 16);
      r_counter[id] = 0;
      r_depth[id] = (uint32_t)(w1 >> 32);
      r_po[id] = (1u << (uint32_t)(w2 >> 32)) - 1u;
      r_inst[id] = (uint32_t)w2;
      r_join[id] = 1u;
      __builtin_amdgcn_s_waitcnt(0);
      lane_put(&slot->flag, lane_slot(ticket + a.queue_cap, a.queue_cap, LANE_EMPTY));   // (the next round's)
    }
    --nfree;
    min_free = min(min_free, nfree);
    push_tasks(lane == 0, id);
  };

  while (!stop) {
    // ---- idle lanes take a task of the wave, an empty wave takes instances, or a ticket of the global queue
    if (sent_mask) poll_replies();
    // (a wave that found work again while it holds a ticket: what is sent to it joins its tasks)
    if (have_ticket) {
      LaneMail* const slot = mail_slot(my_queue, ticket);
      const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)lane_ld(&slot->flag));
      if (lane_is_pill(v)) break;
      if (v == lane_slot(ticket, a.queue_cap, LANE_TASK)) take_mail(slot);
    }
    {
      const unsigned long long idle = ~__ballot(active);
      if (idle) {
        const uint32_t nq = qt - qh;
        if (nq) {
          // (the last lanes work for waves without work only: see the sharing below)
          const unsigned long long can = hungry || idle == ~0ull ? idle : idle & ~exporter;
          const uint32_t r = (uint32_t)__popcll(can & lanemask_lt()), n = min(nq, (uint32_t)__popcll(can));
          const bool on = ((can >> lane) & 1ull) && r < n;
          const uint32_t id = on ? lq[(qh + r) % LANE_QUEUE] : 0;
          qh += n;
          load_rec(on, id);
        } else if (idle == ~0ull) {
          if (more_inst) {
            // instances q, q + n_queues, ... belong to queue q
            const uint32_t in_queue = (a.n_inst + a.n_queues - 1u - my_queue) / a.n_queues;
            uint32_t base = in_queue;
            if (lane == 0 && in_queue) base = lane_add(&a.queues[my_queue].next_inst, a.per_grab);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            if (base >= in_queue) {
              more_inst = false;
              continue;
            }
            const uint32_t got = min(a.per_grab, in_queue - base);
            n_own += got;
            n_mine += got;
            if (lane < got) {
              const uint32_t b = my_queue + a.n_queues * (base + lane);
#pragma unroll
              for (int k = 0; k < NS; ++k)
                x.sv[k] = k < a.n_args ? a.args[(size_t)b * a.n_args + k] : 0ll;
              x.present = (1u << a.n_args) - 1u;
              x.st = lane_state(SW::kResultFn, 0u, 0u);
              x.label = x.counter = x.depth = 0;
              x.inst = b;
              rec = parent = LANE_NONE;
              sp = bs = lo = slack = 0;
              resumed = false;
              active = x.run = true;
            }
            continue;
          }
          // nothing left in this wave: wait for a task, for a value, or to be sent home
          if (!have_ticket && nfree) {
            uint32_t t = 0;
            if (lane == 0) t = lane_add(&a.queues[my_queue].head, 1u);
            ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
            have_ticket = true;
          }
          LaneMail* const slot = mail_slot(my_queue, ticket);
          const long long t0 = wall_clock64();
          uint32_t v = LANE_EMPTY;
          bool task = false, home = false;
          uint32_t beat_seen = 0xFFFFFFFFu;   // the beat of the waves that work, and when it was new
          long long t_beat = t0;
          for (;;) {
            if (have_ticket) {
              v = (uint32_t)__builtin_amdgcn_readfirstlane((int)lane_ld(&slot->flag));
              task = v == lane_slot(ticket, a.queue_cap, LANE_TASK);
              home = lane_is_pill(v);
              if (task || home) break;
            }
            if (sent_mask) {
              poll_replies();
              if (qt != qh) break;
            }
            home = !have_ticket && given_up() != 0;   // (with a ticket it is sent home)
            if (home) break;
            __builtin_amdgcn_s_sleep(4);
            if (__builtin_expect(wall_clock64() - t0 > a.idle_ticks, 0)) {
              if (sent_mask || nfree != LANE_RECS) {   // others still work on what this wave waits for: look whether they gave up
                const uint32_t beat = (uint32_t)__builtin_amdgcn_readfirstlane((int)lane_ld(&ctl->beat));
                if (beat != beat_seen) {
                  beat_seen = beat;
                  t_beat = wall_clock64();
                }
                if (given_up() != 0 || wall_clock64() - t_beat > a.dead_ticks) {
                  if (lane == 0) x.bad = TDF_ERR_STEP_LIMIT;
                  raise_status();
                  home = true;
                  break;
                }
                continue;
              }
              uint32_t left = 0;   // leave; whoever comes to this slot sees that
              if (lane == 0) {
                uint32_t expect = lane_slot(ticket, a.queue_cap, LANE_EMPTY);
                left = __hip_atomic_compare_exchange_strong(&slot->flag, &expect, lane_slot(ticket, a.queue_cap, LANE_LEFT), __ATOMIC_RELAXED,
                                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 1u : 0u;
              }
              home = __builtin_amdgcn_readfirstlane((int)left) != 0;
              if (home) break;
            }
          }
          if (home) break;
          if (task) take_mail(slot);
          continue;
        }
      }
    }

    // ---- a few sweeps
    bool any_done = false;
    const uint32_t n_run = (uint32_t)__popcll(__ballot(x.run));
    const bool spread = SW::kBranching && lane_spreads(a.n_waves, a.n_inst, a.tags_at_once, a.log_cap, n_run, iter,
                                                       [&] { return (uint32_t)wall_clock64() - t_begin; });
    const uint32_t n_sweeps = spread ? 1u : n_run >= 48 ? LANE_SYNC_FULL : hungry ? 2u : LANE_SYNC;
#pragma unroll 1
    for (uint32_t k = 0; k < n_sweeps; ++k) {
      if (__ballot(x.run) == 0) break;
      ++iter;
      if (x.run) x.act = ACT_NONE;
      SW::sweep(x);
      if (hungry) {
        // Waves without work: a call of a frame that has a record goes there, as far as there are reply places.
        const bool can = x.run && x.act == ACT_CALL && sp == bs && rec != LANE_NONE;
        const unsigned long long cm = __ballot(can);
        const uint32_t r = (uint32_t)__popcll(cm & lanemask_lt());
        const uint32_t n = min(min((uint32_t)__popcll(cm), hungry), 64u - (uint32_t)__popcll(sent_mask));
        if (n) {
          unsigned long long places = ~sent_mask;   // the lane's: the r-th free one
          for (uint32_t k2 = 0; k2 < n; ++k2) places = k2 < r ? places & (places - 1ull) : places;
          const uint32_t place = (uint32_t)__ffsll((long long)places) - 1u;
          // tickets without a call, reserved: never more calls than tickets, so that no call waits for a wave
          // (the flags of the slots are requested meanwhile: one that is found empty for its ticket stays so)
          uint32_t t0 = 0, n_got = 0;
          unsigned long long* const q = reinterpret_cast<unsigned long long*>(&a.queues[send_queue].head);
          unsigned long long was = lane_ld(q);
          const uint32_t guess = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(was >> 32));
          uint32_t f = can && r < n ? lane_ld(&mail_slot(send_queue, guess + r)->flag) : 0u;
          if (lane == 0) {
            for (int tries = 0; tries < 16; ++tries) {
              const int open = (int)((uint32_t)was - (uint32_t)(was >> 32));
              if (open <= 0) break;
              const uint32_t m = min((uint32_t)open, n);
              if (__hip_atomic_compare_exchange_strong(q, &was, was + ((unsigned long long)m << 32), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT)) {
                t0 = (uint32_t)(was >> 32);
                n_got = m;
                break;
              }
            }
          }
          t0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)t0);
          n_got = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_got);
          bool on = can && r < n_got;
          // The slot of ticket t belongs to the call with that ticket from the moment on that the one a round before has
          // been taken out (there are far more slots than waves at the queue: practically always).  While a lane waits for
          // that, its wave goes on taking what is sent to itself: so no waves wait for one another in a circle.
          auto not_there = [&]() {   // that wave has left: the slot is free again, the call stays here
            lane_put(&mail_slot(send_queue, t0 + r)->flag, lane_slot(t0 + r + a.queue_cap, a.queue_cap, LANE_EMPTY));
            on = false;
          };
          const uint32_t mine = lane_slot(t0 + r, a.queue_cap, LANE_EMPTY);
          LaneMail* const slot = mail_slot(send_queue, t0 + r);
          if (t0 != guess) f = ~mine;   // (another ticket's)
          long long w0 = 0;
          while (__builtin_expect(__ballot(on && f != mine) != 0, 0)) {
            if (on && f != mine) {
              f = lane_ld(&slot->flag);
              if (f == lane_slot(t0 + r, a.queue_cap, LANE_LEFT)) not_there();
              else if (lane_is_pill(f)) on = false;   // (another wave has met an error)
              else if (w0 == 0) w0 = wall_clock64();
              else if (wall_clock64() - w0 > a.idle_ticks) {
                x.bad = TDF_ERR_DEVICE;
                on = false;
              }
            }
            if (have_ticket) {
              LaneMail* const own = mail_slot(my_queue, ticket);
              if ((uint32_t)__builtin_amdgcn_readfirstlane((int)lane_ld(&own->flag)) == lane_slot(ticket, a.queue_cap, LANE_TASK)) take_mail(own);
            }
          }
          if (on) {
            lane_put(&slot->from, (unsigned long long)(LANE_REMOTE | (wave << 6) | place) | ((unsigned long long)x.c_st << 32));
            lane_put(&slot->meta, (unsigned long long)x.c_label | ((unsigned long long)(x.depth + 1u) << 32));
            lane_put(&slot->inst_np, (unsigned long long)x.inst | ((unsigned long long)x.c_np << 32));
#pragma unroll
            for (int k2 = 0; k2 < NS; ++k2) lane_put(&slot->arg[k2], (unsigned long long)x.arg[k2]);
            __builtin_amdgcn_s_waitcnt(0);
            uint32_t expect = mine;
            if (!__hip_atomic_compare_exchange_strong(&slot->flag, &expect, lane_slot(t0 + r, a.queue_cap, LANE_TASK), __ATOMIC_RELAXED,
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
              if (lane_is_pill(expect)) on = false;
              else not_there();
            }
          }
          if (on) {
            sent[place] = rec | (((x.c_back >> 20) & 31u) << 16);
            // the call is opened; its value is outstanding
            ++x.n_tags;
            x.n_tokens += x.c_np;
            x.mx_depth = x.depth + 1u > x.mx_depth ? x.depth + 1u : x.mx_depth;
            atomicAdd(&r_join[rec], 1u);
            const uint32_t fn = lane_fn(x.st), opened = lane_opened(x.c_back);
            x.st = lane_state(fn, opened, SW::outstanding(fn, opened, x.present));
            x.act = ACT_NONE;
            resumed = false;
          }
          for (unsigned long long m = __ballot(on); m; m &= m - 1ull)   // (the places of the calls that went)
            sent_mask |= 1ull << (uint32_t)__builtin_amdgcn_readlane((int)place, __ffsll((long long)m) - 1);
          hungry = n_got < n ? 0u : hungry - n_got;
        }
      }
      {
        if (x.run && x.act == ACT_CALL) {
          if (sp - lo == LANE_WINDOW) evict();   // (the window's oldest frame makes room)
          uint4 c[NC];
          pack(c, x.c_back, x.more);
          win_put(sp, c);
          slack += x.more ? 1u : 0u;
          ++sp;
          mx_sp = sp - bs > mx_sp ? sp - bs : mx_sp;
          x.st = x.c_st;
          x.label = x.c_label;
          x.counter = 0;
          x.depth += 1;
          x.present = (1u << x.c_np) - 1u;
#pragma unroll
          for (int j = 0; j < NS; ++j) x.sv[j] = x.arg[j];
          ++x.n_tags;
          x.n_tokens += x.c_np;
          x.mx_depth = x.depth > x.mx_depth ? x.depth : x.mx_depth;
        } else if (x.run && x.act == ACT_RET) {
          if (sp > bs) {
            ++x.n_tokens;
            pop(x.ret);
          } else {
            x.run = false;   // to a record or another wave: below
          }
        }
      }
      if (__ballot(x.run && x.act > ACT_RET)) {
        bool done = false, next_bottom = false;
        if (!x.run) {
        } else if (x.act == ACT_NEXT) {
          if (x.counter >= 0xFFFFFFu) x.bad = TDF_ERR_STEP_LIMIT;
          ++x.counter;
          x.st = x.c_st;
          x.present = (1u << x.c_np) - 1u;
#pragma unroll
          for (int j = 0; j < NS; ++j) x.sv[j] = x.arg[j];
          ++x.n_tags;
          x.n_tokens += x.c_np;
          x.mx_depth = x.depth > x.mx_depth ? x.depth : x.mx_depth;
          next_bottom = sp == bs && rec != LANE_NONE;
        } else if (x.act == ACT_DONE) {
          x.run = active = false;
          done = true;
        } else if (x.act == ACT_WAIT && sp == bs && rec != LANE_NONE && !resumed) {
          x.run = false;     // below
        } else if (x.act > ACT_RET) {
          x.bad = x.bad ? x.bad : TDF_ERR_UNSUPPORTED;
          x.run = false;
        }
        n_own -= (uint32_t)__popcll(__ballot(done));
        any_done = any_done || __ballot(done) != 0;
        // a finished iteration, or instance, whose frame had a record
        free_recs((done || next_bottom) && rec != LANE_NONE, rec);
        if (done || next_bottom) rec = LANE_NONE;
      }
    }
    ++syncs;

    // ---- values for records and for other waves, and frames that wait for others
    {
      const bool ret = active && !x.run && x.act == ACT_RET && x.bad == 0;
      const bool wait = active && !x.run && x.act == ACT_WAIT && x.bad == 0;
      if (__ballot(ret || wait)) {
        const bool out = ret;
        free_recs(out && rec != LANE_NONE, rec);
        if (out) ++x.n_tokens;
        const bool remote = out && (parent & LANE_REMOTE) != 0;
        if (remote) {
          LaneReply* const rp = a.reply + (parent & ~LANE_REMOTE);
          lane_put(&rp->value, (unsigned long long)x.ret);
          __builtin_amdgcn_s_waitcnt(0);
          lane_put(&rp->flag, 1ull);
        }
        // to a stack that nobody runs: it is this lane's from now on
        const bool stack = out && !remote && (parent & LANE_STACK) != 0;
        const uint32_t stack_rec = parent & ~LANE_STACK;
        if (__builtin_expect(__ballot(stack) != 0, 0)) {
          if (stack) {
            const uint32_t m = r_meta[stack_rec];
            bs = r_counter[stack_rec];
            sp = lo = r_depth[stack_rec];
            seg = r_po[stack_rec];
            seg_b = r_join[stack_rec];
            parent = r_parent[stack_rec];
            rec = (m & 0xFFFFu) == 0xFFFFu ? LANE_NONE : m & 0xFFFFu;
            resumed = (m >> 31) != 0;
            slack = 0;
            pop(x.ret);
            x.run = true;
            x.act = ACT_NONE;
          }
          free_recs(stack, stack_rec);
        }
        bool last = false;
        uint32_t id = rec;
        if (out && !remote && !stack) {
          id = parent;
          last = deliver(id, SW::ret_slot(x.label), x.ret);
        }
        if (wait) {   // (values of this lane; those outstanding may be written by others meanwhile)
#pragma unroll
          for (int k = 0; k < NS; ++k)
            if ((x.present >> k) & 1) r_val[k * LANE_RECS + id] = (unsigned long long)x.sv[k];
          atomicOr(&r_po[id], x.present | (lane_opened(x.st) << 24));
          last = atomicSub(&r_join[id], 1u) == 1u;
        }
        if ((out && !stack) || wait) {
          active = x.run = false;
          x.act = ACT_NONE;
        }
        resume(last, id);   // (taken at once, most likely by this lane)
      }
    }
    raise_status();   // (before the instances that it concerns count as done)
    if (stop) break;
    if (any_done && n_own == 0) {
      instances_done();
      if (stop) break;
    }
    if (__builtin_expect((syncs & 15u) == 0, 0)) {
      if (given_up() != 0) break;
    }
    if (__builtin_expect((syncs & 63u) == 0, 0)) {   // (rarely: a run that is refused may as well be a little longer)
      if (lane == 0) (void)lane_add(&ctl->beat, 1u);   // (a clock and the time of the last beat cost 20 registers, fib(0..20) 4 %)
      const unsigned long long told = lane_ld(&ctl->n_tags);
      const uint32_t n = wave_usum(x.n_tags);   // (modulo 2^32, like the difference)
      if (n - n_told >= a.tags_at_once) {
        if (lane == 0) (void)lane_add(&ctl->n_tags, (unsigned long long)(n - n_told));
        n_told = n;
      }
      if (__ballot(told > a.max_tags)) {
        x.bad = TDF_ERR_TABLE_FULL;
        raise_status();
        break;
      }
    }

    // ---- sharing
    {
      const uint32_t nq = qt - qh;
      const unsigned long long rich = __ballot(x.run && slack > 0);
      const uint32_t n_idle = 64u - (uint32_t)__popcll(__ballot(active) | exporter);
      // Calls go to other waves early on, while many of them have nothing, and later from waves whose own lanes
      // have work: a wave with a handful of them keeps what it has (it is little by then).  That a wave looks for
      // others at every sharing, with up to 56 lanes idle, and not only with 16 at most and on every fourth, takes
      // fib(30) + fib(31) + fib(32) from 7.4 to 5.9 ms on average and 256 instances of tak from 5.4 to 3.4 (with 32: 6.7 and
      // 4.7, with 64: 6.6 and 3.6); one large frame on a lane of a wave that has little else was where a run ended.
      const bool early = iter < LANE_EARLY;
      hungry = n_idle <= LANE_GIVE || early ? hungry : 0u;
      if (exporter && (rich || nq) && (early || n_idle <= LANE_GIVE)) {
        const unsigned long long ht = lane_ld(reinterpret_cast<const unsigned long long*>(&a.queues[look].head));
        send_queue = look;
        look = look + 1u == a.n_queues ? 0u : look + 1u;
        const int d = (int)((uint32_t)ht - (uint32_t)(ht >> 32));   // tickets without a task
        hungry = (uint32_t)__builtin_amdgcn_readfirstlane(d > 0 ? d : 0);
        if (early && n_idle > LANE_GIVE && hungry < 8u) hungry = 0;
      }
      // Tasks wanted: for the wave's idle lanes, and some for waves without work.  A lane gives the oldest
      // frame of its stack that has a ready call left (the largest piece of work).
      const uint32_t want = n_idle + min(hungry, 16u);
      bool going = x.run && slack > 0 && want > nq && (uint32_t)__popcll(rich & lanemask_lt()) < want - nq;
      // the values of a frame for its record: all but those outstanding, which others may have put there already; what
      // is not present may be the argument of a call that waits
      auto put_frame = [&](const uint4 (&c)[NC], uint32_t id, uint32_t below, bool fresh, bool more) {
        const uint32_t fn = lane_fn(c[0].x), opened = lane_opened(c[0].x), present = c[0].w;
        if (fresh) {
          r_parent[id] = below;
          r_meta[id] = (c[0].x >> 26) | (fn << 16);
          r_counter[id] = c[0].y;
          r_depth[id] = c[0].z;
          r_inst[id] = x.inst;
          r_join[id] = more ? 2u : 1u;   // the call that the frame waits for, and the task
          r_po[id] = present | (opened << 24);
        } else {
          r_meta[id] &= ~(1u << 31);
          atomicOr(&r_po[id], present | (opened << 24));
          if (more) atomicAdd(&r_join[id], 1u);   // one more call outstanding; the lane's own part goes to the task
        }
        const uint32_t others = SW::ret_bits(fn, opened) & ~present;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const uint4 w = c[1 + k / 2];
          const unsigned long long v = k & 1 ? ((unsigned long long)w.z | ((unsigned long long)w.w << 32))
                                             : ((unsigned long long)w.x | ((unsigned long long)w.y << 32));
          if (!((others >> k) & 1)) r_val[k * LANE_RECS + id] = v;
        }
      };
      // Frames below it become records of their own as far as they are few and records plenty: a value for a record
      // costs a few LDS accesses, one for a stack a round trip to memory (with stacks alone fib(30) + fib(31) + fib(32)
      // takes 7.2 ms instead of 5.2, 256 instances of tak 3.4 instead of 2.7).
      if (spare_recs() >= LANE_SCARCE && __ballot(going)) {
        uint32_t below = parent, d = bs;   // the caller of frame d
        bool moved = false;
        for (uint32_t few = 0; few < LANE_FEW; ++few) {
          if (__ballot(going) == 0) break;
          // a record each (as far as there are any: a lane without one keeps its frames)
          const bool fresh = going && !(d == bs && rec != LANE_NONE);
          const unsigned long long rm = __ballot(fresh);
          const uint32_t rr = (uint32_t)__popcll(rm & lanemask_lt()), n_spare = spare_recs();
          const bool ok = going && (!fresh || rr < n_spare);
          const uint32_t id = !fresh ? rec : ok ? lfree[nfree - 1 - rr] : 0u;
          nfree -= min(n_spare, (uint32_t)__popcll(rm));
          min_free = min(min_free, nfree);
          bool more = false;
          if (ok) {
            uint4 c[NC];
            if (d >= lo) {
              win_get(d, c);
            } else {
              mem_get(seg_b, d, c);
              if (d % LANE_SEG == LANE_SEG - 1u || d + 1u == lo) {   // that was the segment's last frame
                const uint32_t sid = seg_b;
                seg_b = d + 1u == lo ? LANE_NONE : seg_at(sid)[0].y;
                if (d + 1u == lo) seg = LANE_NONE;
                drop_seg(sid);
              }
            }
            more = ((c[0].x >> 25) & 1u) != 0;   // it becomes a task
            put_frame(c, id, below, fresh, more);
            slack -= more ? 1u : 0u;
            below = id;
            ++d;
            moved = true;
          }
          push_tasks(ok && more, id);
          going = ok && d < sp && !more;
        }
        if (moved) {
          bs = d;
          lo = lo > d ? lo : d;
          parent = below;
          rec = LANE_NONE;
          resumed = false;
        }
      }
      // Else all of them stay a stack, with one record.
      if (__builtin_expect(spare_recs() >= 2 && __ballot(going) != 0, 0)) {
        uint32_t d = bs, in = seg_b;   // the frame, and the segment it is in if it is in memory
        if (going) {
          while (!(((d >= lo ? win[((d % LANE_WINDOW) * NC) * 64 + lane].x : seg_at(in)[1 + (d % LANE_SEG) * NC].x) >> 25) & 1u)) {
            ++d;
            if (d < lo && d % LANE_SEG == 0) in = seg_at(in)[0].y;
          }
        }
        // a record for the frame, unless it has one, and one for the stack, unless there is none (a lane for which there
        // are not enough keeps its frames)
        const bool fresh = going && !(d == bs && rec != LANE_NONE), stack = going && d > bs;
        const unsigned long long fm = __ballot(fresh), sm = __ballot(stack);
        const uint32_t before = (uint32_t)__popcll(fm & lanemask_lt()) + (uint32_t)__popcll(sm & lanemask_lt());
        const uint32_t need = (fresh ? 1u : 0u) + (stack ? 1u : 0u);
        const bool ok = going && (need == 0 || before + need <= spare_recs());
        uint32_t id = rec, below = parent;
        if (ok && fresh) id = lfree[nfree - 1 - before];
        if (ok && stack) {
          const uint32_t s_id = lfree[nfree - 2 - before];   // (a frame above others is fresh)
          uint32_t top = seg, bottom = seg_b;   // the stack's segments
          if (d >= lo) {   // in the window, like all frames above it
            while (lo < d && x.bad == 0) evict();
            top = seg;
            bottom = seg_b;
          } else if (d % LANE_SEG == 0) {
            top = seg_at(in)[0].x;
          } else {
            top = in;
            if (d + 1 < lo && d % LANE_SEG != LANE_SEG - 1u) {   // the lane has frames above it in the same segment: a copy for the stack
              const bool all = d / LANE_SEG == bs / LANE_SEG;
              const uint32_t under = all ? LANE_NONE : seg_at(in)[0].x;
              top = new_seg();
              if (top != LANE_NONE) {
                seg_at(top)[0].x = under;
                if (all) bottom = top;
                else seg_at(under)[0].y = top;
              }
              for (uint32_t k = all ? bs % LANE_SEG : 0u; top != LANE_NONE && k < d % LANE_SEG; ++k) {
#pragma unroll
                for (int j = 0; j < NC; ++j) seg_at(top)[1 + k * NC + j] = seg_at(in)[1 + k * NC + j];
              }
            }
          }
          r_parent[s_id] = parent;
          r_counter[s_id] = bs;
          r_depth[s_id] = d;
          r_po[s_id] = top;
          r_join[s_id] = bottom;
          r_meta[s_id] = (rec & 0xFFFFu) | (resumed ? 1u << 31 : 0u);
          below = LANE_STACK | s_id;
        }
        if (sm) __builtin_amdgcn_s_waitcnt(0);   // (a stack's frames are in memory before anybody can see its record)
        if (ok) {
          uint4 c[NC];
          if (d >= lo) {
            win_get(d, c);
            seg = seg_b = LANE_NONE;   // (all that was in memory, if anything, is the stack's)
          } else {
            mem_get(in, d, c);
            if (d + 1u == lo) {
              seg = seg_b = LANE_NONE;
              if (d == bs || d % LANE_SEG == 0) drop_seg(in);   // (no frame of the stack is in it)
            } else if (d % LANE_SEG == LANE_SEG - 1u) {
              seg_b = seg_at(in)[0].y;
              if (d == bs) drop_seg(in);
            } else {
              seg_b = in;
            }
          }
          put_frame(c, id, below, fresh, true);
          --slack;
          bs = d + 1u;
          lo = max(lo, bs);
          parent = id;
          rec = LANE_NONE;
          resumed = false;
        }
        const unsigned long long om = __ballot(ok);
        nfree -= (uint32_t)__popcll(fm & om) + (uint32_t)__popcll(sm & om);
        min_free = min(min_free, nfree);
        push_tasks(ok, id);
        raise_status();   // (no segment for a stack: nobody may go on with it)
      }
    }
  }

  // ---- the wave's part of the log that was not used, and its counts
  {
    const uint32_t h0 = x.log_next;
    for (uint32_t h = h0 + lane; h < x.log_end; h += 64)
      if (h < a.log_cap) a.log[h].z = LANE_LOG_HOLE;
    unsigned long long tags = x.n_tags, tokens = x.n_tokens;
    uint32_t leaf = x.n_leaf, cell = x.n_cell, priv = mx_sp;
    for (int off = 32; off > 0; off >>= 1) {
      tags += __shfl_xor(tags, off);
      tokens += __shfl_xor(tokens, off);
      leaf += __shfl_xor(leaf, off);
      cell += __shfl_xor(cell, off);
      priv += __shfl_xor(priv, off);
    }
    const uint32_t md = wave_umax(x.mx_depth), ml = wave_umax(x.mx_level);
    if (lane == 0 && iter) {   // (per queue, summed by the host)
      LaneQueue* q = &a.queues[my_queue];
      (void)lane_add(&q->n_tags, tags);
      (void)lane_add(&q->n_tokens, tokens);
      (void)lane_add(reinterpret_cast<unsigned long long*>(&q->n_leaf), (unsigned long long)leaf | ((unsigned long long)cell << 32));
      (void)lane_add(reinterpret_cast<unsigned long long*>(&q->n_rec), (unsigned long long)(LANE_RECS - min_free) | ((unsigned long long)priv << 32));
      atomicMax(&q->max_depth, md);
      if (ml) atomicMax(&q->max_level, ml);
      atomicMax(&q->max_iter, iter);
    }
  }
}

#endif
}  // namespace tdf
