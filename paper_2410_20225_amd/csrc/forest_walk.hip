// Structural recursion over the forest: the tag phase of programs whose calls follow the children of a tree node.
//
// A function f(v) = cell(f(left v), f(right v)) at inner nodes, embed(token v) at leaves, has one tag per visit of a node:
// Call_i of its two calls are the edges to the children, Return_i the edges back.  Where every node is visited at most
// once, tags and nodes are the same thing, and what the tag machine would log (lane_device.h) follows from the forest
// alone: a leaf fires its EMBED, an inner node its cell when both children have, one level above the higher of them.
// A tree that lies in one piece is numbered where it lies (tree_in_piece).  Any other one wave walks, an instance each: a
// lane goes down to the left child and leaves the right one on a stack in LDS, which lanes without a node take from; a
// leaf turns the lane round, and the second of two children that arrive at their parent goes on up.  The schedule log is
// indexed by node, so a value's name is its node.
//
// The rule: programs of that form (walk_form, below) and forests of at most as many nodes as the log has entries.  One wave
// works on an instance, at 32 nodes a step where the tree is wide, 0.02 to 0.03 us a node; the lanes share a tree
// between waves, at some 3 us a level and, with all of them busy, 0.003 us a node of all instances.  So a wave leaves a wide tree to
// them (16 nodes a step and more) once it is, or the trees are on average, of more than 6,000 nodes, 150 for every level down and a
// twelfth of the forest.  us of an evaluation, all nodes walked -> left to the lanes (and the call whose walk is left): one complete
// tree of 16,384 leaves 850 -> 287 (397), a random one of 16,384 1,197 -> 611 (763), of 8,192 665 -> 522, a complete one of 30,000
// with 63 of 20 beside it 1,539 -> 366 (803), eight complete ones of 16,384 777 -> 465 (575), eight random ones 1,205 -> 1,340.
// Walked all the same (lanes): a complete tree of 4,096 leaves 248 us (226), a random one of 4,096 377 (450), 64 complete ones of
// 16,384 1,035 (849), 64 random ones 1,463 (2,372); chains of any length, 16,384 leaves 40.1 ms (66.8).  More than WALK_NODES
// nodes an instance on average, more than those, were not measured and go to the lanes.
// A forest whose nodes are shared (between parents or instances), or have bad entries, leaves a status, and the lanes run the
// evaluation; what they make of it counts.  (The figures here and below are of trees that are walked; for those in one
// piece see tree_in_piece.)
//
// What bounds the walk: the latency of one request per level down (the node's entries) and one up (the parent's word, in the die's
// L2), and some 150 instructions a step: 1.4 us a level there and back, where the lanes' sweeps take 3.3.
// The tag phase, lanes -> walk: one tree of 35 leaves 94 -> 22 us, 50 trees of up to 50 leaves 128 -> 28, 1,024 trees 205 ->
// 37, 4,096 trees of up to 128 leaves, a fifth of them chains, 620 -> 240, 64 chains of 4,096 leaves 13.5 -> 5.8 ms.
#include "engine.h"
#include "lane_device.h"
#include "tdf_internal.h"

namespace tdf {

// ---- which programs ---------------------------------------------------------------------------------
// The instruction that makes value v of function f, looking through identities; null: none.
static const Instr* maker(const DevProgram& P, int f, int v) {
  for (int hops = 0; v < SRC_NONE && hops < MAX_VALUES; ++hops) {
    const Instr* found = nullptr;
    for (int i = 0; i < P.fn[f].count; ++i) {
      const Instr& I = P.instr[P.fn[f].first + i];
      if (I.op == D_CALL || I.op == D_OUT || I.op == D_NEXT) continue;   // (no value)
      if (I.dst == v || (I.op == D_SWITCH && I.dst + 1 == v)) found = &I;
    }
    if (!found || found->op != D_ID) return found;
    v = found->src[0];
  }
  return nullptr;
}
static int count_of(const DevProgram& P, int f, DevOp op) {
  int n = 0;
  for (int i = 0; i < P.fn[f].count; ++i) n += P.instr[P.fn[f].first + i].op == op;
  return n;
}
static const Instr* only(const DevProgram& P, int f, DevOp op) {
  for (int i = 0; i < P.fn[f].count; ++i)
    if (P.instr[P.fn[f].first + i].op == op) return &P.instr[P.fn[f].first + i];
  return nullptr;
}
// the argument of the one-parameter call with this label; its callee must be g
static const Instr* call_of(const DevProgram& P, int f, int label, int g) {
  const Instr* c = nullptr;
  for (int i = 0; i < P.fn[f].count; ++i) {
    const Instr& I = P.instr[P.fn[f].first + i];
    if (I.op != D_CALL || I.aux != label) continue;
    if (c) return nullptr;
    c = &I;
  }
  return c && P.label_callee[label] == g ? c : nullptr;
}
WalkForm walk_form(const DevProgram& P) {
  WalkForm w;
  if (P.n_fn != 2) return w;
  const int r = P.result_fn, f = 1 - r;
  if (P.fn[f].n_params != 1) return w;
  // result: IN.., one call of f with a parameter, OUT of its value or of HEAD(value, parameter)
  const Instr* out = only(P, r, D_OUT);
  if (!out || count_of(P, r, D_CALL) != 1 || count_of(P, r, D_RET) != 1 || count_of(P, r, D_HEAD) > 1) return w;
  const Instr *head = only(P, r, D_HEAD), *ret = only(P, r, D_RET);
  int others = P.fn[r].count - count_of(P, r, D_IN) - count_of(P, r, D_ID) - 3 - (head ? 1 : 0);
  if (others != 0 || maker(P, r, out->src[0]) != (head ? head : ret)) return w;
  const Instr* call = call_of(P, r, ret->aux2, f);
  const Instr* arg = call ? maker(P, r, call->src[0]) : nullptr;
  if (!arg || arg->op != D_IN) return w;
  w.root_arg = arg->aux;
  if (head) {
    const Instr *row = maker(P, r, head->src[0]), *label = maker(P, r, head->src[1]);
    if (row != ret || !label || label->op != D_IN) return w;
    w.label_arg = label->aux;
  }
  // f: IN v, ISLEAF v, SWITCH(isleaf, v), TOKEN(leaf side) -> EMBED, LEFT and RIGHT(inner side) -> two calls of f -> CELL,
  // MERGE of the two rows, CE_NODE(row, v) if any, OUT
  for (DevOp op : {D_IN, D_ISLEAF, D_SWITCH, D_TOKEN, D_EMBED, D_LEFT, D_RIGHT, D_CELL, D_MERGE, D_OUT})
    if (count_of(P, f, op) != 1) return w;
  const Instr *v = only(P, f, D_IN), *sw = only(P, f, D_SWITCH), *cell = only(P, f, D_CELL), *merge = only(P, f, D_MERGE);
  const Instr *ce = only(P, f, D_CE_NODE), *embed = only(P, f, D_EMBED), *token = only(P, f, D_TOKEN);
  if (count_of(P, f, D_CALL) != 2 || count_of(P, f, D_RET) != 2 || count_of(P, f, D_CE_NODE) > 1) return w;
  others = P.fn[f].count - count_of(P, f, D_ID) - 10 - 4 - (ce ? 1 : 0);
  if (others != 0) return w;
  auto side = [&](int value, int which) {   // value is that side of the switch (identities in between)
    for (int hops = 0; value < SRC_NONE && hops < MAX_VALUES; ++hops) {
      if (value == sw->dst + which) return true;
      const Instr* id = nullptr;
      for (int i = 0; i < P.fn[f].count; ++i) {
        const Instr& I = P.instr[P.fn[f].first + i];
        if (I.op == D_ID && I.dst == value) id = &I;
      }
      if (!id) return false;
      value = id->src[0];
    }
    return false;
  };
  const Instr* isleaf = maker(P, f, sw->src[0]);
  if (!isleaf || isleaf->op != D_ISLEAF || maker(P, f, isleaf->src[0]) != v || maker(P, f, sw->src[1]) != v) return w;
  if (!side(token->src[0], 0) || maker(P, f, embed->src[0]) != token) return w;
  const Instr* kids[2] = {maker(P, f, cell->src[0]), maker(P, f, cell->src[1])};
  const Instr* ends[2] = {nullptr, nullptr};
  for (int k = 0; k < 2; ++k) {
    if (!kids[k] || kids[k]->op != D_RET) return w;
    const Instr* c = call_of(P, f, kids[k]->aux2, f);
    ends[k] = c ? maker(P, f, c->src[0]) : nullptr;
    if (!ends[k] || (ends[k]->op != D_LEFT && ends[k]->op != D_RIGHT) || !side(ends[k]->src[0], 1)) return w;
  }
  if (ends[0]->op == ends[1]->op) return w;
  int rows = 0, from = 0;   // the merge's inputs: the two rows, nothing else
  for (int k = 0; k < 4; ++k) {
    if (merge->src[k] == SRC_NONE) continue;
    const Instr* m = maker(P, f, merge->src[k]);
    ++rows;
    from |= m == embed ? 1 : m == cell ? 2 : 4;
  }
  if (rows != 2 || from != 3) return w;
  const Instr* end = maker(P, f, only(P, f, D_OUT)->src[0]);
  if (ce ? end != ce || maker(P, f, ce->src[0]) != merge || maker(P, f, ce->src[1]) != v : end != merge) return w;
  w.swapped = ends[0]->op == D_RIGHT;
  w.ok = true;
  return w;
}

// ---- the walk ----------------------------------------------------------------------------------------
constexpr uint32_t WALK_STACK = 512;            // nodes on a wave's stack in LDS
constexpr uint32_t WALK_ROOT = 0xFFFFFFFEu;     // parent of an instance's root
constexpr uint32_t WALK_NONE = 0xFFFFFFFFu;     // no node

// On entry log[v].z is LANE_LOG_HOLE for all nodes.  row_of[v] becomes v's parent (until the rows are numbered), log[v] the
// entry of v's EMBED or cell; before that log[v].z is the level of the first child that is through.  All that concerns a
// tree is written and read by its wave, in one die's L2: past the L1 where it is read.
// A node that is visited twice is not noticed here: its leaves count twice then, and the pass over the log, which meets
// every node once, finds fewer.  What has to hold is that nothing leaves the arrays and that the walk ends, on any forest and
// whatever waves with the same nodes write: indices are checked, and no wave makes more visits or cells than there are nodes.
template <typename T> __device__ __forceinline__ T* at32(T* base, uint32_t i) {   // (a uniform base and 32 bits of offset)
  return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (uint32_t)(i * (uint32_t)sizeof(T)));
}
template <typename T> __device__ __forceinline__ const T* at32(const T* base, uint32_t i) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (uint32_t)(i * (uint32_t)sizeof(T)));
}
__device__ __forceinline__ void walk_root(const LaneArgs& a, const WalkForm& w, uint32_t b, uint32_t name, uint32_t level) {
  a.root_lvl[b] = level;
  if (w.label_arg >= 0) {
    a.head_row[b] = name;
    a.head_label[b] = (uint32_t)a.args[(size_t)b * a.n_args + w.label_arg];
  } else {
    a.root_ref[b] = name;
  }
}
// An instance's part of the totals, by one lane.
__device__ __forceinline__ void walk_count(const LaneArgs& a, uint32_t b, uint32_t leaves, uint32_t cells, uint32_t frames, uint32_t depth,
                                           uint32_t level, uint32_t steps) {
  LaneQueue* q = &a.queues[b % a.n_queues];
  const unsigned long long tags = (unsigned long long)leaves + cells;
  (void)lane_add(&q->n_tags, tags);
  (void)lane_add(&q->n_tokens, 2ull * tags);   // an argument and a value each
  (void)lane_add(reinterpret_cast<unsigned long long*>(&q->n_leaf), leaves | ((unsigned long long)cells << 32));
  (void)lane_add(reinterpret_cast<unsigned long long*>(&q->n_rec), (unsigned long long)frames);
  atomicMax(&q->max_depth, depth);
  if (level) atomicMax(&q->max_level, level);
  atomicMax(&q->max_iter, steps);
}

// ---- trees that lie in one piece -----------------------------------------------------------------------
// A tree whose nodes are neighbours in memory, the root at one end and every parent on the root's side of its children
// (depth first or level by level, from the first node on or from the last), needs no walk: its workgroup holds it in LDS, where
// it ends follows from counting (the nodes still open: one more with every inner node, one less with every leaf), and the
// heights come from doubling: every node knows an ancestor 2^k edges up and tells it the height of what is below itself, then
// takes that ancestor's ancestor.  ceil(log2 depth) rounds of LDS instead of two requests to the L2 a level.
// What the nodes are taken for is checked: n - 1 links that all lead to different nodes of the piece, and from all of which the root
// is reached, are a tree.  Whatever fails (another order, nodes in between, shared nodes, bad entries, more than WINDOW nodes)
// is walked, which says what is wrong.
// What bounds it: a dozen LDS accesses a node and round, and the barriers of the rounds where a workgroup has more than one wave.
// The tag phase in us, walked -> this: one tree of 35 leaves 24 -> 14.5 (two launches), 256 trees of up to 50 leaves 26 -> 14, 1,024 of
// up to 60 33 -> 15, 4,096 of up to 128, a fifth of them chains, 240 -> 23, 64 chains of 4,096 leaves and 64 complete trees of as many
// 5,894 -> 68.
constexpr uint32_t WALK_ANC = 0xFFFFu;   // low half of a node's word: the ancestor it has got to; high half: how far that is
template <int THREADS, int WINDOW>
__device__ __forceinline__ bool tree_in_piece(const LaneArgs& a, const WalkForm& w, uint32_t b, uint32_t root, uint32_t* s_up, uint32_t* s_high,
                                              uint32_t* s_tot, uint32_t* s_end) {
  constexpr int K = WINDOW / THREADS, NW = THREADS / 64;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, n_nodes = (uint32_t)a.n_tree_nodes;
  const int first = a.left[root];
  const bool ahead = first < 0 || (uint32_t)first > root;   // the children lie behind their parent, or all the other way round
  const uint32_t room = min((uint32_t)WINDOW, ahead ? n_nodes - root : root + 1u);
  auto node = [&](uint32_t i) { return ahead ? root + i : root - i; };
  auto place = [&](int v) { return ahead ? (uint32_t)v - root : root - (uint32_t)v; };   // (a huge one if it is not there)
  int el[K], er[K];   // left and right child of the thread's nodes; a leaf: negative, token
  auto entries = [&](int c) {
    const uint32_t i = (uint32_t)c * THREADS + tid;
    el[c] = -1;
    er[c] = 0;
    if (i < room) {
      const uint32_t v = node(i);
      const int l = *at32(a.left, v), r = *at32(a.right, v), t = *at32(a.token, v);
      el[c] = l;
      er[c] = l < 0 ? t : r;
    }
  };
  // ---- the nodes' links, up to the one that leaves nothing open
  if (tid == 0) *s_end = WALK_NONE;
  uint32_t n = WALK_NONE;   // (uniform, as are the trip counts)
  int open = 1;
  entries(0);
#pragma unroll
  for (int c = 0; c < K; ++c) {
    if (n != WALK_NONE || (uint32_t)c * THREADS >= room) break;
    if (c + 1 < K) entries(c + 1);   // (on their way meanwhile)
    const uint32_t i = (uint32_t)c * THREADS + tid;
    const unsigned long long inner = __ballot(i < room && el[c] >= 0);
    int at = open, after = open;   // open before the wave's first node, and behind the last of all
    if constexpr (NW > 1) {
      if ((tid & 63u) == 0) s_tot[wave] = (uint32_t)__popcll(inner);
      __syncthreads();
#pragma unroll
      for (uint32_t k = 0; k < NW; ++k) {
        const int d = 2 * (int)s_tot[k] - 64;
        if (k < wave) at += d;
        after += d;
      }
    } else {
      after += 2 * (int)__popcll(inner) - 64;
    }
    const unsigned long long upto = lanemask_lt() | (1ull << (tid & 63u));
    const unsigned long long closed = __ballot(i < room && at + 2 * (int)__popcll(inner & upto) - (int)(tid & 63u) - 1 == 0);
    if constexpr (NW > 1) {
      if (closed && (tid & 63u) == 0) atomicMin(s_end, (uint32_t)c * THREADS + wave * 64u + (uint32_t)__ffsll((long long)closed));
      __syncthreads();
      n = (uint32_t)__builtin_amdgcn_readfirstlane((int)*s_end);
    } else if (closed) {
      n = (uint32_t)c * THREADS + (uint32_t)__ffsll((long long)closed);
    }
    open = after;
    if (i < min(n, room)) {
      s_high[i] = 0;
      if (el[c] >= 0) {
        const uint32_t l = place(el[c]), r = place(er[c]);
        if (l < (uint32_t)WINDOW) s_up[l] = i | 0x10000u;
        if (r < (uint32_t)WINDOW) s_up[r] = i | 0x10000u;
      }
    }
  }
  if (n == WALK_NONE) return false;
  __syncthreads();
  bool good = true;
  uint32_t up[K];
#pragma unroll
  for (int c = 0; c < K; ++c) {
    const uint32_t i = (uint32_t)c * THREADS + tid;
    up[c] = 0;
    if ((uint32_t)c * THREADS < n && i < n) {
      if (i) up[c] = s_up[i];
      if (el[c] >= 0) {
        const uint32_t l = place(el[c]), r = place(er[c]), me = i | 0x10000u;
        good = good && l - 1u < n - 1u && r - 1u < n - 1u && l != r && s_up[min(l, n - 1u)] == me && s_up[min(r, n - 1u)] == me;
      }
    }
  }
  if (!__syncthreads_and(good)) return false;
  // ---- every node tells an ancestor twice as far away as in the round before
  uint32_t rounds = 0;
  for (;; ++rounds) {
    if (rounds > 31u - (uint32_t)__builtin_clz((uint32_t)WINDOW)) return false;   // (a cycle: the piece has no more edges in a row)
    bool on = false;
#pragma unroll
    for (int c = 0; c < K; ++c) {
      const uint32_t p = up[c] & WALK_ANC;
      if ((uint32_t)c * THREADS < n && p) {   // (the root's own height is the greatest distance from it)
        const uint32_t q = s_up[p];
        atomicMax(&s_high[p], s_high[(uint32_t)c * THREADS + tid] + (up[c] >> 16));
        up[c] = (q & WALK_ANC) | ((up[c] & ~WALK_ANC) + (q & ~WALK_ANC));
        on = on || (q & WALK_ANC) != 0;
      }
    }
    if (!__syncthreads_or(on)) break;
#pragma unroll
    for (int c = 0; c < K; ++c)
      if ((uint32_t)c * THREADS < n && (uint32_t)c * THREADS + tid < n) s_up[(uint32_t)c * THREADS + tid] = up[c];
    __syncthreads();
  }
  uint32_t far = 0;
#pragma unroll
  for (int c = 0; c < K; ++c) far = max(far, up[c] >> 16);
  far = wave_umax(far);
  if ((tid & 63u) == 0) atomicMax(&s_high[0], far);
  __syncthreads();
  const uint32_t high = s_high[0];   // of the root
  // ---- the schedule
  bool bad = false;
#pragma unroll
  for (int c = 0; c < K; ++c) {
    const uint32_t i = (uint32_t)c * THREADS + tid;
    if ((uint32_t)c * THREADS < n && i < n) {
      const uint32_t v = node(i);
      const bool leaf = el[c] < 0;
      bad = bad || (leaf && (er[c] < 0 || er[c] >= a.vocab));
      const uint32_t x = (uint32_t)(leaf || w.swapped ? er[c] : el[c]), y = leaf ? 0u : (uint32_t)(w.swapped ? el[c] : er[c]);
      *at32(a.log, v) = make_uint4(x, y, s_high[i], b);
      if (a.row_node) *at32(a.row_node, v) = v;
    }
  }
  if (bad) lane_put(&a.ctl->status, (uint32_t)(-TDF_ERR_BAD_ARG));
  if (tid == 0) {
    walk_root(a, w, b, root, high);
    walk_count(a, b, (n + 1u) / 2u, n / 2u, n, high + 1u, high, rounds);
  }
  return true;
}

// One wave walks the tree of instance b.  `lds`: 3 * WALK_STACK words.
__device__ __forceinline__ void walk_tree(const LaneArgs& a, const WalkForm& w, uint32_t b, long long root, uint32_t* lds) {
  const uint32_t lane = threadIdx.x, n_nodes = (uint32_t)a.n_tree_nodes;
  uint32_t* const s_node = lds;
  uint32_t* const s_parent = lds + WALK_STACK;
  uint32_t* const s_depth = lds + 2 * WALK_STACK;
  uint32_t n_stack = 0, most = 0, iter = 0;   // (uniform)
  bool down = false, up = false;
  uint32_t v = 0, p = WALK_ROOT, depth = 1, lvl = 0;   // down: node, its parent and depth; up: level of a node that is through, its parent
  uint32_t own = WALK_NONE;                   // nodes for which the stack had no room: a list through the log entries of these
  uint32_t n_leaf = 0, n_inner = 0, n_cell = 0, mx_depth = 0, mx_level = 0;
  int bad = 0;
  if (root < 0 || root >= (long long)n_nodes) bad = TDF_ERR_BAD_ARG;
  else if (lane == 0) {
    v = (uint32_t)root;
    down = true;
  }
  bool lists = false;   // (uniform) a lane has had a list of its own
  const uint32_t average = n_nodes / a.n_inst;
  for (;;) {
    if (__builtin_expect(__ballot(bad != 0) != 0, 0)) break;
    // ---- lanes without a node take one of the stack, or of their own list
    unsigned long long idle = ~__ballot(down || up);
    if (idle != 0 && n_stack != 0) {
      const uint32_t n_take = min(n_stack, (uint32_t)__popcll(idle)), rank = (uint32_t)__popcll(idle & lanemask_lt());
      if (!down && !up && rank < n_take) {
        const uint32_t i = n_stack - 1u - rank;
        v = s_node[i];
        p = s_parent[i];
        depth = s_depth[i];
        down = true;
      }
      n_stack -= n_take;
      idle = ~__ballot(down || up);
    }
    if (__builtin_expect(lists, 0)) {
      if (!down && !up && own != WALK_NONE) {
        v = own;
        const uint4* e = at32(a.log, v);
        own = lane_ld(&e->x);
        p = lane_ld(&e->y);
        depth = lane_ld(&e->w);
        down = p < n_nodes && (own < n_nodes || own == WALK_NONE);   // (else another instance has been here)
        if (!down) bad = TDF_ERR_UNSUPPORTED;
      }
      idle = ~__ballot(down || up || bad != 0);
    }
    if (idle == ~0ull) break;
    ++iter;
    // ---- one request of every lane
    int l = 0, r = 0, t = 0;
    uint32_t was = 0, pp = 0;
    if (down) {
      l = *at32(a.left, v);
      r = *at32(a.right, v);
      t = *at32(a.token, v);
    }
    if (up) {
      pp = lane_ld(at32(a.row_of, p));
      was = __hip_atomic_exchange(&at32(a.log, p)->z, lvl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // (Waited for here, together: the compiler would do so on each way, and on the second behind the first one's stores.)
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    // ---- up: the first child to arrive leaves its level, the second goes on
    bool push = false;
    if (up) {
      up = was != LANE_LOG_HOLE;
      if (up) {
        lvl = 1u + max(lvl, was);
        at32(a.log, p)->z = lvl;
        ++n_cell;
        if (pp >= n_nodes) {
          up = false;
          mx_level = lvl;
          if (pp == WALK_ROOT) walk_root(a, w, b, p, lvl);
          else bad = TDF_ERR_UNSUPPORTED;   // (another instance has been here)
        }
        p = pp;
      }
    } else if (down) {
      // ---- down: the node's entries
      *at32(a.row_of, v) = p;
      if (a.row_node) *at32(a.row_node, v) = v;
      if (l < 0) {
        if (t < 0 || t >= a.vocab) bad = TDF_ERR_BAD_ARG;
        *at32(a.log, v) = make_uint4((uint32_t)t, 0u, 0u, b);
        ++n_leaf;
        mx_depth = max(mx_depth, depth);
        lvl = 0;
        down = false;
        up = p != WALK_ROOT;
        if (!up) walk_root(a, w, b, v, 0u);
      } else if ((uint32_t)l >= n_nodes || (uint32_t)r >= n_nodes) {
        bad = TDF_ERR_BAD_ARG;
      } else {
        uint4* e = at32(a.log, v);
        *reinterpret_cast<uint2*>(e) = w.swapped ? make_uint2((uint32_t)r, (uint32_t)l) : make_uint2((uint32_t)l, (uint32_t)r);
        e->w = b;
        ++n_inner;
        ++depth;
        push = true;
        p = v;
        v = (uint32_t)l;
      }
    }
    // ---- right children for lanes without a node
    const unsigned long long pm = __ballot(push);
    if (pm) {
      const uint32_t room = WALK_STACK - n_stack, k = (uint32_t)__popcll(pm & lanemask_lt()), n = (uint32_t)__popcll(pm);
      if (push && k < room) {
        s_node[n_stack + k] = (uint32_t)r;
        s_parent[n_stack + k] = p;
        s_depth[n_stack + k] = depth;
      }
      if (__builtin_expect(n > room, 0)) {
        lists = true;
        if (push && k >= room) {
          uint4* e = at32(a.log, (uint32_t)r);   // (nobody has visited it; z stays as it is)
          lane_put(&e->x, own);
          lane_put(&e->y, p);
          lane_put(&e->w, depth);
          own = (uint32_t)r;
        }
      }
      n_stack += min(room, n);
      most = max(most, n_stack);
    }
    if (__builtin_expect((iter & 63u) == 0, 0)) {
      // (A step of the wave is a visit, or a cell, or the first child's arrival, of which there is one a visit or cell: on
      // any forest one of the two counts passes the number of nodes if the walk does not end before.)
      const uint32_t seen = wave_usum(n_leaf + n_inner);
      const bool wide = seen > 16u * iter && max(seen, average) > 6000u + 150u * wave_umax(depth) + n_nodes / 12u;   // (see above)
      if (seen > n_nodes || wave_usum(n_cell) > n_nodes || wide) bad = TDF_ERR_UNSUPPORTED;
      if (lane_ld(&a.ctl->status) != 0) break;   // another wave has left
    }
  }
  const uint32_t leaves = wave_usum(n_leaf), inner = wave_usum(n_inner), cells = wave_usum(n_cell);
  if (bad == 0 && inner != cells) bad = TDF_ERR_UNSUPPORTED;
  const unsigned long long bm = __ballot(bad != 0);
  const uint32_t md = wave_umax(mx_depth), ml = wave_umax(mx_level);
  if (bm) {
    const int code = __shfl(bad, __ffsll((long long)bm) - 1);
    if (lane == 0) lane_put(&a.ctl->status, (uint32_t)(-code));
  } else if (lane == 0) {
    walk_count(a, b, leaves, cells, most + 64u, md, ml, iter);
  }
}

// A workgroup an instance: the tree in one piece, or (walks) what fails as one is walked by the first wave, or left to k_forest_walk.
template <int WINDOW> constexpr size_t piece_lds() {
  return sizeof(uint32_t) * (2 * WINDOW > 3 * (int)WALK_STACK ? 2 * WINDOW : 3 * (int)WALK_STACK);
}
template <int THREADS, int WINDOW>
__global__ void __launch_bounds__(THREADS) k_forest_pieces(LaneArgs a, WalkForm w, bool walks, Stamp st) {
  extern __shared__ uint32_t lds[];   // a piece's words and heights, or the walk's stack
  __shared__ uint32_t s_tot[THREADS / 64], s_end;
  stamp_now(st);
  const uint32_t b = blockIdx.x;
  const long long root = a.args[(size_t)b * a.n_args + w.root_arg];
  if (root >= 0 && root < (long long)a.n_tree_nodes &&
      tree_in_piece<THREADS, WINDOW>(a, w, b, (uint32_t)root, lds, lds + WINDOW, s_tot, &s_end))
    return;
  if (!walks) {
    if (threadIdx.x == 0) a.root_lvl[b] = WALK_NONE;
    return;
  }
  __syncthreads();   // (the others are through with the piece's words)
  if (THREADS > 64 && threadIdx.x >= 64u) return;
  walk_tree(a, w, b, root, lds);
}
// The instances that k_forest_pieces has left, in workgroups of the walk's own size.
__global__ void __launch_bounds__(64) k_forest_walk(LaneArgs a, WalkForm w) {
  __shared__ uint32_t lds[3 * WALK_STACK];
  const uint32_t b = blockIdx.x;
  if (a.root_lvl[b] != WALK_NONE) return;
  walk_tree(a, w, b, a.args[(size_t)b * a.n_args + w.root_arg], lds);
}

template <int THREADS, int WINDOW> static void launch_pieces(const LaneArgs& a, const WalkForm& w, bool walks, const Stamp& st, hipStream_t s) {
  constexpr size_t lds = piece_lds<WINDOW>();
  if (lds > 48 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_forest_pieces<THREADS, WINDOW>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_forest_pieces<THREADS, WINDOW>), dim3(a.n_inst), dim3(THREADS), lds, s, a, w, walks, st);
}
// The workgroup and its window by the nodes of an instance on average: room for a few times as many, where that leaves a compute
// unit enough instances to work on.  Number of launches.
// What is no piece is walked in workgroups of 64 threads and 6 KB, 26 of which fit a compute unit, in a launch of its own: one
// wave would hold the 32 or 128 KB of a piece (five or one on a compute unit) for as long as it walks.  In random order, all in
// one launch -> two, tag phase in us: 512 chains of 3,500 leaves 10,190 -> 5,070, 512 random trees of 3,500 567 -> 463, 2,048 of
// 600 550 -> 348, 4,096 of 800 1,316 -> 852 (1,024 of 300 leaves, five a compute unit at once: 87 -> 102).  Up to two instances of
// 32 KB a compute unit all are resident anyway and leave room for two workgroups of another evaluation's level tails (90 KB),
// and the second launch is only in the way: 256 trees of up to 50 leaves 14 -> 20 us in order, 30 -> 39 in random order, 200 of
// 400 21 -> 24 and 68 -> 79.
int launch_forest_walk(const LaneArgs& a, const WalkForm& w, const Stamp& st, hipStream_t s) {
  const uint32_t average = (uint32_t)a.n_tree_nodes / a.n_inst;
  const bool large = average > 1024u, small = average <= 192u && a.n_inst > 256u;
  const bool walks = small || (!large && a.n_inst <= 512u);
  if (large) launch_pieces<1024, 16384>(a, w, walks, st, s);
  else if (small) launch_pieces<64, 512>(a, w, walks, st, s);
  else launch_pieces<256, 4096>(a, w, walks, st, s);
  if (!walks) hipLaunchKernelGGL(k_forest_walk, dim3(a.n_inst), dim3(64), 0, s, a, w);
  return walks ? 1 : 2;
}

}  // namespace tdf
