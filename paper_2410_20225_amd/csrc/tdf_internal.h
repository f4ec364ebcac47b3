// Host-side graph object shared by graph_build.cpp, jit.cpp and eval.hip.
#pragma once
#include <stdint.h>

#include <mutex>
#include <string>
#include <vector>

#include "tdf.h"
#include "tdf_tables.h"

namespace tdf {

// ---- host graph object ----------------------------------------------------------------
struct Graph {
  std::vector<tdf_snode> snodes;
  std::vector<tdf_sedge> sedges;
  DevProgram prog;
  int n_labels = 0;
  int n_result_params = 0;
  int cell_kind = 0;        // 0 none, 1 RNN, 2 LSTM
  bool has_embed = false, has_head = false, has_node_loss = false, want_grad = false;
  int out_type = T_INT;     // type of result's output
};

void set_error(const std::string& msg);

// The end of an evaluation: what its last kernel leaves in pinned memory for the host; `seq` is written last.
struct EndReport {
  LaneTotals t;
  uint32_t sync[32][32];          // DieSync records of the chain launches (forward, gradient; deep instances and others)
  unsigned long long gcount[2];
  unsigned long long stamps[2 * TDF_PHASE_COUNT];
  uint32_t seq;
};
struct EndArgs {
  EndReport* end;
  const unsigned long long* stamps;
  const unsigned long long* gcount;   // null: no gradient pass
  const void* sync;                   // null: no chain launch
  uint32_t seq;
  uint32_t lanes_max_tags;            // 0, or: the lanes' totals are wanted, and this is the limit on tags
};

// Run-time generated step kernels for one program (jit.cpp).  Returns false (and leaves the
// handles null) when the run-time compiler is unavailable, disabled (TDF_NO_JIT=1) or fails;
// the table interpreter is used then.
struct JitKernels {
  void* module = nullptr;   // hipModule_t
  void* step = nullptr;     // hipFunction_t of the grid-wide step kernel
  void* step_local = nullptr;   // ... and of its variant that keeps to one accelerator die
  void* small = nullptr;    // hipFunction_t of the single-workgroup kernel
  bool tried = false;
  void* lanes_module = nullptr;   // hipModule_t of the depth-first lanes, compiled when an evaluation without frames first runs
  void* lanes = nullptr;          // hipFunction_t
  bool lanes_tried = false;
};
bool jit_compile(const DevProgram& P, JitKernels& out, std::string& log);
bool jit_compile_lanes(const DevProgram& P, JitKernels& out, std::string& log);
// Programs that are a recursion over the children of tree nodes (forest_walk.hip).
struct WalkForm {
  int ok = 0;
  int root_arg = 0, label_arg = -1;   // arguments of `result`: the instance's root, its label (-1: no head)
  int swapped = 0;                    // the cell's first operand is the right child
};
WalkForm walk_form(const DevProgram& P);
int lane_stored(const DevProgram& P);   // stored values of a frame (the largest function's)
bool lane_branching(const DevProgram& P);   // a frame (other than of `result`) can have several calls or loops
void jit_release(JitKernels& k);

}  // namespace tdf

struct tdf_graph {
  tdf::Graph g;
  tdf::JitKernels jit;
  bool die_local = true;    // tag machines keep to one accelerator die each (cleared if the GPU spreads them)
  // A run that the depth-first lanes leave to the step machine costs their time too: where that then answers it, the next
  // lanes_skip evaluations do not try them, and twice as many after the next such run (other inputs may be theirs again).
  uint32_t lanes_skip = 0, lanes_skip_next = LANES_SKIP;
  static constexpr uint32_t LANES_SKIP = 8, LANES_SKIP_MOST = 1024;
  // The same for a walk over the forest that was left to the lanes.
  tdf::WalkForm walk;
  bool walk_known = false;
  uint32_t walk_skip = 0, walk_skip_next = LANES_SKIP;
  uint32_t max_dies = 8;    // tag machines a batch is dealt to (set to 1 after a part of the table overflowed)
  void* side_stream = nullptr;                     // hipStream_t for work beside the caller's stream
  void* fork_event = nullptr, *join_event = nullptr;   // embedding gradient beside the weight gradients
  void* fork_deep = nullptr, *join_deep = nullptr;     // deep instances beside the others
  void* sort_stream = nullptr;                     // hipStream_t for the embedding gradient's token sort
  void* fork_sort = nullptr;                       // ... which starts once the leaves are known
  // pinned host memory for what an evaluation reads back or sends (control blocks, level offsets,
  // barrier records, the firing tables): copies to and from pageable memory are staged and slower
  void* pinned = nullptr;
  size_t pinned_bytes = 0;
  uint32_t seq = 0;         // of the last report awaited there
  std::mutex busy;          // one evaluation at a time uses the graph's streams, events and host buffer
  bool prepared = false;    // tdf_graph_prepare has run: kernels compiled, events and host buffers exist
  int prepared_device = -1;
  ~tdf_graph();
};
