// Runs the depth-first lanes on the CPU: lane_device.h and the code generated for one program (generated.inc, as the
// library prints it), on waves of fibers (host_wave.h).  Reads a job of whitespace-separated "key value" pairs and arrays
// ("key n v0 v1 ..."), prints what the run left behind in the same form.
#include "host_wave.h"

#include <map>
#include <string>

static char lds[1];   // (the generated kernel names it; it is not called)
#include "generated.inc"

using namespace tdf;

// An array between inaccessible pages: an index out of range ends the program.
template <typename T> static T* guarded(const std::vector<long long>& v) {
  const size_t page = 4096, room = (size_t)1 << 28, bytes = (v.size() * sizeof(T) + page - 1) / page * page;
  char* p = (char*)mmap(nullptr, 2 * room + bytes, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (p == MAP_FAILED || mprotect(p + room, bytes, PROT_READ | PROT_WRITE)) abort();
  T* a = (T*)(p + room + bytes) - v.size();   // ends at the upper pages
  for (size_t k = 0; k < v.size(); ++k) a[k] = (T)v[k];
  return a;
}

static LaneArgs a;
static void body(uint32_t, char* l) { lanes_run<GeneratedLanes>(a, l); }

int main() {
  std::map<std::string, std::vector<long long>> in;
  char key[64];
  for (long long n; scanf("%63s %lld", key, &n) == 2;) {
    std::vector<long long>& v = in[key];
    for (v.resize((size_t)n); long long& x : v)
      if (scanf("%lld", &x) != 1) return 2;
  }
  auto num = [&](const char* k, long long otherwise) { return in.count(k) ? in[k].at(0) : otherwise; };
  constexpr int NS = GeneratedLanes::kStored;
  a = LaneArgs{};
  a.n_args = (int32_t)num("n_args", 1);
  a.n_inst = (uint32_t)(in["args"].size() / (size_t)max(1, a.n_args));
  if (a.n_args == 0) a.n_inst = (uint32_t)num("n_inst", 1);
  a.n_waves = (uint32_t)num("waves", 1);
  a.per_grab = (uint32_t)num("per_grab", max(1u, min(64u, (a.n_inst + a.n_waves - 1) / a.n_waves)));
  a.n_queues = (uint32_t)num("queues", 1);
  a.queue_cap = (uint32_t)num("queue_cap", 128);
  a.n_segs = (uint32_t)num("segs", 1 << 16);
  a.log_cap = (uint32_t)num("log_cap", 0);
  a.vocab = (int32_t)num("vocab", 0);
  a.idle_ticks = num("idle_ticks", 1ll << 40);
  a.dead_ticks = num("dead_ticks", 1ll << 40);
  a.max_tags = (uint32_t)num("max_tags", 1ll << 30);
  a.tags_at_once = max(64u, a.max_tags / (2u * a.n_waves));
  LaneCtl ctl{};
  std::vector<LaneQueue> queues(a.n_queues);
  std::vector<LaneMail> mail((size_t)a.n_queues * a.queue_cap);
  std::vector<LaneReply> reply(a.n_waves * 64u);
  std::vector<uint4> segs((size_t)a.n_segs * lane_seg_units(NS)), log(max(1u, a.log_cap));
  std::vector<uint32_t> row_node(max(1u, a.log_cap)), head(4 * (size_t)a.n_inst);
  std::vector<long long> out(a.n_inst, -1);
  a.ctl = &ctl; a.queues = queues.data(); a.mail = mail.data(); a.reply = reply.data(); a.segs = segs.data(); a.log = log.data();
  a.row_node = num("node_loss", 0) ? row_node.data() : nullptr;
  if (in.count("left")) {
    a.n_tree_nodes = (int32_t)in["left"].size();
    a.left = guarded<int32_t>(in["left"]);
    a.right = guarded<int32_t>(in["right"]);
    a.token = guarded<int32_t>(in["token"]);
  }
  a.args = in["args"].data();
  a.out_i64 = out.data();
  a.root_ref = head.data(); a.root_lvl = a.root_ref + a.n_inst; a.head_row = a.root_lvl + a.n_inst; a.head_label = a.head_row + a.n_inst;
  lane_init(a, 0, 1);
  hw::world().slow_every = (uint32_t)num("slow", 0);
  if (!hw::run(a.n_waves, lane_lds_bytes(NS), (uint64_t)num("seed", 1), (uint64_t)num("max_turns", 200000000), body)) {
    printf("hung 1 1\n");
    return 0;
  }
  LaneQueue t{};
  for (const LaneQueue& q : queues) {
    t.n_tags += q.n_tags; t.n_tokens += q.n_tokens; t.n_leaf += q.n_leaf; t.n_cell += q.n_cell; t.n_rec += q.n_rec; t.n_private += q.n_private;
    t.max_depth = max(t.max_depth, q.max_depth); t.max_level = max(t.max_level, q.max_level); t.max_iter = max(t.max_iter, q.max_iter);
  }
  auto put = [](const char* k, unsigned long long v) { printf("%s 1 %llu\n", k, v); };
  put("status", ctl.status); put("tags", t.n_tags); put("tokens", t.n_tokens); put("leaves", t.n_leaf); put("cells", t.n_cell);
  put("depth", t.max_depth); put("level", t.max_level); put("sweeps", t.max_iter); put("records", t.n_rec); put("turns", hw::world().turns);
  printf("out %u", a.n_inst);
  for (long long v : out) printf(" %lld", v);
  printf("\nroot %u", a.n_inst);
  for (uint32_t b = 0; b < a.n_inst; ++b) printf(" %u", a.root_ref[b]);
  const uint32_t n_log = min(ctl.log_used, a.log_cap);
  printf("\nlog %u", 4 * n_log);
  for (uint32_t k = 0; k < n_log; ++k) printf(" %u %u %u %u", log[k].x, log[k].y, log[k].z, log[k].w);
  printf("\nmarks %u", a.row_node ? n_log : 0u);
  for (uint32_t k = 0; k < n_log && a.row_node; ++k) printf(" %u", row_node[k]);
  printf("\n");
  return 0;
}
