// Prints the generated lanes of a program (the code that the library hands to the run-time compiler; no GPU is needed).
// Reads: functions, result function; for each function parameters, nodes; for each node op, imm, inputs, (node, port)*.
#include <iostream>

#include "jit.cpp"

tdf_graph::~tdf_graph() {}   // (the library's destructor also releases GPU objects; none exist here)

int main() {
  int n_fn = 0;
  tdf_program_desc prog{};
  std::cin >> n_fn >> prog.result_fn;
  std::vector<tdf_function_desc> fns(n_fn);
  std::vector<std::vector<tdf_node_desc>> nodes(n_fn);
  for (int f = 0; f < n_fn; ++f) {
    int n_nodes = 0;
    std::cin >> fns[f].n_params >> n_nodes;
    nodes[f].resize(n_nodes);
    for (tdf_node_desc& n : nodes[f]) {
      memset(&n, 0, sizeof(n));
      std::cin >> n.op >> n.imm >> n.n_in;
      for (int k = 0; k < n.n_in; ++k) std::cin >> n.in[k].node >> n.in[k].port;
    }
    fns[f].name = "f";
    fns[f].n_nodes = n_nodes;
    fns[f].nodes = nodes[f].data();
  }
  prog.n_functions = n_fn;
  prog.functions = fns.data();
  tdf_graph* g = nullptr;
  if (!std::cin || tdf_graph_build(&prog, 0, &g) != TDF_OK) return 2;   // (not a program)
  if (tdf::lane_stored(g->g.prog) > 8) return 3;                        // (one that runs on the step machine)
  tdf::Gen gen(g->g.prog);
  std::cout << gen.lane_source();
  return 0;
}
