// Prints the launch plan of a lane-kernel sweep, on the host: the library's planning
// code with a handle of 256 compute units and 160 KB of LDS.
//   plan_check {launch|queue} kind precision settings trials max_steps n_bins every
// -> chunk, workgroups, lanes of a draining team, direct counting (0 or 1), scan form (0 or 1)
// or of a rate network:
//   plan_check rnn units precision settings trials 0 0 0
// -> form, workgroups, 0, direct counting, runs dealt out in turn (0 or 1)
#include <cstdlib>

#include "../../paper_2110_15425_amd/csrc/api.hip"

int main(int argc, char** argv) {
  if (argc != 9) return 2;
  const bool queue = argv[1][0] == 'q';
  cm_handle h{};
  h.cu_count = 256;
  h.lds_per_block = 163840;
  const uint32_t kind = atoi(argv[2]), prec = atoi(argv[3]);
  if (argv[1][0] == 'r') {
    const uint64_t S = strtoull(argv[4], nullptr, 10), T = strtoull(argv[5], nullptr, 10);
    const cm::RnnPlan p = cm::plan_rnn(prec, kind, S, S * T, 256);
    printf("%d %u 0 %d %d\n", p.form, p.groups, p.direct ? 1 : 0, p.dealt ? 1 : 0);
    return 0;
  }
  h.tune[kind][prec] = default_tuning(kind, prec);
  double params[16] = {0.1, 0.5, 1.0, 0.1, 0.8};
  cm_model m{};
  m.kind = kind;
  m.precision = prec;
  m.params = params;
  cm_sweep s{};
  s.n_settings = strtoull(argv[4], nullptr, 10);
  s.trials = strtoull(argv[5], nullptr, 10);
  s.max_steps = atoi(argv[6]);
  s.n_bins = atoi(argv[7]);
  TcSpec tc;
  tc.every = atoi(argv[8]);
  const uint64_t runs = s.n_settings * s.trials;
  const bool scan = kind == CM_DDM && !tc.every && !queue && scan_ddm(h.tune[kind][prec], runs);
  cm_result r{};
  Layout L{};
  char ws[256];
  cm::SimArgs a;
  uint64_t groups = 0;
  size_t lds = 0;
  if (plan_lane(&h, &m, &s, &r, ws, L, scan ? 512 : 0, runs, tc, a, groups, lds, queue) != CM_OK) return 1;
  printf("%llu %llu %u %u %d\n", (unsigned long long)a.chunk, (unsigned long long)groups, a.team_lanes, a.direct,
         scan ? 1 : 0);
  return 0;
}
