// Batches of small problems, a workgroup or a team per problem (small.hip).
#pragma once

#include "csipm_internal.h"

#include "../../include/csipm.h"

// csipm_solve_small_batch with the ticks of the 100 MHz clock after which a
// team's barrier gives up (not in csipm.h: the tests make it give up at once)
extern "C" csipm_status csipm_solve_small_batch_wait(int n1, int n2, int n3, int count, const double* d_signals,
                                                     const uint8_t* d_observed, const double* d_lambdas,
                                                     double lambda_frac, const csipm_options* opts,
                                                     double* d_beta_out, double* d_info, void* d_workspace,
                                                     size_t workspace_bytes, void* hip_stream, long long wait);

namespace csipm {

// the largest extent of a small problem
constexpr int kSmallMaxExtent = 64;
// the most problems of a batch whose workgroups form teams: a compute unit has
// the registers for one workgroup (170 for each of eight waves), so 129 teams of
// two are more than the 256 compute units hold together (30 x 28 x 33: 128
// problems 20.9 ms, 129 32.4, 256 37.4)
constexpr int kSmallTeams = 128;
constexpr long long kTeamWait = 500000000ll;   // 5 s

// the options the small solver reads (those of csipm_options it uses)
struct SmallOpts {
  double tol;
  int max_iter;
  int cg_max;
  double cg_rtol;
  double cg_atol;
  double sigma;
  double tau;
};

bool small_supported(int n1, int n2, int n3);
// workspace bytes in front of the problems: the twiddle tables and the team
// counters
size_t small_front_bytes(int n1, int n2, int n3);
// workspace bytes of one problem (a multiple of 256)
size_t small_problem_bytes(int n1, int n2, int n3);
// one launch of a workgroup (or a team) per problem; tw holds the tables
// exp(-2 pi i q / L) of L = n1, n2, n3 in that order, counters kSmallTeams
// zeros 64 bytes apart, wait the patience of a team's barrier
hipError_t small_launch(int n1, int n2, int n3, int count, const double* signals, const uint8_t* observed,
                        const double* lambdas, double lambda_frac, double* beta_out, double* info, char* ws,
                        const cx<double>* tw, unsigned* counters, const SmallOpts& o, long long wait, hipStream_t s);

// The grids that small_tiny.hip solves: at most 400 points, or kTinyMax with
// extents 1, 2, 4, 8 and 16 only.
constexpr int kTinyMax = 1024;
bool tiny_grid(int n1, int n2, int n3);
size_t tiny_problem_bytes(int n1, int n2, int n3);
hipError_t tiny_launch(int n1, int n2, int n3, int count, const double* signals, const uint8_t* observed,
                       const double* lambdas, double lambda_frac, double* beta_out, double* info, char* ws,
                       const cx<double>* tw, const SmallOpts& o, hipStream_t s);

}  // namespace csipm
