// qq_tables.h -- the per-thread constants of the cost tables (qq_kernels.hip).
#pragma once

#include "qq_internal.h"

namespace qq {

// Lane run and register run of each table of a problem.
struct TableRuns {
    int count;
    int lane_q[16], reg_q[16];
};

// out[table][256][8]: entry 0 P(E), the cost of the thread's own bits E (qubits 0..3 and the lane run's
// four), entries 1..4 l_Rj + sum_{q in E} b_{q Rj} for the register run's qubits; ell [n] and the symmetric
// b [n][n] on the device.
hipError_t launch_table_constants(int n, const TableRuns &runs, const double *ell, const double *b, double *out,
                                  hipStream_t s);

}  // namespace qq
