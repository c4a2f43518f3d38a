// Ladder term of the lattice observables, sum_nu nu' L_nu Gamma_nu nu' L_nu' at
// Omega = 0: the ladder kernels with n_om = 1 (launchers).
#pragma once

#include "df_internal.hpp"

namespace df {

// gamma L into W [2][n_nu][N] and the certificate of every item (k_ladder_screen)
hipError_t launch_lattice_screen(const LadderArgs &a, const double *L, hipStream_t s);
// lad [2][N] of the certified items of symmetric vertices
hipError_t launch_lattice_sym(const LadderArgs &a, const double *L, double *lad, hipStream_t s);
// lad of the queued items, by elimination with partial pivoting
hipError_t launch_lattice_rest(const LadderArgs &a, const double *L, double *lad, hipStream_t s);

}  // namespace df
