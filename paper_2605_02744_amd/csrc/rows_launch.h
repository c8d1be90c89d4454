// The row kernels behind one interface: evaluation e (or the one Epi belongs to)
// of the rows of c, followed by epi.  Instantiated for every Epi of row_update.h in
// rows64.hip and rows32.hip, called from rows.hip.
#pragma once

#include "row_update.h"

namespace nb {

template <class Epi>
int rows64(RowEval e, const RowCall& c, const double* x, const double* w, const double* u, const Epi& epi);
template <class Epi>
int rows32(RowEval e, const RowCall& c, const double* x, const double* w, const double* u, const Epi& epi);

}  // namespace nb
