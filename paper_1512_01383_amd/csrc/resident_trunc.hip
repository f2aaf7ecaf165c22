// resident_trunc.hip -- the on-chip iteration (resident.hpp) for truncated-quadratic pieces
#include "resident.hpp"

const void *resident_kernel_trunc(bool add, int ch, int lg, int rp, int phys, int *ph) {
  return add ? resident::kernel_of<SLI_TRUNC, true>(ch, lg, rp, phys, ph)
             : resident::kernel_of<SLI_TRUNC, false>(ch, lg, rp, phys, ph);
}
