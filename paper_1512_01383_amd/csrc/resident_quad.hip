// resident_quad.hip -- the on-chip iteration (resident.hpp) for quadratic pieces
#include "resident.hpp"

const void *resident_kernel_quad(bool add, int ch, int lg, int rp, int phys, int *ph) {
  return add ? resident::kernel_of<SLI_QUAD, true>(ch, lg, rp, phys, ph)
             : resident::kernel_of<SLI_QUAD, false>(ch, lg, rp, phys, ph);
}
