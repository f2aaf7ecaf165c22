// resident_sampled.hip -- the on-chip iteration (resident.hpp) for sampled costs
#include "resident.hpp"

const void *resident_kernel_sampled(bool, int ch, int lg, int rp, int phys, int *ph) {
  return resident::kernel_of<SLI_SAMPLED, false>(ch, lg, rp, phys, ph);
}
