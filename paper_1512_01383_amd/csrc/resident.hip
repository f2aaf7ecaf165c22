// resident.hip -- how a problem is laid over the chip for the on-chip iteration
// (resident.hpp), and its launch.
#include "resident.hpp"

const void *resident_kernel_trunc(bool add, int ch, int lg, int rp, int phys, int *ph);
const void *resident_kernel_quad(bool add, int ch, int lg, int rp, int phys, int *ph);
const void *resident_kernel_sampled(bool add, int ch, int lg, int rp, int phys, int *ph);

namespace {

constexpr int kMaxBlocks = 256;              // compute units of the chip: the exchange is sized for them
constexpr size_t kOneBlock = 82 * 1024;      // LDS of more than half a compute unit: one block on each
constexpr size_t kMaxLds = 160 * 1024 - 16 * SLI_MAXK - 64;   // less the kernels' fixed tables

const void *kernel_for(int piece, bool add, int ch, int lg, int rp, int phys, int *ph) {
  return piece == SLI_TRUNC ? resident_kernel_trunc(add, ch, lg, rp, phys, ph)
         : piece == SLI_QUAD ? resident_kernel_quad(add, ch, lg, rp, phys, ph) : resident_kernel_sampled(add, ch, lg, rp, phys, ph);
}

// fewest wavefronts on top of each other (of rp rows each; two at least: a row is at one rim
// only) with which the tiles fit `cus` blocks, 0 if even `waves` of them do not reach
int tile_waves(int H, int W, int rp, int waves, int cus) {
  const int ntc = (W + 63) / 64;
  for (int th = 2; th <= waves; th++)
    if ((long long)((H + th * rp - 1) / (th * rp)) * ntc <= cus) return th;
  return 0;
}

}  // namespace

// A wavefront per label group where the tiles then fit the chip, else two or four groups per
// thread, else (one group) several rows per thread; small tiles spread over as many compute
// units as there are.
bool resident_plan(int piece, bool add, int H, int W, int k, int G, int qmax, int cus, ResidentPlan *out) {
  if (cus > kMaxBlocks) cus = kMaxBlocks;
  const int cn = (k + G - 1) / G;
  auto plan = [&](int lg, int rp) {
    const int th = tile_waves(H, W, rp, 16 / (G / lg), cus);
    int ph = 0;
    if (th == 0 || !kernel_for(piece, add, cn * lg, lg, rp, G / lg, &ph)) return false;
    ResidentPlan L;
    L.ch = cn * lg;
    L.lg = lg;
    L.rp = rp;
    L.th = th;
    L.blocks = ((H + th * rp - 1) / (th * rp)) * ((W + 63) / 64);
    L.threads = 64 * th * (G / lg);
    L.slots = qmax + 2 < k ? qmax + 2 : k;
    L.lds = resident::lds_bytes(piece, L.ch, lg, rp, ph, G, th, qmax, L.slots);
    if (L.lds > kMaxLds) return false;
    if (L.lds < kOneBlock) L.lds = kOneBlock;
    *out = L;
    return true;
  };
  for (int lg = 1; lg <= G; lg *= 2)
    if (plan(lg, 1)) return true;
  if (G > 1) return false;
  for (int rp : {2, 3, 4, 6, 8, 12})
    if (plan(1, rp)) return true;
  return false;
}

// two slots of every tile's rim words (128 + twice its rows, per label)
size_t resident_rim_bytes(const ResidentPlan &L, int k) {
  return (size_t)2 * L.blocks * k * (128 + 2 * L.th * L.rp) * 8;
}
// the most of those for the label groups a tiling may have; 0 if the problem fits the chip
// with none
size_t resident_exchange_bytes(int piece, bool add, int H, int W, int k, int qmax) {
  size_t most = 0;
  for (int G = 1; G <= 4; G *= 2) {
    ResidentPlan L;
    if (resident_plan(piece, add, H, W, k, G, qmax, kMaxBlocks, &L)) {
      const size_t b = resident_rim_bytes(L, k);
      if (b > most) most = b;
    }
  }
  return most;
}

hipError_t launch_resident(int piece, bool add, const ResidentPlan &L, const ResidentArgs &R, hipStream_t st) {
  int ph = 0;
  const void *f = kernel_for(piece, add, L.ch, L.lg, L.rp, R.G / L.lg, &ph);
  if (!f) return hipErrorInvalidValue;
  void *args[] = {const_cast<ResidentArgs *>(&R)};
  return hipLaunchCooperativeKernel(f, dim3(L.blocks), dim3(L.threads), args, (unsigned)L.lds, st);
}
