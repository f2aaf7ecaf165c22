// resident.hip -- how a problem is laid over the chip for the on-chip iteration
// (resident.hpp), and its launch.
#include "resident.hpp"

const void *resident_kernel_trunc(bool add, int ch, int lg);
const void *resident_kernel_quad(bool add, int ch, int lg);
const void *resident_kernel_sampled(bool add, int ch, int lg);

namespace {

constexpr int kMaxBlocks = 256;              // compute units of the chip: the exchange is sized for them
constexpr size_t kOneBlock = 82 * 1024;      // LDS of more than half a compute unit: one block on each
constexpr size_t kMaxLds = 159 * 1024;       // of 160 KB, less the kernels' fixed tables

const void *kernel_for(int piece, bool add, int ch, int lg) {
  return piece == SLI_TRUNC ? resident_kernel_trunc(add, ch, lg)
         : piece == SLI_QUAD ? resident_kernel_quad(add, ch, lg) : resident_kernel_sampled(add, ch, lg);
}

// fewest tile rows (a tile of two rows at least: a row is at one rim only) with which the
// tiles fit `cus` blocks, 0 if even the most of `waves` wavefronts do not reach
int tile_rows(int H, int W, int waves, int cus) {
  const int ntc = (W + 63) / 64;
  for (int th = 2; th <= waves; th++)
    if ((long long)((H + th - 1) / th) * ntc <= cus) return th;
  return 0;
}

}  // namespace

// A wavefront per label group where the tiles then fit the chip, else two or four groups per
// thread; small tiles spread over as many compute units as there are.
bool resident_plan(int piece, bool add, int H, int W, int k, int G, int cus, ResidentPlan *out) {
  if (cus > kMaxBlocks) cus = kMaxBlocks;
  const int cn = (k + G - 1) / G;
  for (int lg = 1; lg <= G; lg *= 2) {
    const int th = tile_rows(H, W, 16 / (G / lg), cus);
    if (th == 0 || !kernel_for(piece, add, cn * lg, lg)) continue;
    ResidentPlan L;
    L.ch = cn * lg;
    L.lg = lg;
    L.th = th;
    L.blocks = ((H + th - 1) / th) * ((W + 63) / 64);
    L.threads = 64 * th * (G / lg);
    L.lds = resident::lds_bytes(piece, L.ch, lg, G, th);
    if (L.lds > kMaxLds) continue;
    if (L.lds < kOneBlock) L.lds = kOneBlock;
    *out = L;
    return true;
  }
  return false;
}

// two slots of every tile's rim words (128 + 2 TH per label) in the plan that needs most of
// those for the label groups a tiling may have; 0 if the problem fits the chip in none
size_t resident_exchange_bytes(int piece, bool add, int H, int W, int k) {
  size_t most = 0;
  for (int G = 1; G <= 4; G *= 2) {
    ResidentPlan L;
    if (!resident_plan(piece, add, H, W, k, G, kMaxBlocks, &L)) continue;
    const size_t b = (size_t)2 * L.blocks * k * (128 + 2 * L.th) * 8;
    if (b > most) most = b;
  }
  return most;
}

hipError_t launch_resident(int piece, bool add, const ResidentPlan &L, const ResidentArgs &R, hipStream_t st) {
  const void *f = kernel_for(piece, add, L.ch, L.lg);
  if (!f) return hipErrorInvalidValue;
  void *args[] = {const_cast<ResidentArgs *>(&R)};
  return hipLaunchCooperativeKernel(f, dim3(L.blocks), dim3(L.threads), args, (unsigned)L.lds, st);
}
