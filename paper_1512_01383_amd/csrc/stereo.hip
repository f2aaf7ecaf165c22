// stereo.hip -- matching-cost volume of the stereo experiment (Sec. 5.4): for every pixel
// and disparity, a truncated sum of absolute gradient differences over a 4x4 patch.
//
// C(d, r, c) = min(T, sum_{i,j in -1..2} |dxL(p) - dxR(q)| + |dyL(p) - dyR(q)|),
// p = (clamp(r+i), clamp(c+j)), q = (p.r, max(p.c - d, 0)); forward differences, zero on
// the last column / row. The volume is the sampled data term of the stereo problem
// (tau_m = m): D planes of H x W, written once, so the kernel is bound by those writes.
//
// What bounds it is vector issue, so the split is the one with the fewest operations per
// output. A block owns a tile of 64 columns x 4 rows and DC disparities and stages both
// images' gradients in LDS, rows and columns clamped to the image on the way in, so that the
// main loop's LDS addresses are one register plus constants. Each of its four wavefronts
// takes every fourth disparity and all four rows: a lane (one image column) forms the
// per-pixel term e of its column's seven patch rows once, adds four of them for each row
// (a sum per row costs three additions; the seven terms serve all four rows), and the four
// column sums of a patch are then added across lanes with DPP wave shifts (all lanes stay
// active; lanes beyond the image work on the clamped last column and store nothing). The
// column sums just beyond the tile (c0-1, c0+64, c0+65), which enter the shifts at the ends of
// the wave, each wavefront forms ahead of its disparities. The volume is larger than the
// caches and is written once, so it is stored past them. 288x384, 64 disparities (28 MB, 5.5 us
// at a copy's rate): 13.6 us with a wavefront per row and every disparity; 10.9 with the rows
// together, 9.7 with the staging's loads in one go, 8.2 with the stores past the caches.
#include "stereo.hpp"

namespace {

constexpr int TW = 64, TH = 4, PR = TH + 3;   // patch rows: r0-1 .. r0+TH+1
constexpr int DC = 16;                          // disparities per block
constexpr int LW = TW + 3;                      // left columns held: c0-1 .. c0+TW+1, clamped
constexpr int QW = LW + DC - 1;                 // right columns held, from qs on
constexpr int NT = 256, NW = NT / 64;

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// x of the next lane (lane 63 takes `last`) and of the previous lane (lane 0 takes `first`):
// DPP wave shifts by one lane, issued with every lane active
__device__ __forceinline__ float from_right(float x, float last) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, last),
                                                               __builtin_bit_cast(int, x), 0x130, 0xF, 0xF, false));
}
__device__ __forceinline__ float from_left(float x, float first) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, first),
                                                               __builtin_bit_cast(int, x), 0x138, 0xF, 0xF, false));
}

__global__ __launch_bounds__(NT) void k_stereo_costs(const float *__restrict__ left,
                                                     const float *__restrict__ right, int H, int W,
                                                     int D, float trunc, float *out) {
  __shared__ float2 lg[PR][LW], rg[PR][QW];   // gradients (x, y)
  __shared__ float4 ev[NW][DC / NW][TH];      // a wave's column sums beyond the tile
  const int ntc = (W + TW - 1) / TW;
  const int r0 = (int)(blockIdx.x / ntc) * TH, c0 = (int)(blockIdx.x % ntc) * TW;
  const int d0 = (int)blockIdx.y * DC, d1 = min(d0 + DC, D);
  // right columns reached: max(p - d, 0), p the clamped patch columns, d in [d0, d0 + DC);
  // at most LW + DC - 1 of them, from qs on
  const int qs = max(max(c0 - 1, 0) - (d0 + DC - 1), 0);
  const int tid = (int)threadIdx.x;

  // all loads first, none of them under a condition: one latency for the whole staging
  struct Px {
    float v, x, y;
    bool hx, hy;
  };
  auto load = [&](const float *img, int r, int c) {
    Px p;
    p.hx = c < W - 1;
    p.hy = r < H - 1;
    const int x = r * W + c;
    p.v = img[x];
    p.x = img[p.hx ? x + 1 : x];
    p.y = img[p.hy ? x + W : x];
    return p;
  };
  auto grad = [](const Px &p) { return make_float2(p.hx ? p.x - p.v : 0.f, p.hy ? p.y - p.v : 0.f); };
  constexpr int NL = (PR * LW + NT - 1) / NT, NR = (PR * QW + NT - 1) / NT;
  Px pl[NL], pr[NR];
#pragma unroll
  for (int j = 0; j < NL; j++) {
    const int e = min(tid + j * NT, PR * LW - 1), rr = e / LW, cc = e - rr * LW;
    pl[j] = load(left, clampi(r0 - 1 + rr, 0, H - 1), clampi(c0 - 1 + cc, 0, W - 1));
  }
#pragma unroll
  for (int j = 0; j < NR; j++) {
    const int e = min(tid + j * NT, PR * QW - 1), rr = e / QW, cc = e - rr * QW;
    pr[j] = load(right, clampi(r0 - 1 + rr, 0, H - 1), min(qs + cc, W - 1));
  }
#pragma unroll
  for (int j = 0; j < NL; j++)   // (threads past the end write the last element's own value)
    (&lg[0][0])[min(tid + j * NT, PR * LW - 1)] = grad(pl[j]);
#pragma unroll
  for (int j = 0; j < NR; j++) (&rg[0][0])[min(tid + j * NT, PR * QW - 1)] = grad(pr[j]);
  __syncthreads();

  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto term = [](float2 l, float2 r) { return fabsf(l.x - r.x) + fabsf(l.y - r.y); };
  static_assert(DC / NW * TH * 3 <= 64, "one lane per column sum beyond the tile");
  if (lane < DC / NW * TH * 3) {
    const int dd = lane / (TH * 3), rem = lane - dd * (TH * 3), j = rem / 3, k = rem - j * 3;
    const int cc = k == 0 ? 0 : TW + k;   // columns c0-1, c0+TW, c0+TW+1
    const int q = max(clampi(c0 - 1 + cc, 0, W - 1) - (d0 + wv + NW * dd), 0) - qs;
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 4; i++) acc += term(lg[j + i][cc], rg[j + i][q]);
    ((float *)&ev[wv][dd][j])[k] = acc;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");   // read by this wave alone
  __builtin_amdgcn_wave_barrier();

  const int c = c0 + lane, col = min(c, W - 1);
  float2 ol[PR];   // left gradients of the own column
#pragma unroll
  for (int i = 0; i < PR; i++) ol[i] = lg[i][lane + 1];
  const long long N = (long long)H * W;
#pragma unroll
  for (int dd = 0; dd < DC / NW; dd++) {
    const int d = d0 + wv + NW * dd;
    if (d >= d1) break;
    const int q = max(col - d, 0) - qs;
    float e[PR];
#pragma unroll
    for (int i = 0; i < PR; i++) e[i] = term(ol[i], rg[i][q]);
    float *o = out + (long long)d * N + (long long)r0 * W;
#pragma unroll
    for (int j = 0; j < TH; j++) {
      const float v = ((e[j] + e[j + 1]) + e[j + 2]) + e[j + 3];
      const float4 eg = ev[wv][dd][j];
      const float vm1 = from_left(v, eg.x);
      const float vp1 = from_right(v, eg.y);
      const float vp2 = from_right(vp1, eg.z);
      const float acc = ((vm1 + v) + vp1) + vp2;
      if (r0 + j < H) {
        if (c < W) __builtin_nontemporal_store(fminf(acc, trunc), o + j * W + c);
      }
    }
  }
}

}  // namespace

hipError_t launch_stereo_costs(const float *left, const float *right, int H, int W, int D,
                               float trunc, float *out, hipStream_t st) {
  const int ntc = (W + TW - 1) / TW, ntr = (H + TH - 1) / TH;
  hipLaunchKernelGGL(k_stereo_costs, dim3(ntc * ntr, (D + DC - 1) / DC), dim3(NT), 0, st,
                     left, right, H, W, D, trunc, out);
  return hipGetLastError();
}
