// a1: the local AdamW step of every active worker (Eq. 1 inner loop,
// App. B "Optimization": decoupled weight decay, bias-corrected moments).
#pragma clang fp contract(off)

#include "device_common.h"

namespace gasloc {
namespace {

constexpr int64_t kBoundedTiles = 28;

// A CU's 160 KiB of LDS in granules of 1280 bytes hold six of these.
constexpr size_t kTilesPerCu = 6;
constexpr size_t kTileLds = (160 * 1024 / kTilesPerCu) / 1280 * 1280;

// One workgroup per tile of 256 x 4 consecutive columns of one active worker:
// grid (tiles, n_active), tiles = ceil(P / 1024); slot blockIdx.y updates
// worker rep[slot].  The grid is not persistent: workgroups are dispatched in
// tile order, one worker row after the other, so the columns in flight at any
// moment form one compact window that sweeps each row once.  (A grid-stride
// loop over a fixed grid lets its workgroups drift apart over a row; on
// MI355X that spread the accesses over the whole row and made the launch's
// speed depend on where the buffers were placed: 25.4-30.1 ms at n = 16,
// P = 350M, against 24.3-26.0 ms for the tiles in the same processes.)
//
// Concurrency is bounded on purpose: each thread waits for one stream's load
// before the next (the per-lane test of the ragged end does that), and on long
// launches kTilesPerCu workgroups share a CU, by LDS that nothing uses.  With more
// tiles in flight the seven streams' windows grow and HBM pages conflict: n=16,
// P=100M fp32, three buffer sets, 8 workgroups per CU 7.39 / 7.34 / 7.50 ms, 7
// 7.29 / 7.19 / 7.38, 6 7.15 / 7.07 / 7.22 (6.3 TB/s), 5 7.48 / 7.45 / 7.65, 3
// 8.61.  Without the per-lane test, all loads at once: 8 per CU 7.71 / 7.79 /
// 7.78, 3 per CU 7.15 / 7.02 / 7.48.  Workgroups of 512 threads 7.26 ms and
// more, of 128 threads 7.09 to 7.42.  Short launches fit the last-level cache
// and lose by the bound what their last wave of workgroups lacks, so it holds
// from kBoundedTiles workgroups per CU.  With it / without, n=16: 7 per CU
// (P=114624 fp32) 10.0 / 7.3 us, 8 10.9 / 8.0, 13 16.8 / 15.3, 20 24.6 / 23.7, 27
// 32.4 / 32.4, 32 38.6 / 39.0, 64 75.9 / 78.0; bf16 8 10.0 / 7.6, 20 21.6 / 20.6,
// 27 28.3 / 28.1, 32 33.3 / 32.9, 64 64.5 / 66.4.
template <int DT>
__global__ __launch_bounds__(256) void k_local_adamw(AdamArgs a) {
  constexpr int V = 4;
  const int slot = blockIdx.y;
  const int64_t gi = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gi >= (a.P + V - 1) / V) return;
  const int r = a.rep[slot];
  const bool from_x = (a.from_x >> slot) & 1ull;
  const int64_t p = gi * V;
  const int64_t e = static_cast<int64_t>(r) * a.ld + p;
  const int cnt = static_cast<int>(a.P - p < V ? a.P - p : V);
  float w[V], g[V], m[V], v[V], out[V], kept[V];
  load_params<DT, V>(from_x ? a.x : a.y, e, cnt, w);
  load_f32<V>(a.g + static_cast<int64_t>(r) * a.gld + p, cnt, g);
  load_f32<V>(a.m + e, cnt, m);
  load_f32<V>(a.v + e, cnt, v);
  const float s1 = a.s1[slot], c2 = a.c2[slot];
#pragma unroll
  for (int c = 0; c < V; ++c)
    out[c] = adamw_element(w[c], g[c], m[c], v[c], a.c_wd, a.b1, a.omb1, a.b2, a.omb2, a.eps, s1, c2);
  store_params<DT, V>(a.y, e, cnt, out, kept);
  store_f32<V>(a.m + e, cnt, m);
  store_f32<V>(a.v + e, cnt, v);
}

}  // namespace

hipError_t launch_local_adamw(const AdamArgs& a, int dtype, int cus, hipStream_t stream) {
  constexpr int64_t kTile = 256 * 4;  // columns per workgroup
  const dim3 grid(static_cast<unsigned>((a.P + kTile - 1) / kTile), a.n_active);
  return launch_kernel(dtype == GASLOC_BF16 ? k_local_adamw<GASLOC_BF16> : k_local_adamw<GASLOC_F32>, grid, 256,
                       static_cast<int64_t>(grid.x) * grid.y < kBoundedTiles * cus ? 0 : kTileLds, stream, a);
}

}  // namespace gasloc
