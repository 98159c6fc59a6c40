// a2-a5: pseudo-gradient, outer step, neighbour mix, consensus momentum, and
// the consensus-error and squared-pseudo-gradient partials, fused, with the
// workers of a column spread over the waves of a workgroup.  A workgroup takes a
// tile of C = 64 V columns of every worker: wave w owns the workers w, w + W, w
// + 2W, ... (K of them at most, W waves), each lane V consecutive columns of
// each.  The thread that loads a worker's streams also finishes that worker's
// row, so every stream is read once, before or around the first barrier, and
// what the row needs again stays in registers; only the mixed values cross
// waves, through LDS.  The stored rows go through LDS too, so that one thread
// per column sums the consensus error of all workers in worker order.
//
// What a slot holds and how a row is finished depends on the round form:
//   EQ          slot z_j = x_j - eta (delta_j + mu u_j), delta_j = x_j - y_j
//               x_i = sum_k W_ik z_k [+ gamma (z_i - zp_i)]      (Eq. 1, Eq. 2)
//   ALG1        slot y_j;  delta_i = sum_k W_ik (x_i - y_k),
//               x_i = OuterOpt(x_i, delta_i)                      (Algorithm 1)
//   DADAM       slot x_j;  x_i = sum_k W_ik x_k + (y_i - x_i)     (App. C)
//   LOCAL_DADAM slot x_j;  d_i = sum_k W_ik (x_i - x_k),
//               x_i = OuterOpt(y_i, d_i)                          (App. C)
// with OuterOpt(b, d): u = mu u + d; b - eta (d + mu u) (Nesterov) or b - eta u.
//
// What bounds it: HBM, and on short rows the latencies of one tile.  Where a
// thread owns all workers of its columns, LDS (4 n bytes a column) bounds the
// columns in flight and a wave walks n workers in turn, twice (values, then
// rows); here the same LDS serves n times as many lanes, and the time between a
// workgroup's barriers is covered by the other workgroups of the CU.  Measured
// on MI355X on the same buffers against such kernels (up to 16 workers every
// value in LDS, beyond that the live ones in a planned order; the complete graph
// beside them with one running sum), n P = 2.7e8, 2-Peer or ring, in ms, fused
// step + round, gamma = 0.1, unless noted: n=1 fp32 2.08 -> 1.90 (6.2 TB/s); n=4
// 1.97 -> 1.88, 2.20 -> 1.98, bf16 1.78 -> 1.80, 1.81 -> 1.71 (two buffer sets
// each: where the buffers lie decides); n=8 1.98 -> 1.91, 2.31 -> 2.08; n=16 2.60
// -> 2.14, bf16 2.17 -> 1.74; complete n=16 2.59 -> 2.05, n=32 3.03 -> 2.13; n=32
// 2.07 -> 1.91 (6.2 TB/s), bf16 1.98 -> 1.75; n=64 2.34 -> 2.19, bf16 1.97 -> 1.79;
// local step and Local-DAdam round, n=64 2.21 -> 2.05, bf16 1.85 -> 1.68.  Short
// rows, n=16, P=65536 37 -> 14 us, n=64 121 -> 43 us.  Behind them by up to 7%:
// the EQ round alone in bf16, gamma = 0, on long rows at 17 to 24 and 49 to 60
// workers (local step and round, n=17 1.72 -> 1.84, n=52 1.82 -> 1.91).
//
// 4 columns per lane: 2 (half the bytes per access) took 3 to 40% longer; tiles
// of 512 or 1024 columns 1 to 5% longer (n=8, n=16), as did giving each XCD 4 or
// 16 consecutive tiles.
//
// Included by round_tile_f32.hip and round_tile_bf16.hip, which compile the
// kernels of one parameter type each.
#pragma once
#pragma clang fp contract(off)

#include "device_common.h"

namespace gasloc {
namespace {

typedef const __attribute__((address_space(4))) int32_t uniform_i32;
typedef const __attribute__((address_space(4))) float uniform_f32;

constexpr int kWaitVector = 0x0f70;  // s_waitcnt vmcnt(0); the other counters are not waited for

// V parameters as stored: fp32, or two bf16 values to a register.
template <int DT, int V>
struct Held {
  uint32_t w[DT == GASLOC_BF16 ? V / 2 : V];
  __device__ __forceinline__ void set(const float (&v)[V]) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      const uint32_t bits = __float_as_uint(v[c]);
      if constexpr (DT != GASLOC_BF16)
        w[c] = bits;
      else
        w[c / 2] = c % 2 ? w[c / 2] | (bits & 0xffff0000u) : bits >> 16;
    }
  }
  __device__ __forceinline__ float get(int c) const {
    if constexpr (DT != GASLOC_BF16) return __uint_as_float(w[c]);
    return __uint_as_float(c % 2 ? w[c / 2] & 0xffff0000u : w[c / 2] << 16);
  }
};

// The forms whose rows are outer steps from differences: they need u.
template <int FORM>
constexpr bool kOuterRow = FORM == GASLOC_FORM_ALG1 || FORM == GASLOC_FORM_LOCAL_DADAM;

// What a worker's row needs after the barrier, by form: EQ the consensus
// momentum term; ALG1 x and u; DAdam y - x; Local-DAdam x, y and u, where x is
// what its slot holds: LEAN takes it from there (two registers or four per
// worker saved; where they are not short the LDS read costs: n=11, P=1M local
// step + round 99.5 us, 97.3 with x kept).
template <int DT, int V, int FORM, bool LEAN>
struct RowKept {
  static constexpr bool kKeepsX = FORM == GASLOC_FORM_LOCAL_DADAM && !LEAN;
  Held<DT, kOuterRow<FORM> ? V : 2> base;
  Held<DT, kKeepsX ? V : 2> x;
  float v[V];  // u, or the term
};

// The value of a slot, and a stored row's in LDS: 16 bits for what is a bf16
// value already (stored rows; iterates and anchors, the mixed values of every
// form but EQ), else fp32.
template <int DT, int FORM>
constexpr bool kSlot16 = DT == GASLOC_BF16 && FORM != GASLOC_FORM_EQ;

// V values to and from LDS (HALF: as bf16).
template <int V, bool HALF>
__device__ __forceinline__ void lds_put(void* lds, int at, const Held<HALF ? GASLOC_BF16 : GASLOC_F32, V>& v) {
  uint32_t* p = reinterpret_cast<uint32_t*>(static_cast<char*>(lds) + at * (HALF ? 2 : 4));
#pragma unroll
  for (int c = 0; c < (HALF ? V / 2 : V); ++c) p[c] = v.w[c];
}

template <int V, bool HALF>
__device__ __forceinline__ void lds_get(const void* lds, int at, float (&v)[V]) {
  Held<HALF ? GASLOC_BF16 : GASLOC_F32, V> h;
  const uint32_t* p = reinterpret_cast<const uint32_t*>(static_cast<const char*>(lds) + at * (HALF ? 2 : 4));
#pragma unroll
  for (int c = 0; c < (HALF ? V / 2 : V); ++c) h.w[c] = p[c];
#pragma unroll
  for (int c = 0; c < V; ++c) v[c] = h.get(c);
}

// One value.
template <bool HALF>
__device__ __forceinline__ float lds_value(const void* lds, int at) {
  if constexpr (HALF) return bf16_to_f32(static_cast<const uint16_t*>(lds)[at]);
  return static_cast<const float*>(lds)[at];
}

// The streams of one worker as loaded (the forms other than EQ: y and u only
// where the worker has them).
//
// The copy of x into y below makes the compiler wait for x before it issues
// the worker's other loads, and its conservative waits past the branches wait
// for stores as well.  The other forms avoid both (tile_round), which took 1
// to 4% off: n=22, P=17.8M Local-DAdam 3.41 -> 3.31 ms, n=16, P=50M bf16
// Algorithm 1 4.34 -> 4.23.  The EQ form, with more streams, is 1 to 3% faster
// as it is (n=12, P=50M ring 5.74 against 5.93 ms, n=4, P=67M 2.08 against
// 2.12, n=8, P=124M 7.87 against 7.98) except for waves of many workers
// (kDeep in tile_round): more loads in flight than HBM needs make its pages
// conflict.
template <int V, bool FUSED, int FORM>
struct WorkerLoads {
  float x[V], y[V], u[V], zp[V];
  float g[FUSED ? V : 1], m[FUSED ? V : 1], v[FUSED ? V : 1];
};

template <int DT, int V, bool FUSED, int FORM, bool ONCE, bool LATE>
__device__ __forceinline__ void tile_load(const GossipArgs& a, int i, int64_t tile0, int at, int cnt,
                                          WorkerLoads<V, FUSED, FORM>& w) {
  constexpr bool kEq = FORM == GASLOC_FORM_EQ;
  constexpr int sp = DT == GASLOC_BF16 ? 2 : 4;
  const int64_t row = static_cast<int64_t>(i) * a.ld + tile0;  // uniform
  load_params<DT, V>(static_cast<const char*>(a.x) + row * sp, at, cnt, w.x);
  if ((a.stepped >> i) & 1ull) {
    load_params<DT, V>(static_cast<const char*>(a.y) + row * sp, at, cnt, w.y);
  } else if constexpr (!ONCE) {
#pragma unroll
    for (int c = 0; c < V; ++c) w.y[c] = w.x[c];
  }
  if constexpr (FUSED) {
    if ((a.active >> i) & 1ull) {
      load_f32<V>(a.g + static_cast<int64_t>(i) * a.gld + tile0 + at, cnt, w.g);
      load_f32<V>(a.m + row + at, cnt, w.m);
      load_f32<V>(a.v + row + at, cnt, w.v);
    }
  }
  if (FORM != GASLOC_FORM_DADAM && !LATE && a.use_u) {
    load_f32<V>(a.u + row + at, cnt, w.u);
  } else if constexpr (!ONCE) {
#pragma unroll
    for (int c = 0; c < V; ++c) w.u[c] = 0.0f;
  }
  if (kEq && a.apply_gamma) load_f32<V>(a.zp + row + at, cnt, w.zp);
}

template <int DT, int V, bool FUSED, int FORM, bool ONCE, bool LATE, bool LEAN>
__device__ __forceinline__ void tile_produce(const GossipArgs& a, int i, int64_t tile0, int at, int cnt,
                                             WorkerLoads<V, FUSED, FORM>& w, void* slots,
                                             RowKept<DT, V, FORM, LEAN>& kept, double& pg) {
  const int64_t row = static_cast<int64_t>(i) * a.ld + tile0;  // uniform
  if constexpr (ONCE) {
    const bool stepped = (a.stepped >> i) & 1ull;
    const bool with_u = FORM != GASLOC_FORM_DADAM && !LATE && a.use_u;
#pragma unroll
    for (int c = 0; c < V; ++c) {
      w.y[c] = stepped ? w.y[c] : w.x[c];
      w.u[c] = with_u ? w.u[c] : 0.0f;
    }
  }
  if constexpr (FUSED) {
    if ((a.active >> i) & 1ull) {
      const float s1 = a.s1[i], c2 = a.c2[i];
#pragma unroll
      for (int c = 0; c < V; ++c)
        w.y[c] = as_stored<DT>(adamw_element(w.y[c], w.g[c], w.m[c], w.v[c], a.c_wd, a.b1, a.omb1, a.b2, a.omb2,
                                             a.eps, s1, c2));
      if constexpr (!ONCE) {
        store_f32<V>(a.m + row + at, cnt, w.m);
        store_f32<V>(a.v + row + at, cnt, w.v);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < V; ++c) {
    const double d = static_cast<double>(w.x[c] - w.y[c]);
    if (c < cnt) pg += d * d;
  }
  float out[V];
  if constexpr (FORM == GASLOC_FORM_EQ) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      out[c] = outer_step(w.x[c], w.x[c] - w.y[c], w.u[c], a.mu, a.eta, a.nesterov);
      kept.v[c] = a.gamma * (out[c] - w.zp[c]);
    }
    if (a.use_u) store_f32<V>(a.u + row + at, cnt, w.u);
    if (a.store_zp) store_f32<V>(a.zp + row + at, cnt, out);
  } else {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      out[c] = FORM == GASLOC_FORM_ALG1 ? w.y[c] : w.x[c];
      if constexpr (FORM == GASLOC_FORM_DADAM)
        kept.v[c] = w.y[c] - w.x[c];
      else if constexpr (!LATE)
        kept.v[c] = w.u[c];
    }
    if constexpr (FORM == GASLOC_FORM_ALG1) kept.base.set(w.x);
    if constexpr (FORM == GASLOC_FORM_LOCAL_DADAM) kept.base.set(w.y);
    if constexpr (RowKept<DT, V, FORM, LEAN>::kKeepsX) kept.x.set(w.x);
  }
  Held<kSlot16<DT, FORM> ? GASLOC_BF16 : GASLOC_F32, V> held;
  held.set(out);
  lds_put<V, kSlot16<DT, FORM>>(slots, i * kWave * V + at, held);
}

// Row i from the slots: res, and u where the form updates it there.
template <int DT, int V, int FORM, bool LEAN, bool SHARED>
__device__ __forceinline__ void tile_row(const GossipArgs& a, uniform_i32* rp, uniform_i32* col, uniform_f32* val,
                                         int i, const void* slots, const float* sums, int at,
                                         RowKept<DT, V, FORM, LEAN>& kept, float (&res)[V]) {
  constexpr int C = kWave * V;
  constexpr bool kHalf = kSlot16<DT, FORM>;
  constexpr bool kDiff = kOuterRow<FORM>;
  float own[V];  // x, which the forms on differences measure them from
  if constexpr (RowKept<DT, V, FORM, LEAN>::kKeepsX) {
#pragma unroll
    for (int c = 0; c < V; ++c) own[c] = kept.x.get(c);
  } else if constexpr (FORM == GASLOC_FORM_LOCAL_DADAM) {
    lds_get<V, kHalf>(slots, i * C + at, own);
  } else if constexpr (FORM == GASLOC_FORM_ALG1) {
#pragma unroll
    for (int c = 0; c < V; ++c) own[c] = kept.base.get(c);
  }
#pragma unroll
  for (int c = 0; c < V; ++c) res[c] = 0.0f;
  if constexpr (SHARED) {
#pragma unroll
    for (int c = 0; c < V; ++c) res[c] = sums[at + c];
  } else {
    const int kb = rp[i], ke = rp[i + 1];
    for (int k0 = kb; k0 < ke; k0 += 4) {
      float zk[4][V], wk[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (k0 + t >= ke) break;
        lds_get<V, kHalf>(slots, col[k0 + t] * C + at, zk[t]);
        wk[t] = val[k0 + t];
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (k0 + t >= ke) break;
#pragma unroll
        for (int c = 0; c < V; ++c) res[c] = res[c] + wk[t] * (kDiff ? own[c] - zk[t][c] : zk[t][c]);
      }
    }
  }
  if constexpr (FORM == GASLOC_FORM_EQ) {
    if (a.apply_gamma) {
#pragma unroll
      for (int c = 0; c < V; ++c) res[c] = res[c] + kept.v[c];
    }
  } else if constexpr (FORM == GASLOC_FORM_DADAM) {
#pragma unroll
    for (int c = 0; c < V; ++c) res[c] = res[c] + kept.v[c];
  } else {
#pragma unroll
    for (int c = 0; c < V; ++c)
      res[c] = outer_step(kept.base.get(c), res[c], kept.v[c], a.mu, a.eta, a.nesterov);
  }
}

// One tile.  TAIL: the tile runs past P (cnt < V in some lanes).  SHARED: every
// row is `sum`, plus its own term.
template <int DT, int V, int K, bool FUSED, int FORM, bool SHARED, bool TAIL>
__device__ __forceinline__ void tile_round(const GossipArgs& a, const RowSum* sum, unsigned char* lds, int64_t tile0,
                                           double& ce, double& pg) {
  constexpr int C = kWave * V;
  constexpr int sp = DT == GASLOC_BF16 ? 2 : 4;
  constexpr int B = K < 2 ? K : 2;  // workers whose loads are issued together (4: up to 20% slower)
  // A wave with many workers of few streams (the round alone) waits for memory
  // more than it loads: there all loads of a batch go out at once with one wait
  // in every form, and u, which only the rows need, is loaded for all of the
  // wave's workers together after the values, in flight across the barrier.
  // Local step, then round, n=40, P=6.7M bf16 2-Peer: EQ, gamma = 0, 2.02 -> 1.86
  // ms; Algorithm 1 1.86 -> 1.76.  With four workers in fp32 neither helps (EQ,
  // gamma = 0.1, n=17, P=15.8M 2.58 -> 2.68).  Eight workers and the fused step
  // take u late for the registers' sake: u and x of all eight next to a
  // batch's six streams do not fit 128.
  constexpr bool kDeep = !FUSED && (K >= 5 || (K == 4 && DT == GASLOC_BF16));
  constexpr bool kOnce = FORM != GASLOC_FORM_EQ || kDeep;
  constexpr bool kLate = kOuterRow<FORM> && (kDeep || K == 8);
  const int n = a.n;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int waves = blockDim.x / kWave;
  const int at = lane * V;
  int cnt = V;
  if constexpr (TAIL) {
    const int64_t left = a.P - tile0 - at;
    cnt = left >= V ? V : (left > 0 ? static_cast<int>(left) : 0);
  }
  constexpr bool kHalf = kSlot16<DT, FORM>;
  constexpr bool kHalfRows = DT == GASLOC_BF16;
  unsigned char* slots = lds;
  unsigned char* xs = lds + a.kept_off;
  float* sums = reinterpret_cast<float*>(lds + a.sums_off);
  uniform_i32* rp = (uniform_i32*)(a.row_ptr);
  uniform_i32* col = (uniform_i32*)(a.col);
  uniform_f32* val = (uniform_f32*)(a.val);

  RowKept<DT, V, FORM, kDeep> kept[K];
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += B) {
    WorkerLoads<V, FUSED, FORM> w[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int i = wave + (k0 + b) * waves;
      if (k0 + b < K && i < n) tile_load<DT, V, FUSED, FORM, kOnce, kLate>(a, i, tile0, at, cnt, w[b]);
    }
    // One wait for the batch, after which no load is pending on any path
    if constexpr (kOnce) __builtin_amdgcn_s_waitcnt(kWaitVector);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int i = wave + (k0 + b) * waves;
      if (k0 + b < K && i < n)
        tile_produce<DT, V, FUSED, FORM, kOnce, kLate, kDeep>(a, i, tile0, at, cnt, w[b], slots, kept[k0 + b], pg);
    }
    if constexpr (FUSED && kOnce) {  // the batch's moments, once all its values are computed
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int i = wave + (k0 + b) * waves;
        if (k0 + b < K && i < n && ((a.active >> i) & 1ull)) {
          const int64_t e = static_cast<int64_t>(i) * a.ld + tile0 + at;
          store_f32<V>(a.m + e, cnt, w[b].m);
          store_f32<V>(a.v + e, cnt, w[b].v);
        }
      }
    }
  }
  if constexpr (kLate) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = wave + k * waves;
      if (i >= n) break;
      if (a.use_u) {
        load_f32<V>(a.u + static_cast<int64_t>(i) * a.ld + tile0 + at, cnt, kept[k].v);
      } else {
#pragma unroll
        for (int c = 0; c < V; ++c) kept[k].v[c] = 0.0f;
      }
    }
  }
  __syncthreads();  // every worker's value is in its slot
  if constexpr (SHARED) {
    for (int c = threadIdx.x; c < C; c += blockDim.x) {
      float s = 0.0f;
      for (int k = 0; k < sum->entries; ++k) s = s + sum->w[k] * lds_value<kHalf>(slots, sum->col[k] * C + c);
      sums[c] = s;
    }
    __syncthreads();
  }
  // Rows.  With up to four workers per wave they are all summed before any is
  // stored, which shortens the chain of a short round (EQ, n=63, P=56784 32.5 ->
  // 31.0 us; Algorithm 1 alone, n=48, P=100000 71 -> 67) and costs the fused
  // Algorithm 1 up to 2% in long bf16 ones (n=36, P=7.4M 1.82 -> 1.86 ms); with
  // more each is stored as soon as it is summed, for the registers.  In LDS they
  // may take the slots' place, once every slot has been read.
  const bool in_place = K >= kInPlaceWorkers && a.kept_off == 0;
  auto store_row = [&](int i, int k, const float (&res)[V], Held<DT, V>& held) {
    const int64_t row = static_cast<int64_t>(i) * a.ld + tile0;
    float as_kept[V];
    store_params<DT, V>(static_cast<char*>(a.x) + row * sp, at, cnt, res, as_kept);
    held.set(as_kept);
    if constexpr (kOuterRow<FORM>) {
      if (a.use_u) store_f32<V>(a.u + row + at, cnt, kept[k].v);
    }
  };
  if constexpr (K <= 4) {
    float res[K][V];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = wave + k * waves;
      if (i < n) tile_row<DT, V, FORM, kDeep, SHARED>(a, rp, col, val, i, slots, sums, at, kept[k], res[k]);
    }
    if (in_place) __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = wave + k * waves;
      if (i >= n) break;
      Held<DT, V> held;
      store_row(i, k, res[k], held);
      lds_put<V, kHalfRows>(xs, i * C + at, held);
    }
  } else {  // rows in place only
    Held<DT, V> stored[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = wave + k * waves;
      if (i >= n) break;
      float res[V];
      tile_row<DT, V, FORM, kDeep, SHARED>(a, rp, col, val, i, slots, sums, at, kept[k], res);
      store_row(i, k, res, stored[k]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = wave + k * waves;
      if (i >= n) break;
      lds_put<V, kHalfRows>(xs, i * C + at, stored[k]);
    }
  }
  __syncthreads();
  // consensus error, one column per thread, workers in order
  const double inv_n = 1.0 / static_cast<double>(n);
  const int cols = TAIL ? static_cast<int>(a.P - tile0 < C ? a.P - tile0 : C) : C;
  for (int c = threadIdx.x; c < cols; c += blockDim.x) {
    auto value = [&](int i) { return static_cast<double>(lds_value<kHalfRows>(xs, i * C + c)); };
    const double shift = value(0);
    double s = 0.0, q = 0.0;
    for (int i = 1; i < n; ++i) {
      const double d = value(i) - shift;
      s += d;
      q += d * d;
    }
    ce += q - s * s * inv_n;
  }
}

template <int DT, int V, int K, bool FUSED, int FORM, bool SHARED>
__device__ __forceinline__ void tile_rounds(const GossipArgs& a, const RowSum* sum, unsigned char* lds) {
  constexpr int C = kWave * V;
  const int64_t tiles = (a.P + C - 1) / C;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * a.tile_groups;
  const int64_t t1 = tiles - t0 < a.tile_groups ? tiles : t0 + a.tile_groups;
  double ce = 0.0, pg = 0.0;
  for (int64_t t = t0; t < t1; ++t) {
    // in place: the stored rows of the tile before have been summed
    if (K >= kInPlaceWorkers && a.kept_off == 0 && t > t0) __syncthreads();
    const int64_t tile0 = t * C;
    if (tile0 + C <= a.P)
      tile_round<DT, V, K, FUSED, FORM, SHARED, false>(a, sum, lds, tile0, ce, pg);
    else
      tile_round<DT, V, K, FUSED, FORM, SHARED, true>(a, sum, lds, tile0, ce, pg);
  }
  double total_ce, total_pg;
  block_sum2(ce, pg, total_ce, total_pg);
  if (threadIdx.x == 0) {
    a.partials[blockIdx.x] = total_ce;
    a.pg_partials[blockIdx.x] = total_pg;
  }
}

// Waves per SIMD.  The fused EQ kernel with two workers per wave needs 95
// registers, which let a fifth wave in: its eight streams are then faster with
// four (n=4, P=60M 1.87 -> 1.84 ms; n=2, P=100M bf16 1.39 -> 1.35).
template <int K, bool FUSED, int FORM>
constexpr int kMaxWaves = FUSED && FORM == GASLOC_FORM_EQ && K == 2 ? 4 : 8;

template <int DT, int V, int K, bool FUSED, int FORM>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, kMaxWaves<K, FUSED, FORM>))) void
k_gossip_tile(GossipArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  tile_rounds<DT, V, K, FUSED, FORM, false>(a, nullptr, lds);
}

// Rounds whose rows are all equal.  The entries are an argument of their own: in
// the other kernels' arguments they would cost every launch about 1 us of host
// time (512 bytes more: a round on a graph that changes, n=17, P=47504 20.5 ->
// 22.1 us).
template <int DT, int V, int K, bool FUSED, int FORM>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, kMaxWaves<K, FUSED, FORM>))) void
k_gossip_tile_shared(GossipArgs a, RowSum sum) {
  extern __shared__ __align__(16) unsigned char lds[];
  tile_rounds<DT, V, K, FUSED, FORM, true>(a, &sum, lds);
}

template <int DT, int K, bool FUSED, int FORM>
hipError_t launch_tile_kernel(const GossipArgs& a, const RowSum& sum, const LaunchShape& s, size_t lds,
                              hipStream_t stream) {
  if constexpr (!kOuterRow<FORM>) {
    if (sum.entries > 0)
      return launch_kernel(k_gossip_tile_shared<DT, kTileVec, K, FUSED, FORM>, dim3(s.blocks), s.threads, lds, stream,
                           a, sum);
  }
  return launch_kernel(k_gossip_tile<DT, kTileVec, K, FUSED, FORM>, dim3(s.blocks), s.threads, lds, stream, a);
}

template <int DT, bool FUSED, int FORM>
hipError_t launch_tile_workers(const GossipArgs& a, const RowSum& sum, const LaunchShape& s, size_t lds,
                               hipStream_t stream) {
  switch (s.batch) {
    case 1: return launch_tile_kernel<DT, 1, FUSED, FORM>(a, sum, s, lds, stream);
    case 2: return launch_tile_kernel<DT, 2, FUSED, FORM>(a, sum, s, lds, stream);
    case 3:
      if constexpr (FUSED && FORM == GASLOC_FORM_EQ)
        return launch_tile_kernel<DT, 3, FUSED, FORM>(a, sum, s, lds, stream);
      return hipErrorInvalidValue;
    case 4: return launch_tile_kernel<DT, 4, FUSED, FORM>(a, sum, s, lds, stream);
    case 5: return launch_tile_kernel<DT, 5, FUSED, FORM>(a, sum, s, lds, stream);
    case 6: return launch_tile_kernel<DT, 6, FUSED, FORM>(a, sum, s, lds, stream);
    case 7: return launch_tile_kernel<DT, 7, FUSED, FORM>(a, sum, s, lds, stream);
    default: return launch_tile_kernel<DT, 8, FUSED, FORM>(a, sum, s, lds, stream);
  }
}

template <int DT>
hipError_t launch_tile_form(const GossipArgs& a, const RowSum& sum, bool fused, int form, const LaunchShape& s,
                            size_t lds, hipStream_t stream) {
  switch (form) {
    case GASLOC_FORM_ALG1:
      return fused ? launch_tile_workers<DT, true, GASLOC_FORM_ALG1>(a, sum, s, lds, stream)
                   : launch_tile_workers<DT, false, GASLOC_FORM_ALG1>(a, sum, s, lds, stream);
    case GASLOC_FORM_DADAM:
      return launch_tile_workers<DT, false, GASLOC_FORM_DADAM>(a, sum, s, lds, stream);
    case GASLOC_FORM_LOCAL_DADAM:
      return launch_tile_workers<DT, false, GASLOC_FORM_LOCAL_DADAM>(a, sum, s, lds, stream);
    default:
      return fused ? launch_tile_workers<DT, true, GASLOC_FORM_EQ>(a, sum, s, lds, stream)
                   : launch_tile_workers<DT, false, GASLOC_FORM_EQ>(a, sum, s, lds, stream);
  }
}

}  // namespace
}  // namespace gasloc
