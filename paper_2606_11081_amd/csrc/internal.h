// Internal interfaces between the C ABI (runtime.cpp), the schedule
// generator (topology.cpp), the visit planner (plan.cpp) and the HIP kernels
// (adamw.hip, round_tile.h, round_planned.hip, reductions.hip, with the device
// helpers of device_common.h).  Not installed.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <string>
#include <vector>

#include "gasloc.h"

namespace gasloc {

constexpr int kMaxReplicas = 64;

// Message of the last failing context-free call on this thread (what
// gasloc_last_error(NULL) returns).
void set_thread_error(const std::string& msg);

bool make_topology(const gasloc_topology& topo, int n, uint64_t t, int32_t* row_ptr, int32_t* col,
                   float* val, int32_t cap, int32_t* nnz, std::string* err);
// Visit plan of a round for the slot-reusing kernel (plan.cpp): super-steps
// of at most kPlanBatch new z values and at most kPlanRows rows; the plan is
// checked by verify_plan before it is returned.  With reuse_mix, a row whose
// CSR entries equal those of the row summed just before it is encoded with
// kPlanReuseMix in place of its entry count and takes that row's sum (only
// for round forms whose neighbour sum does not depend on the row itself).
constexpr int kPlanBatch = 4;
constexpr int kPlanRows = 4;
constexpr int32_t kPlanReuseMix = -1;
bool plan_round(int n, const int32_t* rp, const int32_t* col, const float* val, bool reuse_mix,
                std::vector<int32_t>* ops, int* slots_used, std::string* err);
bool verify_plan(int n, const int32_t* rp, const int32_t* col, const float* val, bool reuse_mix,
                 const int32_t* ops, int len, int slots, std::string* err);
// The plan as the kernel reads it: every slot word (new values, each row's
// own slot, each entry's slot) multiplied by `unit`, the byte stride between
// a thread's slots in LDS.  For a plan verify_plan accepted.
bool scale_plan_slots(std::vector<int32_t>* ops, int32_t unit, std::string* err);
// Upper bound on the words of a plan for n workers.
size_t plan_words_max(int n);
bool skip_exchanges(int n, const int32_t* rp, const int32_t* col, const float* val, const uint8_t* alive,
                    const uint8_t* link_ok, int32_t* out_rp, int32_t* out_col, float* out_val, int32_t cap,
                    int32_t* nnz, std::string* err);

// ---------------------------------------------------------------------------
// kernel arguments (passed by value)
// ---------------------------------------------------------------------------

// One local AdamW step over the active workers.  Slot s of the launch works
// on worker rep[s]; bit s of from_x says that worker's live iterate is still
// the round anchor x (first step after a round), so the step reads x.
struct AdamArgs {
  const void* x;
  void* y;
  float* m;
  float* v;
  const float* g;
  int64_t ld, gld, P;
  float c_wd, b1, omb1, b2, omb2, eps;
  int32_t n_active;
  uint64_t from_x;
  int32_t rep[kMaxReplicas];
  float s1[kMaxReplicas];  // lr / (1 - b1^k)
  float c2[kMaxReplicas];  // sqrt(1 - b2^k)
};

// One gossip round; the consensus-error partial of every workgroup goes to
// partials[blockIdx.x], its partial sum of squared pseudo-gradients to
// pg_partials[blockIdx.x].  Workgroup b takes the column groups [b * tile_groups,
// (b + 1) * tile_groups) (a multiple of the workgroup size), in steps of one
// group per thread.
struct GossipArgs {
  void* x;
  const void* y;
  float* u;
  float* zp;
  const int32_t* row_ptr;
  const int32_t* col;
  const float* val;
  double* partials;
  double* pg_partials;
  int64_t ld, P;
  int64_t tile_groups;
  int32_t n;
  float mu, eta, gamma;
  int32_t nesterov;
  int32_t use_u;        // outer momentum buffer present (mu != 0)
  int32_t apply_gamma;  // gamma term of Eq. 2 (not in the first round)
  int32_t store_zp;     // keep z for the next round's gamma term
  uint64_t stepped;     // bit i: worker i took local steps since the last round

  // planned visit order (k_gossip_planned only): see plan.cpp
  const int32_t* ops;
  int32_t slots;

  // tile kernels only: byte offsets in LDS of the stored rows (0: they take the
  // slots' place, from kInPlaceWorkers per wave) and of the shared sums
  int32_t kept_off, sums_off;

  // Fused last local step (the fused kernel only): every worker i with bit i
  // of `active` first takes one AdamW step from its live iterate; the new
  // iterate feeds delta directly and is never written back (it is logically
  // reset to the new x by the round).  Scalars are indexed by worker.
  const float* g;
  float* m;
  float* v;
  int64_t gld;
  uint64_t active;
  float c_wd, b1, omb1, b2, omb2, eps;
  float s1[kMaxReplicas];
  float c2[kMaxReplicas];
};

// The entries that every row of a round holds, where the form sums them the same
// way for each (EQ, DADAM); `entries` is 0 where the rows differ and are read
// from the CSR.  A kernel argument: a launch recorded in a graph keeps them,
// whatever the context's CSR holds when it is replayed.
struct RowSum {
  int32_t entries;
  int32_t col[kMaxReplicas];
  float w[kMaxReplicas];
};

struct LaunchShape {
  int vec;      // columns per thread per step (1, 2 or 4)
  int threads;  // workgroup size
  int blocks;   // workgroups: one per tile of `per` steps of the workgroup
  int batch;    // tile kernel: workers per wave; planned kernel: workers whose loads are issued together
  int per;      // steps (threads * vec columns each) per workgroup
};

// Launchers: enqueue on `stream`, return the launch status.
hipError_t launch_local_adamw(const AdamArgs& a, int dtype, int cus, hipStream_t stream);
hipError_t launch_gossip_planned(const GossipArgs& a, int dtype, bool fused, int form, const LaunchShape& shape,
                                 hipStream_t stream);
// Rounds with the workers spread over the waves of a workgroup
// (round_tile.h): shape.threads / 64 waves with shape.batch workers each (1
// to 8; 3 in the fused EQ kernel only), kTileVec columns per lane, a.tile_groups tiles per workgroup;
// `lds`: the bytes a.kept_off and a.sums_off were laid out in.
constexpr int kTileVec = 4;
constexpr int kInPlaceWorkers = 4;  // the fewest per wave that may store rows in the slots' place
// Bytes of one slot: the mixed values are parameters as stored except in the EQ form.
constexpr size_t tile_slot_bytes(int dtype, int form) {
  return dtype == GASLOC_BF16 && form != GASLOC_FORM_EQ ? 2 : 4;
}
hipError_t launch_gossip_tile_f32(const GossipArgs& a, const RowSum& sum, bool fused, int form,
                                  const LaunchShape& shape, size_t lds, hipStream_t stream);
hipError_t launch_gossip_tile_bf16(const GossipArgs& a, const RowSum& sum, bool fused, int form,
                                   const LaunchShape& shape, size_t lds, hipStream_t stream);
// Workgroups of the selected planned round kernel that one CU holds at once,
// given its registers, LDS and wave limits (0 if the query fails).
int planned_blocks_per_cu(int dtype, bool fused, int form, const LaunchShape& shape, size_t dyn_lds);
// Dynamic LDS bytes of one workgroup of the planned kernel (z slots only).
size_t planned_lds_bytes(int slots, const LaunchShape& shape);
// The standalone consensus error of columns [p_begin, p_end): one partial per
// workgroup of reduce_threads(dtype) threads, each taking `per` consecutive
// steps of kReduceVec columns; consensus_error_blocks gives the count.  A step
// of a workgroup is 1024 fp32 or 2048 bf16 columns.
constexpr int kReduceVec = 4;
constexpr int reduce_threads(int dtype) { return dtype == GASLOC_BF16 ? 512 : 256; }
constexpr int reduce_step(int dtype) { return kReduceVec * reduce_threads(dtype); }
int consensus_error_blocks(int dtype, int64_t p_begin, int64_t p_end, int per);
hipError_t launch_consensus_error(const void* x, int dtype, int64_t ld, int n, int64_t p_begin,
                                  int64_t p_end, int per, double* partials, hipStream_t stream);
hipError_t launch_finalize(const double* partials, int count, double* out, hipStream_t stream);
// out[0] = sum of a[0..count), out[1] = sum of b[0..count), each as launch_finalize sums.
hipError_t launch_finalize2(const double* a, const double* b, int count, double* out, hipStream_t stream);
// The same sums for up to kMaxPartials partials per array, in a fixed order
// that depends only on count: beyond kFinalizeSegment partials, segments of
// kFinalizeSegment consecutive partials are summed first (into seg[0..S) and
// seg[S..2S), S = ceil(count / kFinalizeSegment)), then the segment sums.
constexpr int kFinalizeSegment = 4096;
constexpr int kMaxPartials = 1 << 20;
hipError_t launch_finalize2_large(const double* a, const double* b, int count, double* seg, double* out,
                                  hipStream_t stream);
// *out = the sum of a[0..count), count <= kMaxPartials, in the same
// segmented order (seg: at least ceil(count / kFinalizeSegment) doubles).
hipError_t launch_finalize_large(const double* a, int count, double* seg, double* out, hipStream_t stream);
// Zeros columns [0, P) of each of the n rows of x.
hipError_t launch_zero_rows(float* x, int64_t ld, int n, int64_t P, hipStream_t stream);
// The network average of columns [0, P), one step per workgroup.
hipError_t launch_replica_mean(const void* x, int dtype, int64_t ld, int n, int64_t P, void* out,
                               hipStream_t stream);

// LDS bytes of a round kernel's own reduction, beside its dynamic LDS.
constexpr size_t kStaticLds = 2 * 1024 / 64 * sizeof(double);

}  // namespace gasloc
