// omerf_launch.h -- host-side launchers shared between the translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "omerf_device.h"

namespace omerf {

// Whether the marches address a scene's rows with 32-bit byte offsets.
bool narrow_scene(const SceneDev& sc, int dtype);

hipError_t launch_place(const SceneDev& sc, const RayParams& rp, const float* o, const float* d, int64_t n,
                        int32_t* k_out, int32_t* n_placed, hipStream_t s);
hipError_t launch_mark(const SceneDev& sc, const RayParams& rp, const float* o, const float* d, int64_t n,
                       const int32_t* n_eval, uint8_t* fg, uint8_t* fxy, uint8_t* fxz, uint8_t* fyz, hipStream_t s);

// Batch records of a training step (float32 [slots][kRecFloats]): the forward
// leaves one per 16-sample batch of a ray, and the backward works from them
// instead of replaying the samples.
//   [0, 128)    [8][16]: channel 0 the samples' optical depths, 1..7 their
//               activated features, from the forward in record_place order;
//               then dL/dt of the 8 channels, in sample order, from k_grad
//   [128, 176)  [3][16]: the sample points (z, which both the XZ and the YZ sums
//               read, NaN: nothing to add)
//   176         the optical depth in front of the batch
constexpr int kRecPoint = 8 * kGroup, kRecCarry = 11 * kGroup, kRecFloats = 12 * kGroup;
// A fused step keeps records where n rays of at most n_max samples may have
// more than kRecordBatches batches and the placement counts find at least
// kRecordMin.  Steps with and without them: 423,000 batches (of 524,288)
// 1.83 and 1.78 ms, 637,000 (of 2^20) 3.29 and 3.43, 1.27 million 5.7 and 6.4,
// 2.54 million 10.4 and 12.3, 5.1 million in bfloat16 18.9 and 23.0; below, the
// planes' tiles are too thinly covered to pay for their sums (212,000: 1.22 and
// 1.07).  And only where a step crosses 0.4 of a plane's texel or more on every
// axis: on coarser planes a batch touches few texels and the scatter is cheap.
// 104,487 rays in float32 and bfloat16: planes of 3072 x 3069 texels 4.14 and
// 4.58 ms, 3.91 and 4.28; 2048 3.48 and 3.77, 3.23 and 3.36; 1536 3.28 and
// 3.37, 3.04 and 3.02; 700 2.83 and 2.72, 2.65 and 2.46; 359 2.75 and 2.50,
// 2.60 and 2.32.  And only without early termination: a ray's records are handed
// out for the samples that it places, a replay is over the samples that it
// reaches.  2^18 rays in float32 that stop at T < 1e-4 / 1e-3 / 1e-2 / 0.1 (918,000
// to 768,000 of 1,116,000 to 966,000 batches evaluated) 5.43 and 5.08, 5.42 and
// 4.90, 5.26 and 4.66, 4.72 and 4.23 ms; 2^20 of the towers in bfloat16 at 1e-4 /
// 1e-2 (1,096,000 of 1,892,000, 881,000 of 1,678,000) 6.46 and 6.03, 5.57 and 5.08.
//
// The placed batches are known on the device only.  A step that turns out to
// have fewer than kRecordMin has ordered and counted its rays and runs the
// kernels' record forms for nothing: 16,500 / 24,000 / 32,000 / 40,000 / 48,000 rays
// in float32 (169,000 to 490,000 of more than 2^20 batches) 1.69 ms and 1.61 without
// a workspace for records, 2.15 and 2.09, 2.34 and 2.26, 2.52 and 2.48, 2.76 and
// 2.71.  Where most rays miss the box it is more, since their keys collide in the
// locality order (1.1 ms each for its histogram and scatter): 2^20 rays of which 1 %
// meet it 3.81 and 1.41, none 2.70 and 0.35; with 10 % (1,017,000 batches, records
// kept) 7.43 and 6.63.
constexpr int64_t kRecordBatches = 1 << 20, kRecordMin = 1 << 19;
constexpr float kRecordTexels = 0.4f;
struct BatchRecords {
    float* rec;
    int32_t* slot_of_ray;  // [n] first record of each ray, -1: none
    int32_t* ray_at;       // [n] locality order of the rays, for the passes over the scene
    int* hist;             // its histogram (order_hist_bytes)
    uint16_t* keys;        // [n] and keys
    int cap;               // records
};
// Where sample i of a batch stands in a channel row as the forward writes it:
// the lane that holds it in the float32 forward.
__host__ __device__ constexpr int record_place(int i) { return 4 * (i & 3) + (i >> 2); }

// Texels of a plane that a step crosses at most, of the axis with the fewest.
float texels_per_step(const SceneDev& sc, float delta);
// br: NULL, or the records; rays without one get the per-batch sums.
hipError_t launch_march_fwd(const SceneDev& sc, int dtype, const RayParams& rp, const float* o, const float* d,
                            int64_t n, float* F, float* T, int32_t* n_placed, int32_t* n_eval, float* batch_wv,
                            const BatchRecords* br, hipStream_t s);
// Samples placed per ray; ray_at: a permutation of the rays to take them in.
hipError_t launch_count(const SceneDev& sc, const RayParams& rp, const float* o, const float* d, int64_t n,
                        const int32_t* ray_at, int32_t* n_placed, hipStream_t s);
// Scheduling words (int32) of the march backward in its workspace: the
// ray-order histogram, its cursors and the hand-out counters, and the slots of
// the rays' records.
constexpr int kBwdSchedWords = 256;
constexpr int kOrderRecords = 198;  // records in use

// Longest-first order of the rays by `counts`; with br, also their records
// (br->slot_of_ray), handed out to whole rays in that order.
hipError_t launch_bwd_order(const int32_t* counts, int64_t n, int n_max, int32_t* order, int* sched,
                            const BatchRecords* br, hipStream_t s);
// The march backward over that order; br: the rays with records go through
// them, the others replay their samples.
hipError_t launch_march_bwd(const SceneDev& sc, bool bf16, const RayParams& rp, const float* o, const float* d,
                            int64_t n, const float* T, const int32_t* n_eval, const float* batch_wv, const float* G8,
                            const int32_t* order, int* sched, const BatchRecords* br, float* gV, float* gxy,
                            float* gxz, float* gyz, float* gocc, hipStream_t s);

// Sums of the recorded XZ and YZ gradients (bwd_tiles.hip).
constexpr int kTileU = 17, kTileV = 20;  // base texels per tile
constexpr int kTileKeys = 4;             // tiles a batch may be listed under, per plane
constexpr int kNoTile = 0xffff;
struct TileLists {
    uint16_t* keys;   // [cap][2 kTileKeys]: the tile ids of a batch on XZ and YZ
    int32_t* listed;  // [2 kTileKeys cap]: records by tile
    int* bins;        // [nbins] entries per tile, then [nbins] cursors (in the end: where each tile's list ends)
    int* total;       // entries
    int nbins, yz;    // tiles, and the first of YZ
    int nu_x, nu_y;   // tiles per row of XZ and of YZ
};
// Workspace bytes of the records and lists for n rays of at most n_max
// samples, or 0 where they do not pay; fills *br and *tl when base is non-NULL.
int64_t record_workspace(const SceneDev& sc, const RayParams& rp, int64_t n, void* base, BatchRecords* br,
                         TileLists* tl);
hipError_t launch_tile_sums(const SceneDev& sc, const BatchRecords& br, const TileLists& tl, const int* records,
                            float* gxz, float* gyz, hipStream_t s);
hipError_t launch_mlp_bwd(const float* W, int mlp_in, const RayParams& rp, const float* F, const float* d,
                          const int32_t* n_eval, const float* dC, const float* dF, int64_t n, float* G8, float* gmlp,
                          hipStream_t s);
hipError_t launch_smooth(const float* W, int mlp_in, const float* F, const float* d, int64_t n, const float* perturb,
                         int P, float weight, float* loss, float* dF, float* gmlp, hipStream_t s);
hipError_t launch_mlp(const float* W, int mlp_in, bool bf16, const RayParams& rp, const float* d, int64_t n,
                      const float* F, const float* T, const int32_t* n_eval, float* C, hipStream_t s);
hipError_t launch_occ_pyramid(const float2* occ, int Mx, int My, float2* mips, int levels, hipStream_t s);
hipError_t launch_occ_loss(const float* occ, int64_t cells, float weight, float* loss, float* grad, hipStream_t s);
hipError_t launch_range(const float* x, int64_t n, float* minmax, uint32_t* keys, hipStream_t s);
hipError_t launch_quantize(const float* x, int64_t n, const float* lo, const float* inv, uint8_t* out, hipStream_t s);
hipError_t launch_blocks_mark(const SceneDev& sc, int shift, int bnx, int bny, int bnz, int32_t* mark, hipStream_t s);
hipError_t launch_blocks_number(int32_t* mark, int64_t n, hipStream_t s);
hipError_t launch_blocks_first(int32_t* mark, hipStream_t s);
hipError_t launch_blocks_fill(const SceneDev& sc, int shift, int bnx, int bny, int bnz, const int32_t* idx,
                              int64_t n_blocks, int units, void* atlas, hipStream_t s);
hipError_t launch_cast_bf16(const float* src, int64_t n, uint16_t* dst, hipStream_t s);
hipError_t launch_l2(const float* C, const float* tgt, int64_t n, float* dC, float* loss, hipStream_t s);
// Ray locality order (order.hip): histogram bytes of its workspace, the
// order with the reordered rays, and row gathers / scatters.
int64_t order_hist_bytes();
hipError_t launch_order_rays(const float* box_lo, const float* box_hi, const float* o, const float* d, int64_t n,
                             int32_t* order, float* o_out, float* d_out, int* hist, uint16_t* keys,
                             hipStream_t s);
hipError_t launch_rows_gather(const float* src, int64_t src_rows, int cols, const int32_t* idx, int64_t n,
                              float* dst, hipStream_t s);
hipError_t launch_rows_scatter(const float* src, int cols, const int32_t* idx, int64_t n, float* dst,
                               int64_t dst_rows, hipStream_t s);
hipError_t launch_l2_fp64(const float* C, const float* tgt, int64_t n, double* loss, hipStream_t s);

}  // namespace omerf
