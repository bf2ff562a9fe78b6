// march_fwd.hip -- occupancy-plane ray marching kernels for gfx950 (forward).
//
// k_place      : sample placement only (k-lists), Sec. 4.1 Eq. 6-7 / Sec. 4.4
// k_march_fwd_f32q / k_march_fwd_lane : placement + feature gather (Eq. 2)
//                + activations (Eq. 3) + compositing (Eq. 1) -> F, T, counts
//                per ray (float32 lane quads; bfloat16 and 8-bit one lane
//                per sample)
//
// One ray per 16-lane group; see omerf_device.h for the decomposition.
#include "../../include/omerf.h"
#include "omerf_device.h"
#include "omerf_launch.h"

#include <type_traits>

namespace omerf {

// ---------------------------------------------------------------------------
// Placement only.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_place(SceneDev sc, RayParams rp, const float* __restrict__ o_,
                                                  const float* __restrict__ d_, int64_t n,
                                                  int32_t* __restrict__ k_out, int32_t* __restrict__ n_placed) {
    __shared__ int qs[kGroupsPerBlock][kQueue];
    const int lane = threadIdx.x & 63;
    const int gl = lane & (kGroup - 1);
    const int gid = threadIdx.x / kGroup;
    const int64_t ray = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kGroupsPerBlock + gid;
    if (ray >= n) return;
    const float3 o = load3(o_, ray), d = load3(d_, ray);
    int32_t* kr = k_out + ray * rp.n_max;
    int written = 0;
    const int cnt = march_candidates(sc, rp, o, d, qs[gid], gl, gl, lane, [&](int kq, int nb) {
        if (gl < nb) kr[written + gl] = kq;
        written += nb;
        return false;
    });
    for (int i = cnt + gl; i < rp.n_max; i += kGroup) kr[i] = -1;
    if (gl == 0) n_placed[ray] = cnt;
}

// The counts alone, ahead of a training step that gives every batch a record.
__global__ __launch_bounds__(kBlock) void k_count(SceneDev sc, RayParams rp, const float* __restrict__ o_,
                                                  const float* __restrict__ d_, int64_t n,
                                                  const int32_t* __restrict__ ray_at, int32_t* __restrict__ n_placed) {
    const int lane = threadIdx.x & 63;
    const int gl = lane & (kGroup - 1);
    const int64_t at = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kGroupsPerBlock + threadIdx.x / kGroup;
    if (at >= n) return;
    const int64_t ray = ray_at[at];
    const int cnt = count_candidates(sc, rp, load3(o_, ray), load3(d_, ray), gl, lane);
    if (gl == 0) n_placed[ray] = cnt;
}

// What a forward leaves for the backward: nothing, the per-batch sums of w v,
// or a record per batch (the sums for rays without records).  With records,
// batches of many rays, the rays are taken in the locality order: the forward
// of 2^18 rays of 16 cameras in float32 3.31 ms as they come and 2.61 so, of
// 2^20 of 64 in bfloat16 6.5 and 4.7, for the 0.08 and 0.19 ms that ordering them
// costs.
enum { kSaveNone, kSaveSums, kSaveRecords };

// ---------------------------------------------------------------------------
// Rows read by a render: for every evaluated sample (the first n_eval placed
// samples of the ray, or all placed samples without n_eval), a byte 1 is
// stored at each of its 8 grid vertices and 12 plane texels (Eq. 2).
// Plain byte stores: marking is idempotent, so no atomics are needed.
// ---------------------------------------------------------------------------
template <bool kSparse>
__global__ __launch_bounds__(kBlock) void k_mark(SceneDev sc, RayParams rp, const float* __restrict__ o_,
                                                 const float* __restrict__ d_, int64_t n,
                                                 const int32_t* __restrict__ n_eval, uint8_t* __restrict__ fg,
                                                 uint8_t* __restrict__ fxy, uint8_t* __restrict__ fxz,
                                                 uint8_t* __restrict__ fyz) {
    __shared__ int qs[kGroupsPerBlock][kQueue];
    const int lane = threadIdx.x & 63;
    const int gl = lane & (kGroup - 1);
    const int gid = threadIdx.x / kGroup;
    const int64_t ray = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kGroupsPerBlock + gid;
    if (ray >= n) return;
    const float3 o = load3(o_, ray), d = load3(d_, ray);
    const int ne = n_eval ? n_eval[ray] : rp.n_max;
    if (ne <= 0) return;
    int done = 0;
    march_candidates(sc, rp, o, d, qs[gid], gl, gl, lane, [&](int kq, int nb) {
        const int nbe = min(nb, ne - done);
        if (gl < nbe) {
            const Corners c = corners_of<kSparse>(sc, lattice_point(kq, o, d, rp.delta));
            const uint32_t nx = (uint32_t)sc.Nx, ny = (uint32_t)sc.Ny;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t b = c.g + ((q & 1) ? sc.gsy : 0u) + ((q >> 1) ? sc.gsz : 0u);
                fg[b] = 1;
                fg[b + 1] = 1;
            }
            fxy[c.xy] = 1;
            fxy[c.xy + 1] = 1;
            fxy[c.xy + nx] = 1;
            fxy[c.xy + nx + 1] = 1;
            fxz[c.xz] = 1;
            fxz[c.xz + 1] = 1;
            fxz[c.xz + nx] = 1;
            fxz[c.xz + nx + 1] = 1;
            fyz[c.yz] = 1;
            fyz[c.yz + 1] = 1;
            fyz[c.yz + ny] = 1;
            fyz[c.yz + ny + 1] = 1;
        }
        done += nbe;
        return done >= ne;
    });
}

// ---------------------------------------------------------------------------
// Forward marches: write F [n][7], T [n], n_placed [n], n_eval [n] (and, with
// kSaveSums, the per-batch sums of w v, or with kSaveRecords the records).
// ---------------------------------------------------------------------------
// Group total of x (inclusive DPP scan; the row's last lane holds it) stored
// by that lane at dst, for the optional per-batch sums of w v.
__device__ __forceinline__ void store_group_total(float x, int gl, float* dst) {
    x = g_scan_incl(x, gl);
    if (gl == kGroup - 1) *dst = x;
}

// ---------------------------------------------------------------------------
// Forward march with one lane per sample, for 8-bit and bfloat16 features.
// A corner pair is 16 (8-bit) or 32 (bfloat16) contiguous bytes, so lane s
// of the group shades sample s of the batch on its own (10 or 20 loads),
// and the batch of 16 samples is composited with one 16-lane scan.  8-bit is
// bound by vector instructions: reading the decoding from the argument
// segment instead of spilled scalar registers, and xcd_block's runs, took a
// 1920x1080 frame with sparse blocks and early termination from 3.66 to 2.57 ms.
// (The sources' four offsets are not summed first, which takes 2.53: a feature
// then has the rounding of their sum, up to four times its own range.)
// bfloat16 is bound by L1 line lookups (1.19 per clock, 36 per load instruction).
// ---------------------------------------------------------------------------
// A sample as the lane that owns it holds it for the other lanes of its quad.
struct QuadSample {
    uint32_t g, xy, xz, yz;              // row keys (RowAddr)
    float fx, fy, fz, ux, uy, uz;        // grid and plane fractions
};

template <bool kNarrow, int kBytes>
__device__ __forceinline__ QuadSample quad_sample(const Corners& c) {
    using A = RowAddr<kNarrow, kBytes>;
    return QuadSample{A::key(c.g), A::key(c.xy), A::key(c.xz), A::key(c.yz), c.fx, c.fy, c.fz, c.ux, c.uy, c.uz};
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// kLanes: the lanes that gather together, which all have to be there; kStage:
// bytes of LDS per wave.
struct GatherU8 {
    static constexpr int kLanes = 1, kStage = 0;
    template <bool kNarrow>
    static __device__ __forceinline__ void run(const SceneDev& sc, const Corners& c, int, char*, float* t) {
        gather_u8<kNarrow>(sc, c, t);
    }
};
struct GatherBF16 {
    static constexpr int kLanes = 1, kStage = 0;
    template <bool kNarrow>
    static __device__ __forceinline__ void run(const SceneDev& sc, const Corners& c, int, char*, float* t) {
        gather_features_split<BF16Store, kNarrow>(sc, c, t);
    }
};

// Rows through LDS: lanes 2i and 2i + 1 of a quad load the two texels of a
// corner pair straight into LDS, first for samples 0 and 1 of the quad, then
// for 2 and 3, so that a load has 32 contiguous bytes of two samples per quad
// and not 16 of four; each lane then reads its own sample's two texels there.
// Where consecutive samples lie in different texel rows the L1 looks up 25
// lines per load instead of 36, and three rows are in flight without holding
// registers (two: 25.8 ms for 3840x2160, four at fewer waves: 28.3).  The sums
// are those of GatherBF16 in the same order.
//
// One lane per sample and this, by the texels per step and axis: 1 (planes of
// 4096 x 4096 x 512) 31.3 and 25.6 ms for 3840x2160, 8.07 and 6.69 for
// 1920x1080, 0.617 and 0.625 for 333x251, sparse blocks 7.71 and 6.83; 0.5
// 1.69 and 1.49 (960x540), 0.291 and 0.266 (333x251); 0.19 1.53 and 1.47, 0.283
// and 0.277; 0.12 1.46 and 1.45, 0.271 and 0.273; 0.06 1.41 and 1.44, 0.253 and
// 0.263.  A training step's rays share few lines, and its forward gains nothing
// (2^20 rays 21.4 and 21.5 ms).
struct GatherBF16Lds {
    static constexpr int kLanes = 4;
    static constexpr int kAhead = 3;                // rows in flight
    static constexpr int kHalf = 64 * 16 + 16;      // a load; 16 bytes keep the quad's reads off each other's banks
    static constexpr int kRow = kHalf + 64 * 16;
    static constexpr int kStage = kAhead * kRow;    // with the queues 26,816 bytes per block: six per CU

    template <int kPerm, bool kNarrow>
    static __device__ __forceinline__ void load(const void* base, uint32_t stride, uint32_t key, uint32_t lane_off,
                                                char* dst) {
        using A = RowAddr<kNarrow, BF16Store::kBytes>;
        const uint32_t k = quad_perm<kPerm>(key);
        const char* p = kNarrow ? A::at(base, stride, k + lane_off) : A::at(base, stride, k) + lane_off;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                         (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    }

    // The lane's two texels of a row once at most kNewer later loads are out.
    template <int kNewer>
    static __device__ __forceinline__ void read(uint32_t at, u32x4& x0, u32x4& x1) {
        asm volatile(
            "s_waitcnt vmcnt(%3)\n\tds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)"
            : "=&v"(x0), "=&v"(x1)
            : "v"(at), "n"(kNewer)
            : "memory");
    }

    template <bool kNarrow>
    static __device__ __forceinline__ void run(const SceneDev& sc, const Corners& c, int lane, char* stage, float* t) {
        const QuadSample o = quad_sample<kNarrow, BF16Store::kBytes>(c);
        const uint32_t lane_off = lane & 1 ? 16u : 0u;
        const uint32_t sy = sc.gsy, sz = sc.gsz, nx = (uint32_t)sc.Nx, ny = (uint32_t)sc.Ny;
        const void* base[10] = {sc.grid, sc.grid, sc.grid, sc.grid, sc.pxy, sc.pxy, sc.pxz, sc.pxz, sc.pyz, sc.pyz};
        const uint32_t stride[10] = {0u, sy, sz, sz + sy, 0u, nx, 0u, nx, 0u, ny};
        const uint32_t key[10] = {o.g, o.g, o.g, o.g, o.xy, o.xy, o.xz, o.xz, o.yz, o.yz};
        auto issue = [&](int j) {
            char* dst = stage + j % kAhead * kRow;
            load<0x50, kNarrow>(base[j], stride[j], key[j], lane_off, dst);          // samples 0, 0, 1, 1
            load<0xFA, kNarrow>(base[j], stride[j], key[j], lane_off, dst + kHalf);  // 2, 2, 3, 3
        };
        const uint32_t own = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)stage +
                             (uint32_t)((lane & 2 ? kHalf : 0) + ((lane & ~3) + (lane & 1) * 2) * 16);
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = 0.0f;
        auto row = [&](auto jc, float w0, float w1) {
            constexpr int j = decltype(jc)::value, newer = 2 * (j + kAhead <= 10 ? kAhead - 1 : 9 - j);
            u32x4 x0, x1;
            read<newer>(own + j % kAhead * kRow, x0, x1);
            if (j + kAhead < 10) issue(j + kAhead);
            BF16Store::acc(make_uint4(x0.x, x0.y, x0.z, x0.w), w0, t);
            BF16Store::acc(make_uint4(x1.x, x1.y, x1.z, x1.w), w1, t);
        };
#pragma unroll
        for (int j = 0; j < kAhead; ++j) issue(j);
        const float x0 = 1.0f - c.fx, x1 = c.fx, y0 = 1.0f - c.fy, y1 = c.fy, z0 = 1.0f - c.fz, z1 = c.fz;
        const float a0 = 1.0f - c.ux, a1 = c.ux, b0 = 1.0f - c.uy, b1 = c.uy, e0 = 1.0f - c.uz, e1 = c.uz;
        row(std::integral_constant<int, 0>{}, x0 * (y0 * z0), x1 * (y0 * z0));
        row(std::integral_constant<int, 1>{}, x0 * (y1 * z0), x1 * (y1 * z0));
        row(std::integral_constant<int, 2>{}, x0 * (y0 * z1), x1 * (y0 * z1));
        row(std::integral_constant<int, 3>{}, x0 * (y1 * z1), x1 * (y1 * z1));
        row(std::integral_constant<int, 4>{}, a0 * b0, a1 * b0);
        row(std::integral_constant<int, 5>{}, a0 * b1, a1 * b1);
        row(std::integral_constant<int, 6>{}, a0 * e0, a1 * e0);
        row(std::integral_constant<int, 7>{}, a0 * e1, a1 * e1);
        row(std::integral_constant<int, 8>{}, b0 * e0, b1 * e0);
        row(std::integral_constant<int, 9>{}, b0 * e1, b1 * e1);
    }
};

// Waves per SIMD the one-lane-per-sample forwards are compiled for: without
// the soft occupancy and with 32-bit addresses they fit 6 (<= 80 VGPRs)
// without spilling, with records 5; the other forms keep the compiler's choice.
template <int kSave, bool kSoft, bool kNarrow>
constexpr int lane_min_waves() {
    return !kSoft && kNarrow ? (kSave == kSaveRecords ? 5 : 6) : 1;
}

template <class Gather, int kSave, bool kSoft, bool kSparse, bool kNarrow>
__global__ __launch_bounds__(kBlock, (lane_min_waves<kSave, kSoft, kNarrow>())) void k_march_fwd_lane(
    SceneDev sc, RayParams rp, const float* __restrict__ o_, const float* __restrict__ d_, int64_t n,
    float* __restrict__ F, float* __restrict__ T, int32_t* __restrict__ n_placed, int32_t* __restrict__ n_eval,
    float* __restrict__ BW, BatchRecords br) {
    __shared__ int qs[kGroupsPerBlock][kQueue];
    __shared__ __attribute__((aligned(16))) char stages[Gather::kStage ? kBlock / 64 * Gather::kStage : 16];
    char* stage = stages + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) * Gather::kStage;
    const int lane = threadIdx.x & 63;
    const int gl = lane & (kGroup - 1);
    const int gid = threadIdx.x / kGroup;
    const int64_t at = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kGroupsPerBlock + gid;
    if (at >= n) return;
    const int64_t ray = kSave == kSaveRecords ? (int64_t)br.ray_at[at] : at;
    const float3 o = load3(o_, ray), d = load3(d_, ray);
    float acc[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) acc[c] = 0.0f;
    float carry = 0.0f;
    int evals = 0, batch = 0;
    const int slots = (rp.n_max + kGroup - 1) / kGroup;
    const int slot = kSave == kSaveRecords ? br.slot_of_ray[ray] : -1;
    const int placed = march_candidates(sc, rp, o, d, qs[gid], gl, gl, lane, [&](int kq, int nb) {
        const bool act = gl < nb;
        float t[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) t[c] = 0.0f;
        float msoft = 0.0f;
        if ((gl & -Gather::kLanes) < nb) {
            const float3 p = lattice_point(kq, o, d, rp.delta);
            const SceneDev& sa = scene_argument();
            Gather::template run<kNarrow>(sa, corners_of<kSparse, kNarrow>(sa, p), lane, stage, t);
            if (kSoft) msoft = occ_value(sc, p, rp.occ_inv_eps).m;
        }
        float a = 0.0f;
        float v[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) v[c] = 0.0f;
        if (act) {
            a = __expf(t[0]) * rp.delta;
#pragma unroll
            for (int c = 0; c < 7; ++c) v[c] = sigmoidf_fast(t[c + 1]);
        }
        const float incl = g_scan_incl(a, gl);
        const float excl = g_shift_up1(incl);
        float w = __expf(-(carry + excl)) * (-expm1f(-a));
        int nb_eff = nb;
        bool stop = false;
        if (rp.t_term > 0.0f) {
            const float Tnext = __expf(-(carry + incl));
            const uint32_t m = g_ballot(act && Tnext < rp.t_term, lane);
            if (m) {
                nb_eff = __ffs(m);
                stop = true;
            }
        }
        if (kSoft) w *= msoft;  // Eq. 8: the weight, not T
        if (gl >= nb_eff) w = 0.0f;
#pragma unroll
        for (int c = 0; c < 7; ++c) acc[c] += w * v[c];
        if (kSave == kSaveRecords && slot >= 0) {
            float* r = br.rec + (size_t)(slot + batch) * kRecFloats;
            float* own = r + record_place(gl);
            own[0] = a;
#pragma unroll
            for (int c = 0; c < 7; ++c) own[(c + 1) * kGroup] = v[c];
            const float3 p = lattice_point(kq, o, d, rp.delta);
            r[kRecPoint + gl] = p.x;
            r[kRecPoint + kGroup + gl] = p.y;
            r[kRecPoint + 2 * kGroup + gl] = p.z;
            if (gl == 0) r[kRecCarry] = carry;
        } else if (kSave != kSaveNone) {
            float* dst = BW + ((size_t)ray * slots + batch) * 7;
#pragma unroll
            for (int c = 0; c < 7; ++c) store_group_total(w * v[c], gl, dst + c);
        }
        carry += __shfl(incl, nb_eff - 1, kGroup);
        evals += nb_eff;
        ++batch;
        return stop;
    });
    float f[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) f[c] = g_sum(acc[c]);
    if (gl == 0) {
#pragma unroll
        for (int c = 0; c < 7; ++c) F[ray * 7 + c] = f[c];
        T[ray] = __expf(-carry);
        n_placed[ray] = placed;
        n_eval[ray] = evals;
    }
}

// ---------------------------------------------------------------------------
// Forward march for float32 features, lane-quad shading.  A queued batch of
// up to 16 samples is shaded in four quarters; in quarter j, lanes
// 4s..4s+3 of the group shade sample 4j + s, lane 4s+q taking x-offset
// (q & 1) and channel half (q >> 1).  A float32 corner pair is 64
// contiguous bytes, so each gather instruction reads one 64-byte span for
// each of 4 consecutive samples of the ray.
//
// A load instruction moves 1,024 bytes, 16 cycles of the L1 at 64 bytes each;
// the kernel starts one every 18.5 (1920x1080 frame), and a SIMD a vector
// instruction every 4.8.  So whatever a sample needs once is computed on one lane:
// lane 4s + j holds sample 4j + s from the start -- its point, row offsets and
// fractions, density, optical depth and weight -- and hands it to the quad
// that shades it with DPP quad broadcasts, which cost one instruction or ride
// on the one that uses the value.  The two x-offset lanes of a channel half
// end with two channels each, so an activation is evaluated once.  With all
// of that on all four lanes, 64-bit vector addresses and scalar registers
// spilled to vector lanes, 64 samples took 1240 vector instructions and a
// 1920x1080 frame of the full-size scene 13.98 ms; with some 600 10.52 ms, and
// 9.14 with the rays dealt to the XCDs in short runs (xcd_block).
// ---------------------------------------------------------------------------
// Sample 4j + s of the quad, j = kJ: the lane's half of the channels, summed
// over the rows at its x-offset.  lane_off: the lane's 16 bytes within a
// corner pair; hs, h0: its x weight is h0 + hs * fraction.
template <int kJ, bool kNarrow>
__device__ __forceinline__ void quad_gather(const SceneDev& sc, const QuadSample& o, uint32_t lane_off, float hs,
                                            float h0, float* t) {
    using A = RowAddr<kNarrow, 32>;
    const uint32_t sy = sc.gsy, sz = sc.gsz, nx = (uint32_t)sc.Nx, ny = (uint32_t)sc.Ny;
    const uint32_t kg = quad_bcast<kJ>(o.g), kxy = quad_bcast<kJ>(o.xy), kxz = quad_bcast<kJ>(o.xz),
                   kyz = quad_bcast<kJ>(o.yz);
    auto row = [&](const void* base, uint32_t stride, uint32_t key) {
        // narrow: the lane's offset joins the 32-bit key
        return *reinterpret_cast<const float4*>(kNarrow ? A::at(base, stride, key + lane_off)
                                                        : A::at(base, stride, key) + lane_off);
    };
    float4 r[10];
    r[0] = row(sc.grid, 0u, kg);
    r[1] = row(sc.grid, sy, kg);
    r[2] = row(sc.grid, sz, kg);
    r[3] = row(sc.grid, sz + sy, kg);
    r[4] = row(sc.pxy, 0u, kxy);
    r[5] = row(sc.pxy, nx, kxy);
    r[6] = row(sc.pxz, 0u, kxz);
    r[7] = row(sc.pxz, nx, kxz);
    r[8] = row(sc.pyz, 0u, kyz);
    r[9] = row(sc.pyz, ny, kyz);
    const float wx = fmaf(hs, quad_bcast<kJ>(o.fx), h0);
    const float wa = fmaf(hs, quad_bcast<kJ>(o.ux), h0);  // x for XY / XZ
    const float wb = fmaf(hs, quad_bcast<kJ>(o.uy), h0);  // y for YZ
    const float y1 = quad_bcast<kJ>(o.fy), z1 = quad_bcast<kJ>(o.fz), y0 = 1.0f - y1, z0 = 1.0f - z1;
    const float b1 = quad_bcast<kJ>(o.uy), e1 = quad_bcast<kJ>(o.uz), b0 = 1.0f - b1, e0 = 1.0f - e1;
    const float xy0 = wx * y0, xy1 = wx * y1;
    const float w[10] = {xy0 * z0, xy1 * z0, xy0 * z1, xy1 * z1, wa * b0, wa * b1, wa * e0, wa * e1, wb * e0, wb * e1};
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < 10; ++j) {
        t[0] += w[j] * r[j].x;
        t[1] += w[j] * r[j].y;
        t[2] += w[j] * r[j].z;
        t[3] += w[j] * r[j].w;
    }
}

template <int kSave, bool kSoft, bool kSparse, bool kNarrow>
__global__ __launch_bounds__(kBlock, 4) void k_march_fwd_f32q(
    SceneDev sc, RayParams rp, const float* __restrict__ o_, const float* __restrict__ d_, int64_t n,
    float* __restrict__ F, float* __restrict__ T, int32_t* __restrict__ n_placed, int32_t* __restrict__ n_eval,
    float* __restrict__ BW, BatchRecords br) {
    __shared__ int qs[kGroupsPerBlock][kQueue];
    const int lane = threadIdx.x & 63;
    const int gl = lane & (kGroup - 1);
    const int gid = threadIdx.x / kGroup;
    const int h = gl & 1, q = gl & 3;
    const int pos = 4 * q + (gl >> 2);  // the lane's own sample of a batch
    const uint32_t lane_off = (uint32_t)(h * 32 + (gl & 2) * 8);
    const float hs = h ? 1.0f : -1.0f, h0 = h ? 0.0f : 1.0f;
    const int64_t at = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kGroupsPerBlock + gid;
    if (at >= n) return;
    const int64_t ray = kSave == kSaveRecords ? (int64_t)br.ray_at[at] : at;
    const float3 o = load3(o_, ray), d = load3(d_, ray);
    float acc0 = 0.0f, acc1 = 0.0f;  // channels 2q and 2q + 1 (0 is the density)
    float carry = 0.0f;
    int evals = 0, batch = 0;
    const int slots = (rp.n_max + kGroup - 1) / kGroup;
    const int slot = kSave == kSaveRecords ? br.slot_of_ray[ray] : -1;
    const int placed = march_candidates(sc, rp, o, d, qs[gid], gl, pos, lane, [&](int kq, int nb) {
        const QuadSample own = quad_sample<kNarrow, 32>(
            corners_of<kSparse, kNarrow>(scene_argument(), lattice_point(kq, o, d, rp.delta)));
        const SceneDev& sa = scene_argument();
        float v0[4], v1[4], t0 = 0.0f;
        auto quarter = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
            v0[j] = v1[j] = 0.0f;
            if (4 * j < nb) {
                float t[4];
                quad_gather<j, kNarrow>(sa, own, lane_off, hs, h0, t);
                // The other x-offset's sums, two channels to each lane.
                const float u0 = (h ? t[2] : t[0]) + pair_swap(h ? t[0] : t[2]);
                const float u1 = (h ? t[3] : t[1]) + pair_swap(h ? t[1] : t[3]);
                const float dens = quad_bcast<0>(u0);
                t0 = q == j ? dens : t0;
                v0[j] = sigmoidf_fast(u0);
                v1[j] = sigmoidf_fast(u1);
            }
        };
        quarter(std::integral_constant<int, 0>{});
        quarter(std::integral_constant<int, 1>{});
        quarter(std::integral_constant<int, 2>{});
        quarter(std::integral_constant<int, 3>{});
        const bool act = pos < nb;
        const float a = act ? __expf(t0) * rp.delta : 0.0f;
        // Optical depth in front of the lane's sample: carry + the earlier
        // quarters one after another (their totals are in the last quad) +
        // the samples before it in its own quarter (lower quads, same q).
        float col = a;
        col += dpp_row<kRowShr | 4>(col);
        col += dpp_row<kRowShr | 8>(col);
        const float run1 = carry + row_bcast<12>(col), run2 = run1 + row_bcast<13>(col);
        const float run3 = run2 + row_bcast<14>(col);
        const float run = q == 0 ? carry : q == 1 ? run1 : q == 2 ? run2 : run3;
        const float pre = run + dpp_row<kRowShr | 4>(col);
        int nb_eff = nb;
        bool stop = false;
        if (rp.t_term > 0.0f) {
            const int first = g_min(act && __expf(-(pre + a)) < rp.t_term ? pos : kGroup);
            if (first < nb) {
                nb_eff = first + 1;
                stop = true;
            }
        }
        float w = __expf(-pre) * (-expm1f(-a));
        if (kSoft) w *= occ_value(sc, lattice_point(kq, o, d, rp.delta), rp.occ_inv_eps).m;  // Eq. 8: the weight, not T
        if (pos >= nb_eff) w = 0.0f;
        float b0 = quad_bcast<0>(w) * v0[0], b1 = quad_bcast<0>(w) * v1[0];
        b0 += quad_bcast<1>(w) * v0[1];
        b1 += quad_bcast<1>(w) * v1[1];
        b0 += quad_bcast<2>(w) * v0[2];
        b1 += quad_bcast<2>(w) * v1[2];
        b0 += quad_bcast<3>(w) * v0[3];
        b1 += quad_bcast<3>(w) * v1[3];
        acc0 += b0;
        acc1 += b1;
        if (kSave == kSaveRecords && slot >= 0) {
            float* r = br.rec + (size_t)(slot + batch) * kRecFloats;
            float4* rows = reinterpret_cast<float4*>(r + 2 * q * kGroup + (gl & ~3));  // the quad's four samples
            const float4 depth = make_float4(quad_bcast<0>(a), quad_bcast<1>(a), quad_bcast<2>(a), quad_bcast<3>(a));
            rows[0] = q == 0 ? depth : make_float4(v0[0], v0[1], v0[2], v0[3]);
            rows[kGroup / 4] = make_float4(v1[0], v1[1], v1[2], v1[3]);
            int kr = kq;  // the point is formed again, not held across the gather
            asm volatile("" : "+v"(kr));
            const float3 p = lattice_point(kr, o, d, rp.delta);
            r[kRecPoint + pos] = p.x;
            r[kRecPoint + kGroup + pos] = p.y;
            r[kRecPoint + 2 * kGroup + pos] = p.z;
            if (gl == 0) r[kRecCarry] = carry;
        } else if (kSave != kSaveNone) {
            b0 = quad_column_sum(b0);
            b1 = quad_column_sum(b1);
            float* dst = BW + ((size_t)ray * slots + batch) * 7 + 2 * gl;
            if (gl < 4) {
                if (gl > 0) dst[-1] = b0;
                dst[0] = b1;
            }
        }
        ++batch;
        // depth through the last evaluated sample
        const int last = nb_eff - 1;
        carry = nb_eff == kGroup ? row_bcast<kGroup - 1>(pre + a)
                                 : __shfl(pre + a, 4 * (last & 3) + (last >> 2), kGroup);
        evals += nb_eff;
        return stop;
    });
    acc0 = quad_column_sum(acc0);
    acc1 = quad_column_sum(acc1);
    if (gl < 4) {
        float* dst = F + ray * 7 + 2 * gl;
        if (gl > 0) dst[-1] = acc0;
        dst[0] = acc1;
    }
    if (gl == 0) {
        T[ray] = __expf(-carry);
        n_placed[ray] = placed;
        n_eval[ray] = evals;
    }
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
static inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kGroupsPerBlock - 1) / kGroupsPerBlock); }

hipError_t launch_count(const SceneDev& sc, const RayParams& rp, const float* o, const float* d, int64_t n,
                        const int32_t* ray_at, int32_t* n_placed, hipStream_t s) {
    hipLaunchKernelGGL(k_count, dim3(blocks_for(n)), dim3(kBlock), 0, s, sc, rp, o, d, n, ray_at, n_placed);
    return hipGetLastError();
}

hipError_t launch_place(const SceneDev& sc, const RayParams& rp, const float* o, const float* d, int64_t n,
                        int32_t* k_out, int32_t* n_placed, hipStream_t s) {
    hipLaunchKernelGGL(k_place, dim3(blocks_for(n)), dim3(kBlock), 0, s, sc, rp, o, d, n, k_out, n_placed);
    return hipGetLastError();
}

hipError_t launch_mark(const SceneDev& sc, const RayParams& rp, const float* o, const float* d, int64_t n,
                       const int32_t* n_eval, uint8_t* fg, uint8_t* fxy, uint8_t* fxz, uint8_t* fyz, hipStream_t s) {
    if (sc.blk_shift > 0)
        hipLaunchKernelGGL(k_mark<true>, dim3(blocks_for(n)), dim3(kBlock), 0, s, sc, rp, o, d, n, n_eval, fg, fxy,
                           fxz, fyz);
    else
        hipLaunchKernelGGL(k_mark<false>, dim3(blocks_for(n)), dim3(kBlock), 0, s, sc, rp, o, d, n, n_eval, fg, fxy,
                           fxz, fyz);
    return hipGetLastError();
}

// Whether every feature source can be addressed with 32-bit byte offsets and
// 24-bit index factors (RowAddr<true>): the full-size scenes of the benchmark
// can, in every storage type (their float32 grid is 4 GiB exactly).
bool narrow_scene(const SceneDev& sc, int dtype) {
    const uint64_t bytes = dtype == OM_F32 ? 32 : dtype == OM_BF16 ? 16 : 8, most = 1ull << 32, f24 = 1ull << 24;
    const uint64_t grid = sc.blk_shift > 0 ? ((uint64_t)sc.n_blocks + 1) * sc.blk_verts
                                           : (uint64_t)sc.Lx * (uint64_t)sc.Ly * (uint64_t)sc.Lz;
    const bool factors = sc.blk_shift > 0 ? sc.n_blocks < f24
                                          : (uint64_t)sc.Ly * (uint64_t)sc.Lz <= f24 && (uint64_t)sc.Lx < f24;
    return factors && grid * bytes <= most && (uint64_t)sc.Nx * (uint64_t)sc.Ny * bytes <= most &&
           (uint64_t)sc.Nx * (uint64_t)sc.Nz * bytes <= most && (uint64_t)sc.Ny * (uint64_t)sc.Nz * bytes <= most;
}

float texels_per_step(const SceneDev& sc, float delta) { return fminf(sc.px.s, fminf(sc.py.s, sc.pz.s)) * delta; }

template <bool kSoft, bool kSparse, bool kNarrow>
static void launch_fwd_form(const SceneDev& sc, int dtype, const RayParams& rp, const float* o, const float* d,
                            int64_t n, float* F, float* T, int32_t* n_placed, int32_t* n_eval, float* batch_wv,
                            const BatchRecords* br, hipStream_t s) {
    // Sparse blocks and 8-bit features are render only (the API refuses
    // per-batch sums for them).
    constexpr int kSums = kSparse ? kSaveNone : kSaveSums, kRecs = kSparse ? kSaveNone : kSaveRecords;
    typedef void (*Kernel)(SceneDev, RayParams, const float*, const float*, int64_t, float*, float*, int32_t*,
                           int32_t*, float*, BatchRecords);
    static constexpr Kernel f32[3] = {k_march_fwd_f32q<kSaveNone, kSoft, kSparse, kNarrow>,
                                      k_march_fwd_f32q<kSums, kSoft, kSparse, kNarrow>,
                                      k_march_fwd_f32q<kRecs, kSoft, kSparse, kNarrow>};
    static constexpr Kernel bf16[3] = {k_march_fwd_lane<GatherBF16, kSaveNone, kSoft, kSparse, kNarrow>,
                                       k_march_fwd_lane<GatherBF16, kSums, kSoft, kSparse, kNarrow>,
                                       k_march_fwd_lane<GatherBF16, kRecs, kSoft, kSparse, kNarrow>};
    // Rows through LDS: plain renders of scenes with 32-bit addresses.
    constexpr bool kLds = kNarrow && !kSoft;
    static constexpr Kernel bf16_lds =
        k_march_fwd_lane<std::conditional_t<kLds, GatherBF16Lds, GatherBF16>, kSaveNone, kSoft, kSparse, kNarrow>;
    const int save = br ? kSaveRecords : batch_wv ? kSaveSums : kSaveNone;
    // Below 0.15 texels per step the samples of a quad share their rows anyway.
    const bool lds = kLds && save == kSaveNone && texels_per_step(sc, rp.delta) >= 0.15f;
    const Kernel k = dtype == OM_U8 ? k_march_fwd_lane<GatherU8, kSaveNone, kSoft, kSparse, kNarrow>
                                    : dtype == OM_BF16 ? (lds ? bf16_lds : bf16[save]) : f32[save];
    hipLaunchKernelGGL(k, dim3(blocks_for(n)), dim3(kBlock), 0, s, sc, rp, o, d, n, F, T, n_placed, n_eval, batch_wv,
                       br ? *br : BatchRecords{});
}

hipError_t launch_march_fwd(const SceneDev& sc, int dtype, const RayParams& rp, const float* o, const float* d,
                            int64_t n, float* F, float* T, int32_t* n_placed, int32_t* n_eval, float* batch_wv,
                            const BatchRecords* br, hipStream_t s) {
    // The per-batch sums, the soft occupancy, the sparse blocks and the wide
    // addresses are separate specialisations, so the plain path carries none.
    typedef void (*Form)(const SceneDev&, int, const RayParams&, const float*, const float*, int64_t, float*, float*,
                         int32_t*, int32_t*, float*, const BatchRecords*, hipStream_t);
    static constexpr Form forms[2][2][2] = {
        {{launch_fwd_form<false, false, false>, launch_fwd_form<false, false, true>},
         {launch_fwd_form<false, true, false>, launch_fwd_form<false, true, true>}},
        {{launch_fwd_form<true, false, false>, launch_fwd_form<true, false, true>},
         {launch_fwd_form<true, true, false>, launch_fwd_form<true, true, true>}}};
    forms[rp.occ_inv_eps > 0.0f][sc.blk_shift > 0][narrow_scene(sc, dtype)](sc, dtype, rp, o, d, n, F, T, n_placed,
                                                                           n_eval, batch_wv, br, s);
    return hipGetLastError();
}

}  // namespace omerf
