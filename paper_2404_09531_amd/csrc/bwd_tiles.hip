// bwd_tiles.hip -- XZ and YZ gradients of the march backward, from its batch
// records, summed by tiles.
//
// The terrain band leaves few rows of the XZ and YZ planes in use, and a
// training step's samples fall on those tens of times per texel, from rays
// that are nowhere near one another in the batch.  Added one 64-byte segment
// per batch and row they are half of the backward's float atomics, whose rate
// beyond L2 bounds it.  So the recorded batches are listed by the tiles of
// kTileU x kTileV texels that their samples fall in, and each tile is summed
// in LDS and added to its plane once.
//
// k_tile_keys : the tiles of each batch and the number of entries per tile;
// k_tile_scan : start of each tile's list;
// k_tile_list : lists the batches by tile;
// k_tile_sum  : sums the tiles, each wave over an equal share of the lists.
//
// 2^18 rays in float32 (2.5 million batches): keys 0.26 ms, list 0.09, sum
// 2.50, of which the records' reads at the large copy's rate are about 0.9 and the
// rest the four read-add-write steps per batch and plane in LDS, one after
// another.
#include "omerf_launch.h"

namespace omerf {

constexpr int kListThreads = 1024;
constexpr int kListBlocks = 256;
constexpr int kTileMaxBins = 16384;  // a block's counters: 64 KB of LDS
constexpr int kKeysPerBatch = 2 * kTileKeys;

__global__ __launch_bounds__(kListThreads) void k_tile_clear(int* __restrict__ bins, int nbins) {
    const int i = blockIdx.x * kListThreads + threadIdx.x;
    if (i < nbins) bins[i] = 0;
}

// Records [s, e) of those in use that this block handles.
__device__ __forceinline__ void record_range(int records, int& s, int& e) {
    const int per = (records + (int)gridDim.x - 1) / (int)gridDim.x;
    s = (int)min((int64_t)records, (int64_t)blockIdx.x * per);
    e = min(records, s + per);
}

// Lane `first` + t of the group gets the t-th tile of one plane that the
// batch's samples fall in, in their order, kNoTile past the last.  A sample in
// a further one, rare since a batch spans few texels, is added to the plane
// here: 16 lanes take its pair of texels in each of its two rows.
__device__ __forceinline__ void batch_tiles(const float* __restrict__ rec, float* G, int bin0, int nu,
                                            const AxisMap& mu, const AxisMap& mv, float pu, float pv, bool add,
                                            int first, int gl, int lane, int& mine) {
    int ju = 0, jv = 0;
    float fu = 0.0f, fv = 0.0f;
    if (add) {
        axis_coord(pu, mu, ju, fu);
        axis_coord(pv, mv, jv, fv);
    }
    const int tile = bin0 + jv / kTileV * nu + ju / kTileU;
    bool left = add;
#pragma unroll
    for (int t = 0; t < kTileKeys; ++t) {
        const uint32_t m = g_ballot(left, lane);
        if (!m) return;
        const int k = __shfl(tile, __ffs(m) - 1, kGroup);
        if (gl == first + t) mine = k;
        left = left && tile != k;
    }
    const int n = (int)mu.top + 2;
    for (uint32_t m = g_ballot(left, lane); m; m &= m - 1) {
        const int s = __ffs(m) - 1;
        const float u = __shfl(fu, s, kGroup), v = __shfl(fv, s, kGroup);
        const float x = (gl & 8 ? u : 1.0f - u) * rec[(gl & 7) * kGroup + s];
        float* dst = G + ((size_t)__shfl(jv, s, kGroup) * (size_t)n + (size_t)__shfl(ju, s, kGroup)) * 8 + gl;
        unsafeAtomicAdd(dst, x * (1.0f - v));
        unsafeAtomicAdd(dst + (size_t)n * 8, x * v);
    }
}

__global__ __launch_bounds__(kListThreads) void k_tile_keys(SceneDev sc, const float* __restrict__ recs, TileLists tl,
                                                            const int* __restrict__ records, float* __restrict__ gxz,
                                                            float* __restrict__ gyz) {
    extern __shared__ int cnt[];
    for (int i = threadIdx.x; i < tl.nbins; i += kListThreads) cnt[i] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, gl = lane & (kGroup - 1);
    int s, e;
    record_range(*records, s, e);
    for (int i = s + (int)threadIdx.x / kGroup; i < e; i += kListThreads / kGroup) {
        const float* r = recs + (size_t)i * kRecFloats;
        const float px = r[kRecPoint + gl], py = r[kRecPoint + kGroup + gl], pz = r[kRecPoint + 2 * kGroup + gl];
        const bool add = pz == pz;
        int mine = kNoTile;
        batch_tiles(r, gxz, 0, tl.nu_x, sc.px, sc.pz, px, pz, add, 0, gl, lane, mine);
        batch_tiles(r, gyz, tl.yz, tl.nu_y, sc.py, sc.pz, py, pz, add, kTileKeys, gl, lane, mine);
        if (gl < kKeysPerBatch) {
            tl.keys[(size_t)i * kKeysPerBatch + gl] = (uint16_t)mine;
            if (mine != kNoTile) atomicAdd(&cnt[mine], 1);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < tl.nbins; i += kListThreads)
        if (cnt[i]) atomicAdd(&tl.bins[i], cnt[i]);
}

// Exclusive sum over the block; `all` receives the total.
__device__ __forceinline__ int block_scan(int x, int* part, int& all) {
    const int t = threadIdx.x;
    part[t] = x;
    __syncthreads();
    for (int off = 1; off < kListThreads; off <<= 1) {
        const int v = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    const int r = part[t] - x;
    all = part[kListThreads - 1];
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kListThreads) void k_tile_scan(int* __restrict__ bins, int nbins,
                                                            int* __restrict__ total) {
    __shared__ int part[kListThreads];
    const int per = (nbins + kListThreads - 1) / kListThreads;
    const int b0 = min(nbins, (int)threadIdx.x * per), b1 = min(nbins, b0 + per);
    int entries = 0, all;
    for (int b = b0; b < b1; ++b) entries += bins[b];
    int at = block_scan(entries, part, all);
    for (int b = b0; b < b1; ++b) {
        bins[nbins + b] = at;
        at += bins[b];
    }
    if (threadIdx.x == 0) *total = all;
}

// Two keys per word.
__global__ __launch_bounds__(kListThreads) void k_tile_list(TileLists tl, const int* __restrict__ records) {
    extern __shared__ int cnt[];  // entries of this block, then its next place, per tile
    for (int i = threadIdx.x; i < tl.nbins; i += kListThreads) cnt[i] = 0;
    __syncthreads();
    int s, e;
    record_range(*records, s, e);
    constexpr int kWords = kKeysPerBatch / 2;
    const uint32_t* words = reinterpret_cast<const uint32_t*>(tl.keys);
    const int64_t w0 = (int64_t)s * kWords, w1 = (int64_t)e * kWords;
    for (int64_t i = w0 + threadIdx.x; i < w1; i += kListThreads) {
        const uint32_t k = words[i], a = k & 0xffffu, b = k >> 16;
        if (a != kNoTile) atomicAdd(&cnt[a], 1);
        if (b != kNoTile) atomicAdd(&cnt[b], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < tl.nbins; i += kListThreads)
        if (cnt[i]) cnt[i] = atomicAdd(&tl.bins[tl.nbins + i], cnt[i]);
    __syncthreads();
    for (int64_t i = w0 + threadIdx.x; i < w1; i += kListThreads) {
        const uint32_t k = words[i], a = k & 0xffffu, b = k >> 16;
        if (a != kNoTile) tl.listed[atomicAdd(&cnt[a], 1)] = (int32_t)(i / kWords);
        if (b != kNoTile) tl.listed[atomicAdd(&cnt[b], 1)] = (int32_t)(i / kWords);
    }
}

// ---------------------------------------------------------------------------
// Tile sums.  A wave owns a tile in LDS (18 x 21 texels with the next row and
// column of each base texel: 12.7 KB with a spare row, twelve waves per CU)
// and adds its batches with plain reads and writes: LDS float atomics are
// performed one lane at a time on this chip (195 cycles per wave instruction,
// against 10 for a read and a write), so nothing is shared between waves.
// Each of the wave's four 16-lane rows takes four samples of a batch and adds
// one per step, so a step adds samples i, i + 4, i + 8 and i + 12: a lane two
// channels (lane % 4) of one of the sample's four texels (lane / 4 % 4).  The
// four are kept apart where they touch the same texels.
// ---------------------------------------------------------------------------
constexpr int kTilePitch = (kTileU + 1) * 8;
constexpr int kTileFloats = (kTileV + 1) * kTilePitch;

// One batch as a wave holds it: the coordinates of sample lane % 4 of the
// row's four, and two channels of all four.
struct TileBatch {
    float pu, pv;
    float4 a, b;
};

__device__ __forceinline__ TileBatch load_batch(const float* __restrict__ recs, int at, int ou, int ov, int lane) {
    const float* r = recs + (size_t)at * kRecFloats + (lane >> 4) * 4;
    const int k = lane & 3;
    TileBatch t;
    t.pu = r[ou + k];
    t.pv = r[ov + k];
    const float4* g = reinterpret_cast<const float4*>(r + 2 * k * kGroup);
    t.a = g[0];
    t.b = g[kGroup / 4];
    return t;
}

// Sample kS of each row, whose texel offset is `off` and whose weights for
// the four texels are `w` on the lanes that hold it.  A sample outside the
// tile adds to the spare row behind it.
template <int kS>
__device__ __forceinline__ void add_step(float* tile, uint32_t used, uint32_t clash, uint32_t off, float w, int place,
                                         float ga, float gb, int lane) {
    if (!((used >> kS) & 0x1111u)) return;
    const float wk = quad_bcast<kS>(w);
    float2* dst = reinterpret_cast<float2*>(tile + quad_bcast<kS>(off) + place);
    if (!((clash >> kS) & 0x1111u)) {
        float2 t = *dst;
        t.x = fmaf(wk, ga, t.x);
        t.y = fmaf(wk, gb, t.y);
        *dst = t;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (lane >> 4 == k) {
                float2 t = *dst;
                t.x = fmaf(wk, ga, t.x);
                t.y = fmaf(wk, gb, t.y);
                *dst = t;
            }
            wave_order();
        }
    }
    wave_order();
}

// Whether two samples share a texel, by their keys: 64 row + column, with
// fewer than 32 columns, and far apart for samples outside.
__device__ __forceinline__ bool touching(int a, int b) {
    const uint32_t d = (uint32_t)abs(a - b);
    return d <= 1u || d - 63u <= 2u;
}

// Bits 0..3 of each row, as 16 bits.
__device__ __forceinline__ uint32_t row_bits(bool x) {
    const uint64_t m = __ballot(x);
    return (uint32_t)(m & 0xfu) | (uint32_t)((m >> 12) & 0xf0u) | (uint32_t)((m >> 24) & 0xf00u) |
           (uint32_t)((m >> 36) & 0xf000u);
}

__global__ __launch_bounds__(64) void k_tile_sum(SceneDev sc, const float* __restrict__ recs, TileLists tl,
                                                 float* __restrict__ gxz, float* __restrict__ gyz) {
    __shared__ __attribute__((aligned(16))) float tile[kTileFloats + kTilePitch + 16];  // + spare
    const int lane = threadIdx.x;
    for (int i = lane; i < kTileFloats; i += 64) tile[i] = 0.0f;
    wave_order();
    const float hs = lane & 4 ? 1.0f : -1.0f, h0 = lane & 4 ? 0.0f : 1.0f;  // weights of the lane's texel
    const float vs = lane & 8 ? 1.0f : -1.0f, v0 = lane & 8 ? 0.0f : 1.0f;
    const int place = (lane & 3) * 2 + (lane & 4 ? 8 : 0) + (lane & 8 ? kTilePitch : 0);
    // Every wave takes an equal share of the listed batches, whatever tiles
    // they lie in, and adds a tile to its plane where the next one begins:
    // shorter pieces cost more in flushed tiles than they even out (5.4 ms
    // with pieces of 128, 3.2 with 256 handed out one by one, 2^18 rays).
    const int total = *tl.total, waves = (int)gridDim.x;
    int e0 = (int)((int64_t)total * blockIdx.x / waves);
    const int stop = (int)((int64_t)total * (blockIdx.x + 1) / waves);
    const int* ends = tl.bins + tl.nbins;  // of each tile's entries
    int b = 0;
    for (int hi = tl.nbins - 1; b < hi;) {  // first tile that ends past e0
        const int mid = (b + hi) >> 1;
        if (ends[mid] > e0)
            hi = mid;
        else
            b = mid + 1;
    }
    for (; e0 < stop; ++b) {
        const int tile_end = min(stop, ends[b]);
        if (tile_end <= e0) continue;
        const bool yz = b >= tl.yz;
        const int nu = yz ? tl.nu_y : tl.nu_x, id = yz ? b - tl.yz : b;
        const int tv = id / nu, u0 = (id - tv * nu) * kTileU, w0 = tv * kTileV;
        const AxisMap mu = yz ? sc.py : sc.px, mv = sc.pz;
        const int ou = kRecPoint + (yz ? kGroup : 0), ov = kRecPoint + 2 * kGroup;
        for (; e0 < tile_end; e0 += 64) {
            const int cnt = min(64, tile_end - e0);
            const int ids = tl.listed[e0 + min(lane, cnt - 1)];
            TileBatch nx = load_batch(recs, __builtin_amdgcn_readlane(ids, 0), ou, ov, lane);
            for (int k = 0; k < cnt; ++k) {
                const TileBatch t = nx;
                if (k + 1 < cnt) nx = load_batch(recs, __builtin_amdgcn_readlane(ids, k + 1), ou, ov, lane);
                int iu = 0, iv = 0;
                float fu = 0.0f, fv = 0.0f;
                axis_coord(t.pu, mu, iu, fu);
                axis_coord(t.pv, mv, iv, fv);
                iu -= u0;
                iv -= w0;
                const bool in = t.pv == t.pv && (unsigned)iu < (unsigned)kTileU && (unsigned)iv < (unsigned)kTileV;
                const uint32_t off = in ? (uint32_t)(iv * kTilePitch + iu * 8) : (uint32_t)kTileFloats;
                const float w = fmaf(hs, fu, h0) * fmaf(vs, fv, v0);
                const int key = in ? iv * 64 + iu : (100 + 4 * lane) * 64;
                const int k1 = __shfl_xor(key, 16), k2 = __shfl_xor(key, 32), k3 = __shfl_xor(key, 48);
                const uint32_t used = row_bits(in);
                const uint32_t clash = row_bits(touching(key, k1) || touching(key, k2) || touching(key, k3));
                add_step<0>(tile, used, clash, off, w, place, t.a.x, t.b.x, lane);
                add_step<1>(tile, used, clash, off, w, place, t.a.y, t.b.y, lane);
                add_step<2>(tile, used, clash, off, w, place, t.a.z, t.b.z, lane);
                add_step<3>(tile, used, clash, off, w, place, t.a.w, t.b.w, lane);
            }
        }
        float* G = yz ? gyz : gxz;
        const int nu_t = (int)mu.top + 2, nv_t = (int)mv.top + 2;  // texels of the plane
        const int cols = min(kTileU + 1, nu_t - u0) * 8, rows = min(kTileV + 1, nv_t - w0);
        for (int i = lane; i < kTileFloats; i += 64) {
            const float v = tile[i];
            tile[i] = 0.0f;
            const int r = i / kTilePitch, x = i - r * kTilePitch;
            if (v != 0.0f && r < rows && x < cols)
                unsafeAtomicAdd(G + ((size_t)(w0 + r) * (size_t)nu_t + (size_t)u0) * 8 + x, v);
        }
        wave_order();
        e0 = tile_end;
    }
}

namespace {
constexpr int64_t align256(int64_t b) { return (b + 255) / 256 * 256; }
}  // namespace

int64_t record_workspace(const SceneDev& sc, const RayParams& rp, int64_t n, void* base, BatchRecords* br,
                         TileLists* tl) {
    // At most 6 Mi records (4.5 GB): rays take them longest first, and what is
    // left replays its samples.
    const int64_t batches = n * ((rp.n_max + kGroup - 1) / kGroup);
    const int64_t cap = batches < (6ll << 20) ? batches : (6ll << 20);
    const int64_t nu_x = (sc.Nx - 2) / kTileU + 1, nu_y = (sc.Ny - 2) / kTileU + 1, nv = (sc.Nz - 2) / kTileV + 1;
    const int64_t bins = (nu_x + nu_y) * nv;
    if (rp.t_term > 0.0f || batches <= kRecordBatches || bins > kTileMaxBins ||
        texels_per_step(sc, rp.delta) < kRecordTexels)
        return 0;
    const int64_t parts[9] = {cap * kRecFloats * (int64_t)sizeof(float),
                              n * (int64_t)sizeof(int32_t),
                              cap * kKeysPerBatch * (int64_t)sizeof(uint16_t),
                              cap * kKeysPerBatch * (int64_t)sizeof(int32_t),
                              2 * bins * (int64_t)sizeof(int),
                              (int64_t)sizeof(int),
                              n * (int64_t)sizeof(int32_t),
                              order_hist_bytes(),
                              n * (int64_t)sizeof(uint16_t)};
    char* p = static_cast<char*>(base);
    int64_t at[9], total = 0;
    for (int i = 0; i < 9; ++i) {
        at[i] = total;
        total += align256(parts[i]);
    }
    if (p) {
        *br = BatchRecords{reinterpret_cast<float*>(p + at[0]), reinterpret_cast<int32_t*>(p + at[1]),
                           reinterpret_cast<int32_t*>(p + at[6]), reinterpret_cast<int*>(p + at[7]),
                           reinterpret_cast<uint16_t*>(p + at[8]), (int)cap};
        *tl = TileLists{reinterpret_cast<uint16_t*>(p + at[2]), reinterpret_cast<int32_t*>(p + at[3]),
                        reinterpret_cast<int*>(p + at[4]),   reinterpret_cast<int*>(p + at[5]),
                        (int)bins,                           (int)(nu_x * nv),
                        (int)nu_x,                           (int)nu_y};
    }
    return total;
}

hipError_t launch_tile_sums(const SceneDev& sc, const BatchRecords& br, const TileLists& tl, const int* records,
                            float* gxz, float* gyz, hipStream_t s) {
    const size_t lds = (size_t)tl.nbins * sizeof(int);
    hipLaunchKernelGGL(k_tile_clear, dim3((unsigned)((tl.nbins + kListThreads - 1) / kListThreads)), dim3(kListThreads),
                       0, s, tl.bins, tl.nbins);
    hipLaunchKernelGGL(k_tile_keys, dim3(kListBlocks), dim3(kListThreads), lds, s, sc, br.rec, tl, records, gxz, gyz);
    hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(kListThreads), 0, s, tl.bins, tl.nbins, tl.total);
    hipLaunchKernelGGL(k_tile_list, dim3(kListBlocks), dim3(kListThreads), lds, s, tl, records);
    hipLaunchKernelGGL(k_tile_sum, dim3(3072), dim3(64), 0, s, sc, br.rec, tl, gxz, gyz);
    return hipGetLastError();
}

}  // namespace omerf
