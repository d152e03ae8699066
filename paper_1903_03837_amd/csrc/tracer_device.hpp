// tracer_device.hpp -- building blocks of the volumetric path tracer behind
// lf_generate and lf_generate_backward (the kernel itself is in wave.hip).
//
// Each ray r_k of the SF ray set (Sec. 2, ray equation) is traced by one
// lane, all of its samples in order, so the FP32 sum per texel is
// deterministic.  Transport (the volumetric reading of Sec. 2's "conventional
// path tracer"):
//   - origin jitter on the disk of area 4 pi R^2 / M in the tangent plane;
//   - delta tracking against a majorant: one global sigma_bar, or a grid of
//     cell majorants walked cell by cell;
//   - real collision: throughput times the albedo, next-event estimation
//     towards the light with ratio-tracking transmittance, Henyey-Greenstein
//     direction for the next segment; escape: constant environment.
// Random numbers: Philox4x32-10 keyed by the seed, counter (ray, sample,
// bounce << 8 | purpose, block); a block holds two word pairs.  Purpose 1
// ("flight" of segment b): pair 0 of segment 0 jitters the origin, then one
// pair per tentative collision (distance, acceptance).  Purpose 2 ("vertex"
// b): pair 0 samples the light, pair 1 the phase function, then one pair per
// shadow step (first word: distance).
//
// The kernel runs in three modes:
//   kFwd     plain estimator;
//   kFrozen  decisions with the sampling medium, importance weights to the
//            evaluated medium (finite-difference hook of the adjoint);
//   kGrad    path replay: every event scatters its score times the radiance
//            gathered after it into LDS accumulators (dLUT, dscale).
#pragma once

#include <hip/hip_fp16.h>

#include "sf_device.hpp"

namespace lp {

enum { kFwd = 0, kFrozen = 1, kGrad = 2 };
enum { kPurFlight = 1, kPurVertex = 2 };
// At most 2^20 word pairs (2^19 blocks) per stream.  Valid scenes stay orders
// of magnitude below; a segment that reaches it ends absorbed (free flight)
// or fully blocked (shadow), so no lane can spin.
constexpr uint32_t kMaxBlocks = 1u << 19;

// Pinhole view for ground-truth rendering: eye, orthonormal basis and the
// half-extents tan(vfov / 2) * aspect, tan(vfov / 2) of the image plane.
struct ViewCam {
    float eye[3], fwd[3], right[3], up[3];
    float sx, sy;
};

struct TraceParams {
    // volume: the library's halo-brick copy (4^3-voxel bricks every 3
    // voxels, bricks x-fastest, voxels x-fastest inside a brick)
    const void* vol;
    int32_t nx, ny;
    int32_t nbx, nby;                // bricks along x and y
    float ga[3], gb[3];              // grid coordinate = x * ga + gb
    float gmax[3];                   // n - 1
    int32_t imax[3];                 // n - 2
    float vmin, vscale;              // s = (v - vmin) * vscale
    int32_t lut_n;
    float lut_last;                  // lut_n - 1
    const float* lut_e;              // [lut_n][4]
    const float* lut_s;
    float scale_e, scale_s;
    float bmin[3], bmax[3];
    // light
    int32_t light_kind, light_on;
    float ldir[3], lcorner[3], le1[3], le2[3], lrad[3], lnrm[3];
    float larea;
    float env[3];
    // ray set
    int32_t M, N;
    float O[3], R;
    int32_t spp, maxb;
    float g;
    uint32_t key0, key1;
    int32_t jitter;
    float jit_rad;                   // 2 R / sqrt(M)
    int32_t row_begin, row_end;
    const float* sigbar;             // device scalar
    // outputs
    void* out;
    int32_t dtype;
    unsigned long long* stats;
    int32_t part_log2;  // work items per ray = 2^part_log2 sample ranges
    float* part_sums;   // forward with several ranges: [rows][N][ranges][3]
    // forward: the last fine_units ray tiles of each part of the queue have
    // 2^fine_log2 work items per ray; every sample of theirs is kept in
    // `samples` [kParts][fine_units][spp][64][3] (workspace), and a second
    // kernel sums it
    int32_t fine_units, fine_log2;
    float* samples;
    // SF points of both sets (workspace tables filled by sf_point with
    // inv_n = 1/n in FP32, the values the kernel would compute)
    const float4* tab_o;
    const float4* tab_d;
    // per-sample radiance [rows][N][spp][3]: written by the forward,
    // read by the adjoint in place of its first pass (or NULL)
    float* srad;
    // adjoint
    const float* d_lf;
    float* d_lut;
    float* d_scale;
    // persistent forward kernel: spatial orders of the origin rows and the
    // directions, and the per-XCD tile counters (workspace)
    const int32_t* perm_o;
    const int32_t* perm_d;
    unsigned int* tile_ctr;
    int32_t ctr_stride;              // counters' distance (a cache line each where waves contend for them)
    // majorant grid: grid_n^3 cell majorants (x fastest) over the volume box;
    // grid_n = 1 with maj = sigbar is the global majorant
    int32_t grid_n, nz;
    // isosurface variant: isovalue, half the smallest voxel extent, raw
    // [lo, hi] per grid cell
    int32_t surface;
    float iso, half_voxel;
    const float* srange;
    // its march's blocks: block_bricks bricks along each axis, blocks_n of them,
    // two bits per block; inv_block = 1 / (3 block_bricks)
    int32_t block_bricks[3], blocks_n[3];
    float inv_block[3];
    const uint32_t* sblocks;
    // ground-truth views (views != nullptr): camera rays instead of the SF ray
    // set, 8 x 8 pixel tiles, stream key = (view * H + y) * W + x
    const ViewCam* views;
    int32_t nviews, W, H;
    int32_t vtx, vtiles;             // tiles per image row, tiles per view
    float gcell[3];                  // cells per world unit
    float gcw[3];                    // cell width
    float glast, gpitch;             // grid_n - 1, grid_n + 2 (the padded grid's pitch)
    const float* maj;
    // adjoint: compacted list of rays with a nonzero adjoint and its length
    uint32_t* ray_list;
    unsigned int* ray_count;
    // adjoint: kRecords records for each lane of record_groups workgroups
    float4* records;
    int32_t record_groups;
};

// The kernel arguments seen through the kernarg segment (constant address
// space): fields read through such a reference load with scalar loads.  The
// persistent kernels read their parameters this way inside their main loop,
// behind an empty asm barrier per iteration that keeps the loads from being
// hoisted: the compiler then reloads parameters where they are needed
// instead of holding ~100 uniform values in scalar registers and spilling
// them to vector-register lanes (one VALU instruction per spilled read).
typedef const __attribute__((address_space(4))) TraceParams KTraceParams;

// Ray tiles: 8 origins x 8 directions, taken in groups of 16 origin tiles
// sweeping the direction tiles; the tile sequence is cut into 8 parts, one
// per XCD (workgroups are dispatched round-robin over the XCDs).
constexpr int kGroupTiles = 16;
constexpr int kParts = 8;

// Tile t of the row slab -> (origin tile, direction tile).  Tile counts are
// below 2^32 (M, N <= 65535), so 32-bit unsigned division suffices.
__device__ __forceinline__ void tile_coords(long long t, int tiles_i, int tiles_j, int& ti, int& tj) {
    const uint32_t tu = (uint32_t)t;
    const uint32_t per_group = (uint32_t)kGroupTiles * (uint32_t)tiles_j;
    const uint32_t gi = tu / per_group;
    const uint32_t gsz = (uint32_t)min(kGroupTiles, tiles_i - (int)gi * kGroupTiles);
    const uint32_t off = tu - gi * per_group;
    const uint32_t q = off / gsz;
    tj = (int)q;
    ti = (int)(gi * kGroupTiles + (off - q * gsz));
}

// Lane states of the persistent kernels (kDone: the sample's radiance is
// complete and waits to be added to its texel; kScore: the adjoint's recorded
// events are being scored).
enum : int {
    kIdle = 0, kStart = 1, kFlight = 2, kVertex = 3, kShadow = 4, kShadow2 = 5, kScatter = 6, kDone = 7, kScore = 8
};
// Records a lane can keep for scoring (adjoint; 64, the bits of a mask: 97 % of
// the events of a 128^3 training pass lie in paths that fit, two thirds of
// a 256^3 one with eight bounces), and the lanes of 64 live ones that wait
// before a wave scores (dense adjoint of the 128^3 blobs, N = 1024, 32 spp: 5.79
// ms; 8 lanes 5.85, 32 lanes 6.10).
constexpr int kRecords = 64;
constexpr int kScoreLanes = 16;
// Divisor of a point that is not on its segment (the bits of a NaN that no
// arithmetic returns).
constexpr uint32_t kNoPoint = 0x7fc0a11eu;
// Workgroups that have records: a full grid of the MI355X (256 CUs, three
// each), so that the workspace has a fixed bound.  The launch never exceeds it.
constexpr int kRecordGroups = 768;
// A further tracking pass runs while at least this many lanes of a wave are
// still tracking a segment.
constexpr int kTrackPass = 36;

// Kept sample s of ray r of the samples buffer (a tile's 64 rays side by side:
// the summing kernel reads a tile's samples in whole lines.  With each ray's
// samples side by side instead its pass over 403 MB took 0.51 ms, now 0.09).
template <class PT>
__device__ __forceinline__ float* kept_sample(const PT& P, uint32_t r, int s) {
    return P.samples + 3 * (((uint64_t)(r >> 6) * (uint32_t)P.spp + (uint32_t)s) * 64 + (r & 63));
}

// First sample of item `item` of the 2^log2 that a ray's spp samples are split
// into (the item ends where the next begins).  The product is formed in 64
// bits: finely split rays have up to spp items, and 32 bits overflow from 65536
// samples on.
__host__ __device__ __forceinline__ int item_sample(int item, int spp, int log2) {
    return (int)(((long long)item * spp) >> log2);
}

// The work queue: `units` in kParts contiguous parts of equal length.  A unit
// is a ray tile (64 rays), of which each part hands out the first ones with
// 2^log2 items per ray and the last `fine` ones with 2^fine_log2 (in the
// adjoint: 64 items of the ray list, log2 = fine = 0), 64 items at a time.
struct Queue {
    long long units, part;   // units in all, and per part (the last parts may be shorter)
    int log2, fine, fine_log2;
    __host__ __device__ __forceinline__ Queue(long long n, int l, int f, int fl)
        : units(n), part((n + kParts - 1) / kParts), log2(l), fine(f), fine_log2(fl) {}
    __host__ __device__ __forceinline__ long long first(int p) const { return (long long)p * part; }
    __host__ __device__ __forceinline__ long long count(int p) const {
        const long long n = units - first(p);
        return n < 0 ? 0 : (n < part ? n : part);
    }
    __host__ __device__ __forceinline__ long long coarse(int p) const {
        const long long n = count(p);
        return n > fine ? n - fine : 0;
    }
    __host__ __device__ __forceinline__ long long tiles(int p) const {
        const long long c = coarse(p);
        return (c << log2) + ((count(p) - c) << fine_log2);
    }
};

// 64 items of the queue: items [cur, end), 2^log2 of them per ray slot; fine
// items keep their samples at ray `slot + shift` of the samples buffer.
struct Tile {
    long long cur, end, shift;
    int log2;
    bool fine;
};

// Next tile for a wave whose home part is `home` (called by the whole wave):
// false when all are taken.  The wave's first tile is its own by position
// (idx: its place among the waves of its home part), the rest come from the
// part's counter, one atomic each.  A wave that finds a part taken looks at
// all counters with one load before it tries another part: with every wave
// trying every part in turn, and the counters in one cache line, the atomics
// held small launches (10 us and more per refill).  With the counters in one
// line and a line apart: 64^3 blobs, N = 256, 16 spp 0.62 and 0.43 ms; two 480 x
// 270 views of the 256^3 phantom at 256 spp 3.9 and 2.4 ms; its field, N = 2048,
// 64 spp 10.6 and 8.6 ms.
__device__ __forceinline__ bool next_tile(unsigned int* ctr, int stride, const Queue& Q, int home, int idx, bool& begun,
                                          unsigned& dry, Tile& T) {
    const int lane = threadIdx.x & 63;
    const int groups = (int)gridDim.x;
    while (dry != (1u << kParts) - 1u) {
        const unsigned open = ~dry & ((1u << kParts) - 1u);
        const unsigned turned = (open | (open << kParts)) >> home;
        const int p = (home + __ffs((int)turned) - 1) % kParts;
        const long long own = 4ll * ((groups - p + kParts - 1) / kParts);  // tiles taken by position
        long long got;
        if (!begun) {
            got = idx;
            begun = true;
        } else {
            unsigned g = 0;
            if (lane == 0) g = atomicAdd(&ctr[p * stride], 1u);
            got = own + (unsigned)__builtin_amdgcn_readfirstlane((int)g);
        }
        if (got < Q.tiles(p)) {
            const long long c = Q.coarse(p), ct = c << Q.log2;
            T.fine = got >= ct;
            T.log2 = T.fine ? Q.fine_log2 : Q.log2;
            const long long u0 = Q.first(p) + (T.fine ? c : 0);  // first unit of this kind
            T.cur = ((u0 << T.log2) + (T.fine ? got - ct : got)) * 64;
            T.end = T.cur + 64;
            T.shift = ((long long)p * Q.fine - u0) * 64;
            return true;
        }
        unsigned c = 0;
        bool empty = false;
        if (lane < kParts) {
            c = __hip_atomic_load(&ctr[lane * stride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            empty = 4ll * ((groups - lane + kParts - 1) / kParts) + c >= Q.tiles(lane);
        }
        dry |= (unsigned)__ballot(empty) | (got >= own ? 1u << p : 0u);
    }
    return false;
}

// Hardware reciprocal / reciprocal square root (1 ulp).  Used where the
// result only moves a continuous quantity (slab bounds, frames, directions);
// the texel mean and the importance weights keep IEEE division.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }

struct Counters {
    uint32_t tent, shadow, real, samples, cells;
};

// ---------------------------------------------------------------------------
// Medium
// ---------------------------------------------------------------------------
// The 2 x 2 voxels (x, x + 1) of rows y and y + 1 of one brick layer, from the
// address of the first: each row's pair is one load (4 bytes for u16, 2 for
// u8, 8 for f32), half as many load instructions and destination registers
// as voxel by voxel.  A pair lies inside its brick row, so it is in range and
// never crosses a cache line; it is aligned to the voxel size only (the
// types below), which global loads allow.  The fetch was bound by its load
// and address instructions: 16 loads per pair of points, each with a 64-bit
// address of its own, against 8 now at fixed offsets from one address.  On the
// synthetic phantoms at their default settings: 256^3 u16, N = 2048, 64 spp
// 10.0 -> 9.5 ms; 512^3, N = 32768, 16 spp, 2048 rows 292 -> 251 ms (278 -> 265
// where the kernel then had 3 waves per SIMD); isosurface of the 256^3 one, N =
// 1024, 16 spp 52.2 -> 44.8 ms; 128^3 f32 training pass 14.3 -> 13.9 ms; two 480
// x 270 views at 256 spp 2.4 ms with either.
typedef uint16_t u16_at1 __attribute__((aligned(1)));
typedef uint32_t u32_at2 __attribute__((aligned(2)));
typedef float f32x2_at4 __attribute__((ext_vector_type(2), aligned(4)));
template <int VT>
__device__ __forceinline__ void vox_quad(const char* p, float& a0, float& a1, float& b0, float& b1) {
    if constexpr (VT == 0) {
        const uint32_t a = *(const u16_at1*)p, b = *(const u16_at1*)(p + 4);
        a0 = (float)(a & 255u);
        a1 = (float)(a >> 8);
        b0 = (float)(b & 255u);
        b1 = (float)(b >> 8);
    } else if constexpr (VT == 1) {
        const uint32_t a = *(const u32_at2*)p, b = *(const u32_at2*)(p + 8);
        a0 = (float)(a & 65535u);
        a1 = (float)(a >> 16);
        b0 = (float)(b & 65535u);
        b1 = (float)(b >> 16);
    } else {
        const f32x2_at4 a = *(const f32x2_at4*)p, b = *(const f32x2_at4*)(p + 16);
        a0 = a.x;
        a1 = a.y;
        b0 = b.x;
        b1 = b.y;
    }
}

// Trilinear raw value at world point y (edge-clamped grid coordinates) from
// the library's halo-brick copy of the volume: bricks of 4^3 voxels placed
// every 3 voxels, so that neighbouring bricks share one layer.  The 2 x 2 x 2
// footprint of base voxel (ix, iy, iz) then lies whole in brick
// (ix/3, iy/3, iz/3) at local offset (ix%3, iy%3, iz%3): one 128-byte line
// for u16, half a line for u8, and one of two lines for f32 (or both, in one
// case of three).  Its eight voxels sit at fixed offsets from the first, so
// one 64-bit address serves all loads.
struct VoxelPoint {
    uint32_t base;      // first voxel of the footprint in the copy
    float fx, fy, fz;   // position inside it
};
template <class PT>
__device__ __forceinline__ VoxelPoint voxel_point(const PT& P, f3 y) {
    // clamp to [0, n - 1] as one median-of-three
    const float gx = __builtin_amdgcn_fmed3f(fmaf(y.x, P.ga[0], P.gb[0]), 0.0f, P.gmax[0]);
    const float gy = __builtin_amdgcn_fmed3f(fmaf(y.y, P.ga[1], P.gb[1]), 0.0f, P.gmax[1]);
    const float gz = __builtin_amdgcn_fmed3f(fmaf(y.z, P.ga[2], P.gb[2]), 0.0f, P.gmax[2]);
    const int ix = min((int)gx, P.imax[0]);
    const int iy = min((int)gy, P.imax[1]);
    const int iz = min((int)gz, P.imax[2]);
    // i / 3 as (i * 43691) >> 17, exact for i < 2^17.  Dimensions are below
    // 2^16 and brick counts below 2^15 (stated here so that these products
    // become full-rate 24-bit multiplies); only the last one, whose brick row
    // may pass 2^24 in a thin volume, takes the quarter-rate 32-bit multiply.
    __builtin_assume((uint32_t)ix < 65536u && (uint32_t)iy < 65536u && (uint32_t)iz < 65536u);
    const uint32_t bx = ((uint32_t)ix * 43691u) >> 17, by = ((uint32_t)iy * 43691u) >> 17,
                   bz = ((uint32_t)iz * 43691u) >> 17;
    const uint32_t nbx = (uint32_t)P.nbx, nby = (uint32_t)P.nby;
    __builtin_assume(nby < 32768u);
    // voxel index 64 ((bz nby + by) nbx + bx) + 16 (iz - 3 bz) + 4 (iy - 3 by) + (ix - 3 bx),
    // regrouped to shifts and adds: 16 (iz - 3 bz) = 16 (iz + bz) - 64 bz, and
    // so on down the axes
    const uint32_t brick = (bz * nby + by) * nbx + (bx - bz);
    const uint32_t base = ((((((brick << 2) + ((uint32_t)iz + bz - by)) << 2) + ((uint32_t)iy + by - bx)) << 2)) +
                          ((uint32_t)ix + bx);
    return {base, gx - (float)ix, gy - (float)iy, gz - (float)iz};
}
template <int VT, class PT>
__device__ __forceinline__ void load_footprint(const PT& P, uint32_t base, float& v000, float& v100, float& v010,
                                               float& v110, float& v001, float& v101, float& v011, float& v111) {
    constexpr int ESZ = VT == 0 ? 1 : VT == 1 ? 2 : 4;
    const char* const p = (const char*)P.vol + (uint64_t)base * ESZ;
    vox_quad<VT>(p, v000, v100, v010, v110);
    vox_quad<VT>(p + 16 * ESZ, v001, v101, v011, v111);
}
__device__ __forceinline__ float lerp_footprint(const VoxelPoint& p, float v000, float v100, float v010, float v110,
                                                float v001, float v101, float v011, float v111) {
    const float c00 = fmaf(p.fx, v100 - v000, v000), c10 = fmaf(p.fx, v110 - v010, v010);
    const float c01 = fmaf(p.fx, v101 - v001, v001), c11 = fmaf(p.fx, v111 - v011, v011);
    const float c0 = fmaf(p.fy, c10 - c00, c00), c1 = fmaf(p.fy, c11 - c01, c01);
    return fmaf(p.fz, c1 - c0, c0);
}
template <int VT, class PT>
__device__ __forceinline__ float sample_volume(const PT& P, f3 y) {
    const VoxelPoint p = voxel_point(P, y);
    float v000, v100, v010, v110, v001, v101, v011, v111;
    load_footprint<VT>(P, p.base, v000, v100, v010, v110, v001, v101, v011, v111);
    return lerp_footprint(p, v000, v100, v010, v110, v001, v101, v011, v111);
}
// Voxel (x, y, z) of the copy.
template <int VT, class PT>
__device__ __forceinline__ float voxel_at(const PT& P, int x, int y, int z) {
    // (the last voxel of an axis is the fourth of its brick)
    const int bx = min(x / 3, P.nbx - 1), by = min(y / 3, P.nby - 1), bz = z / 3 - (z == P.nz - 1 && z % 3 == 0 ? 1 : 0);
    const uint64_t i = 64ull * (((uint64_t)bz * (uint32_t)P.nby + (uint32_t)by) * (uint32_t)P.nbx + (uint32_t)bx) +
                       (uint32_t)(16 * (z - 3 * bz) + 4 * (y - 3 * by) + (x - 3 * bx));
    if constexpr (VT == 0) return (float)((const uint8_t*)P.vol)[i];
    else if constexpr (VT == 1) return (float)((const uint16_t*)P.vol)[i];
    else return ((const float*)P.vol)[i];
}

struct TF {
    int l0;
    float w;
    float a;        // alpha of the evaluated medium
    float a_s;      // alpha of the sampling medium (kFrozen)
};

// Post-classification: window, clamp, linear LUT interpolation (LUT in LDS).
// The alpha of the point; its colour (needed at real collisions only) comes
// from tf_rgb with the same entries and weight.
template <int MODE, class PT>
__device__ __forceinline__ TF classify(const PT& P, const float4* lut_e, const float4* lut_s, float raw) {
    TF t;
    const float s = __builtin_amdgcn_fmed3f((raw - P.vmin) * P.vscale, 0.0f, 1.0f);
    const float u = s * P.lut_last;
    t.l0 = min((int)u, P.lut_n - 2);
    t.w = fmaf(s, P.lut_last, -(float)t.l0);
    const float Aw = lut_e[t.l0].w, Bw = lut_e[t.l0 + 1].w;
    t.a = fmaf(t.w, Bw - Aw, Aw);
    if constexpr (MODE == kFrozen) {
        const float4 C = lut_s[t.l0], D = lut_s[t.l0 + 1];
        t.a_s = fmaf(t.w, D.w - C.w, C.w);
    } else {
        t.a_s = t.a;
    }
    return t;
}

// Evaluated colour (unclamped) of a classified point.
__device__ __forceinline__ f3 tf_rgb(const float4* lut_e, const TF& t) {
    const float4 A = lut_e[t.l0], B = lut_e[t.l0 + 1];
    return mk3(fmaf(t.w, B.x - A.x, A.x), fmaf(t.w, B.y - A.y, A.y), fmaf(t.w, B.z - A.z, A.z));
}

// ---------------------------------------------------------------------------
// Geometry
// ---------------------------------------------------------------------------
// Hardware reciprocals of a direction's components (used by the clip and by
// the majorant-grid walk of the same segment).
__device__ __forceinline__ f3 rcp3(f3 d) { return mk3(rcp(d.x), rcp(d.y), rcp(d.z)); }

// [tn, tf) of o + t d, t >= 0, inside the box; false when empty.  id: the
// reciprocals of d's components (rcp3).
__device__ __forceinline__ bool clip_box(f3 bmin, f3 bmax, f3 o, f3 d, f3 id, float& tn, float& tf) {
    float t0 = 0.0f, t1 = 3.402823466e38f;
    bool in = true;
    const float oo[3] = {o.x, o.y, o.z}, dd[3] = {d.x, d.y, d.z}, ii[3] = {id.x, id.y, id.z};
    const float lo[3] = {bmin.x, bmin.y, bmin.z}, hi[3] = {bmax.x, bmax.y, bmax.z};
    // formed with selects: lanes with a zero component cost the others no
    // divergent branch per axis
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool flat = dd[a] == 0.0f;  // no bounds on t along this axis, in or out
        const float ta = (lo[a] - oo[a]) * ii[a], tb = (hi[a] - oo[a]) * ii[a];
        const bool swap = ta > tb;
        const float near = swap ? tb : ta, far = swap ? ta : tb;
        t0 = flat ? t0 : fmaxf(t0, near);
        t1 = flat ? t1 : fminf(t1, far);
        in = in & !(flat & ((oo[a] < lo[a]) | (oo[a] > hi[a])));
    }
    tn = t0;
    tf = t1;
    return in & (t0 < t1);
}

__device__ __forceinline__ bool clip_box(f3 bmin, f3 bmax, f3 o, f3 d, float& tn, float& tf) {
    return clip_box(bmin, bmax, o, d, rcp3(d), tn, tf);
}

// True when the light-field ray from SF origin po (unit sphere) along d0
// misses the volume box in every sample.  The jitter moves the origin by less
// than jit_rad, so the test clips against the box grown by jit_rad plus a
// margin far above FP32 rounding; without jitter it is the sample's own clip
// (the same function on the same origin).
template <class PT>
__device__ __forceinline__ bool misses_box(const PT& P, f3 O, f3 bmin, f3 bmax, f3 po, f3 d0) {
    const float pad = P.jitter ? P.jit_rad * 1.001f + 1e-5f * P.R : 0.0f;
    float tn, tf;
    return !clip_box(mk3(bmin.x - pad, bmin.y - pad, bmin.z - pad), mk3(bmax.x + pad, bmax.y + pad, bmax.z + pad),
                     O + po * P.R, d0, tn, tf);
}

// Orthonormal completion of unit n (Duff et al. 2017).
__device__ __forceinline__ void frame(f3 n, f3& t1, f3& t2) {
    const float sg = n.z >= 0.0f ? 1.0f : -1.0f;
    const float a = -rcp(sg + n.z);
    const float b = n.x * n.y * a;
    t1 = mk3(1.0f + sg * n.x * n.x * a, sg * b, -sg * n.x);
    t2 = mk3(b, sg + n.y * n.y * a, -n.y);
}

__device__ __forceinline__ float hg_phase(float g, float mu) {
    const float den = 1.0f + g * g - 2.0f * g * mu;
    const float r = rsq(den);
    return (1.0f - g * g) * 0.0795774715459476679f * r * r * r;
}
__device__ __forceinline__ float hg_mu(float g, float u) {
    float mu;
    if (fabsf(g) < 1e-3f) {
        mu = 1.0f - 2.0f * u;
    } else {
        const float s = (1.0f - g * g) * rcp(1.0f - g + 2.0f * g * u);
        mu = (1.0f + g * g - s * s) * rcp(2.0f * g);
    }
    return fminf(fmaxf(mu, -1.0f), 1.0f);
}

// -ln(1 - u) for u = k 2^-24 in [0, 1): 1 - u is exact and a normal number, so
// the hardware base-2 logarithm needs no scaling of denormal arguments and no
// test for infinities (seven instructions of the general logarithm).  ln 2 is
// the sum of two floats (the first rounded towards zero), and the rounding
// error of the first product is added back by a fused multiply-add.
__device__ __forceinline__ float neg_log1m(float u) {
    constexpr float kLn2Hi = 0.6931471228599548f, kLn2Lo = 5.769998878690785e-08f;
    const float y = __builtin_amdgcn_logf(1.0f - u);
    const float p = y * kLn2Hi;
    return -fmaf(y, kLn2Hi, fmaf(y, kLn2Lo, fmaf(y, kLn2Hi, -p)));
}

// ---------------------------------------------------------------------------
// Majorant-grid walk (3-D DDA over the grid_n^3 cells along x + t d).  The
// exponential variate tau of a tentative collision is spent cell by cell at
// each cell's majorant; a cell of majorant 0 spends none.
// The walk is rebuilt from the point reached at the start of each iteration;
// a point that rounds into a neighbouring cell only shortens that cell's
// first piece (the cell majorants cover one voxel beyond each cell).
// ---------------------------------------------------------------------------
struct GridWalk {
    float t, tx, ty, tz, dx, dy, dz;
    int ci;          // LDS address of the cell in the padded grid (one border cell per side, 8 bytes a cell)
    int sx, sy, sz;  // signed steps of it along x, y, z (by the sign of d)

    // mg: LDS address of the padded grid; id: the reciprocals of d's components (rcp3)
    template <class PT>
    __device__ __forceinline__ void init(const PT& P, uint32_t mg, f3 x, f3 d, f3 id, float t0) {
        const f3 p = fma3(d, t0, x);
        const float pp[3] = {p.x, p.y, p.z}, dd[3] = {d.x, d.y, d.z}, xx[3] = {x.x, x.y, x.z};
        const float ii[3] = {id.x, id.y, id.z};
        // cell coordinates stay floats (whole numbers below 16, exact): the
        // clamp is one median-of-three and the cell index two fused
        // multiply-adds, where integers took a conversion per use and
        // quarter-rate multiplies.  Selects instead of a branch per axis.
        float c[3], tm[3], dl[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            c[a] = __builtin_amdgcn_fmed3f(floorf((pp[a] - P.bmin[a]) * P.gcell[a]), 0.0f, P.glast);
            const bool flat = fabsf(dd[a]) < 1e-20f;
            const float plane = fmaf(c[a] + (dd[a] > 0.0f ? 1.0f : 0.0f), P.gcw[a], P.bmin[a]);
            tm[a] = flat ? 3.402823466e38f : (plane - xx[a]) * ii[a];
            dl[a] = flat ? 0.0f : P.gcw[a] * fabsf(ii[a]);
        }
        t = t0;
        const int Gp = 8 * (P.grid_n + 2), Gq = Gp * (P.grid_n + 2);
        ci = 8 * (int)fmaf(fmaf(c[2], P.gpitch, c[1]), P.gpitch, c[0]) + ((int)mg + Gq + Gp + 8);
        sx = d.x > 0.0f ? 8 : -8;
        sy = d.y > 0.0f ? Gp : -Gp;
        sz = d.z > 0.0f ? Gq : -Gq;
        tx = tm[0];
        ty = tm[1];
        tz = tm[2];
        dx = dl[0];
        dy = dl[1];
        dz = dl[2];
    }

    // Both tentative points of one iteration in a single walk: point A for
    // tauA (when wantA), then point B for tauB from A.  One loop for both
    // keeps the wave's trip count at the maximum over lanes of the cells both
    // points need, not the sum of two maxima.  Points past the segment come
    // back as tend (their majorant is then not used).
    // One trip handles one cell: point A if it lies in the cell, then point B
    // if it lies in the rest of the same cell, else the exponential variate
    // left over and either the segment's end or a step into the next cell.
    // The arithmetic is that of one point per trip (B's room in the cell is
    // measured from A, with the same majorant and cell exit), so the points
    // are the same; only trips whose cell holds both points or holds A and is
    // then left are merged.  All outcomes are formed with selects, so lanes
    // that take different ones run a trip's instructions once, and what the
    // code after the loop needs is left in lane values rather than in
    // conditions, which a divergent loop merges into masks on every trip: a
    // target lies in its last cell when the variate left over is negative
    // (while A is sought and not found it never is: tau >= room), and A keeps
    // the segment's end until it is found.
    // The LDS grid at address mg holds each padded cell's majorant s and the
    // hardware reciprocal of s; ci is the cell's LDS address, the read's own.
    // The face crossed first is the one whose boundary
    // equals the minimum, and the cell index moves by that axis's signed
    // stride.  The grid in LDS carries a border of cells that repeat the edge
    // cells, so a step that rounding carries one cell past the grid reads the
    // edge cell's majorant; the segment ends at the box, within rounding of
    // the last face, so no walk goes two cells past it (the index is clamped
    // to the padded grid all the same).  Every step raises the smallest
    // boundary by one cell width along its axis, so the loop reaches tend
    // within 3 (grid_n * segment length / cell width + 2) steps.
    template <class PT>
    __device__ __forceinline__ void next2(const PT& P, uint32_t mg, bool wantA, float tauA,
                                          float tauB, float tend, float& tA, float& sbA, float& tB, float& sbB,
                                          float& rbB, uint32_t& steps) {
        // (no contraction: the variate left over is a rounded product, then a
        // difference, whichever form of the trip computes it)
#pragma clang fp contract(off)
        typedef const __attribute__((address_space(3))) float2 LdsCell;
        const int Gp = P.grid_n + 2;
        const unsigned last = mg + 8u * (unsigned)(Gp * Gp * Gp - 1);
        const int stx = sx, sty = sy, stz = sz;
        bool seekA = wantA;  // still looking for A (else for B)
        float tau = wantA ? tauA : tauB;
        tend = __builtin_canonicalizef(tend);
        tA = wantA ? tend : t;
        float2 m;
        float from, taub;
        for (;;) {
            m.x = ((LdsCell*)(uintptr_t)(uint32_t)ci)->x;
            m.y = ((LdsCell*)(uintptr_t)(uint32_t)ci)->y;
            const float s = m.x;
            const float tmin = fminf(fminf(tx, ty), tz);
            const float te = __builtin_amdgcn_fmed3f(tmin, tend, -3.402823466e38f);  // min(tmin, tend)
            const float room = s * fmaxf(te - t, 0.0f);
            const float th = fmaf(tau, m.y, t);        // A's point, if it lies here (then s > 0)
            const bool hitA = seekA && tau < room;     // A lies in this cell
            // B from A in the same cell, or the current target from the cell's entry
            from = hitA ? th : t;
            taub = hitA ? tauB : tau;
            const float roomb = s * fmaxf(te - from, 0.0f);
            const bool hit = taub < roomb;             // B lies in this cell
            const bool step = !hit && te < tend;       // on into the next cell
            tA = hitA ? th : tA;
            sbA = hitA ? s : sbA;
            t = te;
            tau = taub - roomb;
            seekA = seekA && !hitA;
            steps += step ? 1u : 0u;
            const bool bx = tx == tmin, by = !bx && ty == tmin, bz = !bx && !by;
            ci = (int)min((unsigned)(ci + (bx ? stx : (by ? sty : stz))), last);  // (a wrapped index clamps to last)
            tx += bx ? dx : 0.0f;
            ty += by ? dy : 0.0f;
            tz += bz ? dz : 0.0f;
            if (!step) break;
        }
        tB = tau < 0.0f ? fmaf(taub, m.y, from) : tend;
        sbB = m.x;
        rbB = m.y;
    }
};

// ---------------------------------------------------------------------------
// Gradient accumulation (kGrad): per-lane cache of the alpha gradient of the
// last LUT pair, flushed into the workgroup's LDS accumulator when the pair
// changes; scale gradient kept in a register.
// ---------------------------------------------------------------------------
struct GradAcc {
    float* lds;     // [lut_n][4]
    int cl0;
    float c0, c1;
    float dscale;
    __device__ __forceinline__ void flush() {
        if (cl0 >= 0) {
            atomicAdd(&lds[cl0 * 4 + 3], c0);
            atomicAdd(&lds[cl0 * 4 + 7], c1);
        }
        cl0 = -1;
        c0 = c1 = 0.0f;
    }
    // d(sigma) = scale * ((1-w) d alpha[l0] + w d alpha[l0+1]) + alpha d scale,
    // scattered with factor f.
    __device__ __forceinline__ void sigma(const TF& t, float scale, float f) {
        if (t.l0 != cl0) {
            flush();
            cl0 = t.l0;
        }
        c0 = fmaf(f * scale, 1.0f - t.w, c0);
        c1 = fmaf(f * scale, t.w, c1);
        dscale = fmaf(f, t.a, dscale);
    }
    // albedo scores d rho_c / rho_c of a real collision, times the channel's
    // later radiance (adjoint included)
    __device__ __forceinline__ void albedo(const TF& t, f3 rgb, f3 after) {
        const float ra[3] = {rgb.x, rgb.y, rgb.z};
        const float af[3] = {after.x, after.y, after.z};
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (ra[c] > 0.0f && ra[c] < 1.0f && af[c] != 0.0f) {
                const float f = af[c] / ra[c];
                atomicAdd(&lds[t.l0 * 4 + c], f * (1.0f - t.w));
                atomicAdd(&lds[t.l0 * 4 + 4 + c], f * t.w);
            }
    }
};

// ---------------------------------------------------------------------------
// Texel store (FP32 / FP16 / BF16, round to nearest even) and wave sums
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint16_t bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ void store_texel(void* out, int dtype, uint64_t k, f3 v) {
    if (dtype == 0) {
        float* o = (float*)out + 3 * k;
        o[0] = v.x;
        o[1] = v.y;
        o[2] = v.z;
    } else if (dtype == 1) {
        __half* o = (__half*)out + 3 * k;
        o[0] = __float2half_rn(v.x);
        o[1] = __float2half_rn(v.y);
        o[2] = __float2half_rn(v.z);
    } else {
        uint16_t* o = (uint16_t*)out + 3 * k;
        o[0] = bf16_rne(v.x);
        o[1] = bf16_rne(v.y);
        o[2] = bf16_rne(v.z);
    }
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ unsigned long long wave_sum64(uint32_t v) {
    unsigned long long w = v;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) w += __shfl_xor(w, o, 64);
    return w;
}
__device__ __forceinline__ float wave_sumf(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

}  // namespace lp
