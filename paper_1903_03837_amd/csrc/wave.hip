// wave.hip -- persistent light-field generation kernel (forward, frozen
// sampling, and the path-replay adjoint).
//
// Paths differ wildly in cost: a ray that misses the volume is done after
// one clip, a ray through dense tissue scatters and casts shadow rays.  With
// one ray per lane and all of a ray's samples in a loop, a wave64 runs as
// long as its most expensive lane; measured lane utilisation was 17 %.  Here
// every lane runs its own state machine
//     IDLE -> START -> FLIGHT -> VERTEX -> SHADOW -> SCATTER -> FLIGHT ... -> IDLE
// and each loop iteration advances every lane by one Philox4x32-10 block
// (further passes of the same iteration advance only the lanes still
// tracking a segment, while at least kTrackPass of the 64 do):
//   START   pair 0 jitters the origin, pair 1 is the first tentative collision;
//   FLIGHT  two tentative collisions (delta tracking; the majorant grid is
//           walked from the current point to each of them);
//   VERTEX  light sample and phase-function words (NEE set-up);
//   SHADOW  two ratio-tracking steps towards the light;
//   SCATTER the new direction from the phase words, then as FLIGHT (pairs 0
//           and 1 of the next segment's block 0).
// START, SCATTER and VERTEX run one shared rotation and one shared clip, so
// a wave that holds all three pays for each once.
// Both tentative points of a block are fetched before either is classified,
// so a lane keeps 16 voxel loads in flight.  A lane whose sample ends starts
// the next sample of its work item (a range of one ray's samples) in the
// next iteration; a lane whose work item is done takes the next one of its
// wave's current 8 x 8 tile of rays, and the wave takes a new tile when the
// current one is used up (one atomic per tile).
//
// Ray order: origins and directions are each sorted into latitude bands of
// ~5 sqrt(n) consecutive SF indices, by azimuth inside a band, so a tile's
// 64 rays run between two small patches of S; tiles are taken in groups of 16
// origin tiles sweeping the direction tiles, and the tile sequence is cut into
// 8 contiguous parts, one per XCD (workgroups are dispatched round-robin over
// the XCDs), so each XCD's L2 sees a narrow bundle of rays.  A part that runs
// dry hands out tiles of the next parts.  Results do not depend on the order:
// every random number is keyed by (ray, sample, bounce).
//
// Adjoint mode: the rays with a nonzero adjoint are first compacted into a
// list (in the same spatial order) and the waves take 64-ray chunks of that
// list.  An event's score times the radiance gathered after it (adjoint .
// (L_tot - L_so_far)) is added to per-workgroup LDS gradients: real collision
// d sigma / sigma, null collision and ratio-tracking step -d sigma /
// (sigma_bar - sigma) (a shadow ray's steps multiply only its own light
// sample's term), albedo d rho / rho.  That radiance is known only at the
// path's end, so a path's events are recorded as they happen and scored
// afterwards: up to kRecords of 16 bytes per lane (in memory; LDS has room for
// an eighth of them), one per block (its two points' raw values and their
// scores' divisors) and one per vertex (its light sample's contribution and
// the number of its shadow ray's records).  Lanes whose path is done wait
// until a quarter of the wave does; then the wave scores their lists as one,
// 64 records at a time, a lane each.  A path with more records is traced
// again with its radiance known, its flights scored as they happen, and so is
// every sample whose radiance the forward kept; a shadow ray's steps are then
// recorded in the same way, and traced again if they are too many.
// The tracing bounds it, as it does the forward.  Dense adjoint of the 128^3
// blobs, N = 1024, 32 spp: 7.9 ms when every sample was traced a second time and
// its shadow rays a third, 5.8 now.  The training step of a denser scene of
// these sizes (10 events per sample, 7.5 of them in shadow rays): 19.2 ms
// before, 18.1 when each lane scored its own list (a quarter of the lanes
// busy), 15.3 when the lists are shared, 14.4 at three waves per SIMD; 11.6
// with the scoring left out.  Several copies of the LDS sums against
// conflicting atomics: no difference.
#include "internal.hpp"

namespace lp {

// Orders the wave's memory accesses before and after it across its lanes.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Adds a light sample's term C Tr to the sample's radiance L and returns the
// rounded product.  The adjoint multiplies scores by the radiance gathered
// after an event, the total less the sum so far, so both must be formed alike
// or a rounding residue is left after the last term.  Totals from the forward
// (srad) hold fused sums; without them the recorded terms are added up, which
// are rounded products, so a path traced again adds the same.
template <int MODE, class PT>
__device__ __forceinline__ f3 add_light(const PT& P, f3 C, float Tr, f3& L) {
#pragma clang fp contract(off)
    const f3 p = {C.x * Tr, C.y * Tr, C.z * Tr};
    const bool rounded = MODE == kGrad && !P.srad;
    L = rounded ? f3{L.x + p.x, L.y + p.y, L.z + p.z} : fma3(C, Tr, L);
    return p;
}

// STATS: the work counters of `stats` are kept (a separate instantiation, so
// the plain kernel spends no registers on them).  VIEWS: ground-truth views
// (pinhole rays of pixel tiles) instead of light-field rays, also a separate
// instantiation so that the light-field kernel carries none of its code.
// Registers are budgeted for four resident waves per SIMD (128 VGPRs; the plain
// forward spills 9 to 13 values by voxel type, the views 6 to 8, frozen sampling
// 15 or 16, the instantiations with work counts 26 to 34), the adjoint's for
// three (166 or 168, none spilled).  Other budgets, on the synthetic phantoms at
// their default settings: 256^3, N = 2048, 64 spp 8.5 ms, with five waves (96
// VGPRs) 11.4, with three 9.2; two 480 x 270 views of it at 256 spp 2.4, 3.3 and
// 2.3; 512^3, N = 32768, 2048 rows 249, 307 and 248; the 128^3 dense adjoint 5.8
// ms, 7.8 with four waves.
template <int VT, int MODE, bool STATS, bool VIEWS>
__global__ __launch_bounds__(256, MODE == kGrad ? 3 : 4) void gen_wave_kernel(TraceParams P) {
    // LDS: cell majorants and their reciprocals (first, so that the grid walk's
    // byte offsets are its addresses), then the tables
    extern __shared__ float4 smem[];
    const int ncell = (P.grid_n + 2) * (P.grid_n + 2) * (P.grid_n + 2);  // padded grid
    float2* mg = (float2*)smem;
    const uint32_t mga = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float2*)mg;  // its LDS address
    float4* lut_e = smem + (ncell + 1) / 2;
    float4* lut_s = lut_e + (MODE == kFrozen ? P.lut_n : 0);
    float* glds = (float*)(lut_e + P.lut_n);  // kGrad: dLUT [lut_n][4], dscale
    for (int e = threadIdx.x; e < P.lut_n; e += blockDim.x) {
        lut_e[e] = ((const float4*)P.lut_e)[e];
        if constexpr (MODE == kFrozen) lut_s[e] = ((const float4*)P.lut_s)[e];
    }
    // the cell majorants with a border that repeats the edge cells
    for (int e = threadIdx.x; e < ncell; e += blockDim.x) {
        const int Gp = P.grid_n + 2, ex = e % Gp, ey = (e / Gp) % Gp, ez = e / (Gp * Gp);
        const int G1 = P.grid_n - 1;
        const int cx = min(max(ex - 1, 0), G1), cy = min(max(ey - 1, 0), G1), cz = min(max(ez - 1, 0), G1);
        const float m = P.maj[(cz * P.grid_n + cy) * P.grid_n + cx];
        mg[e] = make_float2(m, rcp(m));
    }
    if constexpr (MODE == kGrad)
        for (int e = threadIdx.x; e < 4 * P.lut_n + 1; e += blockDim.x) glds[e] = 0.0f;
    __syncthreads();

    const float sigbar = *P.sigbar;
    const int lane = threadIdx.x & 63;
    // Each ray is split into 2^part_log2 work items, ranges of its samples,
    // for load balance (the rays of the last tiles would otherwise hold the
    // grid long after most waves are done).  Adjoint: the scores add up in
    // any order.  Forward with more than one range: each item leaves its
    // partial sum in part_sums, and a second kernel adds the ranges in order.
    // The last rays of each part of the queue are split further, down to a
    // sample or two per item: their samples are kept, and summed by a second
    // kernel in the same order.
    const long long nlist = MODE == kGrad ? (long long)*P.ray_count << P.part_log2 : 0;
    const Queue Q(MODE == kGrad ? (nlist + 63) / 64
                  : VIEWS       ? (long long)P.nviews * P.vtiles
                                : (long long)((P.row_end - P.row_begin + 7) / 8) * ((P.N + 7) / 8),
                  MODE == kGrad ? 0 : P.part_log2, MODE == kGrad ? 0 : P.fine_units, P.fine_log2);
    const int home = blockIdx.x % kParts;
    const int place = (int)(blockIdx.x / kParts) * 4 + (int)(threadIdx.x >> 6);  // among the part's waves
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    // wave-uniform queue cursor
    Tile tile = {0, 0, 0, 0, false};
    unsigned dry = 0;
    bool begun = false, drained = false;

    // lane state
    int mode = kIdle;
    uint32_t k = 0, blk = 0;
    int s = 0, b = 0;
    int s_end = P.spp;  // end of this work item's sample range
    int part = 0;       // its range index, or (fine items) the ray in the samples buffer with the top bit set
    f3 po = mk3(0, 0, 0), d0 = po, acc = po, x = po, dir = po, T = po, L = po, om = po, C = po;
    float W = 1.0f, t = 0.0f, tend = 0.0f, Tr = 1.0f, up0 = 0.0f, up1 = 0.0f;
    f3 isd = po;  // reciprocals of the current segment's direction (dir or om)
    Counters cnt = {0, 0, 0, 0, 0};
    // adjoint state: texel adjoint / spp, the sample's radiance, pass (0: radiance not known yet, 1: known,
    // scored on the way, 2: whole path recorded), score weight of the light sample
    f3 adj = po, ltot = po;
    int pass = 0;
    float rc = 0.0f;
    GradAcc G;
    G.lds = glds;
    G.cl0 = -1;
    G.c0 = G.c1 = 0.0f;
    G.dscale = 0.0f;
    // recorded events: nrec of them, `heads` the vertices among them (bit per
    // record), `mark` the latest vertex
    int nrec = 0, mark = 0;
    uint64_t heads = 0;
    const uint32_t rec_at = ((uint32_t)blockIdx.x * 256u + threadIdx.x) * (uint32_t)kRecords;

    KTraceParams* Pk = (KTraceParams*)__builtin_amdgcn_kernarg_segment_ptr();
    for (;;) {
        // parameters reloaded in each iteration (scalar loads; see KTraceParams)
        asm volatile("" : "+s"(Pk));
        const KTraceParams& P = *Pk;
        const uint32_t K0 = P.key0, K1 = P.key1;
        const int rows = P.row_end - P.row_begin;
        const int tiles_i = (rows + 7) / 8, tiles_j = (P.N + 7) / 8;
        const int plog = P.part_log2;
        const int parts = 1 << plog;
        const float inv_spp = 1.0f / (float)P.spp;
        const f3 O = mk3(P.O[0], P.O[1], P.O[2]);
        const f3 env = mk3(P.env[0], P.env[1], P.env[2]);
        // adding a zero environment leaves a sum of +0 at +0: such sums are skipped
        const bool env_zero = env.x == 0.0f && env.y == 0.0f && env.z == 0.0f;
        const f3 bmin = mk3(P.bmin[0], P.bmin[1], P.bmin[2]), bmax = mk3(P.bmax[0], P.bmax[1], P.bmax[2]);
        // ------------------------------------------------------ sample end
        // (of the samples that ended in the previous iteration's passes)
        if (mode == kDone) {
            bool next = true;
            if constexpr (MODE == kGrad) {
                if (pass == 0) {  // radiance known: score the recorded events
                    ltot = L;
                    next = nrec == 0;
                    pass = 1;  // (too many to keep: replay the sample with scores)
                    if (nrec > 0 && nrec <= kRecords) {
                        pass = 2;
                        mode = kScore;
                    }
                }
                if (next) pass = P.srad ? 1 : 0;
            } else {
                acc = acc + L;
                if (P.srad && !VIEWS) {
                    float* o = P.srad + 3 * ((uint64_t)k * (uint32_t)P.spp + (uint32_t)s);
                    o[0] = L.x;
                    o[1] = L.y;
                    o[2] = L.z;
                }
                if (part < 0) {
                    float* o = kept_sample(P, part & 0x7fffffff, s);
                    o[0] = L.x;
                    o[1] = L.y;
                    o[2] = L.z;
                }
            }
            if (next && ++s == s_end) {
                if constexpr (MODE != kGrad) {
                    if (part < 0) {  // fine item: its samples are summed later
                    } else if (parts == 1) {
                        const float fs = (float)P.spp;
                        store_texel(P.out, P.dtype, k, mk3(acc.x / fs, acc.y / fs, acc.z / fs));
                    } else {  // this range's sum, for the combining kernel
                        const uint64_t kl = (uint64_t)k - (uint64_t)P.row_begin * (uint32_t)P.N;
                        float* o = P.part_sums + 3 * (kl * parts + part);
                        o[0] = acc.x;
                        o[1] = acc.y;
                        o[2] = acc.z;
                    }
                }
                mode = kIdle;
            } else if (MODE != kGrad || mode != kScore) {
                mode = kStart;
                b = 0;
                blk = 0;
            }
        }

        // ------------------------------------------------------------ refill
        const uint64_t idle = __ballot(mode == kIdle);
        if (idle) {
            const int nidle = __popcll(idle);
            const int rank = __popcll(idle & lt_mask);
            const long long avail = tile.end - tile.cur;
            Tile fresh;
            bool more = false;
            if (nidle > avail && !drained) {
                more = next_tile(P.tile_ctr, P.ctr_stride, Q, home, place, begun, dry, fresh);
                drained = !more;
            }
            long long q = -1;
            bool fine = tile.fine;
            int lg = MODE == kGrad ? plog : tile.log2;
            long long shift = tile.shift;
            if (mode == kIdle) {
                if (rank < avail) {
                    q = tile.cur + rank;
                } else if (more) {
                    q = fresh.cur + (rank - avail);
                    if constexpr (MODE != kGrad) {
                        fine = fresh.fine;
                        lg = fresh.log2;
                        shift = fresh.shift;
                    }
                }
            }
            if (more) {
                tile = fresh;
                tile.cur += nidle - avail;
            } else {
                tile.cur += min((long long)nidle, avail);
            }
            if (q >= 0) {
                int i = -1, j = -1;
                // work item q: sample range q mod 2^lg of ray slot q >> lg
                const long long slot = q >> lg;
                const int item = (int)q & ((1 << lg) - 1);
                const int s_first = item_sample(item, P.spp, lg);
                s_end = item_sample(item + 1, P.spp, lg);
                part = fine ? (int)(0x80000000u | (uint32_t)(slot + shift)) : item;
                if constexpr (MODE == kGrad) {
                    if (q < nlist) {
                        const uint32_t kk = P.ray_list[slot];
                        i = (int)(kk / (uint32_t)P.N);
                        j = (int)(kk - (uint32_t)i * (uint32_t)P.N);
                        const float* a = P.d_lf + 3 * (uint64_t)kk;
                        adj = mk3(a[0] * inv_spp, a[1] * inv_spp, a[2] * inv_spp);
                        pass = P.srad ? 1 : 0;
                    }
                } else if constexpr (VIEWS) {
                    // pixel of an 8 x 8 tile of a view: the ray from the eye through its centre
                    const uint32_t t = (uint32_t)(slot >> 6);
                    const uint32_t v = t / (uint32_t)P.vtiles, rem = t - v * (uint32_t)P.vtiles;
                    const uint32_t ty = rem / (uint32_t)P.vtx, tx = rem - ty * (uint32_t)P.vtx;
                    const int py = (int)ty * 8 + (int)((slot >> 3) & 7), px = (int)tx * 8 + (int)(slot & 7);
                    if (py < P.H && px < P.W) {
                        const ViewCam& cam = P.views[v];
                        const float ndx = (2.0f * ((float)px + 0.5f) / (float)P.W - 1.0f) * cam.sx;
                        const float ndy = (1.0f - 2.0f * ((float)py + 0.5f) / (float)P.H) * cam.sy;
                        k = (v * (uint32_t)P.H + (uint32_t)py) * (uint32_t)P.W + (uint32_t)px;
                        po = mk3(cam.eye[0], cam.eye[1], cam.eye[2]);
                        d0 = normalize(mk3(cam.fwd[0], cam.fwd[1], cam.fwd[2]) +
                                       mk3(cam.right[0], cam.right[1], cam.right[2]) * ndx +
                                       mk3(cam.up[0], cam.up[1], cam.up[2]) * ndy);
                        acc = mk3(0.0f, 0.0f, 0.0f);
                        s = s_first;
                        b = 0;
                        blk = 0;
                        mode = kStart;
                    }
                } else {
                    int ti, tj;
                    tile_coords(slot >> 6, tiles_i, tiles_j, ti, tj);
                    const int oi = ti * 8 + (int)((slot >> 3) & 7), dj = tj * 8 + (int)(slot & 7);
                    if (oi < rows && dj < P.N) {
                        i = P.perm_o[oi];
                        j = P.perm_d[dj];
                    }
                }
                if (i >= 0) {
                    k = (uint32_t)i * (uint32_t)P.N + (uint32_t)j;
                    if (P.M == P.N && i == j) {
                        // no direction: texel 0 (never listed for the adjoint;
                        // with several ranges or kept samples the summing kernel
                        // writes it)
                        if constexpr (MODE != kGrad)
                            if (parts == 1 && !fine) store_texel(P.out, P.dtype, k, mk3(0.0f, 0.0f, 0.0f));
                    } else {
                        const float4 a = P.tab_o[i], c = P.tab_d[j];
                        po = mk3(a.x, a.y, a.z);
                        d0 = normalize(mk3(c.x, c.y, c.z) - po);
                        acc = mk3(0.0f, 0.0f, 0.0f);
                        s = s_first;
                        b = 0;
                        blk = 0;
                        mode = kStart;
                        // A ray that misses the volume box in every sample: all
                        // samples of the range but the last are added here (each
                        // is the environment radiance), and the last one runs as
                        // usual.  (The adjoint's ray list leaves such rays out.)
                        if constexpr (MODE != kGrad) {
                            if (misses_box(P, O, bmin, bmax, po, d0)) {
                                if (fine) {  // all of the item's samples
                                    for (int s2 = s_first; s2 < s_end; ++s2) {
                                        float* o = kept_sample(P, part & 0x7fffffff, s2);
                                        o[0] = env.x;
                                        o[1] = env.y;
                                        o[2] = env.z;
                                    }
                                    // (of the kept sample radiance, the last one of each range)
                                    if (P.srad && ((item + 1) & ((1 << (lg - plog)) - 1)) == 0) {
                                        float* r = P.srad + 3 * ((uint64_t)k * (uint32_t)P.spp + (uint32_t)(s_end - 1));
                                        r[0] = env.x;
                                        r[1] = env.y;
                                        r[2] = env.z;
                                    }
                                    cnt.samples++;
                                    mode = kIdle;
                                } else if (!env_zero) {
                                    for (int s2 = s_first + 1; s2 < s_end; ++s2) acc = acc + env;
                                }
                                cnt.samples += (uint32_t)(s_end - 1 - s_first);
                                s = s_end - 1;
                            }
                        }
                    }
                }
            }
        }
        const int live = __popcll(__ballot(mode != kIdle));
        if (live == 0) {
            if (drained && tile.end <= tile.cur) break;
            continue;
        }

        // ------------------------------------------------------------- score
        if constexpr (MODE == kGrad) {
            const int scoring = __popcll(__ballot(mode == kScore));
            if (scoring != 0 && scoring * 64 >= kScoreLanes * live) {
                // the lanes' lists as one, 64 records at a time (read by other
                // lanes than wrote them, and written anew afterwards: both
                // orders are stated, at no instruction's cost within a wave)
                wave_fence();
                const int mine = mode == kScore ? nrec : 0;
                int end = mine;  // inclusive prefix sum
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int v = __shfl_up(end, o, 64);
                    end += lane >= o ? v : 0;
                }
                const int total = __builtin_amdgcn_readlane(end, 63);
                const uint32_t wave_at = rec_at - (uint32_t)lane * (uint32_t)kRecords;
                for (int first = 0; first < total; first += 64) {
                    const int g = first + lane;
                    // the list that holds record g: the number of lists that end at or before it
                    int own = 0;
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1)
                        if (__shfl(end, own + o - 1, 64) <= g) own += o;
                    own = min(own, 63);
                    const int at = g - (__shfl(end, own, 64) - __shfl(mine, own, 64));
                    const f3 adj1 = mk3(__shfl(adj.x, own, 64), __shfl(adj.y, own, 64), __shfl(adj.z, own, 64));
                    const f3 ltot1 = mk3(__shfl(ltot.x, own, 64), __shfl(ltot.y, own, 64), __shfl(ltot.z, own, 64));
                    const uint64_t heads1 = (uint64_t)__shfl((uint32_t)heads, own, 64) |
                                            (uint64_t)__shfl((uint32_t)(heads >> 32), own, 64) << 32;
                    const float rc1 = __shfl(rc, own, 64);
                    const bool path = __shfl(pass, own, 64) == 2;  // a whole path (else a shadow ray only)
                    if (g < total && !((heads1 >> at) & 1)) {
                        const float4* const list =
                            (const float4*)((const char*)P.records + (wave_at + (uint32_t)own * (uint32_t)kRecords) * 16u);
                        const float4 q = list[at];
                        // the radiance gathered before the record, and whether a shadow ray's
                        f3 L1 = mk3(0.0f, 0.0f, 0.0f);
                        bool shadow = !path;
                        float gain = rc1;
                        for (uint64_t hs = heads1 & ((1ull << at) - 1ull); hs; hs &= hs - 1) {
                            const int h = __ffsll((long long)hs) - 1;
                            const float4 v = list[h];
                            L1 = L1 + mk3(v.x, v.y, v.z);
                            shadow = at <= h + __float_as_int(v.w);
                            gain = dot(adj1, mk3(v.x, v.y, v.z));
                        }
                        const bool on = !shadow || gain != 0.0f;
                        if (!shadow) gain = dot(adj1, ltot1 - L1);
                        const bool inA = __float_as_uint(q.y) != kNoPoint, inB = __float_as_uint(q.w) != kNoPoint;
                        const TF fA = classify<MODE>(P, lut_e, lut_s, q.x), fB = classify<MODE>(P, lut_e, lut_s, q.z);
                        if (on && inA) G.sigma(fA, P.scale_e, gain / q.y);
                        if (on && inB) G.sigma(fB, P.scale_e, gain / q.w);
                        if (at < kRecords - 1 && ((heads1 >> (at + 1)) & 1)) {  // its last point is a real collision
                            TF te;
                            te.l0 = inB ? fB.l0 : fA.l0;
                            te.w = inB ? fB.w : fA.w;
                            G.albedo(te, tf_rgb(lut_e, te), (ltot1 - L1) * adj1);
                        }
                    }
                }
                wave_fence();
                if (mode == kScore) {
                    mode = kDone;
                    if (pass == 1) {  // the shadow ray's light, and the path goes on
                        add_light<MODE>(P, C, Tr, L);
                        if (b != P.maxb - 1) {
                            ++b;
                            blk = 0;
                            mode = kScatter;
                        }
                    }
                }
            }
        }

        // Passes: the first one draws a block for every lane and runs the
        // set-up of START, SCATTER and VERTEX lanes; further passes, while at
        // least kTrackPass lanes are still tracking a segment, advance only
        // those lanes by one block each.  A lane whose segment needs a set-up
        // or whose sample ended waits for the next iteration, so the set-up
        // and sample-end code runs once per iteration for all such lanes.
        // Every lane still takes the same steps in the same order.
        for (bool first = true;; first = false) {
            // ------------------------------------------------------ one block
            const bool vstream = mode == kVertex || mode == kShadow || mode == kShadow2;
            const u4 r = philox(k, (uint32_t)s, ((uint32_t)b << 8) | (vstream ? kPurVertex : kPurFlight), blk, K0, K1);
            bool stepA = mode == kFlight || mode == kShadow || mode == kShadow2;
            bool stepB = stepA;
            bool sample_done = false, after_shadow = false;

            if (first) {
                // --------------------------------------------------- segment set-up
                // A sample's first segment (START), the segment after a scatter
                // (SCATTER: b already advanced) and the shadow ray of a vertex
                // (VERTEX) share one rotation (START's jitter disk, SCATTER's phase
                // direction) and one clip against the box.
                const bool seg = mode == kStart || mode == kScatter;
                const bool shadow_ray = mode == kVertex && P.light_on;
                f3 Le = mk3(0.0f, 0.0f, 0.0f);
                float dist = 0.0f;
                if (mode == kVertex) {
                    // next-event estimation: light sample (pair 0); phase words (pair 1) kept for the scatter
                    up0 = u01(r.z);
                    up1 = u01(r.w);
                    if (P.light_on) {
                        if (P.light_kind == 0) {
                            om = mk3(P.ldir[0], P.ldir[1], P.ldir[2]);
                            Le = mk3(P.lrad[0], P.lrad[1], P.lrad[2]);
                        } else {
                            const f3 yl = mk3(P.lcorner[0], P.lcorner[1], P.lcorner[2]) +
                                          mk3(P.le1[0], P.le1[1], P.le1[2]) * u01(r.x) +
                                          mk3(P.le2[0], P.le2[1], P.le2[2]) * u01(r.y);
                            const f3 v = yl - x;
                            const float d2 = dot(v, v);
                            const float rinv = rsq(d2);
                            dist = d2 * rinv;
                            om = v * rinv;
                            const float cl = fmaxf(0.0f, -dot(mk3(P.lnrm[0], P.lnrm[1], P.lnrm[2]), om));
                            Le = mk3(P.lrad[0], P.lrad[1], P.lrad[2]) * (cl * P.larea * rcp(d2));
                        }
                    } else {
                        after_shadow = true;
                    }
                } else if (seg) {
                    // base + A (cos(2 pi u) t1 + sin(2 pi u) t2), (t1, t2) completing n
                    f3 n, base;
                    float A, ua;
                    if (mode == kStart) {
                        cnt.samples++;
                        if constexpr (MODE == kGrad) {
                            if (P.srad) {  // the sample's total radiance, kept by the forward
                                const float* lt = P.srad + 3 * ((uint64_t)k * (uint32_t)P.spp + (uint32_t)s);
                                ltot = mk3(lt[0], lt[1], lt[2]);
                            }
                        }
                        // light-field ray: origin on S (jittered); view ray: the eye
                        base = VIEWS ? po : O + po * P.R;
                        n = po;
                        A = (P.jitter && !VIEWS) ? P.jit_rad * sqrtf(u01(r.x)) : 0.0f;
                        ua = u01(r.y);
                        T = mk3(1.0f, 1.0f, 1.0f);
                        W = 1.0f;
                        nrec = 0;
                        heads = 0;
                        L = mk3(0.0f, 0.0f, 0.0f);
                    } else {
                        const float mu = hg_mu(P.g, up0);
                        A = sqrtf(fmaxf(0.0f, 1.0f - mu * mu));
                        base = dir * mu;
                        n = dir;
                        ua = up1;
                    }
                    float sa, ca;
                    sincospif(2.0f * ua, &sa, &ca);
                    f3 t1, t2;
                    frame(n, t1, t2);
                    const f3 v = base + t1 * (A * ca) + t2 * (A * sa);
                    if (mode == kStart) {
                        x = v;
                        dir = d0;
                    } else {
                        dir = v;
                    }
                }
                if (seg || shadow_ray) {
                    float tn, tf;
                    const f3 cd = shadow_ray ? om : dir;
                    isd = rcp3(cd);  // kept for the grid walks of this segment
                    const bool hit = clip_box(bmin, bmax, x, cd, isd, tn, tf);
                    if (shadow_ray) {
                        const float te = hit ? (P.light_kind == 0 ? tf : fminf(dist, tf)) : 0.0f;
                        C = T * Le * (W * hg_phase(P.g, dot(dir, om)));
                        Tr = 1.0f;
                        if (sigbar > 0.0f) {
                            t = 0.0f;
                            tend = te;
                            mode = kShadow;
                            blk = 1;
                            if (pass) nrec = 0;
                        } else {
                            L = L + C;
                            after_shadow = true;
                        }
                    } else if (hit && sigbar > 0.0f) {
                        // START: pair 1 is the first tentative collision (pair 0 was the
                        // jitter); SCATTER: pairs 0 and 1
                        stepA = mode == kScatter;
                        stepB = true;
                        t = tn;
                        tend = tf;
                        mode = kFlight;
                    } else {
                        L = L + T * env * W;
                        sample_done = true;
                    }
                }

            }

            // -------------------------------------------- two tentative points
            if (stepA || stepB) {
                // (stepB always holds here; stepA is off for the first point of a sample)
                const bool flight = mode == kFlight;
                const f3 sd = flight ? dir : om;
                GridWalk gw;
                gw.init(P, mga, x, sd, isd, t);
                float sbA = 0.0f, sbB = 0.0f, rbB = 0.0f, tA, tB;
                // The walk is a chain of dependent steps (an LDS read of the
                // cell's majorant, then ~30 instructions) that the wave's
                // slowest lane drags out; raised wave priority lets it issue
                // ahead of the other waves of its SIMD, whose volume loads are
                // in flight meanwhile (forward modes: 0.5-1 %; the adjoint
                // keeps the default).  Scheduling only: the same instructions
                // and results.
                if constexpr (MODE != kGrad) __builtin_amdgcn_s_setprio(2);
                gw.next2(P, mga, stepA, neg_log1m(u01(r.x)), neg_log1m(u01(r.z)), tend, tA, sbA, tB, sbB, rbB,
                         cnt.cells);
                if constexpr (MODE != kGrad) __builtin_amdgcn_s_setprio(0);
                // (without a point A both fetches read point B's line)
                const f3 yA = fma3(sd, stepA ? tA : tB, x), yB = fma3(sd, tB, x);
                const float rawA = sample_volume<VT>(P, yA);
                const float rawB = sample_volume<VT>(P, yB);
                // Both points are classified and decided in straight-line code:
                // lanes in flight, in shadow or with one point only differ by
                // selects (nested branches ran every side in nearly every wave,
                // with copies of the values that cross them).
                const TF fA = classify<MODE>(P, lut_e, lut_s, rawA), fB = classify<MODE>(P, lut_e, lut_s, rawB);
                const float sgA = P.scale_e * fA.a, sgB = P.scale_e * fB.a;
                const float ssA = MODE == kFrozen ? P.scale_s * fA.a_s : sgA;
                const float ssB = MODE == kFrozen ? P.scale_s * fB.a_s : sgB;
                const bool inA = stepA && !(tA >= tend);                       // A lies on the segment
                const bool realA = inA && flight && u01(r.y) * sbA < ssA;      // and is a real collision
                const bool reachB = !stepA || (inA && !realA);                 // B is looked at
                const bool inB = reachB && !(tB >= tend);
                const bool realB = inB && flight && u01(r.w) * sbB < ssB;
                const bool ev_end = (stepA && !inA) || (reachB && !inB), ev_real = realA || realB;
                t = inB ? tB : (inA ? tA : t);
                if (flight) cnt.tent += (inA ? 1u : 0u) + (inB ? 1u : 0u);
                if (mode == kShadow) cnt.shadow += (inA ? 1u : 0u) + (inB ? 1u : 0u);
                // ratio tracking (Tr is set anew for each shadow ray, so lanes in
                // flight may spoil it; the replay of a shadow ray may not)
                const bool ratio = MODE != kGrad || mode == kShadow;
                Tr *= inA && ratio ? fmaf(-rcp(sbA), sgA, 1.0f) : 1.0f;
                Tr *= inB && ratio ? fmaf(-rbB, sgB, 1.0f) : 1.0f;
                if constexpr (MODE == kFrozen) {
                    if (inA && flight) W *= realA ? sgA / ssA : (sbA - sgA) / (sbA - ssA);
                    if (inB && flight) W *= realB ? sgB / ssB : (sbB - sgB) / (sbB - ssB);
                }
                if constexpr (MODE == kGrad) {
                    // scores: d sigma / sigma at a real collision, -d sigma /
                    // (sigma_bar - sigma) at a null one and at a shadow step
                    const bool on = flight ? pass != 0 : mode == kShadow2;
                    const float gain = flight ? dot(adj, ltot - L) : rc;
                    const float divA = realA ? sgA : sgA - sbA, divB = realB ? sgB : sgB - sbB;
                    if (on && inA) G.sigma(fA, P.scale_e, gain / divA);
                    if (on && inB) G.sigma(fB, P.scale_e, gain / divB);
                    // where the factor is not known yet, the points are recorded
                    if ((pass == 0 || mode == kShadow) && (inA || inB)) {
                        if (nrec < kRecords)
                            *(float4*)((char*)P.records + (rec_at + (uint32_t)nrec) * 16u) =
                                make_float4(rawA, inA ? divA : __uint_as_float(kNoPoint), rawB,
                                            inB ? divB : __uint_as_float(kNoPoint));
                        ++nrec;
                    }
                }
                if (ev_end) {
                    if (mode == kFlight) {
                        L = L + T * env * W;
                        sample_done = true;
                    } else if (MODE == kGrad && mode == kShadow && pass) {
                        // transmittance known: replay the shadow ray for its scores
                        rc = dot(adj, C * Tr);
                        if (rc != 0.0f && nrec > 0 && nrec <= kRecords) {
                            mode = kScore;
                            heads = 0;
                        } else if (rc != 0.0f && nrec > 0) {
                            mode = kShadow2;
                            blk = 1;
                            t = 0.0f;
                        } else {
                            add_light<MODE>(P, C, Tr, L);
                            after_shadow = true;
                        }
                    } else {
                        const f3 p = add_light<MODE>(P, C, Tr, L);
                        if constexpr (MODE == kGrad)
                            if (mode == kShadow && mark < kRecords)  // the vertex's record
                                *(float4*)((char*)P.records + (rec_at + (uint32_t)mark) * 16u) =
                                    make_float4(p.x, p.y, p.z, __int_as_float(nrec - mark - 1));
                        after_shadow = true;
                    }
                } else if (ev_real) {
                    cnt.real++;
                    TF te;
                    te.l0 = realB ? fB.l0 : fA.l0;
                    te.w = realB ? fB.w : fA.w;
                    const f3 rgb = tf_rgb(lut_e, te);
                    if constexpr (MODE == kGrad) {
                        if (pass) {
                            G.albedo(te, rgb, (ltot - L) * adj);
                        } else {
                            if (nrec < kRecords) {
                                heads |= 1ull << nrec;
                                *(float4*)((char*)P.records + (rec_at + (uint32_t)nrec) * 16u) =
                                    make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                            }
                            mark = nrec++;
                        }
                    }
                    x = realB ? yB : yA;
                    T = T * mk3(__builtin_amdgcn_fmed3f(rgb.x, 0.0f, 1.0f), __builtin_amdgcn_fmed3f(rgb.y, 0.0f, 1.0f),
                                __builtin_amdgcn_fmed3f(rgb.z, 0.0f, 1.0f));
                    if (T.x == 0.0f && T.y == 0.0f && T.z == 0.0f) {
                        sample_done = true;
                    } else {
                        mode = kVertex;
                        blk = 0;
                    }
                } else if (++blk >= kMaxBlocks) {
                    // stream exhausted: the segment ends absorbed / blocked
                    if (mode == kFlight) {
                        sample_done = true;
                    } else {
                        Tr = 0.0f;  // C * 0 adds nothing
                        after_shadow = true;
                    }
                }
            }

            // ------------------------------------------------ scatter direction
            // (drawn at the start of the next iteration, from the phase words)
            if (after_shadow) {
                if (b == P.maxb - 1) {
                    sample_done = true;
                } else {
                    ++b;
                    blk = 0;
                    mode = kScatter;
                }
            }

            if (sample_done) mode = kDone;
            if (__popcll(__ballot(mode == kFlight || mode == kShadow || mode == kShadow2)) * 64 < kTrackPass * live) break;
        }
    }

    if constexpr (MODE == kGrad) {
        G.flush();
        const float ds = wave_sumf(G.dscale);
        if (lane == 0) atomicAdd(&glds[4 * P.lut_n], ds);
        __syncthreads();
        for (int e = threadIdx.x; e < 4 * P.lut_n; e += blockDim.x)
            if (glds[e] != 0.0f) atomicAdd(&P.d_lut[e], glds[e]);
        if (threadIdx.x == 0 && glds[4 * P.lut_n] != 0.0f) atomicAdd(P.d_scale, glds[4 * P.lut_n]);
        return;
    }

    if (STATS) {
        const uint32_t a = wave_sum(cnt.tent), c = wave_sum(cnt.shadow), e = wave_sum(cnt.real),
                       f = wave_sum(cnt.samples);
        const unsigned long long cs = wave_sum64(cnt.cells);
        if (lane == 0) {
            atomicAdd(&P.stats[0], (unsigned long long)a);
            atomicAdd(&P.stats[1], (unsigned long long)c);
            atomicAdd(&P.stats[2], (unsigned long long)e);
            atomicAdd(&P.stats[3], (unsigned long long)f);
            atomicAdd(&P.stats[4], cs);
        }
    }
}

// Compacts the rays (in the spatial tile order) whose adjoint is nonzero and
// which can reach the volume box (a ray that misses it in every sample has no
// collision and so no score).
// One atomic per workgroup and trip claims the list slots of its four waves
// (one per wave made the single counter the bottleneck).
__global__ __launch_bounds__(256) void active_rays_kernel(TraceParams P) {
    __shared__ unsigned wave_n[4], wave_at[4];
    const int rows = P.row_end - P.row_begin;
    const int tiles_i = (rows + 7) / 8, tiles_j = (P.N + 7) / 8;
    const long long total = (long long)tiles_i * tiles_j * 64;
    const int lane = threadIdx.x & 63;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long base = (long long)blockIdx.x * blockDim.x; base < total; base += stride) {
        const long long q = base + threadIdx.x;
        bool take = false;
        uint32_t k = 0;
        if (q < total) {
            int ti, tj;
            tile_coords(q >> 6, tiles_i, tiles_j, ti, tj);
            const int oi = ti * 8 + (int)((q >> 3) & 7), dj = tj * 8 + (int)(q & 7);
            if (oi < rows && dj < P.N) {
                const int i = P.perm_o[oi], j = P.perm_d[dj];
                k = (uint32_t)i * (uint32_t)P.N + (uint32_t)j;
                const float* a = P.d_lf + 3 * (uint64_t)k;
                take = !(P.M == P.N && i == j) && (a[0] != 0.0f || a[1] != 0.0f || a[2] != 0.0f);
                if (take) {
                    const float4 a = P.tab_o[i], c = P.tab_d[j];
                    const f3 po = mk3(a.x, a.y, a.z);
                    const f3 d0 = normalize(mk3(c.x, c.y, c.z) - po);
                    take = !misses_box(P, mk3(P.O[0], P.O[1], P.O[2]), mk3(P.bmin[0], P.bmin[1], P.bmin[2]),
                                       mk3(P.bmax[0], P.bmax[1], P.bmax[2]), po, d0);
                }
            }
        }
        const uint64_t m = __ballot(take);
        const int wave = threadIdx.x >> 6;
        if (lane == 0) wave_n[wave] = (unsigned)__popcll(m);
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned n0 = wave_n[0], n1 = wave_n[1], n2 = wave_n[2], n3 = wave_n[3];
            const unsigned tot = n0 + n1 + n2 + n3;
            const unsigned at = tot ? atomicAdd(P.ray_count, tot) : 0u;
            wave_at[0] = at;
            wave_at[1] = at + n0;
            wave_at[2] = at + n0 + n1;
            wave_at[3] = at + n0 + n1 + n2;
        }
        __syncthreads();
        if (take) P.ray_list[wave_at[wave] + __popcll(m & lt_mask)] = k;
        __syncthreads();  // wave_n / wave_at are rewritten by the next trip
    }
}

// What the persistent kernels need beside the volume, in one launch: the
// global majorant and the cleared counters (the last workgroup), the spatial
// orders of origin rows and directions (one workgroup per band) and both
// point tables.  Each part is latency: as five launches they were 7 % of a
// small field's call (256 x 256 rays, 16 spp, 64^3: 0.53 ms).
struct SetupParams {
    const float* lut;
    int lut_n;
    float scale, given;
    float* sigbar;
    unsigned int *ctr, *ray_count;
    int ctr_stride;
    // order and table of the origin rows and of the directions
    struct Set {
        int base, count, band;  // indices ordered, in bands
        int32_t* perm;
        int n;                  // points of the set
        float inv_n;
        float4* table;
        unsigned order_groups, table_groups;
    } set[2];
};

// Spatial order of count consecutive SF indices base..base+count-1 of a set
// of n points: bands of B indices, each sorted by azimuth (rank counting).
// One workgroup per band, its azimuths staged in LDS (B <= 1272 for
// n <= 65535).
constexpr int kMaxBand = 1280;
__device__ __forceinline__ void order_band(const SetupParams::Set& S, unsigned group, float* fr) {
    const int lo = (int)group * S.band;
    const int cnt = min(S.count - lo, S.band);
    for (int t = (int)threadIdx.x; t < cnt; t += 256) fr[t] = sf_frac(S.base + lo + t);
    __syncthreads();
    for (int t = (int)threadIdx.x; t < cnt; t += 256) {
        const float fe = fr[t];
        int rank = 0;
        for (int f = 0; f < cnt; ++f) {
            const float ff = fr[f];
            rank += ff < fe || (ff == fe && f < t);
        }
        S.perm[lo + rank] = S.base + lo + t;
    }
}

__global__ __launch_bounds__(256) void setup_kernel(SetupParams P) {
    __shared__ float lds[kMaxBand];
    unsigned g = blockIdx.x;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const SetupParams::Set& S = P.set[a];
        if (g < S.order_groups) return order_band(S, g, lds);
        g -= S.order_groups;
        if (g < S.table_groups) return sf_table_entry(S.n, S.inv_n, S.table, g * 256u + threadIdx.x);
        g -= S.table_groups;
    }
    float m = 0.0f;
    for (int e = threadIdx.x; e < P.lut_n; e += 256) m = fmaxf(m, P.lut[4 * e + 3]);
    lds[threadIdx.x] = m;
    if (threadIdx.x < kParts) P.ctr[threadIdx.x * P.ctr_stride] = 0u;
    if (threadIdx.x == kParts && P.ray_count) *P.ray_count = 0u;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) lds[threadIdx.x] = fmaxf(lds[threadIdx.x], lds[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) P.sigbar[0] = P.given > 0.0f ? P.given : 1.25f * P.scale * lds[0];
}

static int band_size(int n) {
    int b = (int)(5.0 * std::sqrt((double)n));
    b &= ~7;
    return b < 8 ? 8 : b;
}

hipError_t launch_wave_setup(const TraceParams& P, const float* sample_lut, int lut_n, float sample_scale,
                             float given, float* sigbar, int32_t* perm_o, int32_t* perm_d, hipStream_t s) {
    SetupParams S = {sample_lut, lut_n, sample_scale, given, sigbar, P.tile_ctr, P.ray_count, P.ctr_stride, {}};
    const int rows = P.row_end - P.row_begin;
    auto fill = [](int base, int count, int n, int32_t* perm, const float4* table) {
        SetupParams::Set t = {base, count, band_size(n), perm, n, 1.0f / (float)n, (float4*)table, 0, 0};
        if (count > 0) t.order_groups = (unsigned)((count + t.band - 1) / t.band);
        if (table) t.table_groups = (unsigned)(n + 255) / 256;
        return t;
    };
    S.set[0] = fill(P.row_begin, rows, P.M, perm_o, P.tab_o);
    S.set[1] = fill(0, P.N, P.N, perm_d, P.tab_d);
    unsigned groups = 1;
    for (const auto& t : S.set) groups += t.order_groups + t.table_groups;
    setup_kernel<<<groups, 256, 0, s>>>(S);
    return hipGetLastError();
}

hipError_t launch_active_rays(const TraceParams& P, hipStream_t s) {
    const long long rows = P.row_end - P.row_begin;
    const long long total = ((rows + 7) / 8) * (long long)((P.N + 7) / 8) * 64;
    if (total <= 0) return hipSuccess;
    long long blocks = (total + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    active_rays_kernel<<<(unsigned)blocks, 256, 0, s>>>(P);
    return hipGetLastError();
}

static long long ray_tiles(const TraceParams& P) {
    return P.views ? (long long)P.nviews * P.vtiles
                   : (long long)((P.row_end - P.row_begin + 7) / 8) * ((P.N + 7) / 8);
}

template <int VT, int MODE, bool STATS, bool VIEWS>
static hipError_t launch_wave_t(const TraceParams& P, hipStream_t s) {
    // (adjoint: the list's length is only known on the device)
    long long ntiles = 0;
    if (MODE == kGrad) {
        ntiles = ray_tiles(P) << P.part_log2;
    } else {
        const Queue Q(ray_tiles(P), P.part_log2, P.fine_units, P.fine_log2);
        for (int p = 0; p < kParts; ++p) ntiles += Q.tiles(p);
    }
    if (ntiles <= 0) return hipSuccess;
    const size_t ncell = (size_t)(P.grid_n + 2) * (P.grid_n + 2) * (P.grid_n + 2);  // padded grid in LDS
    const size_t lds = sizeof(float4) * (size_t)P.lut_n * (MODE == kFrozen ? 2 : 1) +
                       (MODE == kGrad ? sizeof(float) * (4 * (size_t)P.lut_n + 1) : 0) +
                       sizeof(float4) * ((ncell + 1) / 2);
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gen_wave_kernel<VT, MODE, STATS, VIEWS>, 256,
                                                         lds);
    if (e != hipSuccess) return e;
    long long blocks = (long long)cus * (per_cu > 0 ? per_cu : 1);
    if (MODE == kGrad && blocks > P.record_groups) blocks = P.record_groups;
    // at least one tile per wave (list lengths are only known on the device;
    // waves that find no chunk exit at once)
    const long long need = (ntiles + 3) / 4;
    if (blocks > need) blocks = need;
    gen_wave_kernel<VT, MODE, STATS, VIEWS><<<(unsigned)blocks, 256, lds, s>>>(P);
    return hipGetLastError();
}

template <int VT>
static hipError_t launch_wave_mode(const TraceParams& P, int mode, hipStream_t s) {
    if (P.views) return launch_wave_t<VT, kFwd, false, true>(P, s);  // ground-truth views: plain forward
    if (mode == kGrad) return launch_wave_t<VT, kGrad, false, false>(P, s);
    if (P.stats)
        return mode == kFrozen ? launch_wave_t<VT, kFrozen, true, false>(P, s)
                               : launch_wave_t<VT, kFwd, true, false>(P, s);
    return mode == kFrozen ? launch_wave_t<VT, kFrozen, false, false>(P, s)
                           : launch_wave_t<VT, kFwd, false, false>(P, s);
}

// Light-field texels from the sample ranges: the ranges' sums in range
// order, divided by spp (texels i == j are 0).
__global__ void combine_parts_kernel(TraceParams P, long long n) {
    const long long kl = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (kl >= n) return;
    const int parts = 1 << P.part_log2;
    bool none = false;  // texel i == j of the light field
    uint32_t k = (uint32_t)kl;  // views: the pixel
    if (!P.views) {
        const uint32_t i = (uint32_t)P.row_begin + (uint32_t)(kl / P.N), j = (uint32_t)(kl % P.N);
        k = i * (uint32_t)P.N + j;
        none = P.M == P.N && i == j;
    }
    f3 acc = mk3(0.0f, 0.0f, 0.0f);
    if (!none) {
        const float* p = P.part_sums + 3 * (uint64_t)kl * parts;
        acc = mk3(p[0], p[1], p[2]);
        for (int q = 1; q < parts; ++q) acc = acc + mk3(p[3 * q], p[3 * q + 1], p[3 * q + 2]);
        const float fs = (float)P.spp;
        acc = mk3(acc.x / fs, acc.y / fs, acc.z / fs);
    }
    store_texel(P.out, P.dtype, k, acc);
}

// Texels of the rays whose samples were kept (the last fine_units ray tiles
// of each part of the queue): each range's sum in sample order, as the tracer
// forms it, then the ranges in order, divided by spp.
__global__ __launch_bounds__(256) void combine_samples_kernel(TraceParams P, Queue Q) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;  // ray of the samples buffer
    const long long per_part = 64ll * Q.fine;
    const int p = (int)(e / per_part);
    if (p >= kParts) return;
    const long long r = e - p * per_part, u = r >> 6, c = Q.coarse(p);
    if (u >= Q.count(p) - c) return;
    const long long slot = (Q.first(p) + c + u) * 64 + (r & 63);
    bool none = false;
    uint32_t k;
    if (P.views) {
        const uint32_t t = (uint32_t)(slot >> 6), v = t / (uint32_t)P.vtiles, rem = t - v * (uint32_t)P.vtiles;
        const uint32_t ty = rem / (uint32_t)P.vtx, tx = rem - ty * (uint32_t)P.vtx;
        const int py = (int)ty * 8 + (int)((slot >> 3) & 7), px = (int)tx * 8 + (int)(slot & 7);
        if (py >= P.H || px >= P.W) return;
        k = (v * (uint32_t)P.H + (uint32_t)py) * (uint32_t)P.W + (uint32_t)px;
    } else {
        const int rows = P.row_end - P.row_begin;
        int ti, tj;
        tile_coords(slot >> 6, (rows + 7) / 8, (P.N + 7) / 8, ti, tj);
        const int oi = ti * 8 + (int)((slot >> 3) & 7), dj = tj * 8 + (int)(slot & 7);
        if (oi >= rows || dj >= P.N) return;
        const int i = P.perm_o[oi], j = P.perm_d[dj];
        k = (uint32_t)i * (uint32_t)P.N + (uint32_t)j;
        none = P.M == P.N && i == j;
    }
    f3 acc = mk3(0.0f, 0.0f, 0.0f);
    if (!none) {
        const float* s = kept_sample(P, (uint32_t)e, 0);
        for (int q = 0; q < 1 << P.part_log2; ++q) {
            const int s1 = item_sample(q + 1, P.spp, P.part_log2);
            f3 sum = mk3(0.0f, 0.0f, 0.0f);
#pragma unroll 8
            for (int i = item_sample(q, P.spp, P.part_log2); i < s1; ++i)
                sum = sum + mk3(s[192 * i], s[192 * i + 1], s[192 * i + 2]);
            acc = q ? acc + sum : sum;
        }
        const float fs = (float)P.spp;
        acc = mk3(acc.x / fs, acc.y / fs, acc.z / fs);
    }
    store_texel(P.out, P.dtype, k, acc);
}

hipError_t launch_combine_parts(const TraceParams& P, hipStream_t s) {
    const long long n = P.views ? (long long)P.nviews * P.H * P.W : (long long)(P.row_end - P.row_begin) * P.N;
    if (n <= 0) return hipSuccess;
    const Queue Q(ray_tiles(P), P.part_log2, P.fine_units, P.fine_log2);
    // (texels of kept samples are written last: part_sums has none of theirs)
    if (P.part_log2 > 0 && Q.part > Q.fine) combine_parts_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(P, n);
    if (Q.fine > 0) combine_samples_kernel<<<(unsigned)((64ll * Q.fine * kParts + 255) / 256), 256, 0, s>>>(P, Q);
    return hipGetLastError();
}

hipError_t launch_generate_wave(const TraceParams& P, int vtype, int mode, hipStream_t s) {
    switch (vtype) {
        case 0: return launch_wave_mode<0>(P, mode, s);
        case 1: return launch_wave_mode<1>(P, mode, s);
        default: return launch_wave_mode<2>(P, mode, s);
    }
}

}  // namespace lp
