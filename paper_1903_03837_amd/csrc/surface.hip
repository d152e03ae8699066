// surface.hip -- isosurface variant of generation and of the ground-truth
// views: the paper path-traces segmented surfaces; here the surface is where
// the trilinear raw field crosses an isovalue, shaded as a Lambertian
// reflector with the LUT colour at the isovalue.
//
// Path (per sample, up to max_bounces vertices):
//   - first crossing along the segment inside the box: the field minus the
//     isovalue is sampled every half voxel from the segment start, the first
//     pair of samples with different signs is bisected, and the bracket end
//     on the incoming side is the vertex (a path always continues on the
//     side it came from);
//   - normal: central differences of the field over a quarter voxel, turned
//     to face the incoming ray;
//   - next-event estimation: one light sample (vertex stream, pair 0) with a
//     visibility march towards it, BRDF rho / pi;
//   - bounce: cosine-weighted about the normal (pair 1), throughput * rho;
//   - a segment with no crossing adds the environment.
// Samples inside a majorant-grid cell whose raw range excludes the isovalue
// have a known sign and are not fetched: the cell range covers every point
// of the cell plus a voxel, so the march finds the same crossing as a march
// that fetches every sample.
//
// A work item is a ray (light-field ray or view pixel) with its samples in
// order, so the texel sum is deterministic; the last rays of the queue are
// split into items of a sample or two, kept and summed in order afterwards
// (the work queue is the volume tracer's).  Paths differ in length and marches
// in steps, and with one ray per lane and nested loops an eighth of the lanes
// were active; so every lane runs its own state machine
//     IDLE -> INIT -> MARCH -> HIT -> INIT (shadow) -> MARCH -> INIT ... -> DONE -> IDLE
// in a persistent grid: the march advances all marching lanes by one step
// while enough of the wave marches, and what interrupts it (sample ends,
// refills, segment set-up, bisection and shading) runs for all waiting lanes
// together.
#include <algorithm>

#include "internal.hpp"

namespace lp {

struct SurfCtx {
    const TraceParams& P;
    const float2* rng;      // LDS: raw [lo, hi] per grid cell
    const uint32_t* blocks; // LDS: two bits per block (kAbove, kBelow or neither)
    float iso, h;
};

enum : uint32_t { kMixed = 0, kAbove = 1, kBelow = 2 };
// Voxels from here on count as not finite (the differences that interpolation
// forms of smaller ones are finite).
constexpr float kLargeVoxel = 1.7e38f;
// Kind of a block whose voxels lie in [lo, hi].
__device__ __forceinline__ uint32_t block_kind(float lo, float hi, bool finite, float iso) {
    const float gap = 1e-5f * (fmaxf(fabsf(lo), fabsf(hi)) + fabsf(iso));
    return !finite ? kMixed : lo - iso > gap ? kAbove : iso - hi > gap ? kBelow : kMixed;
}

template <int VT>
__device__ __forceinline__ float field(const SurfCtx& S, f3 y) {
    return sample_volume<VT>(S.P, y) - S.iso;
}

// Raw range of the majorant-grid cell that holds y.
__device__ __forceinline__ float2 cell_range(const SurfCtx& S, f3 y) {
    const TraceParams& P = S.P;
    const int G = P.grid_n, Gm = G - 1;
    const int cx = min(max((int)floorf((y.x - P.bmin[0]) * P.gcell[0]), 0), Gm);
    const int cy = min(max((int)floorf((y.y - P.bmin[1]) * P.gcell[1]), 0), Gm);
    const int cz = min(max((int)floorf((y.z - P.bmin[2]) * P.gcell[2]), 0), Gm);
    return S.rng[(cz * G + cy) * G + cx];
}

// Sign of field - iso at y: from the cell range when it excludes the
// isovalue, else fetched.  Returns true for "non-negative".
template <int VT>
__device__ __forceinline__ bool field_sign(const SurfCtx& S, f3 y) {
    const float2 r = cell_range(S, y);
    if (S.iso < r.x) return true;
    if (S.iso > r.y) return false;
    return field<VT>(S, y) >= 0.0f;
}

// The trilinear value with its eight voxels kept: a bisection shrinks into
// one footprint after a few steps, and most of its steps then load nothing.
// The arithmetic is sample_volume's.
template <int VT>
struct Footprint {
    uint32_t base = 0xFFFFFFFFu;
    float v000, v100, v010, v110, v001, v101, v011, v111;
    __device__ __forceinline__ float at(const TraceParams& P, f3 y) {
        const VoxelPoint p = voxel_point(P, y);
        if (p.base != base) {
            base = p.base;
            load_footprint<VT>(P, base, v000, v100, v010, v110, v001, v101, v011, v111);
        }
        return lerp_footprint(p, v000, v100, v010, v110, v001, v101, v011, v111);
    }
};

// The march along x + t d over [t0, t1] (the definition: samples at t0 + m h,
// the last one at t1, up to the first whose sign differs from the start's).
//
// Its length bounds it (up to 900 half-voxel samples a segment, each at least
// a cell test and mostly a fetch with its latency).  So inside a block of known
// sign equal to the current one the march goes on at the first sample past
// the block's exit, which skips only samples of that sign: the block's
// voxels, and one more on each side, are clear of the isovalue by more than
// the rounding of positions and interpolation.  (In mixed blocks one sample a
// step: fetching two or four together took 16 and 36 % longer, their waves
// being kept busy by the other lanes' steps.)  256^3 u16 phantom, N = 1024, 16
// spp: 45 ms as nested loops of one ray per lane, 18.6 with the blocks and
// without bisecting visibility rays, 5.7 as a state machine (an eighth of the
// lanes were active before it).
enum class Step { kOn, kMiss, kCross };
template <int VT>
__device__ __forceinline__ Step march_step(const SurfCtx& S, f3 x, f3 d, float t0, float t1, bool sa, int& m) {
    const TraceParams& P = S.P;
    float tb = fmaf((float)m, S.h, t0);
    if (tb > t1) tb = t1;
    // the sample's block: grid coordinates in blocks, o + t s
    const f3 ib = mk3(P.inv_block[0], P.inv_block[1], P.inv_block[2]);
    const f3 o = mk3(fmaf(x.x, P.ga[0], P.gb[0]), fmaf(x.y, P.ga[1], P.gb[1]), fmaf(x.z, P.ga[2], P.gb[2])) * ib;
    const f3 v = d * mk3(P.ga[0], P.ga[1], P.ga[2]) * ib;
    const int nx = P.blocks_n[0], ny = P.blocks_n[1], nz = P.blocks_n[2];
    const float bx = floorf(__builtin_amdgcn_fmed3f(fmaf(v.x, tb, o.x), 0.0f, (float)nx - 0.5f));
    const float by = floorf(__builtin_amdgcn_fmed3f(fmaf(v.y, tb, o.y), 0.0f, (float)ny - 0.5f));
    const float bz = floorf(__builtin_amdgcn_fmed3f(fmaf(v.z, tb, o.z), 0.0f, (float)nz - 0.5f));
    const int e = ((int)bz * ny + (int)by) * nx + (int)bx;
    const uint32_t kind = (S.blocks[e >> 4] >> (2 * (e & 15))) & 3u;
    if (kind == (sa ? kAbove : kBelow)) {
        // the block's exit (an axis the ray does not move along has none)
        const float ex = v.x != 0.0f ? (bx + (v.x > 0.0f ? 1.0f : 0.0f) - o.x) * rcp(v.x) : 3.402823466e38f;
        const float ey = v.y != 0.0f ? (by + (v.y > 0.0f ? 1.0f : 0.0f) - o.y) * rcp(v.y) : 3.402823466e38f;
        const float ez = v.z != 0.0f ? (bz + (v.z > 0.0f ? 1.0f : 0.0f) - o.z) * rcp(v.z) : 3.402823466e38f;
        const float te = fminf(fminf(ex, ey), ez);
        if (tb >= t1 || te >= t1) return Step::kMiss;
        m = max(m + 1, (int)((te - t0) * rcp(S.h)) + 1);
        return Step::kOn;
    }
    if (field_sign<VT>(S, fma3(d, tb, x)) != sa) return Step::kCross;
    if (tb >= t1) return Step::kMiss;
    ++m;
    return Step::kOn;
}

// Incoming-side end of the crossing between samples m - 1 and m: 24 bisections.
template <int VT>
__device__ __forceinline__ float bisect(const SurfCtx& S, f3 x, f3 d, float t0, float t1, bool sa, int m) {
    float lo = m == 1 ? t0 : fmaf((float)(m - 1), S.h, t0), hi = fminf(fmaf((float)m, S.h, t0), t1);
    Footprint<VT> F;
    for (int it = 0; it < 24; ++it) {
        const float mid = 0.5f * (lo + hi);
        if ((F.at(S.P, fma3(d, mid, x)) - S.iso >= 0.0f) == sa) lo = mid;
        else hi = mid;
    }
    return lo;
}

template <int VT>
__device__ __forceinline__ f3 surface_normal(const SurfCtx& S, f3 y, f3 d) {
    const float e = 0.5f * S.h;
    const float gx = sample_volume<VT>(S.P, mk3(y.x + e, y.y, y.z)) - sample_volume<VT>(S.P, mk3(y.x - e, y.y, y.z));
    const float gy = sample_volume<VT>(S.P, mk3(y.x, y.y + e, y.z)) - sample_volume<VT>(S.P, mk3(y.x, y.y - e, y.z));
    const float gz = sample_volume<VT>(S.P, mk3(y.x, y.y, y.z + e)) - sample_volume<VT>(S.P, mk3(y.x, y.y, y.z - e));
    f3 n = mk3(gx, gy, gz);
    const float l2 = dot(n, n);
    if (!(l2 > 0.0f)) return d * -1.0f;
    n = n * rsq(l2);
    return dot(n, d) > 0.0f ? n * -1.0f : n;
}

enum : int { kSIdle = 0, kSInit = 1, kSInitShadow = 2, kSMarch = 3, kSMarchShadow = 4, kSHit = 5, kSDone = 6 };
// The march goes on while at least this many of 64 live lanes march (16 and
// 32: within 1 %; so are five and six waves per SIMD instead of four).
constexpr int kMarchLanes = 24;

template <int VT>
__global__ __launch_bounds__(256, 4) void surface_kernel(TraceParams P) {
    extern __shared__ float2 rng[];
    const int ncell = P.grid_n * P.grid_n * P.grid_n;
    const int nblock = (P.blocks_n[0] * P.blocks_n[1] * P.blocks_n[2] + 15) / 16;  // words
    uint32_t* blocks = (uint32_t*)(rng + ncell);
    for (int e = threadIdx.x; e < ncell; e += blockDim.x) rng[e] = ((const float2*)P.srange)[e];
    for (int e = threadIdx.x; e < nblock; e += blockDim.x) blocks[e] = P.sblocks[e];
    __syncthreads();
    const SurfCtx S{P, rng, blocks, P.iso, P.half_voxel};
    // albedo: the LUT colour at the isovalue's window position, clamped
    f3 rho;
    {
        const float sw = fminf(fmaxf((P.iso - P.vmin) * P.vscale, 0.0f), 1.0f);
        const float u = sw * P.lut_last;
        const int l0 = min((int)u, P.lut_n - 2);
        const float w = u - (float)l0;
        const float4 A = ((const float4*)P.lut_e)[l0], B = ((const float4*)P.lut_e)[l0 + 1];
        rho = mk3(fminf(fmaxf(fmaf(w, B.x - A.x, A.x), 0.0f), 1.0f), fminf(fmaxf(fmaf(w, B.y - A.y, A.y), 0.0f), 1.0f),
                  fminf(fmaxf(fmaf(w, B.z - A.z, A.z), 0.0f), 1.0f));
    }

    const int lane = threadIdx.x & 63;
    const uint32_t K0 = P.key0, K1 = P.key1;
    const f3 bmin = mk3(P.bmin[0], P.bmin[1], P.bmin[2]), bmax = mk3(P.bmax[0], P.bmax[1], P.bmax[2]);
    const f3 env = mk3(P.env[0], P.env[1], P.env[2]), O = mk3(P.O[0], P.O[1], P.O[2]);
    const int rows = P.row_end - P.row_begin;
    const int tiles_i = (rows + 7) / 8, tiles_j = (P.N + 7) / 8;
    const Queue Q(P.views ? (long long)P.nviews * P.vtiles : (long long)tiles_i * tiles_j, 0, P.fine_units, P.fine_log2);
    const int home = blockIdx.x % kParts;
    const int place = (int)(blockIdx.x / kParts) * 4 + (int)(threadIdx.x >> 6);
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    Tile tile = {0, 0, 0, 0, false};
    unsigned dry = 0;
    bool begun = false, drained = false;

    // lane state: the work item, then the path, then the march
    int mode = kSIdle, s = 0, s_end = 0, b = 0, part = 0, m = 0;
    uint32_t k = 0;
    bool fresh = false, sa = false;
    f3 po = mk3(0, 0, 0), d0 = po, acc = po, x = po, dir = po, T = po, L = po, om = po, C = po;
    float t0 = 0.0f, t1 = 0.0f, cw = 0.0f;  // cw, C: the light sample's contribution is cw C
    Counters cnt = {0, 0, 0, 0, 0};

    for (;;) {
        // ------------------------------------------------------ sample end
        if (mode == kSDone) {
            acc = acc + L;
            if (part < 0) {
                float* o = kept_sample(P, part & 0x7fffffff, s);
                o[0] = L.x;
                o[1] = L.y;
                o[2] = L.z;
            }
            if (++s == s_end) {
                if (part >= 0) {
                    const float fs = (float)P.spp;
                    store_texel(P.out, P.dtype, k, mk3(acc.x / fs, acc.y / fs, acc.z / fs));
                }
                mode = kSIdle;
            } else {
                mode = kSInit;
                fresh = true;
            }
        }

        // ---------------------------------------------------------- refill
        const uint64_t idle = __ballot(mode == kSIdle);
        if (idle) {
            const int nidle = __popcll(idle), rank = __popcll(idle & lt_mask);
            const long long avail = tile.end - tile.cur;
            Tile next;
            bool more = false;
            if (nidle > avail && !drained) {
                more = next_tile(P.tile_ctr, P.ctr_stride, Q, home, place, begun, dry, next);
                drained = !more;
            }
            long long q = -1, shift = tile.shift;
            bool fine = tile.fine;
            int lg = tile.log2;
            if (mode == kSIdle) {
                if (rank < avail) {
                    q = tile.cur + rank;
                } else if (more) {
                    q = next.cur + (rank - avail);
                    fine = next.fine;
                    lg = next.log2;
                    shift = next.shift;
                }
            }
            if (more) {
                tile = next;
                tile.cur += nidle - avail;
            } else {
                tile.cur += min((long long)nidle, avail);
            }
            if (q >= 0) {
                const long long slot = q >> lg;
                const int item = (int)q & ((1 << lg) - 1);
                s = item_sample(item, P.spp, lg);
                s_end = item_sample(item + 1, P.spp, lg);
                part = fine ? (int)(0x80000000u | (uint32_t)(slot + shift)) : 0;
                bool active = false;
                int skip = 0;  // environment samples at the item's start
                if (P.views) {
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
                        active = true;
                    }
                } else {
                    int ti, tj;
                    tile_coords(slot >> 6, tiles_i, tiles_j, ti, tj);
                    const int oi = ti * 8 + (int)((slot >> 3) & 7), dj = tj * 8 + (int)(slot & 7);
                    if (oi < rows && dj < P.N) {
                        const int i = P.perm_o[oi], j = P.perm_d[dj];
                        k = (uint32_t)i * (uint32_t)P.N + (uint32_t)j;
                        if (P.M == P.N && i == j) {
                            // no direction: texel 0 (of kept samples, the summing kernel writes it)
                            if (!fine) store_texel(P.out, P.dtype, k, mk3(0.0f, 0.0f, 0.0f));
                        } else {
                            po = sf_point(P.M, i, 1.0f / (float)P.M);
                            d0 = normalize(sf_point(P.N, j, 1.0f / (float)P.N) - po);
                            active = true;
                            // a ray that misses the box in every sample: the
                            // item's samples but the last are added here
                            if (misses_box(P, O, bmin, bmax, po, d0)) skip = s_end - 1 - s;
                        }
                    }
                }
                if (active) {
                    acc = mk3(0.0f, 0.0f, 0.0f);
                    for (; skip > 0; --skip, ++s) {
                        acc = acc + env;
                        cnt.samples++;
                        if (fine) {
                            float* o = kept_sample(P, part & 0x7fffffff, s);
                            o[0] = env.x;
                            o[1] = env.y;
                            o[2] = env.z;
                        }
                    }
                    mode = kSInit;
                    fresh = true;
                }
            }
        }
        const int live = __popcll(__ballot(mode != kSIdle));
        if (live == 0) {
            if (drained && tile.end <= tile.cur) break;
            continue;
        }

        // ------------------------------------------------- segment set-up
        if (mode == kSInit || mode == kSInitShadow) {
            if (fresh) {
                fresh = false;
                cnt.samples++;
                x = po;
                dir = d0;
                T = mk3(1.0f, 1.0f, 1.0f);
                L = mk3(0.0f, 0.0f, 0.0f);
                b = 0;
                if (!P.views) {
                    x = O + po * P.R;
                    if (P.jitter) {
                        const u4 rj = philox(k, (uint32_t)s, kPurFlight, 0u, K0, K1);
                        const float rr = P.jit_rad * sqrtf(u01(rj.x));
                        float sn, cs;
                        sincospif(2.0f * u01(rj.y), &sn, &cs);
                        f3 e1, e2;
                        frame(po, e1, e2);
                        x = x + (e1 * (rr * cs) + e2 * (rr * sn));
                    }
                }
            }
            const bool shadow = mode == kSInitShadow;
            const f3 d = shadow ? om : dir;
            float tn, tf;
            // a direction that is not a number (the normal beside an infinite
            // voxel) leaves the interval open, and the march without an end:
            // such a segment meets nothing
            const bool hit = clip_box(bmin, bmax, x, d, tn, tf) && tf < 3.402823466e38f;
            if (shadow) {  // t1 holds the light's distance (directional: infinity)
                tn = 0.0f;
                tf = hit ? fminf(t1, tf) : 0.0f;
            }
            if (shadow ? tf > 0.0f : hit) {
                t0 = tn;
                t1 = tf;
                m = 1;
                sa = field_sign<VT>(S, fma3(d, t0, x));
                mode = shadow ? kSMarchShadow : kSMarch;
            } else if (shadow) {  // nothing in the way
                L = fma3(C, cw, L);
                mode = kSHit;     // (the path goes on below)
                m = -1;
            } else {
                L = L + T * env;
                mode = kSDone;
            }
        }

        // ----------------------------------------------------------- march
        for (;;) {
            if (mode == kSMarch || mode == kSMarchShadow) {
                const bool shadow = mode == kSMarchShadow;
                const Step r = march_step<VT>(S, x, shadow ? om : dir, t0, t1, sa, m);
                if (r != Step::kOn) {
                    if (shadow) {
                        if (r == Step::kMiss) L = fma3(C, cw, L);
                        mode = kSHit;
                        m = -1;
                    } else if (r == Step::kCross) {
                        mode = kSHit;
                    } else {
                        L = L + T * env;
                        mode = kSDone;
                    }
                }
            }
            const int marching = __popcll(__ballot(mode == kSMarch || mode == kSMarchShadow));
            if (marching == 0 || marching * 64 < kMarchLanes * live) break;
        }

        // ------------------------------------------- vertex, and what follows it
        if (mode == kSHit) {
            if (m > 0) {
                // the vertex of a crossing: light sample, and the bounce's direction
                cnt.real++;
                const f3 y = fma3(dir, bisect<VT>(S, x, dir, t0, t1, sa, m), x);
                const f3 n = surface_normal<VT>(S, y, dir);
                const u4 r = philox(k, (uint32_t)s, ((uint32_t)b << 8) | kPurVertex, 0u, K0, K1);
                x = y;
                // cosine-weighted bounce about n
                const float u0 = u01(r.z), rr = sqrtf(u0);
                float sp, cp;
                sincospif(2.0f * u01(r.w), &sp, &cp);
                f3 b1, b2;
                frame(n, b1, b2);
                dir = normalize(b1 * (rr * cp) + b2 * (rr * sp) + n * sqrtf(fmaxf(0.0f, 1.0f - u0)));
                bool lit = false;
                if (P.light_on) {
                    f3 Le;
                    if (P.light_kind == 0) {
                        om = mk3(P.ldir[0], P.ldir[1], P.ldir[2]);
                        Le = mk3(P.lrad[0], P.lrad[1], P.lrad[2]);
                        t1 = 3.402823466e38f;
                    } else {
                        const f3 yl = mk3(P.lcorner[0], P.lcorner[1], P.lcorner[2]) +
                                      mk3(P.le1[0], P.le1[1], P.le1[2]) * u01(r.x) +
                                      mk3(P.le2[0], P.le2[1], P.le2[2]) * u01(r.y);
                        const f3 v = yl - y;
                        const float d2 = dot(v, v);
                        const float rinv = rsq(d2);
                        t1 = d2 * rinv;
                        om = v * rinv;
                        const float cl = fmaxf(0.0f, -dot(mk3(P.lnrm[0], P.lnrm[1], P.lnrm[2]), om));
                        Le = mk3(P.lrad[0], P.lrad[1], P.lrad[2]) * (cl * P.larea * rcp(d2));
                    }
                    const float cosl = fmaf(n.z, om.z, fmaf(n.x, om.x, n.y * om.y));
                    C = T * rho * Le;
                    cw = cosl * 0.318309886183790672f;
                    lit = cosl > 0.0f;
                }
                if (lit) mode = kSInitShadow;
                else m = -1;
            }
            if (m < 0) {
                // the light is accounted for: the last vertex, or the next segment
                mode = kSDone;
                if (b != P.maxb - 1) {
                    T = T * rho;
                    if (!(T.x == 0.0f && T.y == 0.0f && T.z == 0.0f)) {
                        ++b;
                        mode = kSInit;
                    }
                }
            }
        }
    }
    if (P.stats) {
        const uint32_t r = wave_sum(cnt.real), n = wave_sum(cnt.samples);
        if (lane == 0) {
            atomicAdd(&P.stats[2], (unsigned long long)r);
            atomicAdd(&P.stats[3], (unsigned long long)n);
        }
    }
}

// Kinds of the march's blocks, from the halo-brick copy: block (x, y, z) spans
// block_bricks bricks along each axis, and its kind covers one voxel more on
// each side (a march point is assigned to a block to within rounding).  kAbove /
// kBelow: every voxel is clear of the isovalue by more than the rounding of a
// trilinear value; a voxel that is not finite makes the block mixed.  A
// workgroup forms one byte: four blocks, a wave each.  It is the latency of a
// lane's loads one after the other, so four are in flight.  Against a wave for
// four blocks in turn, u8: 64^3 19.8 -> 6.3 us, 256^3 103 -> 102, 512^3 375 ->
// 354, 1024 x 1024 x 512 1.43 -> 1.02 ms; with a block length per axis besides,
// 2048 x 128 x 128 1.53 -> 0.11, 6000 x 500 x 100 27.1 -> 0.78 ms.  (Four waves a
// block: 256^3 236 us, 6000 x 500 x 100 0.75 ms.)
template <int VT>
__global__ __launch_bounds__(256) void surface_blocks_kernel(TraceParams P, uint8_t* out) {
    __shared__ uint32_t kinds[4];
    const int nx = P.blocks_n[0], ny = P.blocks_n[1], total = nx * ny * P.blocks_n[2];
    const int wave = (int)threadIdx.x >> 6, lane = threadIdx.x & 63, e = (int)blockIdx.x * 4 + wave;
    float vlo = 3.402823466e38f, vhi = -3.402823466e38f;
    bool finite = true;
    if (e < total) {
        const int b[3] = {e % nx, e / nx % ny, e / (nx * ny)}, n[3] = {P.nx, P.ny, P.nz};
        int lo[3], cnt[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int span = 3 * P.block_bricks[a];
            lo[a] = max(span * b[a] - 1, 0);
            cnt[a] = min(span * (b[a] + 1) + 1, n[a] - 1) - lo[a] + 1;
        }
        // a lane takes every 64th voxel, x-fastest: the place of the next one is
        // a sum with carries.  Past the end they are voxels of the last layer
        // once more.
        const int plane = cnt[0] * cnt[1];
        const int step[3] = {64 % plane % cnt[0], 64 % plane / cnt[0], 64 / plane};
        int p[3] = {lane % plane % cnt[0], lane % plane / cnt[0], lane / plane};
        while (p[2] < cnt[2]) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = voxel_at<VT>(P, lo[0] + p[0], lo[1] + p[1], lo[2] + min(p[2], cnt[2] - 1));
                p[0] += step[0];
                const bool cx = p[0] >= cnt[0];
                p[0] -= cx ? cnt[0] : 0;
                p[1] += step[1] + (cx ? 1 : 0);
                const bool cy = p[1] >= cnt[1];
                p[1] -= cy ? cnt[1] : 0;
                p[2] += step[2] + (cy ? 1 : 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                finite = finite && fabsf(v[i]) < kLargeVoxel;
                vlo = fminf(vlo, v[i]);
                vhi = fmaxf(vhi, v[i]);
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        vlo = fminf(vlo, __shfl_xor(vlo, o, 64));
        vhi = fmaxf(vhi, __shfl_xor(vhi, o, 64));
    }
    const bool all_finite = __ballot(!finite) == 0;
    if (lane == 0) kinds[wave] = e < total ? block_kind(vlo, vhi, all_finite, P.iso) : kMixed;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = (uint8_t)(kinds[0] | kinds[1] << 2 | kinds[2] << 4 | kinds[3] << 6);
}

hipError_t launch_surface_blocks(const TraceParams& P, int vtype, uint32_t* out, hipStream_t s) {
    const unsigned bytes = 4 * (unsigned)((P.blocks_n[0] * P.blocks_n[1] * P.blocks_n[2] + 15) / 16);
    if (vtype == 0) surface_blocks_kernel<0><<<bytes, 256, 0, s>>>(P, (uint8_t*)out);
    else if (vtype == 1) surface_blocks_kernel<1><<<bytes, 256, 0, s>>>(P, (uint8_t*)out);
    else surface_blocks_kernel<2><<<bytes, 256, 0, s>>>(P, (uint8_t*)out);
    return hipGetLastError();
}

template <int VT>
static hipError_t launch_surface_t(const TraceParams& P, hipStream_t s) {
    const long long rows = P.row_end - P.row_begin;
    const Queue Q(P.views ? (long long)P.nviews * P.vtiles : ((rows + 7) / 8) * (long long)((P.N + 7) / 8), 0,
                  P.fine_units, P.fine_log2);
    long long ntiles = 0;
    for (int p = 0; p < kParts; ++p) ntiles += Q.tiles(p);
    if (ntiles <= 0) return hipSuccess;
    const size_t lds = sizeof(float2) * (size_t)P.grid_n * P.grid_n * P.grid_n +
                       4 * (((size_t)P.blocks_n[0] * P.blocks_n[1] * P.blocks_n[2] + 15) / 16);
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, surface_kernel<VT>, 256, lds);
    if (e != hipSuccess) return e;
    const long long blocks = std::min((long long)cus * std::max(per_cu, 1), (ntiles + 3) / 4);
    surface_kernel<VT><<<(unsigned)blocks, 256, lds, s>>>(P);
    return hipGetLastError();
}

hipError_t launch_surface(const TraceParams& P, int vtype, hipStream_t s) {
    switch (vtype) {
        case 0: return launch_surface_t<0>(P, s);
        case 1: return launch_surface_t<1>(P, s);
        default: return launch_surface_t<2>(P, s);
    }
}

}  // namespace lp
