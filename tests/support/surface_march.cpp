// Host build of the isosurface march and the halo-brick indexing.
//
// "march": reads a scene from stdin (nx ny nz type iso bx by bz rays seed, then
// the voxels as floats), marches rays through it twice, stepping over blocks of
// known sign and cell ranges, and fetching every sample, and prints the rays
// that hit the box, the crossings, the rays on which the two differ in outcome
// or crossing sample, and the steps of either.
// "index": reads "nx ny nz" lines and prints, for each, the points whose
// footprint voxel_point places elsewhere than 64-bit arithmetic does.
#include "host_device.hpp"

#include "../../paper_1903_03837_amd/csrc/api.cpp"
#include "../../paper_1903_03837_amd/csrc/surface.hip"

#include <cstdio>
#include <random>

namespace {

lf_volume volume(const int n[3], int type, const float box[3]) {
    lf_volume v = {};
    v.data = nullptr;
    v.type = type;
    v.nx = n[0], v.ny = n[1], v.nz = n[2];
    v.vmin = 0.0f, v.vmax = 4095.0f;
    for (int a = 0; a < 3; ++a) v.box_min[a] = -box[a], v.box_max[a] = box[a];
    return v;
}

lp::TraceParams params(const lf_volume& v, float iso, int cells) {
    lf_medium m = {};
    m.lut_size = 2;
    lf_light l = {};
    lf_gen_params p = {};
    p.M = p.N = 8;
    p.radius = 1.0f;
    p.spp = p.max_bounces = 1;
    p.surface = 1;
    p.iso = iso;
    p.majorant_grid = cells;
    lp::TraceParams T;
    pack_trace(T, &v, &m, nullptr, &l, &p);
    set_surface_blocks(T, &v);
    return T;
}

template <int VT, class E>
void march(const int n[3], float iso, const float box[3], int rays, unsigned seed, const std::vector<float>& vox) {
    const int G = 5;
    const lf_volume v = volume(n, VT, box);
    lp::TraceParams P = params(v, iso, G);
    auto at = [&](int x, int y, int z) {
        return vox[((size_t)std::min(z, n[2] - 1) * n[1] + std::min(y, n[1] - 1)) * n[0] + std::min(x, n[0] - 1)];
    };
    // the halo-brick copy
    std::vector<E> copy(brick_voxels(&v));
    const int nbz = lp::halo_bricks(n[2]);
    for (int bz = 0; bz < nbz; ++bz)
        for (int by = 0; by < P.nby; ++by)
            for (int bx = 0; bx < P.nbx; ++bx)
                for (int i = 0; i < 64; ++i)
                    copy[(((size_t)bz * P.nby + by) * P.nbx + bx) * 64 + i] =
                        (E)at(3 * bx + i % 4, 3 * by + i / 4 % 4, 3 * bz + i / 16);
    P.vol = copy.data();
    auto range = [&](const int lo[3], const int hi[3], float& a, float& b, bool& finite) {
        a = 3.4e38f, b = -3.4e38f, finite = true;
        for (int z = std::max(lo[2], 0); z <= std::min(hi[2], n[2] - 1); ++z)
            for (int y = std::max(lo[1], 0); y <= std::min(hi[1], n[1] - 1); ++y)
                for (int x = std::max(lo[0], 0); x <= std::min(hi[0], n[0] - 1); ++x) {
                    const float f = at(x, y, z);
                    finite = finite && fabsf(f) < lp::kLargeVoxel;
                    a = fminf(a, f);
                    b = fmaxf(b, f);
                }
    };
    // kinds of the blocks (one voxel more on each side) and ranges of the cells
    const int nb = P.blocks_n[0] * P.blocks_n[1] * P.blocks_n[2];
    std::vector<uint32_t> kinds(nb / 16 + 1, 0), mixed(nb / 16 + 1, 0);
    for (int e = 0; e < nb; ++e) {
        const int b[3] = {e % P.blocks_n[0], e / P.blocks_n[0] % P.blocks_n[1], e / (P.blocks_n[0] * P.blocks_n[1])};
        int lo[3], hi[3];
        for (int a = 0; a < 3; ++a) {
            const int span = 3 * P.block_bricks[a];
            lo[a] = span * b[a] - 1;
            hi[a] = span * (b[a] + 1) + 1;
        }
        float a, c;
        bool finite;
        range(lo, hi, a, c, finite);
        kinds[e >> 4] |= lp::block_kind(a, c, finite, iso) << (2 * (e & 15));
    }
    std::vector<float2> cells, all;
    for (int e = 0; e < G * G * G; ++e) {
        const int c[3] = {e % G, e / G % G, e / (G * G)};
        int lo[3], hi[3];
        for (int a = 0; a < 3; ++a) {
            lo[a] = (int)std::floor((double)c[a] * n[a] / G - 0.5) - 1;
            hi[a] = (int)std::floor((double)(c[a] + 1) * n[a] / G - 0.5) + 2;
        }
        float a, b;
        bool finite;
        range(lo, hi, a, b, finite);
        cells.push_back(finite ? make_float2(a, b) : make_float2(-INFINITY, INFINITY));
        all.push_back(make_float2(-INFINITY, INFINITY));
    }
    for (int a = 0; a < 3; ++a) {
        const double ext = (double)v.box_max[a] - (double)v.box_min[a];
        P.gcell[a] = (float)(G / ext);
    }
    P.grid_n = G;
    const lp::SurfCtx skip{P, cells.data(), kinds.data(), iso, P.half_voxel}, full{P, all.data(), mixed.data(), iso, P.half_voxel};

    std::mt19937 rng(seed);
    std::uniform_real_distribution<float> U(-1.0f, 1.0f);
    long long met = 0, crossings = 0, differ = 0, steps[2] = {0, 0};
    for (int r = 0; r < rays; ++r) {
        // origins outside and inside the box, every third on a voxel plane or a
        // block border; directions any, every fourth along an axis or nearly so
        lp::f3 x = {U(rng), U(rng), U(rng)}, d = {U(rng), U(rng), U(rng)};
        const float reach = r % 2 ? 1.0f : 3.0f;
        x = {x.x * box[0] * reach, x.y * box[1] * reach, x.z * box[2] * reach};
        if (r % 2 == 0) d = lp::f3{U(rng) * box[0], U(rng) * box[1], U(rng) * box[2]} - x;
        if (r % 3 == 0) {
            const int a = r / 3 % 3, i = (int)((U(rng) + 1.0f) * 0.5f * n[a]);
            const float g = r % 2 ? (float)i : (float)(i / (3 * P.block_bricks[a]) * (3 * P.block_bricks[a]));
            (&x.x)[a] = (g - P.gb[a]) / P.ga[a];
        }
        if (r % 4 == 0) {
            (&d.x)[r / 4 % 3] = r % 8 ? 0.0f : 1e-7f * U(rng);
            (&d.x)[r / 12 % 3] = r % 8 ? 0.0f : 1e-7f * U(rng);
        }
        d = lp::normalize(d);
        float tn, tf;
        const lp::f3 lo = {P.bmin[0], P.bmin[1], P.bmin[2]}, hi = {P.bmax[0], P.bmax[1], P.bmax[2]};
        if (!lp::clip_box(lo, hi, x, d, tn, tf) || !(tf < 3.4e38f)) continue;
        if (r % 5 == 0) tf = tn + (tf - tn) * 0.7f;  // (a light in the box)
        ++met;
        lp::Step out[2];
        int m[2];
        for (int k = 0; k < 2; ++k) {
            const lp::SurfCtx& S = k ? full : skip;
            const bool sa = lp::field_sign<VT>(S, lp::fma3(d, tn, x));
            m[k] = 1;
            do {
                out[k] = lp::march_step<VT>(S, x, d, tn, tf, sa, m[k]);
                ++steps[k];
            } while (out[k] == lp::Step::kOn);
        }
        crossings += out[1] == lp::Step::kCross;
        differ += out[0] != out[1] || (out[0] == lp::Step::kCross && m[0] != m[1]);
    }
    std::printf("%lld %lld %lld %lld %lld\n", met, crossings, differ, steps[0], steps[1]);
}

void index_check(const int n[3]) {
    const float box[3] = {1.0f, 1.0f, 1.0f};
    const lf_volume v = volume(n, 0, box);
    const lp::TraceParams P = params(v, 0.0f, 1);
    std::mt19937 rng(7);
    long long bad = 0;
    for (int r = 0; r < 200000; ++r) {
        int i[3];
        lp::f3 y;
        for (int a = 0; a < 3; ++a) {
            // any voxel, or one of the first or last four
            const unsigned u = rng();
            i[a] = u % 3 == 0 ? (int)(rng() % 4) : u % 3 == 1 ? n[a] - 1 - (int)(rng() % 4) : (int)(rng() % (unsigned)n[a]);
            i[a] = std::min(std::max(i[a], 0), n[a] - 1);
            (&y.x)[a] = ((float)i[a] + 0.5f - P.gb[a]) / P.ga[a];  // the middle of its footprint
        }
        const lp::VoxelPoint p = lp::voxel_point(P, y);
        // the footprint that the rounded position lies in
        unsigned long long b[3], l[3];
        for (int a = 0; a < 3; ++a) {
            const float g = std::min(std::max(fmaf((&y.x)[a], P.ga[a], P.gb[a]), 0.0f), (float)(n[a] - 1));
            const int base = std::min((int)g, n[a] - 2);
            b[a] = (unsigned)base / 3;
            l[a] = (unsigned)base % 3;
        }
        const unsigned long long want =
            64 * ((b[2] * (unsigned long long)P.nby + b[1]) * (unsigned long long)P.nbx + b[0]) + 16 * l[2] + 4 * l[1] + l[0];
        bad += want != p.base;
    }
    std::printf("%lld %llu\n", bad, (unsigned long long)brick_voxels(&v));
}

}  // namespace

int main(int argc, char** argv) {
    if (argc == 2 && std::string(argv[1]) == "index") {
        int n[3];
        while (std::scanf("%d %d %d", n, n + 1, n + 2) == 3) index_check(n);
        return 0;
    }
    int n[3], type, rays;
    unsigned seed;
    float iso, box[3];
    if (std::scanf("%d %d %d %d %f %f %f %f %d %u", n, n + 1, n + 2, &type, &iso, box, box + 1, box + 2, &rays, &seed) != 10)
        return 1;
    std::getchar();
    std::vector<float> vox((size_t)n[0] * n[1] * n[2]);
    if (std::fread(vox.data(), 4, vox.size(), stdin) != vox.size()) return 1;
    if (type == 1) march<1, uint16_t>(n, iso, box, rays, seed, vox);
    else march<2, float>(n, iso, box, rays, seed, vox);
    return 0;
}
