// Per-tile visibility resolve: ray-cast every pixel of a tile against the
// primitives binned to it and keep the nearest hit (paper, Methods,
// "Meshless Representations": ray-casting evaluates the implicit equation of
// each primitive, which makes the display pixel-exact).
//
// One workgroup owns one tile.  The tile's list holds 8-byte entries (source
// index, footprint clipped to the tile); each chunk of 256 entries is turned
// back into view-space records from the sources and staged in LDS.  The
// records' footprint pixel counts are prefix-summed and the resulting
// (record, pixel) fragments are dealt to the 256 lanes round-robin, so the
// load is balanced whatever the mix of tiny and large primitives, and lanes of
// one wave work on neighbouring pixels of the same few records.  A hit is
// folded into the tile's depth buffer in LDS with one 64-bit atomicMin of the
// packed key (float bits of z) << 32 | id: positive floats order like their
// bit patterns, so the minimum key is the nearest hit and equal depths go to
// the smaller id, in any order of evaluation.
//
// Depth early-outs, all conservative (statistics frames switch them off):
// a record whose nearest possible depth lies behind everything the 4x4-pixel
// blocks under its footprint hold is dropped; a fragment whose pixel holds a
// nearer hit is skipped; chunks of large footprints run front to back, each
// 8x8-pixel block on its own, without the records behind everything the block
// holds; a resident scene's list, ordered front to back by layers, ends
// once every layer left lies behind the whole tile.
#include "prims.h"

namespace vtx {

namespace {

constexpr int kChunk = kBlock;
constexpr int kBuckets = 64;      // depth buckets of the front-to-back record order
static_assert(kBuckets == 64, "a wave scans the buckets, one per lane");
// A chunk is ordered and resolved by blocks (resolve_blocks) when its kept
// records average more than kSortArea pixels and cover the tile more than
// kSortDepth times: a block's wave spends a pass of 64 lanes on a record
// however few of its pixels the footprint has, which pays only where the
// order hides records behind it.  kSortArea 20 to 40 measure the same on
// spheres (4,096 at 256x256, 16-pixel tiles: 9.9 us of resolve; 64: 22); on
// bonds small areas lose (in image order, 107,500 atoms with bonds at 1080p:
// 58 us with 32, 69 to 79 with 16; 1M dust with bonds: 96 with 32, 103 with 16, 153 with 8).
// kSortDepth 2, 4, 8: 191, 192, 207 us on 11M spheres at 4K.
constexpr int kSortArea = 32;
constexpr int kSortDepth = 2;
constexpr int kKeptShift = 21;    // packed scan: footprint area (<= 256 * 64 * 64) below, kept count above
constexpr uint32_t kAreaMask = (1u << kKeptShift) - 1u;
static_assert(kBlock == kChunk, "one 64-slot window per wave in the order array");
template <int TS>
struct HzGrid {
    static constexpr int kBlocks = (TS / 4) * (TS / 4);
};

struct Rec {
    float4 a;          // sphere: centre (view), radius | cylinder: A (view), radius
    float4 b;          // cylinder: unit axis (view), length
    float zcull;       // lower bound of the depth of any hit of this record
    uint32_t id;
    uint32_t rect;     // tile-local x0 | y0 << 8 | w << 16 | h << 24
    float inv_w;       // 1 / w (hardware reciprocal): splits a footprint offset into row and column
};

// Inclusive max-scan over the 64 lanes of a wave by DPP row shifts and row
// broadcasts (lanes shifted in from outside a row read 0, the identity).
__device__ inline uint32_t wave_incl_max(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return v;
}

// Inclusive sum-scan over the 64 lanes of a wave, the same DPP steps.
__device__ inline uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

// Sphere: front root of |o + t D - c| = r with D = (Dx, Dy, 1), so t is the
// view depth.  Stable form: b = (c-o).D / D.D, q = (c-o) - b D,
// t = b - sqrt((r^2 - q.q) / D.D).
// The hardware reciprocal and square root (<= 1 ulp) are used throughout:
// their error is a few parts in 1e7 of the distance, far inside the 1e-5
// depth tolerance and the grazing band the oracle allows.
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// graze: the hit's n.V (the half chord sqrt(disc) over r) is below
// kGrazeCos, or the sphere is large against its depth (r > z / 4): where the
// FP32 root may miss the depth tolerance (see kGrazeCos).
__device__ inline float hit_sphere(const float4 s, float ox, float oy, float Dx, float Dy, bool& graze) {
    const float cx = s.x - ox, cy = s.y - oy, cz = s.z;
    const float inv_dd = fast_rcp(fmaf(Dx, Dx, fmaf(Dy, Dy, 1.0f)));
    const float b = fmaf(cx, Dx, fmaf(cy, Dy, cz)) * inv_dd;
    const float qx = fmaf(-b, Dx, cx), qy = fmaf(-b, Dy, cy), qz = cz - b;
    const float disc = fmaf(s.w, s.w, -fmaf(qx, qx, fmaf(qy, qy, qz * qz)));
    if (disc < 0.0f) return INFINITY;
    const float t = b - fast_sqrt(disc * inv_dd);
    graze = disc < kGrazeCos * kGrazeCos * (s.w * s.w) || 4.0f * s.w > t;
    return t;
}

// Closed cylinder of radius rho from A along unit axis a for length L: the
// entry point is the lateral front root with 0 <= s <= L, or the plane hit of
// the cap the ray enters through (cap A when D.a > 0, cap B when D.a < 0) if
// it lies within rho of the axis.
__device__ inline float hit_cylinder(const float4 ca, const float4 cb, float ox, float oy, float Dx,
                                     float Dy) {
    const float wx = ox - ca.x, wy = oy - ca.y, wz = -ca.z;
    const float rho2 = ca.w * ca.w;
    const float da = fmaf(Dx, cb.x, fmaf(Dy, cb.y, cb.z));
    const float wa = fmaf(wx, cb.x, fmaf(wy, cb.y, wz * cb.z));
    const float px = fmaf(-da, cb.x, Dx), py = fmaf(-da, cb.y, Dy), pz = fmaf(-da, cb.z, 1.0f);
    const float qx = fmaf(-wa, cb.x, wx), qy = fmaf(-wa, cb.y, wy), qz = fmaf(-wa, cb.z, wz);
    const float k = fmaf(px, px, fmaf(py, py, pz * pz));
    float t = INFINITY;
    if (k > 0.0f) {
        const float inv_k = fast_rcp(k);
        const float tc = -fmaf(qx, px, fmaf(qy, py, qz * pz)) * inv_k;
        const float rx = fmaf(tc, px, qx), ry = fmaf(tc, py, qy), rz = fmaf(tc, pz, qz);
        const float disc = rho2 - fmaf(rx, rx, fmaf(ry, ry, rz * rz));
        if (disc >= 0.0f) {
            const float ts = tc - fast_sqrt(disc * inv_k);
            const float s = fmaf(ts, da, wa);
            if (s >= 0.0f && s <= cb.w) t = ts;
        }
    }
    if (da != 0.0f) {
        const float tp = (da > 0.0f ? -wa : cb.w - wa) * fast_rcp(da);
        const float off = da > 0.0f ? 0.0f : cb.w;
        const float ex = fmaf(tp, Dx, wx) - off * cb.x;
        const float ey = fmaf(tp, Dy, wy) - off * cb.y;
        const float ez = (tp + wz) - off * cb.z;
        if (fmaf(ex, ex, fmaf(ey, ey, ez * ez)) <= rho2) t = fminf(t, tp);
    }
    return t;
}

// Depth of primitive `id` at pixel (px, py), recomputed in FP64 from the
// caller's FP32 inputs.  The FP32 ray test decides which primitive a pixel
// shows; its depth is only good to a few ulps of the distance divided by n.V,
// so towards a silhouette it drifts past any fixed relative tolerance (at
// n.V = 0.01 about 1e-5 of the depth).  The FP64 root loses the same digits
// relative to 2^-53, and rounding it once gives the depth to half an FP32 ulp
// wherever the hit is not within ~1e-7 of grazing.  Where FP64 finds no
// entry (an FP32 hit at the silhouette that FP64 places just outside), the
// depth is the surface's closest approach to the ray: the front root with
// the discriminant taken as zero, or the cap plane's crossing, whichever is
// nearest the FP32 depth.
__device__ inline float refine_depth_at(const Frame& F, const global_t<const float>* __restrict__ pos,
                                       const global_t<const float>* __restrict__ rad,
                                       const global_t<const uint32_t>* __restrict__ bonds, uint32_t id, int px, int py,
                                       float z32) {
    const double ndx = fma((double)px + 0.5, F.inv_w2d, -1.0);
    const double ndy = fma(-((double)py + 0.5), F.inv_h2d, 1.0);
    // ray o + t D with D.z = 1, so t is the view depth
    double ox = 0.0, oy = 0.0, Dx = 0.0, Dy = 0.0;
    if (F.proj == 0) {
        Dx = ndx * F.tx;
        Dy = ndy * F.ty;
    } else {
        ox = ndx * F.hx;
        oy = ndy * F.hy;
    }
    const double dd = fma(Dx, Dx, fma(Dy, Dy, 1.0)), idd = 1.0 / dd;
    double t = (double)z32;
    if (id < F.n_atoms) {
        const size_t i = id;
        double cx, cy, cz;
        to_view(F, pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], cx, cy, cz);
        const double r = (double)atom_radius(F, rad[i]);
        cx -= ox;
        cy -= oy;
        const double b = fma(cx, Dx, fma(cy, Dy, cz)) * idd;
        const double qx = fma(-b, Dx, cx), qy = fma(-b, Dy, cy), qz = cz - b;
        const double disc = fma(r, r, -fma(qx, qx, fma(qy, qy, qz * qz)));
        t = b - sqrt(fmax(disc, 0.0) * idd);
    } else {
        const size_t bi = id - F.n_atoms;
        const uint32_t ia = bonds[2 * bi], ib = bonds[2 * bi + 1];
        double A[3], B[3];
        to_view(F, pos[3 * (size_t)ia], pos[3 * (size_t)ia + 1], pos[3 * (size_t)ia + 2], A[0], A[1], A[2]);
        to_view(F, pos[3 * (size_t)ib], pos[3 * (size_t)ib + 1], pos[3 * (size_t)ib + 2], B[0], B[1], B[2]);
        const double rho = (double)F.bond_radius;
        double ax = B[0] - A[0], ay = B[1] - A[1], az = B[2] - A[2];
        const double L = sqrt(fma(ax, ax, fma(ay, ay, az * az)));
        ax /= L;
        ay /= L;
        az /= L;
        const double wx = ox - A[0], wy = oy - A[1], wz = -A[2];
        const double da = fma(Dx, ax, fma(Dy, ay, az)), wa = fma(wx, ax, fma(wy, ay, wz * az));
        const double px_ = fma(-da, ax, Dx), py_ = fma(-da, ay, Dy), pz_ = fma(-da, az, 1.0);
        const double qx = fma(-wa, ax, wx), qy = fma(-wa, ay, wy), qz = fma(-wa, az, wz);
        const double k = fma(px_, px_, fma(py_, py_, pz_ * pz_));
        double entry = INFINITY, near = INFINITY;
        auto consider = [&](double tt, bool valid) {
            if (valid) entry = fmin(entry, tt);
            if (fabs(tt - (double)z32) < fabs(near - (double)z32)) near = tt;
        };
        if (k > 0.0) {
            const double tc = -fma(qx, px_, fma(qy, py_, qz * pz_)) / k;
            const double rx = fma(tc, px_, qx), ry = fma(tc, py_, qy), rz = fma(tc, pz_, qz);
            const double disc = fma(rho, rho, -fma(rx, rx, fma(ry, ry, rz * rz)));
            const double ts = tc - sqrt(fmax(disc, 0.0) / k);
            const double s = fma(ts, da, wa);
            consider(ts, disc >= 0.0 && s >= 0.0 && s <= L);
        }
        if (da != 0.0) {
            const double cap[2] = {0.0, L};
            for (int c = 0; c < 2; ++c) {
                const double tp = (cap[c] - wa) / da;
                const double ex = fma(tp, Dx, wx) - cap[c] * ax, ey = fma(tp, Dy, wy) - cap[c] * ay,
                             ez = (tp + wz) - cap[c] * az;
                const bool front = c == 0 ? da > 0.0 : da < 0.0;
                consider(tp, front && fma(ex, ex, fma(ey, ey, ez * ez)) <= rho * rho);
            }
        }
        t = entry < INFINITY ? entry : near;
    }
    const float z = (float)t;
    return z > 0.0f && z < INFINITY ? z : z32;
}

// Expand a list record into the LDS form.
__device__ inline Rec make_rec(const Frame& F, const PrimRec& p) {
    Rec r;
    r.id = p.g1.z;
    r.rect = p.g1.w;
    r.inv_w = __builtin_amdgcn_rcpf((float)((r.rect >> 16) & 0xFF));
    if (r.id < F.n_atoms) {
        r.a = p.g0;
        r.b = make_float4(0.f, 0.f, 0.f, 0.f);
        r.zcull = (p.g0.z - p.g0.w) * (1.0f - 1e-5f);
    } else {
        const float dx = p.g0.w, dy = __uint_as_float(p.g1.x), dz = __uint_as_float(p.g1.y);
        const float L = fast_sqrt(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
        const float inv = fast_rcp(L);
        const float rho = F.bond_radius;
        r.a = make_float4(p.g0.x, p.g0.y, p.g0.z, rho);
        r.b = make_float4(dx * inv, dy * inv, dz * inv, L);
        r.zcull = (fminf(p.g0.z, p.g0.z + dz) - rho) * (1.0f - 1e-5f) - 1e-6f;
    }
    return r;
}

// View-space record of a visible primitive, rebuilt from its source (the
// tile lists hold only source indices and footprints).  The count pass has
// culled it already, so the frustum test is not repeated.
__device__ inline bool source_record(JobRef R, uint32_t src, PrimRec& pr) {
    double v[6], rr;
    const Frame F = R.frame();
    const SceneDev S = R.scene();
    const Item it = S.xyzr ? fetch_scene(S, src)
                           : fetch_plain(to_global(R.pos()), to_global(R.rad()), to_global(R.bonds()), F.n_atoms, src);
    return item_view<false>(F, it, pr, v, rr);
}

// Resolves tile t of job J, whose list holds n records from offset o
// (over: the list overflowed and the tile is rebuilt from every binning
// workgroup's visible list; the same for the whole workgroup).  Re-arms the tile's count and cursor for the next
// frame.  The workgroup's LDS holds the tile's depth buffer, one chunk of
// records and their prefix.  Two-pass frames: the front pass also stores the
// farthest depth of each 16x16 cell of the tile; the rest pass starts from the
// front pass's depth and id.
template <int TS, bool kCount, int kPhase>
__device__ __forceinline__ void resolve_tile(JobRef R, int t, uint32_t n, uint64_t o, bool over,
                                             unsigned long long* keys) {
    const JobRef R0 = R.again();
    const Frame F = R0.frame();
    const BinBuffers bb = R0.bins();
    constexpr int phase = kPhase;
    __shared__ Rec recs[kChunk];
    __shared__ uint32_t pref[kChunk + 1];
    __shared__ uint32_t wsum[kBlock / 64];
    constexpr int kHzBlocks = HzGrid<TS>::kBlocks;
    __shared__ uint32_t hz[kHzBlocks];
    __shared__ uint32_t red_lo[kBlock / 64], red_hi[kBlock / 64], bcnt[kBuckets];
    // resident scenes: list position where each layer starts, and the least
    // cull depth (float bits) of the layers from there on
    __shared__ uint32_t lay_start[kLayers], lay_zrest[kLayers];
    // depth-ordered chunk: record slots front to back.  Chunks resolved in
    // list order use it instead as 64 slots per wave, slot i holding j when
    // record j's first fragment is the i-th of the 64 the wave resolves
    // next, else 0 (all 0 between uses).
    __shared__ __align__(16) uint8_t ord[kChunk];

    // record slot j < kChunk, addressed with a 24-bit multiply (full rate)
    auto rec_at = [&](uint32_t j) -> const Rec& {
        return *reinterpret_cast<const Rec*>(reinterpret_cast<const char*>(recs) + __umul24(j, (uint32_t)sizeof(Rec)));
    };
    uint32_t* __restrict__ const cnt = bb.tile_cnt;
    const global_t<const uint2>* __restrict__ const list = to_global(bb.list);
    uint32_t* __restrict__ const fill = bb.tile_fill;
    Counters* const ctr = bb.ctr;
    global_t<float>* __restrict__ const depth = to_global(R0.depth());
    global_t<uint32_t>* __restrict__ const out_id = to_global(R0.id());

    const int tid = threadIdx.x, lane = __lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool stats = kCount && (F.flags & 1u) != 0;
    // counting frames (statistics, or VTX_FLAG_COUNT with the early-outs on):
    // ray tests and hits, and how often each early-out fired
    const bool counting = kCount && (F.flags & (1u | 16u)) != 0;
    unsigned long long n_tested = 0, n_hit = 0, n_hit_bond = 0, n_tested_bond = 0, n_skipped = 0, n_culled = 0;
    uint32_t n_list_stop = 0, n_chunk_stop = 0;

    {
        const int tx = t % F.tiles_x, ty = t / F.tiles_x;
        const int px0 = tx * TS, py0 = ty * TS;
        const int tw = min(TS, F.W - px0), th = min(TS, F.H - py0);
        for (int i = tid; i < TS * TS; i += kBlock) {
            unsigned long long k0 = ~0ull;
            const int ly = i / TS, lx = i - ly * TS;
            if (phase == kPhaseRest && lx < tw && ly < th) {
                const size_t p = (size_t)(py0 + ly) * F.W + (px0 + lx);
                const uint32_t id0 = out_id[p];
                if (id0 != kBackground) k0 = ((unsigned long long)__float_as_uint(depth[p]) << 32) | id0;
            }
            keys[i] = k0;
        }
        if (tid < kChunk / 4) reinterpret_cast<uint32_t*>(ord)[tid] = 0u;
        const uint64_t nsrc = over ? (uint64_t)bb.groups * bb.chunk : n;
        const bool persp = F.proj == 0;
        __syncthreads();
        // every wave has read the tile's count (it sets the trip count of the
        // barrier loop below): re-arm it for the next frame's count kernel
        if (tid == 0) cnt[t] = 0;
        if ((uint32_t)tid < bb.layers) fill[(size_t)tid * F.tiles_x * F.tiles_y + t] = 0;

        // one (record, pixel) ray test folded into the tile's LDS depth buffer
        auto test_pixel = [&](const Rec& rc, int lx, int ly) {
            const int slot = ly * TS + lx;
            if (!stats) {
                const unsigned long long cur = keys[slot];
                if (__uint_as_float((uint32_t)(cur >> 32)) < rc.zcull) {
                    if (counting) n_skipped += 1;
                    return;
                }
            }
            const float ndx = fmaf((float)(px0 + lx) + 0.5f, F.inv_w2, -1.0f);
            const float ndy = fmaf(-((float)(py0 + ly) + 0.5f), F.inv_h2, 1.0f);
            float ox, oy, Dx, Dy;
            if (persp) {
                ox = 0.f; oy = 0.f; Dx = ndx * F.txf; Dy = ndy * F.tyf;
            } else {
                ox = ndx * F.hxf; oy = ndy * F.hyf; Dx = 0.f; Dy = 0.f;
            }
            // cylinder hits are always refined; sphere hits only when grazing
            bool graze = true;
            const bool sphere = rc.id < F.n_atoms;   // ids past the atoms are bonds
            const float z = sphere ? hit_sphere(rc.a, ox, oy, Dx, Dy, graze)
                                         : hit_cylinder(rc.a, rc.b, ox, oy, Dx, Dy);
            bool hit = z >= F.znear && z <= F.zfar;
            // clip plane: the hit point (ox + z Dx, oy + z Dy, z) on the cut side draws nothing
            if (F.clip_on && hit)
                hit = fmaf(F.clip[0], fmaf(z, Dx, ox), fmaf(F.clip[1], fmaf(z, Dy, oy), fmaf(F.clip[2], z, F.clip[3]))) >= 0.0f;
            if (counting) {
                n_tested += 1;
                n_tested_bond += sphere ? 0 : 1;
                n_hit += hit ? 1 : 0;
                n_hit_bond += (hit && !sphere) ? 1 : 0;
            }
            if (hit)
                atomicMin(&keys[slot], ((unsigned long long)__float_as_uint(z) << 32) |
                                           (rc.id | (graze && F.refine_flag ? kRefineBit : 0u)));
        };
        // entry k of the visible lists (tiles whose list overflowed), as the
        // list entry it would have been
        auto fetch_overflow = [&](uint64_t k, uint2& e) -> bool {
            const BinBuffers vb = R.again().bins();
            const uint32_t g = (uint32_t)(k / vb.chunk);
            if ((uint32_t)(k - (uint64_t)g * vb.chunk) >= vb.vis_cnt[g]) return false;
            const uint2 gb = vb.vis_box[g];    // skip workgroups whose primitives cannot touch this tile
            if (tx < (int)(gb.x & 0xFFFF) || tx > (int)(gb.y & 0xFFFF) || ty < (int)(gb.x >> 16) ||
                ty > (int)(gb.y >> 16))
                return false;
            const uint2 r = vb.vis_rect[k];
            const int x0 = max((int)(r.x & 0xFFFF), px0) - px0, y0 = max((int)(r.x >> 16), py0) - py0;
            const int x1 = min((int)(r.y & 0xFFFF), px0 + TS - 1) - px0;
            const int y1 = min((int)(r.y >> 16), py0 + TS - 1) - py0;
            if (x0 > x1 || y0 > y1) return false;
            e.x = vb.vis_src[k];
            e.y = (uint32_t)x0 | ((uint32_t)y0 << 8) | ((uint32_t)(x1 - x0 + 1) << 16) |
                      ((uint32_t)(y1 - y0 + 1) << 24);
            return true;
        };

        // hz[b]: float bits of the farthest depth held by 4x4-pixel block b
        // (+inf while any of its pixels is empty).  It only decreases during
        // the frame, so a stale value is a safe bound.
        for (int i = tid; i < kHzBlocks; i += kBlock) hz[i] = 0x7F800000u;
        // The tile's list is staged 256 records at a time; the next chunk's
        // records are loaded while this chunk is resolved.
        // A list's next chunk is loaded while this one is resolved; the
        // overflow path loads each chunk when it starts.
        uint2 nxt = make_uint2(0u, 0u);
        bool nxt_ok = !over && (uint64_t)tid < nsrc;
        if (nxt_ok) nxt = list[o + tid];
        __syncthreads();
        // record cull against the block depths: its nearest possible depth
        // lies behind everything the 4x4 blocks under its footprint hold
        auto hz_culled = [&](const Rec& rc) -> bool {
            const int x0 = (int)(rc.rect & 0xFF), y0 = (int)((rc.rect >> 8) & 0xFF);
            const int x1 = x0 + (int)((rc.rect >> 16) & 0xFF) - 1, y1 = y0 + (int)(rc.rect >> 24) - 1;
            uint32_t m = 0;
            for (int by = y0 >> 2; by <= (y1 >> 2); ++by)
                for (int bx = x0 >> 2; bx <= (x1 >> 2); ++bx) m = max(m, hz[by * (TS / 4) + bx]);
            return __float_as_uint(rc.zcull) > m && rc.zcull > 0.0f;
        };
        auto rect_area = [](uint32_t rect) -> uint32_t { return ((rect >> 16) & 0xFF) * (rect >> 24); };
        // farthest depth (float bits) that 4 pixels of row r of 4x4 block
        // (bx, by) hold: +inf while one is empty; pixels outside the image
        // never hold a hit and do not bound the block
        auto row_zmax = [&](int bx, int by, int r) -> uint32_t {
            const int ly = by * 4 + r;
            uint32_t m = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int lx = bx * 4 + c;
                const unsigned long long kk = keys[ly * TS + lx];
                const uint32_t zb = (lx < tw && ly < th) ? (kk == ~0ull ? 0x7F800000u : (uint32_t)(kk >> 32)) : 0u;
                m = max(m, zb);
            }
            return m;
        };
        // refresh every block depth from the tile's depth buffer (the whole
        // workgroup, after its writes): four lanes per block, one row each
        auto hz_refresh = [&]() {
            for (int u = tid; u < kHzBlocks * 4; u += kBlock) {
                const int b = u >> 2;
                uint32_t m = row_zmax(b % (TS / 4), b / (TS / 4), u & 3);
                m = max(m, (uint32_t)__shfl_xor((int)m, 1));
                m = max(m, (uint32_t)__shfl_xor((int)m, 2));
                if ((u & 3) == 0) hz[b] = m;
            }
            __syncthreads();
        };
        // exclusive prefix of per-thread fragment counts `a` over the
        // workgroup into pref[0..kChunk]; the high bits of `a` may carry a
        // second count (kept records), summed alongside: returns the packed total
        auto block_scan = [&](uint32_t a) -> uint32_t {
            const uint32_t incl = wave_incl_scan(a);
            if (lane == 63) wsum[wave] = incl;
            __syncthreads();
            uint32_t wb = 0, tot = 0;
            for (int w = 0; w < kBlock / 64; ++w) {
                wb += w < wave ? wsum[w] : 0u;
                tot += wsum[w];
            }
            pref[tid] = (wb + incl - a) & kAreaMask;
            if (tid == kBlock - 1) pref[kChunk] = tot & kAreaMask;
            __syncthreads();
            return tot;
        };
        // fragments f of the chunk's records recs[j] with prefix pref.
        // Each wave takes an equal contiguous share and resolves it 64
        // consecutive fragments at a time (neighbouring pixels of a few
        // adjacent records, so early-out decisions agree across the wave).
        // The owner of a fragment is the last record starting at or before
        // it: one search finds it for the share's first fragment; after
        // that the records starting within each step mark their first
        // fragment in the wave's slots, and a max-scan over the lanes,
        // seeded with the previous owner, gives every lane its record.
        auto resolve_fragments = [&]() {
            constexpr int span = kChunk;
            const uint32_t total = pref[kChunk];
            const uint32_t share = (total + kBlock - 1) / kBlock * 64;
            const uint32_t q0 = min(total, (uint32_t)wave * share), q1 = min(total, q0 + share);
            if (q0 < q1) {
                int lo = 0, hi = span;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (pref[mid] <= q0) lo = mid;
                    else hi = mid;
                }
                uint32_t own = (uint32_t)__builtin_amdgcn_readfirstlane(lo);
                uint8_t* const st = ord + wave * 64;
                for (uint32_t f0 = q0; f0 < q1; f0 += 64) {
                    // records after `own` start at or after f0, in order: mark
                    // those with fragments that start before f0 + 64
                    for (uint32_t j0 = own + 1;; j0 += 64) {
                        const uint32_t j = j0 + (uint32_t)lane;
                        uint32_t e = ~0u;
                        bool some = false;
                        if (j < (uint32_t)span) {
                            e = pref[j];
                            some = pref[j + 1] > e;
                        }
                        const bool in = e < f0 + 64;
                        if (in && some) st[e - f0] = (uint8_t)j;
                        if (!__all(in)) break;
                    }
                    // the wave's own LDS writes are seen by its later reads
                    __builtin_amdgcn_wave_barrier();
                    uint32_t m = st[lane];
                    if (m) st[lane] = 0;
                    m = max(wave_incl_max(m), own);
                    own = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
                    const uint32_t f = f0 + (uint32_t)lane;
                    if (f < q1) {
                        const Rec& rr = rec_at(m);
                        const uint32_t local = f - pref[m];
                        const uint32_t rw = (rr.rect >> 16) & 0xFF;
                        // exact: local < 4096 and rw <= 64, so the rounding error of
                        // (local + 1/2) / rw is far below its distance to an integer
                        const uint32_t dy = (uint32_t)(((float)local + 0.5f) * rr.inv_w);
                        const uint32_t dx = local - __umul24(dy, rw);
                        test_pixel(rr, (int)(rr.rect & 0xFF) + (int)dx, (int)((rr.rect >> 8) & 0xFF) + (int)dy);
                    }
                }
            }
            __syncthreads();
        };
        // The kept records of a chunk in depth order (ord), resolved by 8x8
        // blocks: a wave holds a block's depth buffer in registers, one pixel
        // per lane, and takes the records whose footprint meets the block
        // front to back, one at a time, on the pixels that lie in the
        // footprint and hold nothing nearer.  After each hit the records
        // behind the block's farthest depth leave the wave's list at once.
        // Nothing is shared until the chunk is done, so no wave waits for
        // another, no pixel is searched for its record and no depth goes
        // through an atomic; the rays' reciprocals are taken once per pixel.
        // VALU-bound on batches.  Dealing the fragments of 8 records at a
        // time to the whole workgroup, with a barrier on both sides of a
        // refresh of 4x4 block depths, took (resolve of 4,096 spheres at
        // 256x256 / 11M at 4K / 256 renders of 50,000) 22 us / 275 us / 4.01
        // ms; this takes 10 / 191 / 3.21.  Looking at the farthest depth only
        // after every 8th record: 4.47 ms, 4th: 4.32; of each 4x4 quarter:
        // 3.84 against 3.40; record data through scalar registers instead of
        // one LDS read the lanes share: 3.34 against 3.24.
        auto resolve_blocks = [&](uint32_t nk) {
            constexpr int kSide = TS / 8;
            for (int b = wave; b < kSide * kSide; b += kBlock / 64) {
                const int by = b / kSide, bx = (b + by) % kSide;   // a wave's blocks lie on diagonals
                if (bx * 8 >= tw || by * 8 >= th) continue;
                const int lx = bx * 8 + (lane & 7), ly = by * 8 + (lane >> 3);
                const bool in = lx < tw && ly < th;
                const int slot = ly * TS + lx;
                unsigned long long cur = in ? keys[slot] : 0ull;   // outside the image: nothing is nearer
                const float ndx = fmaf((float)(px0 + lx) + 0.5f, F.inv_w2, -1.0f);
                const float ndy = fmaf(-((float)(py0 + ly) + 0.5f), F.inv_h2, 1.0f);
                float ox, oy, Dx, Dy;
                if (persp) {
                    ox = 0.f; oy = 0.f; Dx = ndx * F.txf; Dy = ndy * F.tyf;
                } else {
                    ox = ndx * F.hxf; oy = ndy * F.hyf; Dx = 0.f; Dy = 0.f;
                }
                // farthest depth the block holds (all ones while a pixel is empty)
                auto block_max = [&]() -> uint32_t {
                    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_max((uint32_t)(cur >> 32)), 63);
                };
                for (uint32_t base = 0; base < nk; base += 64) {
                    const uint32_t zmax0 = block_max();
                    const uint32_t i = base + (uint32_t)lane;
                    // this lane's record: its pixels of the block (bit = lane)
                    unsigned long long m = 0ull;
                    uint32_t rj = 0, rid = 0, zcb = 0;
                    if (i < nk) {
                        rj = ord[i];
                        const Rec& r = rec_at(rj);
                        zcb = r.zcull > 0.0f ? __float_as_uint(r.zcull) : 0u;
                        rid = r.id;
                        const uint32_t rect = r.rect;
                        const int x0 = (int)(rect & 0xFF) - bx * 8, y0 = (int)((rect >> 8) & 0xFF) - by * 8;
                        const int x1 = x0 + (int)((rect >> 16) & 0xFF), y1 = y0 + (int)(rect >> 24);
                        if (zcb <= zmax0 && x0 < 8 && y0 < 8 && x1 > 0 && y1 > 0) {
                            const uint32_t row = (1u << min(x1, 8)) - (1u << max(x0, 0));
                            const uint32_t rows4 = row * 0x01010101u;
                            m = (((unsigned long long)rows4 << 32) | rows4) & (~0ull << (8 * max(y0, 0))) &
                                (~0ull >> (64 - 8 * min(y1, 8)));
                        }
                    }
                    unsigned long long live = __ballot(m != 0ull);
                    const unsigned long long spheres = __ballot(rid < F.n_atoms);
                    while (live) {
                        const int s = __builtin_ctzll(live);
                        live &= live - 1ull;
                        const unsigned long long px =
                            ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), s) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, s);
                        const uint32_t zcs = (uint32_t)__builtin_amdgcn_readlane((int)zcb, s);
                        const unsigned long long open = px & __ballot((uint32_t)(cur >> 32) >= zcs);
                        if (counting && __builtin_amdgcn_inverse_ballot_w64(px & ~open)) n_skipped += 1;
                        if (open == 0ull) continue;
                        if (counting) pref[(uint32_t)__builtin_amdgcn_readlane((int)rj, s)] = 1u;
                        bool better = false;
                        const Rec& rs = rec_at((uint32_t)__builtin_amdgcn_readlane((int)rj, s));
                        const float4 a = rs.a;
                        const uint32_t id = rs.id;
                        const bool sphere = (spheres >> s) & 1ull;
                        if (__builtin_amdgcn_inverse_ballot_w64(open)) {
                            bool graze = true;
                            float z;
                            if (sphere) z = hit_sphere(a, ox, oy, Dx, Dy, graze);
                            else z = hit_cylinder(a, rs.b, ox, oy, Dx, Dy);
                            bool hit = z >= F.znear && z <= F.zfar;
                            if (F.clip_on && hit)
                                hit = fmaf(F.clip[0], fmaf(z, Dx, ox), fmaf(F.clip[1], fmaf(z, Dy, oy), fmaf(F.clip[2], z, F.clip[3]))) >= 0.0f;
                            if (counting) {
                                n_tested += 1;
                                n_tested_bond += sphere ? 0 : 1;
                                n_hit += hit ? 1 : 0;
                                n_hit_bond += (hit && !sphere) ? 1 : 0;
                            }
                            const unsigned long long k = ((unsigned long long)__float_as_uint(z) << 32) |
                                                         (id | (graze && F.refine_flag ? kRefineBit : 0u));
                            better = hit && k < cur;
                            if (better) cur = k;
                        }
                        if (__ballot(better)) live &= __ballot(zcb <= block_max());
                    }
                }
                if (in) keys[slot] = cur;
            }
            __syncthreads();
        };
        // Layered lists (resident scenes) run front to back by layer: once
        // every record from a layer on lies behind all block depths of the
        // tile, the rest of the list is culled whole, unread.
        const uint32_t L = over || stats || n <= (uint32_t)kChunk ? 1u : bb.layers;   // one chunk: nothing to stop
        if (L > 1 && wave == 0) {
            uint32_t zr = lane < (int)L ? ctr->layer_zlo[phase == kPhaseRest ? 1 : 0][lane] : 0x7F800000u;
#pragma unroll
            for (int o2 = 1; o2 < 32; o2 <<= 1) {
                const uint32_t u = (uint32_t)__shfl_down((int)zr, o2);
                if (lane + o2 < 64) zr = min(zr, u);
            }
            if (lane < (int)L) {
                lay_zrest[lane] = zr;
                lay_start[lane] = bb.layer_off[(size_t)lane * F.tiles_x * F.tiles_y + t];
            }
        }
        bool hz_set = false;   // the block depths hold a refresh (uniform)
        if (phase == kPhaseRest) {
            hz_refresh();   // the front pass's depths bound the blocks from the start
            hz_set = true;
        }
        for (uint64_t base = 0; base < nsrc; base += kChunk) {
            if (L > 1 && hz_set) {
                // every wave reads the same LDS after the last barrier: a uniform decision
                uint32_t m = 0;
                for (int i = lane; i < kHzBlocks; i += 64) m = max(m, hz[i]);
                m = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_max(m), 63);
                const unsigned long long started = __ballot(lane < (int)L && lay_start[lane] <= (uint32_t)base);
                const uint32_t zr = lay_zrest[63 - __clzll((long long)started)];
                if (zr > m && zr != 0u) {
                    if (counting && tid == 0) ++n_list_stop;
                    break;
                }
            }
            PrimRec pr;
            bool have;
            uint2 e = nxt;
            if (over) have = base + tid < nsrc && fetch_overflow(base + tid, e);
            else have = nxt_ok;
            have = have && source_record(R.again(), e.x, pr);
            pr.g1.w = e.y;
            nxt_ok = !over && base + kChunk + tid < nsrc;
            if (nxt_ok) nxt = list[o + base + kChunk + tid];
            bool keep = false;
            uint32_t area = 0;
            float zc = INFINITY;
            if (have) {
                const Rec rc = make_rec(F, pr);
                // until a refresh has stored depths every block is +inf: nothing to test
                keep = stats || !hz_set || !hz_culled(rc);
                if (counting && !keep) n_culled += 1;
                if (keep) {
                    area = rect_area(rc.rect);
                    zc = rc.zcull;
                    recs[tid] = rc;
                }
            }
            const bool more = base + kChunk < nsrc;
            // the kept records' depth range, per wave (as bits: depths before
            // the eye count as 0, the order need not be exact), and the
            // buckets cleared, for a chunk that gets ordered
            const float zord = fmaxf(zc, 0.0f);
            {
                const uint32_t zb = __float_as_uint(zord);
                const uint32_t hi = wave_incl_max(keep ? zb : 0u), lo = wave_incl_max(keep ? ~zb : 0u);
                if (lane == 63) {
                    red_hi[wave] = hi;
                    red_lo[wave] = ~lo;
                }
                if (tid < kBuckets) bcnt[tid] = 0u;
            }
            // prefix of the footprint areas, with the kept records counted in
            // the high bits
            const uint32_t packed = block_scan(area | (keep ? 1u << kKeptShift : 0u));
            const uint32_t atot = packed & kAreaMask, nk = packed >> kKeptShift;
            // Large footprints (many records cover each pixel): order the
            // kept records front to back by a counting sort over depth
            // buckets and resolve them block by block, so records behind the
            // first layers are dropped before any of their pixels is tested.
            const bool sorted = TS > 8 && !stats && atot > (uint32_t)kSortArea * nk &&
                                atot > (uint32_t)(kSortDepth * TS * TS);
            if (!sorted) {
                resolve_fragments();
                if (!stats && more) {
                    hz_refresh();
                    hz_set = true;
                }
                continue;
            }
            // A record's rank in its bucket, then (every wave for itself) the
            // buckets' starts: two barriers (with the depth range by shuffles,
            // one wave's scan and a second atomic five, and the resolve of 256
            // renders of 50,000 atoms 3.21 ms instead of 3.12).
            const float zlo = __uint_as_float(min(min(red_lo[0], red_lo[1]), min(red_lo[2], red_lo[3])));
            const float zhi = __uint_as_float(max(max(red_hi[0], red_hi[1]), max(red_hi[2], red_hi[3])));
            const float span = zhi - zlo;
            const float scale = span > 0.0f ? (float)kBuckets / span : 0.0f;
            const int bk = keep ? min(kBuckets - 1, (int)((zord - zlo) * scale)) : 0;
            uint32_t rank = 0;
            if (keep) rank = atomicAdd(&bcnt[bk], 1u);
            __syncthreads();
            {
                const uint32_t c = bcnt[lane];
                const uint32_t at = (uint32_t)__shfl((int)(wave_incl_scan(c) - c), bk) + rank;
                if (keep) ord[at] = (uint8_t)tid;
            }
            if (counting) pref[tid] = 0u;   // marks the records that some pixel tests
            __syncthreads();   // the order is in LDS
            resolve_blocks(nk);
            if (counting && keep && pref[tid] == 0u) {
                n_culled += 1;
                if ((int)ord[nk - 1] == tid) ++n_chunk_stop;
            }
            if (more) {
                hz_refresh();
                hz_set = true;
            }
            if (counting) __syncthreads();   // every thread has read the order
            if (tid < kChunk / 4) reinterpret_cast<uint32_t*>(ord)[tid] = 0u;
        }
        __syncthreads();
        if constexpr (TS >= kHzCell) {
            if (phase == kPhaseFront) {
                // farthest depth of each 16x16 cell of the tile, for the rest
                // pass's cluster test (cells past the image edge are not stored)
                hz_refresh();
                constexpr int kCells = TS / kHzCell, kSub = kHzCell / 4;
                if (tid < kCells * kCells) {
                    const int cy = tid / kCells, cx = tid - cy * kCells;
                    const int gx = tx * kCells + cx, gy = ty * kCells + cy;
                    if (gx < bb.hz16_w && gy < (F.H + kHzCell - 1) / kHzCell) {
                        uint32_t m = 0;
                        for (int by = 0; by < kSub; ++by)
                            for (int bx = 0; bx < kSub; ++bx) m = max(m, hz[(cy * kSub + by) * (TS / 4) + cx * kSub + bx]);
                        bb.hz16[(size_t)gy * bb.hz16_w + gx] = m;
                    }
                }
            }
        }

        // The G-buffer: the winner of each pixel.  The last pass gives the
        // marked winners their depths recomputed in FP64 and plain ids; the
        // front pass of a two-pass frame, which the rest pass continues from,
        // keeps the FP32 depths and the marks.
        const bool finish = phase != kPhaseFront;
        const JobRef Rr = R.again();
        const Frame Fr = Rr.frame();
        auto is_marked = [&](unsigned long long kk) { return kk != ~0ull && (!F.refine_flag || ((uint32_t)kk & kRefineBit)); };
        auto refined = [&](unsigned long long kk, int i) -> unsigned long long {
            const uint32_t id = F.refine_flag ? (uint32_t)kk & ~kRefineBit : (uint32_t)kk;
            const float z = refine_depth_at(Fr, to_global(Rr.pos()), to_global(Rr.rad()), to_global(Rr.bonds()), id, px0 + i % TS, py0 + i / TS,
                                            __uint_as_float((uint32_t)(kk >> 32)));
            return ((unsigned long long)__float_as_uint(z) << 32) | id;
        };
        // About one winner in five is marked, in nearly every wave, so the
        // marked pixels are packed into a list first and only as many waves
        // as they fill run the FP64 code (256 renders of 50,000 atoms, 32-pixel
        // tiles: 3.12 ms, with each thread refining its own pixels 3.39; with
        // one pixel per thread, 16-pixel tiles, the list and its barriers cost
        // as much as they save: 1M atoms and bonds at 1080p 60.5 and 60.9 us).
        if (finish) {
            uint16_t* const todo = reinterpret_cast<uint16_t*>(recs);   // the records are done with
            static_assert(TS * TS * sizeof(uint16_t) <= sizeof(recs), "one list entry per pixel of the tile");
            if (tid == 0) wsum[0] = 0u;
            __syncthreads();
            for (int i = tid; i < TS * TS; i += kBlock) {   // whole waves: TS * TS is a multiple of 64
                const unsigned long long kk = keys[i];
                const unsigned long long mm = __ballot(is_marked(kk));
                uint32_t at = 0;
                if (mm && lane == 0) at = atomicAdd(&wsum[0], (uint32_t)__popcll(mm));
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
                if (is_marked(kk)) todo[at + (uint32_t)__popcll(mm & __lanemask_lt())] = (uint16_t)i;
            }
            __syncthreads();
            const uint32_t n_todo = wsum[0];
#pragma unroll 1
            for (uint32_t e = (uint32_t)tid; e < n_todo; e += kBlock) {
                const int i = todo[e];
                keys[i] = refined(keys[i], i);
            }
            __syncthreads();
        }
#pragma unroll 1
        for (int i = tid; i < TS * TS; i += kBlock) {
            const int ly = i / TS, lx = i - ly * TS;
            if (lx < tw && ly < th) {
                const unsigned long long kk = keys[i];
                const size_t p = (size_t)(py0 + ly) * F.W + (px0 + lx);
                depth[p] = kk == ~0ull ? INFINITY : __uint_as_float((uint32_t)(kk >> 32));
                out_id[p] = (uint32_t)kk;   // no hit: kBackground, the key's low word
            }
        }
    }
    if (counting) {
        unsigned long long a = n_tested, b = n_hit, c = n_hit_bond, d = n_tested_bond, e = n_skipped, g = n_culled;
        for (int o2 = 32; o2 > 0; o2 >>= 1) {
            a += __shfl_xor(a, o2);
            b += __shfl_xor(b, o2);
            c += __shfl_xor(c, o2);
            d += __shfl_xor(d, o2);
            e += __shfl_xor(e, o2);
            g += __shfl_xor(g, o2);
        }
        if (lane == 0) {
            if (a) {
                atomicAdd(&ctr->frag_tested, a);
                atomicAdd(&ctr->frag_hit, b);
                atomicAdd(&ctr->frag_hit_bond, c);
                atomicAdd(&ctr->frag_tested_bond, d);
            }
            if (e) atomicAdd(&ctr->frag_skipped, e);
            if (g) atomicAdd(&ctr->rec_culled, g);
        }
        if (tid == 0 && n_list_stop) atomicAdd(&ctr->lists_stopped, (unsigned long long)n_list_stop);
        if (tid == 0 && n_chunk_stop) atomicAdd(&ctr->chunks_stopped, (unsigned long long)n_chunk_stop);
    }
}

// The rest pass in a tile it adds nothing to: the front pass's marked winners
// get their FP64 depths, the other pixels stay as they are.
template <int TS>
__device__ __forceinline__ void refine_tile(JobRef R, int t, unsigned long long* todo) {
    __shared__ uint32_t n_todo;
    const Frame F = R.frame();
    global_t<float>* __restrict__ const depth = to_global(R.depth());
    global_t<uint32_t>* __restrict__ const out_id = to_global(R.id());
    const int px0 = (t % F.tiles_x) * TS, py0 = (t / F.tiles_x) * TS;
    const int tid = threadIdx.x, lane = __lane_id();
    if (tid == 0) n_todo = 0u;
    __syncthreads();
    for (int i = tid; i < TS * TS; i += kBlock) {
        const int x = px0 + i % TS, y = py0 + i / TS;
        const uint32_t id = x < F.W && y < F.H ? out_id[(size_t)y * F.W + x] : kBackground;
        const bool marked = id != kBackground && (!F.refine_flag || (id & kRefineBit));
        const unsigned long long mm = __ballot(marked);
        uint32_t at = 0;
        if (mm && lane == 0) at = atomicAdd(&n_todo, (uint32_t)__popcll(mm));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(mm & __lanemask_lt());
        if (marked) todo[at] = ((unsigned long long)i << 32) | (F.refine_flag ? id & ~kRefineBit : id);
    }
    __syncthreads();
    for (uint32_t e = (uint32_t)tid; e < n_todo; e += kBlock) {
        const int i = (int)(todo[e] >> 32);
        const uint32_t id = (uint32_t)todo[e];
        const int x = px0 + i % TS, y = py0 + i / TS;
        const size_t p = (size_t)y * F.W + x;
        depth[p] = refine_depth_at(F, to_global(R.pos()), to_global(R.rad()), to_global(R.bonds()), id, x, y, depth[p]);
        out_id[p] = id;
    }
}

// Main launch: work block t of a job is that job's tile t, or the t-th of its
// tile order (see kOrderTiles), so consecutive
// tiles go to different XCDs (the dispatcher deals blocks round-robin).  The
// costly tiles lie together, around the footprints of the nearest atoms:
// contiguous tile ranges per XCD left one XCD with most of them (20 % longer
// on the whole-cell frame).  A tile whose list overflowed the bins
// is rebuilt from the visible lists by the same code: a second launch for
// those tiles costs every frame that has none 1.4 to 2 us (4,096 atoms at
// 256x256: 53.1 us with it, 51.7 without; 1M atoms and bonds at 1080p: 172.9
// and 170.2; four views in a batch: 179.1 and 173.7).
// kCount: the instantiation that can count fragments (jobs with
// VTX_FLAG_STATS); the other one carries no counters.
// kPhase: one pass, or one of a two-pass frame's.
template <int TS, class JS, bool kCount, int kPhase>
__global__ void __launch_bounds__(kBlock, kCount ? 1 : 7) k_resolve(JS js) {
    uint32_t tu;
    const int ji = js.find(blockIdx.x, tu);
    if (ji < 0) return;
    const Job& J = js.job(ji);
    const int T = J.F.tiles_x * J.F.tiles_y;
    if (JS::kOrdered && T > kOrderTiles) tu = (uint32_t)__builtin_amdgcn_readfirstlane((int)tile_order(J.bb, T)[tu]);
    const uint32_t n = J.bb.tile_cnt[tu];
    const uint64_t o = J.bb.tile_off[tu];
    const bool over = o + n > J.bb.capacity;
    if (kPhase == kPhaseAll && n == 0) {   // nothing to cast or to re-arm: background
        const int W = J.F.W, H = J.F.H, tiles_x = J.F.tiles_x;
        const int px0 = ((int)tu % tiles_x) * TS, py0 = ((int)tu / tiles_x) * TS;
        global_t<float>* __restrict__ const depth = to_global(J.depth);
        global_t<uint32_t>* __restrict__ const out_id = to_global(J.id);
        for (int i = threadIdx.x; i < TS * TS; i += kBlock) {
            const int x = px0 + i % TS, y = py0 + i / TS;
            if (x < W && y < H) {
                depth[(size_t)y * W + x] = INFINITY;
                out_id[(size_t)y * W + x] = kBackground;
            }
        }
        return;
    }
    __shared__ unsigned long long keys[TS * TS];   // the tile's depth buffer
    if constexpr (kPhase == kPhaseRest) {
        if (n == 0) {
            refine_tile<TS>(job_ref(js, ji), (int)tu, keys);
            return;
        }
    }
    resolve_tile<TS, kCount, kPhase>(job_ref(js, ji), (int)tu, n, o, over, keys);
}

// Counting frames: the resolve's fragment counters, to every counting job's
// host buffer (one workgroup, queued after the resolve).
template <class JS>
__global__ void __launch_bounds__(kBlock) k_publish(JS js) {
    for (uint32_t j = threadIdx.x; j < js.count(); j += kBlock) {
        const Job& J = js.job((int)j);
        if (!(J.F.flags & (1u | 16u)) || !J.bb.host_ctr) continue;
        const Counters* const src = J.bb.ctr;
        J.bb.host_ctr->frag_tested = src->frag_tested;
        J.bb.host_ctr->frag_hit = src->frag_hit;
        J.bb.host_ctr->frag_hit_bond = src->frag_hit_bond;
        J.bb.host_ctr->frag_tested_bond = src->frag_tested_bond;
        J.bb.host_ctr->frag_skipped = src->frag_skipped;
        J.bb.host_ctr->rec_culled = src->rec_culled;
        J.bb.host_ctr->lists_stopped = src->lists_stopped;
        J.bb.host_ctr->chunks_stopped = src->chunks_stopped;
        stamp_counters(J.bb.host_ctr, J.bb.stamp);
    }
}

}  // namespace

template <int TS, class JS, bool kCount, int kPhase>
hipError_t resolve_pass(const JS& js, unsigned g, hipStream_t stream) {
    const hipError_t e = dispatch(k_resolve<TS, JS, kCount, kPhase>, g, kBlock, 0, stream, js);
    if (e || !kCount) return e;
    return dispatch(k_publish<JS>, 1, kBlock, 0, stream, js);
}

template <int TS, class JS, bool kCount>
hipError_t resolve_launch(const JS& js, int phase, unsigned g, hipStream_t stream) {
    if constexpr (!kCount && TS >= kHzCell) {
        if (phase == kPhaseFront) return resolve_pass<TS, JS, false, kPhaseFront>(js, g, stream);
        if (phase == kPhaseRest) return resolve_pass<TS, JS, false, kPhaseRest>(js, g, stream);
    }
    return resolve_pass<TS, JS, kCount, kPhaseAll>(js, g, stream);
}

template <class JS, bool kCount>
hipError_t resolve_impl(const JS& js, int tile, int phase, uint32_t grid, hipStream_t stream) {
    if (grid == 0) return hipSuccess;
    if (phase != kPhaseAll && (kCount || tile < kHzCell)) return hipErrorInvalidValue;
    const unsigned g = (unsigned)xcd_grid((int)grid);
    switch (tile) {
        case 8: return resolve_launch<8, JS, kCount>(js, phase, g, stream);
        case 16: return resolve_launch<16, JS, kCount>(js, phase, g, stream);
        case 32: return resolve_launch<32, JS, kCount>(js, phase, g, stream);
        case 64: return resolve_launch<64, JS, kCount>(js, phase, g, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_resolve(const OneJob& js, int tile, int phase, uint32_t grid, bool count, hipStream_t stream) {
    return count ? resolve_impl<OneJob, true>(js, tile, phase, grid, stream)
                 : resolve_impl<OneJob, false>(js, tile, phase, grid, stream);
}
hipError_t launch_resolve(const JobList& js, int tile, int phase, uint32_t grid, bool count, hipStream_t stream) {
    return count ? resolve_impl<JobList, true>(js, tile, phase, grid, stream)
                 : resolve_impl<JobList, false>(js, tile, phase, grid, stream);
}

}  // namespace vtx
