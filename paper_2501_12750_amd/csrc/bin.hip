// Screen-tile binning of atoms and bonds: a counting sort by tile.
//
// The paper rasterizes one screen quad per primitive and lets the fixed
// function rasterizer find the pixels it covers (Methods, "Meshless
// Representations").  Here the quad's role, a conservative footprint, becomes
// an exact tile rectangle per primitive, and the rasterizer becomes a
// counting sort of (tile, primitive) pairs:
//   count    G workgroups each own a contiguous run of primitives (resident
//            scenes: of the visible clusters in depth-class order, so the
//            workgroups run front to back): view transform (FP64), culling,
//            footprint rectangle, a compacted per-workgroup list of the
//            visible ones, and a tile histogram in LDS; the histogram row is
//            stored and its non-zero entries are added to the tile totals
//            (resident scenes: to the totals of the workgroup's layer, 1/32
//            of the workgroups), one atomic per touched tile;
//   layers   resident scenes: the per-layer totals become the start of each
//            layer's run in every tile list, and the tile totals;
//   scatter  each workgroup takes the exclusive scan of the tile totals (the
//            list offsets) and reserves, per touched tile, one run of the tile's
//            list inside its layer's run (one atomic), then places its
//            primitives with LDS atomics (one per run of lanes with the same
//            tile): 8 bytes per (primitive, tile), the source index and the
//            footprint clipped to the tile.  The resolve rebuilds each record
//            from its source, so the view-space record is never written out.
// So the global atomics scale with (workgroup, touched tile) pairs rather
// than with (primitive, tile) pairs, and a resident scene's tile lists run
// roughly front to back.  Lists that would not fit the bin
// capacity are left empty; the resolve pass then finds those tiles' primitives
// in the per-workgroup visible lists, so every frame is exact whatever the
// capacity.
#include <algorithm>

#include "prims.h"

namespace vtx {

namespace {

// Zeroes n words (allocation time only: afterwards every frame leaves the
// tile counts and the frame counters at zero for the next one).
__global__ void __launch_bounds__(kBlock) k_zero(uint32_t* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
}

// Footprint of a visible item (its view coordinates from item_view).
__device__ inline bool item_rect(const Frame& F, const Item& it, const double* v, double r, int& x0, int& y0,
                                 int& x1, int& y1) {
    if (it.kind == kAtom) return sphere_rect_fast(F, v[0], v[1], v[2], r, x0, y0, x1, y1);
    return bond_rect_fast(F, v, v + 3, r, x0, y0, x1, y1);
}

// Runs of consecutive lanes whose primitives lie in the same single tile t
// (t < 0: none); Morton-ordered primitives keep them long.  For such a lane
// `head` is its run's first lane, and for a head `len` is the run's length
// (other lanes: head = the lane itself).  Branch-free: one DPP shift, one
// ballot and a few mask operations.  Every lane of the wave calls it.
__device__ inline void lane_run(int t, int& head, uint32_t& len) {
    const int lane = __lane_id();
    const int tp = __builtin_amdgcn_update_dpp(-1, t, 0x138, 0xf, 0xf, false);   // wave_shr:1: lane - 1's t
    const unsigned long long cm = __ballot(t >= 0 && lane > 0 && t == tp);     // lanes continuing a run
    head = 63 - __clzll((long long)(~cm & ((2ull << lane) - 1ull)));            // nearest non-continuing lane <= lane
    len = (uint32_t)__builtin_ctzll(~((cm >> lane) >> 1)) + 1u;                  // continuing lanes after it, + 1
}

// Adds one to the LDS counter of each lane's tile t (t < 0: nothing): one
// atomic per run of lanes with the same tile.
__device__ inline void wave_count(uint32_t* hist, int t) {
    int head;
    uint32_t len;
    lane_run(t, head, len);
    if (t >= 0 && head == (int)__lane_id()) atomicAdd(&hist[t], len);
}

// Inclusive sum over the 64 lanes of a wave by DPP row shifts and row
// broadcasts (lanes shifted in from outside a row read 0).
__device__ inline uint32_t wave_scan_u32(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

// Maximum over the 64 lanes of a wave, the same steps, in every lane.
__device__ inline uint32_t wave_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Tile of entry i of a workgroup's histogram row: the row covers the box of
// tiles [bx0, bx0 + bw) x [by0, ...) its primitives touch, row-major.
__device__ inline int box_tile(int tiles_x, uint32_t bx0, uint32_t by0, int bw, int i) {
    const int q = i / bw;
    return ((int)by0 + q) * tiles_x + (int)bx0 + (i - q * bw);
}

// Count.  Work block b of a job is that job's binning workgroup b.
// kRest: the rest pass of a two-pass frame, over the clusters
// k_cluster_rest kept.  kAtoms: a scene without bonds (no bond path in the
// loop: fewer live registers).  kQuarters: see quarters() for the scenes that
// take it.  kStored (not kScene): a resident scene's primitives in their
// stored order, without its clusters.
template <class JS, bool kScene, bool kRest, bool kAtoms = false, bool kQuarters = false, bool kStored = false>
__global__ void __launch_bounds__(kBinThreads, 8) k_count(JS js, int phase) {
    extern __shared__ uint32_t hist[];
    __shared__ uint32_t local_n, bx0, by0, bx1, by1;
    __shared__ unsigned long long local_pairs;
    __shared__ uint32_t cls_end[kDepthBuckets], cls_all[kRest ? kDepthBuckets : 1];
    __shared__ uint32_t wg_zlo;
    uint32_t blk;
    const int ji = js.find(blockIdx.x, blk);
    if (ji < 0) return;
    const JobRef R = job_ref(js, ji);
    const BinBuffers bb = R.bins();
    const uint32_t chunk = bb.chunk;
    Counters* const ctr = bb.ctr;
    const int tiles_x = R.frame().tiles_x, tsh = R.frame().tile_shift;
    const int T = tiles_x * R.frame().tiles_y;
    const int tid = threadIdx.x;
    for (int t = tid; t < T; t += kBinThreads) hist[t] = 0;
    if constexpr (kScene) {
        // end of each depth class in the front-to-back order of the clusters
        // (rest pass: also where each class's region of the kept ones starts)
        if (tid < 64) {
            class_ends(kRest ? ctr->rest_bucket : ctr->vis_bucket, cls_end);
            if constexpr (kRest) class_ends(ctr->vis_bucket, cls_all);
        }
    }
    if (tid == 0) {
        local_n = 0;
        wg_zlo = 0x7F800000u;
        local_pairs = 0;
        bx0 = 0xFFFF;
        by0 = 0xFFFF;
        bx1 = 0;
        by1 = 0;
    }
    __syncthreads();
    // resident scenes: the least cull depth of this lane's visible primitives
    // (float bits), a bound the resolve may stop a tile's list at.  The
    // resolve culls a record by (z - r)(1 - 1e-5) from FP32 coordinates
    // (bonds: the nearer end's z less the radius, and 1e-6 less); the FP64
    // value here, 2e-5 of the magnitudes and 2e-6 lower and rounded down,
    // stays below it.
    uint32_t my_zlo = 0x7F800000u;
    auto note_z = [&](double zmin, double mag) {
        const float lb = __double2float_rd(zmin - 2e-5 * mag - 2e-6);
        my_zlo = min(my_zlo, lb > 0.0f ? __float_as_uint(lb) : 0u);
    };

    const uint64_t start = (uint64_t)blk * chunk;
    uint32_t bad_count = 0;
    global_t<uint32_t>* __restrict__ const my_src = to_global(bb.vis_src) + start;   // this workgroup's visible list
    global_t<uint2>* __restrict__ const my_rect = to_global(bb.vis_rect) + start;
    // One visible-or-not primitive per lane (every lane of the wave calls
    // it): its slot in the workgroup's visible list, its tile counts.
    auto emit = [&](bool vis, uint32_t sidx, int x0, int y0, int x1, int y1) {
        const unsigned long long vmask = __ballot(vis);
        uint32_t slot_base = 0;
        const int leader = __ffsll((long long)(vmask | 1ull)) - 1;
        if (vmask && (int)__lane_id() == leader) slot_base = atomicAdd(&local_n, (uint32_t)__popcll(vmask));
        slot_base = __shfl(slot_base, leader);
        const int tx0 = x0 >> tsh, tx1 = x1 >> tsh, ty0 = y0 >> tsh, ty1 = y1 >> tsh;
        const bool single = vis && tx0 == tx1 && ty0 == ty1;
        wave_count(hist, single ? ty0 * tiles_x + tx0 : -1);
        if (vis) {
            const uint32_t slot = slot_base + (uint32_t)__popcll(vmask & __lanemask_lt());
            my_src[slot] = sidx;
            my_rect[slot] = make_uint2((uint32_t)x0 | ((uint32_t)y0 << 16), (uint32_t)x1 | ((uint32_t)y1 << 16));
            if (!single)
                for (int ty = ty0; ty <= ty1; ++ty)
                    for (int tx = tx0; tx <= tx1; ++tx) atomicAdd(&hist[ty * tiles_x + tx], 1u);
        }
    };
    // any primitive (the generic path)
    auto emit_item = [&](const Frame& F, const Item& it) {
        int x0 = 0, y0 = 0, x1 = -1, y1 = -1;
        PrimRec rec;
        double v[6], r = 0.0;
        const bool vis = item_view(F, it, rec, v, r) && item_rect(F, it, v, r, x0, y0, x1, y1);
        bad_count += it.kind == kBadBond ? 1u : 0u;
        if (kScene && vis) {
            if (it.kind == kAtom) note_z(v[2] - r, fabs(v[2]) + r);
            else note_z(fmin(v[2], v[5]) - r, fabs(v[2]) + fabs(v[5]) + r);
        }
        emit(vis, it.src, x0, y0, x1, y1);
    };
    if constexpr (kScene) {
        // Resident scene: each wave takes whole clusters or quarters of them
        // (256 primitives of one kind, so the kind is the same across the wave).  An atom
        // cluster's 64-atom quarters take the sphere-only path.
        // Workgroup b takes positions [c0, c1) of the pass's clusters in
        // depth-class order, so the workgroups run front to back.
        const SceneDev S = R.scene();
        const uint32_t stride = S.atom_clusters + S.bond_clusters;
        const uint32_t n = phase == kPhaseFront ? front_clusters(cls_end) : cls_end[kDepthBuckets - 1];
        const uint32_t cpw = (n + bb.groups - 1) / bb.groups;
        const uint32_t c0 = min(n, blk * cpw), c1 = min(n, c0 + cpw);
        int cls = 0;   // class of the positions this wave reads next (they increase)
        auto cluster_at = [&](uint32_t q) -> uint32_t {
            while (cls_end[cls] <= q) ++cls;
            const uint32_t in = q - (cls ? cls_end[cls - 1] : 0u);
            if constexpr (kRest) return S.vis_clusters[(size_t)kDepthBuckets * stride + (cls ? cls_all[cls - 1] : 0u) + in];
            return S.vis_clusters[(size_t)cls * stride + in];
        };
        // kQuarters: the waves take the clusters' 64-primitive quarters in
        // turn, four waves per cluster, else whole clusters.
        constexpr uint32_t kPer = kQuarters ? 4u : 1u;   // waves per cluster
        const uint32_t nw = kBinThreads / 64 / kPer;
        const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
        const uint32_t first = c0 + wave / kPer;
        const uint32_t part = (wave % kPer) * 64u + __lane_id();
        uint32_t cn = first < c1 ? cluster_at(first) : 0u;
        for (uint32_t ci = first; ci < c1; ci += nw) {
            const uint32_t ce = (uint32_t)__builtin_amdgcn_readfirstlane((int)cn);
            const uint32_t c = ce & ~kClusterInside;
            const bool inside = (ce & kClusterInside) != 0u;   // its atoms need no frustum test
            if (ci + nw < c1) cn = cluster_at(ci + nw);   // the next cluster's id, ahead of its use
            if (kAtoms || c < S.atom_clusters) {
                // one quarter at a time: holding more quarters' atoms spills
                // registers, which costs more than the load latency it hides
                for (uint32_t q = 0; q < 4u / kPer; ++q) {
                    const Frame F = R.again().frame();
                    const uint32_t i = c * kCluster + q * 64u + part;
                    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (i < S.n_atoms) a = to_global(S.xyzr)[i];
                    int x0 = 0, y0 = 0, x1 = -1, y1 = -1;
                    double vx, vy, vz;
                    to_view(F, a.x, a.y, a.z, vx, vy, vz);
                    const double r = (double)atom_radius(F, a.w);
                    const bool vis = i < S.n_atoms && r > 0.0 && (inside || sphere_in_frustum(F, vx, vy, vz, r)) &&
                                     sphere_rect_fast(F, vx, vy, vz, r, x0, y0, x1, y1);
                    if (vis) {
                        // in FP32: the resolve takes (z - r)(1 - 1e-5) from
                        // these same rounded z and r; 3e-5 of the magnitudes
                        // covers that and the few roundings here
                        const float zf = (float)vz, rf = (float)r;
                        const float lb = (zf - rf) - 3e-5f * (fabsf(zf) + rf) - 2e-6f;
                        my_zlo = min(my_zlo, lb > 0.0f ? __float_as_uint(lb) : 0u);
                    }
                    emit(vis, i, x0, y0, x1, y1);
                }
            } else if constexpr (!kAtoms) {
                for (uint32_t q = 0; q < 4u / kPer; ++q) {
                    const uint32_t j = (c - S.atom_clusters) * kCluster + q * 64u + part;
                    const JobRef Rq = R.again();
                    const SceneDev Sq = Rq.scene();
                    emit_item(Rq.frame(), j < Sq.n_bonds ? fetch_scene(Sq, Sq.n_atoms + j) : empty_item());
                }
            }
        }
    } else {
        const uint32_t n_atoms = R.frame().n_atoms;
        const uint64_t total = (uint64_t)n_atoms + R.frame().n_bonds;
        const uint32_t nitems = start < total ? (uint32_t)min((uint64_t)chunk, total - start) : 0u;
        auto fetch = [&](uint32_t k) {
            if constexpr (kStored) return fetch_scene(R.scene(), (uint32_t)start + k);
            return fetch_plain(to_global(R.pos()), to_global(R.rad()), to_global(R.bonds()), n_atoms, start + k);
        };
        Item cur = empty_item();
        if ((uint32_t)tid < nitems) cur = fetch(tid);
        for (uint32_t base = 0; base < nitems; base += kBinThreads) {
            // the next iteration's inputs are loaded while this one is processed
            Item nxt = empty_item();
            if (base + kBinThreads + tid < nitems) nxt = fetch(base + kBinThreads + tid);
            emit_item(R.again().frame(), cur);
            cur = nxt;
        }
    }
    if (bad_count) atomicAdd(&ctr->bad_bonds, bad_count);
    if constexpr (kScene) {
        const uint32_t zlo = ~wave_max_u32(~my_zlo);   // the wave's least
        if (__lane_id() == 0 && zlo != 0x7F800000u) atomicMin(&wg_zlo, zlo);
    }
    __syncthreads();   // the histogram is complete
    {
        // the workgroup's box of touched tiles and its pair count, read from
        // the histogram once rather than tracked per primitive; reduced over
        // each wave first (an LDS atomic to one address takes its lanes in
        // turn: with one per thread 4,096 atoms at 256x256 took 16.6 us in
        // this kernel, 6.6 so; 11M spheres at 4K 120 and 94)
        uint32_t mx0 = 0xFFFF, my0 = 0xFFFF, mx1 = 0, my1 = 0;
        unsigned long long my_pairs = 0;
        for (int t = tid; t < T; t += kBinThreads) {
            const uint32_t h = hist[t];
            if (h) {
                const uint32_t ty = (uint32_t)(t / tiles_x), tx = (uint32_t)t - ty * (uint32_t)tiles_x;
                mx0 = min(mx0, tx);
                my0 = min(my0, ty);
                mx1 = max(mx1, tx);
                my1 = max(my1, ty);
                my_pairs += h;
            }
        }
        if (__ballot(my_pairs != 0ull)) {
            // minima as maxima of the complements
            mx0 = 0xFFFFu - wave_max_u32(0xFFFFu - mx0);
            my0 = 0xFFFFu - wave_max_u32(0xFFFFu - my0);
            mx1 = wave_max_u32(mx1);
            my1 = wave_max_u32(my1);
            // 16-bit halves, so that 64 lanes cannot overflow
            const uint32_t lo = wave_scan_u32((uint32_t)my_pairs & 0xFFFFu), hi = wave_scan_u32((uint32_t)(my_pairs >> 16));
            if (__lane_id() == 63) {
                atomicMin(&bx0, mx0);
                atomicMin(&by0, my0);
                atomicMax(&bx1, mx1);
                atomicMax(&by1, my1);
                atomicAdd(&local_pairs, ((unsigned long long)hi << 16) + lo);
            }
        }
    }
    __syncthreads();
    global_t<uint32_t>* const row = to_global(bb.hist) + (size_t)blk * T;
    // layered lists: per-layer totals (the layer kernel turns them into list
    // starts and tile totals); otherwise the tile totals directly
    uint32_t* const tot = kScene && bb.layers > 1
                              ? bb.layer_sum + (size_t)layer_of(blk, bb.groups, bb.layers) * T
                              : bb.tile_cnt;
    // the histogram row holds the tiles of the workgroup's box only (see
    // box_tile), row-major within the box
    const int bw = bx0 <= bx1 ? (int)(bx1 - bx0) + 1 : 0, nb = bw * (bw ? (int)(by1 - by0) + 1 : 0);
    for (int i = tid; i < nb; i += kBinThreads) {
        const int t = box_tile(tiles_x, bx0, by0, bw, i);
        const uint32_t h = hist[t];
        row[i] = h;
        if (h) atomicAdd(&tot[t], h);
    }
    if (tid == 0) {
        if (kScene && bb.layers > 1 && wg_zlo != 0x7F800000u)
            atomicMin(&ctr->layer_zlo[phase == kPhaseRest ? 1 : 0][layer_of(blk, bb.groups, bb.layers)], wg_zlo);
        bb.vis_cnt[blk] = local_n;
        bb.vis_box[blk] = make_uint2(bx0 | (by0 << 16), bx1 | (by1 << 16));
        atomicAdd(&ctr->vis_count, local_n);
        if (local_pairs) atomicAdd(&ctr->pairs_counted, local_pairs);
    }
}

// Layer starts of the tile lists (jobs with layers > 1).  For tile t,
// layer_off[g][t] is the number of t's entries in the layers before g (the
// exclusive prefix over g of the count kernel's per-layer totals), and
// tile_cnt[t] the list's length; the totals are re-zeroed for the next frame.
// With P the power of two >= layers, work block b takes the (1024 / P)-tile
// blocks b, b + groups, ...; thread (g, i) = (tid / W, tid % W) holds layer
// g's total of tile i (loads coalesced along i), and the prefix over g goes
// through LDS.
template <class JS>
__global__ void __launch_bounds__(kBinThreads) k_layers(JS js) {
    static_assert(kBinThreads == 1024 && kLayers <= 32, "tile blocks of 1024 / P tiles, P <= 32");
    __shared__ uint32_t part[kBinThreads + kLayers];
    uint32_t blk;
    const int ji = js.find(blockIdx.x, blk);
    if (ji < 0) return;
    const Job& J = js.job(ji);
    const uint32_t L = J.bb.layers, groups = J.bb.groups;
    if (L <= 1) return;
    const uint32_t T = (uint32_t)(J.F.tiles_x * J.F.tiles_y);
    uint32_t* __restrict__ const sum = J.bb.layer_sum;
    uint32_t* __restrict__ const loff = J.bb.layer_off;
    const uint32_t lsh = 32u - (uint32_t)__builtin_clz(L - 1u);   // P = 1 << lsh >= L (L <= kLayers)
    const uint32_t wsh = 10u - lsh, W = 1u << wsh;                  // tiles per block: kBinThreads / P
    const uint32_t g = threadIdx.x >> wsh, i = threadIdx.x & (W - 1u);
    for (uint32_t tb = blk; tb * W < T; tb += groups) {   // trip count uniform over the workgroup
        const uint32_t t = tb * W + i;
        const bool mine = t < T && g < L;
        uint32_t v = 0;
        if (mine) {
            v = sum[(size_t)g * T + t];
            sum[(size_t)g * T + t] = 0u;
        }
        part[g * (W + 1u) + i] = v;
        __syncthreads();
        uint32_t pre = 0;
        for (uint32_t h = 0; h < g; ++h) pre += part[h * (W + 1u) + i];
        if (mine) {
            loff[(size_t)g * T + t] = pre;
            if (g == L - 1u) J.bb.tile_cnt[t] = pre + v;
        }
        __syncthreads();   // part is rewritten by the next tile block
    }
}

// Scatter cursor of a tile this workgroup has no run in (its list did not
// fit, or it has no primitive there).  Slots are below kMaxCapacity <=
// 2^28, and adding at most a workgroup's pairs keeps the flag bit set.
constexpr uint32_t kNoRun = 0x80000000u;

// Exclusive prefix sum of the counts of T <= kRows * 1024 tiles by one
// workgroup: put(t, start, count) for every tile, and the list total.  The
// counts are read as kRows rows of 1024 consecutive tiles, every load issued
// before the first is used (coalesced, all in flight); each wave scans its
// 64 lanes of every row with DPP steps, and one wave scans the (row, wave)
// totals, which gives every (row, wave) its start.
template <int kRows, class Put>
__device__ __forceinline__ unsigned long long tile_starts(const uint32_t (&v)[kRows], int T, Put put) {
    constexpr int kWaves = kBinThreads / 64;
    constexpr int kPre = (kRows * kWaves + 63) / 64;
    __shared__ uint32_t wsum[kRows][kWaves];
    __shared__ unsigned long long wpre[kRows * kWaves + 1];
    const int tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    const int rows = (T + kBinThreads - 1) / kBinThreads;
    uint32_t incl[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        incl[r] = wave_scan_u32(v[r]);
        if (lane == 63) wsum[r][wave] = incl[r];
    }
    __syncthreads();
    // wave 0: the exclusive prefix of the (row, wave) totals in row-major
    // order, kPre per lane, and the list total after them
    if (wave == 0) {
        unsigned long long part[kPre], s = 0;
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int i = lane * kPre + k;
            part[k] = s;
            s += i < rows * kWaves ? wsum[i / kWaves][i % kWaves] : 0u;
        }
        unsigned long long pre = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long u = __shfl_up(pre, o);
            if (lane >= o) pre += u;
        }
        pre -= s;
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const int i = lane * kPre + k;
            if (i < kRows * kWaves) wpre[i] = pre + part[k];
        }
        if (lane == 63) wpre[kRows * kWaves] = pre + s;
    }
    __syncthreads();
    // start of this thread's tile in each row: the (row, wave) start, then
    // the lanes before it
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        if (r >= rows) break;
        const int t = r * kBinThreads + tid;
        if (t < T) put(t, (uint64_t)(wpre[r * kWaves + wave] + (incl[r] - v[r])), v[r]);
    }
    return wpre[kRows * kWaves];
}

// The tiles by falling list length (4 classes per octave, in any order within
// one; no list: last), by one workgroup beside those of the launch that finds
// the offsets.  A class has kCopies counters, so that fewer lanes of a wave
// meet in one.
__device__ __forceinline__ void order_tiles(const Job& J) {
    constexpr int kClasses = 64, kCopies = 4, kLoads = 4;
    __shared__ uint32_t next[kCopies][kClasses];
    const int T = J.F.tiles_x * J.F.tiles_y;
    const global_t<const uint32_t>* __restrict__ const cnt = to_global((const uint32_t*)J.bb.tile_cnt);
    global_t<uint32_t>* __restrict__ const order = to_global(tile_order(J.bb, T));
    const int tid = threadIdx.x, lane = __lane_id();
    uint32_t* const mine = next[lane & (kCopies - 1)];
    // exponent and two bits of the mantissa, from 1 on
    auto class_of = [](uint32_t n) { return (int)min((__float_as_uint((float)n) >> 21) - (127u << 2) + 1u, (uint32_t)kClasses - 1u); };
    if (tid < kClasses * kCopies) next[tid / kClasses][tid % kClasses] = 0u;
    __syncthreads();
    // every tile's count, kLoads at a time: f(tile, count, whether it exists)
    auto each = [&](auto f) {
        for (int t0 = 0; t0 < T; t0 += kLoads * kBinThreads) {
            uint32_t v[kLoads];
#pragma unroll
            for (int k = 0; k < kLoads; ++k) {
                const int t = t0 + k * kBinThreads + tid;
                v[k] = t < T ? cnt[t] : 0u;
            }
#pragma unroll
            for (int k = 0; k < kLoads; ++k) f(t0 + k * kBinThreads + tid, v[k], t0 + k * kBinThreads + tid < T);
        }
    };
    // the empty tiles, most of many images, are counted once per wave
    uint32_t empty = 0;
    each([&](int, uint32_t n, bool in) {
        if (n) atomicAdd(&mine[class_of(n)], 1u);
        empty += (uint32_t)__popcll(__ballot(in && n == 0u));
    });
    if (empty && lane == 0) atomicAdd(&next[0][0], empty);
    __syncthreads();
    if (tid < 64) {
        uint32_t c[kCopies], sum = 0;
#pragma unroll
        for (int k = 0; k < kCopies; ++k) {
            c[k] = sum;
            sum += next[k][kClasses - 1 - tid];
        }
        const uint32_t start = wave_scan_u32(sum) - sum;
#pragma unroll
        for (int k = 0; k < kCopies; ++k) next[k][kClasses - 1 - tid] = start + c[k];
    }
    __syncthreads();
    uint32_t at = 0;
    if (empty && lane == 0) at = atomicAdd(&next[0][0], empty);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    each([&](int t, uint32_t n, bool in) {
        const unsigned long long none = __ballot(in && n == 0u);
        if (n) order[atomicAdd(&mine[class_of(n)], 1u)] = (uint32_t)t;
        else if (in) order[at + (uint32_t)__popcll(none & __lanemask_lt())] = (uint32_t)t;
        at += (uint32_t)__popcll(none);
    });
}

// The frame counters of a job's lists: their total, whether it passes the
// capacity, and how many tiles' lists do (n_over, per thread; the scatter
// leaves those out).  The whole workgroup.
__device__ __forceinline__ void publish_lists(const Job& J, unsigned long long total, uint32_t n_over) {
    __shared__ uint32_t over_sum;
    if (threadIdx.x == 0) over_sum = 0;
    __syncthreads();
    for (int o = 32; o > 0; o >>= 1) n_over += (uint32_t)__shfl_xor((int)n_over, o);
    if (__lane_id() == 0 && n_over) atomicAdd(&over_sum, n_over);
    __syncthreads();
    if (threadIdx.x == 0) {
        J.bb.ctr->pairs = total;
        J.bb.ctr->overflow = total > J.bb.capacity ? 1u : 0u;
        J.bb.ctr->overflow_tiles = over_sum;
    }
}

// Scatter.  Every workgroup reserves, for each tile its primitives touch,
// one run of that tile's list (one global atomic), then places its visible
// primitives kScatterPer per thread at a time, all their loads issued
// before any is used.  Lanes of a wave whose primitive lies in one tile take
// their slots by runs of consecutive lanes with the same tile (one LDS
// atomic per run, in one instruction for the wave).  Primitives spanning
// several tiles take one LDS atomic per tile.  Workgroup 0 also publishes
// the frame counters.
// List offsets: every workgroup scans the tile counts for itself while its
// reservations are in flight, and workgroup 0 stores the offsets for the
// resolve.  The counts come from L2, which costs less than the 4 to 5 us of a
// launch of one workgroup per job on small frames (4,096 atoms at 256x256:
// 51.5 us with the launch, 48.3 without; 1M atoms and bonds at 1080p: 170.2
// and 167.1) and as much on large ones (four views up to 1440p 158 both; 11M
// spheres at 4K, 512 workgroups: 640 both; 256 renders of 50,000 atoms: 9,430
// to 9,445 both).
// kParts: parts of kScanTiles tiles.  With two the reservations follow the
// scan, part by part: 16 rows of both at once do not fit the 64 registers (44
// to 49 spilled).
constexpr int kScatterPer = 4;
constexpr int kScanTiles = 8 * kBinThreads;
static_assert(kMaxLdsTiles <= 2 * kScanTiles, "one or two parts");

template <class JS, int kParts>
__global__ void __launch_bounds__(kBinThreads, 8) k_scatter(JS js, int phase) {
    constexpr int kRows = kScanTiles / kBinThreads;
    extern __shared__ uint32_t cur[];
    uint32_t blk;
    const int ji = js.find(blockIdx.x, blk);
    if (ji < 0) {
        if (JS::kOrdered) order_tiles(js.job(0));
        return;
    }
    const Job& J = js.job(ji);
    const Frame F = J.F;
    const uint32_t chunk = J.bb.chunk;
    const global_t<const uint32_t>* __restrict__ const vis_src = to_global(J.bb.vis_src);
    const global_t<const uint2>* __restrict__ const vis_rect = to_global(J.bb.vis_rect);
    const global_t<const uint32_t>* __restrict__ const vis_cnt = to_global(J.bb.vis_cnt);
    const global_t<const uint32_t>* __restrict__ const hist_in = to_global(J.bb.hist);
    const global_t<const uint32_t>* __restrict__ const cnt = to_global(J.bb.tile_cnt);
    global_t<uint64_t>* __restrict__ const off = to_global(J.bb.tile_off);
    global_t<uint2>* __restrict__ const list = to_global(J.bb.list);
    const uint64_t capacity = J.bb.capacity;
    Counters* const ctr = J.bb.ctr;
    Counters* const host_ctr = J.bb.host_ctr;
    const int T = F.tiles_x * F.tiles_y;
    // this workgroup's layer: its runs go after those of the layers before it
    const uint32_t lay = J.bb.layers > 1 ? layer_of(blk, J.bb.groups, J.bb.layers) : 0u;
    uint32_t* const fill = J.bb.tile_fill + (size_t)lay * T;
    const global_t<const uint32_t>* __restrict__ const loff =
        J.bb.layers > 1 ? to_global(J.bb.layer_off + (size_t)lay * T) : nullptr;
    const int tid = threadIdx.x;
    const bool lead = blk == 0;
    const global_t<const uint32_t>* const row = hist_in + (size_t)blk * T;
    {
        // the workgroup's tile box (its primitives touch no tile outside it,
        // whose cursors are never read); the box's counts first, then the
        // reservations of the touched tiles, so the loads and atomics overlap
        const uint2 box = to_global(J.bb.vis_box)[blk];
        const uint32_t bx0 = box.x & 0xFFFFu, by0 = box.x >> 16, bx1 = box.y & 0xFFFFu, by1 = box.y >> 16;
        const int bw = bx0 <= bx1 ? (int)(bx1 - bx0) + 1 : 0, nb = bw * (bw ? (int)(by1 - by0) + 1 : 0);
        uint32_t h[kRows], r[kRows], v[kRows];
        // kRows rows of the box from row q0 on: their reservations, and then
        // their cursors
        auto reserve = [&](int q0) {
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                const int i = (q0 + q) * kBinThreads + tid;
                h[q] = i < nb ? row[i] : 0u;
                if (kParts == 1) v[q] = i < T ? cnt[i] : 0u;
            }
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                const int i = (q0 + q) * kBinThreads + tid;
                r[q] = h[q] ? atomicAdd(&fill[box_tile(F.tiles_x, bx0, by0, bw, i)], h[q]) : 0u;
            }
        };
        auto place = [&](int q0) {
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                const int i = (q0 + q) * kBinThreads + tid;
                if (i >= nb) break;
                const int t = box_tile(F.tiles_x, bx0, by0, bw, i);
                const uint32_t run = cur[t];
                if (h[q] && run != kNoRun) cur[t] = run + (loff ? loff[t] : 0u) + r[q];
            }
        };
        if (kParts == 1) reserve(0);   // in flight during the scan
        uint32_t n_over = 0;
        unsigned long long total = 0;
#pragma unroll 1
        for (int part = 0; part < kParts; ++part) {
            const int t0 = part * kScanTiles;
            if (kParts > 1) {
#pragma unroll
                for (int q = 0; q < kRows; ++q) {
                    const int t = t0 + q * kBinThreads + tid;
                    v[q] = t < T ? cnt[t] : 0u;
                }
            }
            total += tile_starts<kRows>(v, T - t0, [&](int t, uint64_t in, uint32_t n) {
                const uint64_t o = total + in;
                const bool fits = o + n <= capacity;   // else the resolve rebuilds this tile from the visible lists
                cur[t0 + t] = fits ? (uint32_t)o : kNoRun;
                if (lead) off[t0 + t] = o;
                n_over += fits ? 0u : 1u;
            });
        }
        if (lead) publish_lists(J, total, n_over);
        __syncthreads();   // every tile's start is in LDS
        if (kParts == 1) place(0);
        else
#pragma unroll 1
            for (int q0 = 0; q0 < kParts * kRows; q0 += kRows) {
                reserve(q0);
                place(q0);
            }
    }
    if (lead) {
        if (tid == 0) {
            const unsigned int vis = ctr->vis_count, bad = ctr->bad_bonds;
            const unsigned long long total = ctr->pairs;   // from publish_lists
            const unsigned int n_over = ctr->overflow_tiles;
            ctr->vis_count = 0;            // the next frame's count kernel adds to these
            ctr->bad_bonds = 0;
            ctr->frag_tested = 0;          // this frame's resolve adds to these
            ctr->frag_hit = 0;
            ctr->frag_hit_bond = 0;
            ctr->frag_tested_bond = 0;
            ctr->frag_skipped = 0;
            ctr->rec_culled = 0;
            ctr->lists_stopped = 0;
            ctr->chunks_stopped = 0;
            ctr->pairs_counted = 0;
            // the next frame's cluster test adds to these (the rest pass reads them)
            if (phase != kPhaseFront)
                for (int k = 0; k < kDepthBuckets; ++k) ctr->vis_bucket[k] = ctr->rest_bucket[k] = 0;
            if (host_ctr && phase == kPhaseRest) {
                // a two-pass frame: visible primitives and overflowed tiles of
                // both passes, the larger list total
                host_ctr->vis_count += vis;
                host_ctr->bad_bonds += bad;
                if (total > host_ctr->pairs) host_ctr->pairs = total;
                host_ctr->overflow |= total > capacity ? 1u : 0u;
                host_ctr->overflow_tiles += n_over;
            } else if (host_ctr) {
                host_ctr->vis_count = vis;
                host_ctr->bad_bonds = bad;
                host_ctr->pairs = total;
                host_ctr->overflow = total > capacity ? 1u : 0u;
                host_ctr->overflow_tiles = n_over;
                host_ctr->frag_tested = 0;
                host_ctr->frag_hit = 0;
                host_ctr->frag_hit_bond = 0;
                host_ctr->frag_tested_bond = 0;
                host_ctr->frag_skipped = 0;
                host_ctr->rec_culled = 0;
                host_ctr->lists_stopped = 0;
                host_ctr->chunks_stopped = 0;
            }
        }
    }
    __syncthreads();
    // at the end of the workgroup's work, when the counters' stores are long
    // done; a counting frame's follow the fragment counters (k_publish)
    auto stamp = [&]() {
        if (lead && tid == 0 && host_ctr && phase != kPhaseFront && !(F.flags & (1u | 16u)))
            stamp_counters(host_ctr, J.bb.stamp);
    };
    const uint32_t n = vis_cnt[blk];
    if (n == 0) {
        stamp();
        return;
    }
    const global_t<const uint32_t>* __restrict__ const my_src = vis_src + (size_t)blk * chunk;
    const global_t<const uint2>* __restrict__ const my_rect = vis_rect + (size_t)blk * chunk;
    const int ts = F.tile, tsh = F.tile_shift;
    // the footprint clipped to tile (tx, ty), in tile-local pixels
    auto local_fp = [&](int x0, int y0, int x1, int y1, int tx, int ty) -> uint32_t {
        const int lx0 = max(x0 - tx * ts, 0), ly0 = max(y0 - ty * ts, 0);
        const int lx1 = min(x1 - tx * ts, ts - 1), ly1 = min(y1 - ty * ts, ts - 1);
        return (uint32_t)lx0 | ((uint32_t)ly0 << 8) | ((uint32_t)(lx1 - lx0 + 1) << 16) |
               ((uint32_t)(ly1 - ly0 + 1) << 24);
    };
    const int lane = __lane_id();
    constexpr uint32_t kSpan = (uint32_t)kBinThreads * kScatterPer;
    for (uint32_t base = 0; base < n; base += kSpan) {   // uniform trip count (wave ops inside)
        uint32_t src[kScatterPer];
        uint2 rc[kScatterPer];
#pragma unroll
        for (int p = 0; p < kScatterPer; ++p) {
            // past the end: a copy of the last entry, dropped below (loads stay in bounds)
            const uint32_t k = min(base + (uint32_t)(p * kBinThreads + tid), n - 1u);
            src[p] = my_src[k];
            rc[p] = my_rect[k];
        }
        // the single-tile primitives of all kScatterPer batches take their
        // slots first (their atomics and slot exchanges overlap), then write
        // their entries; the primitives spanning several tiles follow
        uint32_t slot[kScatterPer];
        bool single[kScatterPer];
#pragma unroll
        for (int p = 0; p < kScatterPer; ++p) {
            const bool have = base + (uint32_t)(p * kBinThreads + tid) < n;
            const int x0 = rc[p].x & 0xFFFF, y0 = rc[p].x >> 16, x1 = rc[p].y & 0xFFFF, y1 = rc[p].y >> 16;
            single[p] = have && (x0 >> tsh) == (x1 >> tsh) && (y0 >> tsh) == (y1 >> tsh);
            const int t1 = single[p] ? (y0 >> tsh) * F.tiles_x + (x0 >> tsh) : -1;
            // one LDS atomic per run of lanes with the same tile; the run's
            // lanes take consecutive slots after its head's
            int head;
            uint32_t len;
            lane_run(t1, head, len);
            const uint32_t first = single[p] && head == lane ? atomicAdd(&cur[t1], len) : 0u;
            slot[p] = (uint32_t)__shfl((int)first, head) + (uint32_t)(lane - head);
        }
#pragma unroll
        for (int p = 0; p < kScatterPer; ++p) {
            if (single[p] && !(slot[p] & kNoRun)) {
                // inside its one tile: the rectangle in tile-local pixels, unclipped
                const uint32_t x0 = rc[p].x & 0xFFFFu, y0 = rc[p].x >> 16, x1 = rc[p].y & 0xFFFFu, y1 = rc[p].y >> 16;
                const uint32_t m = (uint32_t)ts - 1u;
                list[slot[p]] = make_uint2(src[p], (x0 & m) | ((y0 & m) << 8) | ((x1 - x0 + 1u) << 16) |
                                                       ((y1 - y0 + 1u) << 24));
            }
        }
#pragma unroll
        for (int p = 0; p < kScatterPer; ++p) {
            const bool have = base + (uint32_t)(p * kBinThreads + tid) < n;
            if (have && !single[p]) {
                const int x0 = rc[p].x & 0xFFFF, y0 = rc[p].x >> 16, x1 = rc[p].y & 0xFFFF, y1 = rc[p].y >> 16;
                for (int ty = y0 >> tsh; ty <= (y1 >> tsh); ++ty)
                    for (int tx = x0 >> tsh; tx <= (x1 >> tsh); ++tx) {
                        const uint32_t sl = atomicAdd(&cur[ty * F.tiles_x + tx], 1u);
                        if (!(sl & kNoRun)) list[sl] = make_uint2(src[p], local_fp(x0, y0, x1, y1, tx, ty));
                    }
            }
        }
    }
    stamp();
}

}  // namespace

// Two workgroups of 16 waves fill a CU, so a large scene takes 512 workgroups
// of 4096 primitives or more.  Below that the launch leaves CUs idle and each
// workgroup's primitives are a serial chain (four rounds of 1024 threads for
// 4096), so a single render cuts them finer: 512 primitives each up to 128
// workgroups, 1024 up to 256.  Past those the finer cut loses: every
// workgroup adds to, and reserves a run in, each tile it touches (count and
// scatter of a figure of large spheres at 3840x2160: 36 us in 128 workgroups,
// 44 in 256).  4,096 atoms at 256x256 take 29 us in one workgroup and 14 in 8;
// 50,000 at 720p 34 us in 13 and 18 in 98.  A batch's renders share the device: 512 workgroups over all of them
// are enough, and 256 renders of 50,000 atoms lose 8 % with 98 each.
void bin_grid(uint64_t nprim, uint64_t renders, uint32_t* groups, uint32_t* chunk) {
    const uint64_t share = std::max<uint64_t>(1, kMaxBinGroups / std::max<uint64_t>(1, renders));
    auto cut = [&](uint64_t per, uint64_t most) { return std::min((nprim + per - 1) / per, most); };
    uint64_t g = std::max(cut(4096, kMaxBinGroups),
                          std::max(cut(512, std::min<uint64_t>(128, share)), cut(1024, std::min<uint64_t>(256, share))));
    if (g < 1) g = 1;
    uint64_t c = (nprim + g - 1) / g;
    if (c < 1) c = 1;
    *groups = (uint32_t)g;
    *chunk = (uint32_t)c;
}

hipError_t launch_zero(uint32_t* p, size_t n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    size_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > 4096) blocks = 4096;
    k_zero<<<(unsigned)blocks, kBlock, 0, stream>>>(p, n);
    return hipGetLastError();
}

// A render, or a batch, of scenes without bonds takes the atom-only count.
inline bool atoms_only(const OneJob& js) { return js.j.S.bond_clusters == 0; }
inline bool atoms_only(const JobList& js) { return js.no_bonds != 0; }

// A scene of few clusters per binning workgroup is dealt by quarters: whole
// clusters would leave most of the workgroup's 16 waves without work
// (107,500 atoms with bonds, two clusters per workgroup: 16.6 us by clusters,
// 10.7 by quarters).  So is any scene with bonds (1M atoms and bonds: 32 us
// either way); large atom-only scenes are not, whose waves then wait on a
// cluster id per quarter (100M atoms: 170 us by clusters, 185 by quarters;
// 256 renders of 50,000 atoms 121 and 129).
inline bool quarters(const OneJob& js) { return js.j.S.atom_clusters <= kFewClusters * js.j.bb.groups; }
inline bool quarters(const JobList& js) { return js.few_clusters != 0; }

template <class JS>
hipError_t count_impl(const JS& js, BinForm form, int phase, uint32_t grid, int max_tiles, hipStream_t stream) {
    const bool scene = form == kBinClusters;
    if (max_tiles > kMaxLdsTiles) return hipErrorInvalidValue;
    if (phase != kPhaseAll && !scene) return hipErrorInvalidValue;
    if (grid == 0) return hipSuccess;
    const size_t lds = (size_t)max_tiles * sizeof(uint32_t);
    if (form == kBinStored)
        return dispatch(k_count<JS, false, false, false, false, true>, grid, kBinThreads, lds, stream, js, phase);
    if (!scene) return dispatch(k_count<JS, false, false>, grid, kBinThreads, lds, stream, js, phase);
    if (phase == kPhaseRest) return dispatch(k_count<JS, true, true>, grid, kBinThreads, lds, stream, js, phase);
    if (!atoms_only(js)) return dispatch(k_count<JS, true, false, false, true>, grid, kBinThreads, lds, stream, js, phase);
    if (quarters(js) || phase == kPhaseFront) return dispatch(k_count<JS, true, false, true, true>, grid, kBinThreads, lds, stream, js, phase);
    return dispatch(k_count<JS, true, false, true>, grid, kBinThreads, lds, stream, js, phase);
}

template <class JS>
hipError_t scatter_impl(const JS& js, int phase, uint32_t grid, int max_tiles, hipStream_t stream) {
    if (max_tiles > kMaxLdsTiles) return hipErrorInvalidValue;
    if (grid == 0) return hipSuccess;
    const uint32_t lds = (uint32_t)(max_tiles * sizeof(uint32_t));
    // the workgroup that orders the tiles comes after the others: it takes
    // less time than they do, also where it has to wait for a CU
    const uint32_t extra = JS::kOrdered && max_tiles > kOrderTiles ? 1u : 0u;
    if (max_tiles <= kScanTiles) return dispatch(k_scatter<JS, 1>, grid + extra, kBinThreads, lds, stream, js, phase);
    return dispatch(k_scatter<JS, 2>, grid + extra, kBinThreads, lds, stream, js, phase);
}

hipError_t launch_count(const OneJob& js, BinForm form, int phase, uint32_t grid, int max_tiles, hipStream_t stream) {
    return count_impl(js, form, phase, grid, max_tiles, stream);
}
hipError_t launch_count(const JobList& js, BinForm form, int phase, uint32_t grid, int max_tiles, hipStream_t stream) {
    return count_impl(js, form, phase, grid, max_tiles, stream);
}
hipError_t launch_layers(const OneJob& js, uint32_t grid, hipStream_t stream) {
    return dispatch(k_layers<OneJob>, grid, kBinThreads, 0, stream, js);
}
hipError_t launch_layers(const JobList& js, uint32_t grid, hipStream_t stream) {
    return dispatch(k_layers<JobList>, grid, kBinThreads, 0, stream, js);
}
hipError_t launch_scatter(const OneJob& js, int phase, uint32_t grid, int max_tiles, hipStream_t stream) {
    return scatter_impl(js, phase, grid, max_tiles, stream);
}
hipError_t launch_scatter(const JobList& js, int phase, uint32_t grid, int max_tiles, hipStream_t stream) {
    return scatter_impl(js, phase, grid, max_tiles, stream);
}

}  // namespace vtx
