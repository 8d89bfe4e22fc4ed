// Solvent excluded surface on a grid, extracted by marching cubes (paper,
// Methods, "Cartoon and SES representations": a discrete SES, as in Lindow
// et al., extracted with marching cubes).
//
// Readings (the paper gives no formulas):
//  - grid point (i, j, k) is at o + h (i, j, k) in FP64; it lies inside the
//    solvent-accessible region when some atom has |p - c|^2 < (r + rp)^2,
//    each square and sum rounded once in FP64; the others are positions a
//    probe centre can take ("exterior");
//  - f(p) = min(h sqrt(g), W h) - rp, g the least squared grid distance from
//    p to an exterior point, W = ceil(rp / h) + 2 (beyond W h only the sign
//    matters), rounded to FP32; the SES encloses f >= 0;
//  - marching cubes over f >= 0 with a case table built from the cube's
//    faces: each face with two crossing edges gives a segment, a face whose
//    inside corners are diagonal gives two segments cutting off the inside
//    corners; segments close into loops, oriented from the inside corners to
//    the outside ones and started at their lowest edge; a 3-edge loop is a
//    triangle, a longer one a fan around the mean of its vertices.
//
// Passes: mark the SAS interior per atom, one bit per point; the exact
// squared distance to the nearest exterior point within a W-box by three
// separable 1-D passes in integers (x: nearest exterior point on the row; y
// and z: the least of g + d^2 over the window), all three in LDS per brick of
// points when W is small, then the field and one sign bit per point; triangle
// counts per run of cubes from the sign bits, an exclusive scan of those
// (scan.hip), and the triangles of each run's cubes that have any.
#include <mutex>

#include "vtx_internal.h"

namespace vtx {

namespace {

constexpr int kSesBlock = 256;
constexpr int kSesMarkBlock = 64;      // one wave per atom: its box setup is paid once per wave
constexpr int kSesRun = 64;            // words of sign bits (up to 32 cubes each) per run of cubes
// Windows up to which a brick's distances fit LDS, which is also where they
// pay: the whole call for 9.4M points and W = 7, 9, 11, 12 in LDS 116, 153, 176,
// 160 us, through memory 251, 250, 273, 270 (and 288 for 13).
constexpr int kMaxFusedW = 12;
constexpr int32_t kFar = 0x3FFFFFFF;   // no exterior point within the window

// Case table: for each case, one word with its loops' edges in order, 4 bits
// each from bit 0 (12 at most), and the loops' lengths, 4 bits each from bit
// 48 (4 loops at most; 0 ends them), so that a cube's thread reads its case
// at once.  Edges 0-3 run along x, 4-7 along y, 8-11 along z (corner pairs
// below); corner c sits at (c & 1, c >> 1 & 1, c >> 2 & 1).
__constant__ unsigned long long c_cases[256];
__constant__ uint8_t c_case_tris[256];

constexpr int kEdgeA[12] = {0, 2, 4, 6, 0, 1, 4, 5, 0, 1, 2, 3};
constexpr int kEdgeB[12] = {1, 3, 5, 7, 2, 3, 6, 7, 4, 5, 6, 7};
int edge_of(int a, int b) {
    if (a > b) {
        const int t = a;
        a = b;
        b = t;
    }
    for (int e = 0; e < 12; ++e)
        if (kEdgeA[e] == a && kEdgeB[e] == b) return e;
    return -1;
}

// The loops of case m, built as the table's rule states.
void build_case(int m, unsigned long long* out, uint8_t* ntri) {
    static const int faces[6][4] = {{0, 2, 6, 4}, {1, 3, 7, 5}, {0, 1, 5, 4}, {2, 3, 7, 6}, {0, 1, 3, 2}, {4, 5, 7, 6}};
    int in[8];
    for (int c = 0; c < 8; ++c) in[c] = (m >> c) & 1;
    int nb[12][2], deg[12] = {};
    auto link = [&](int a, int b) {
        nb[a][deg[a]++] = b;
        nb[b][deg[b]++] = a;
    };
    for (const auto& f : faces) {
        int e[4], s[4], nc = 0, cr[4];
        for (int i = 0; i < 4; ++i) {
            s[i] = in[f[i]];
            e[i] = edge_of(f[i], f[(i + 1) & 3]);
        }
        for (int i = 0; i < 4; ++i)
            if (s[i] != s[(i + 1) & 3]) cr[nc++] = i;
        if (nc == 2) {
            link(e[cr[0]], e[cr[1]]);
        } else if (nc == 4) {
            for (int i = 0; i < 4; ++i)
                if (s[i]) link(e[(i + 3) & 3], e[i]);
        }
    }
    bool used[12] = {};
    int pos = 0, loops = 0, tris = 0;
    unsigned long long w = 0;
    for (int start = 0; start < 12; ++start) {
        if (deg[start] == 0 || used[start]) continue;
        int loop[12], k = 0;
        loop[k++] = start;
        used[start] = true;
        int prev = start, cur = nb[start][0];
        while (cur != start) {
            loop[k++] = cur;
            used[cur] = true;
            const int nxt = nb[cur][0] == prev ? nb[cur][1] : nb[cur][0];
            prev = cur;
            cur = nxt;
        }
        // orientation: the loop's normal over its edge midpoints against the
        // sum of the inside -> outside directions of its edges
        double mid[12][3], nrm[3] = {0, 0, 0}, dir[3] = {0, 0, 0};
        for (int i = 0; i < k; ++i) {
            const int a = kEdgeA[loop[i]], b = kEdgeB[loop[i]];
            for (int d = 0; d < 3; ++d) {
                const double pa = (a >> d) & 1, pb = (b >> d) & 1;
                mid[i][d] = 0.5 * (pa + pb);
                dir[d] += in[a] ? pb - pa : pa - pb;
            }
        }
        for (int i = 0; i < k; ++i) {
            const double* p = mid[i];
            const double* q = mid[(i + 1) % k];
            nrm[0] += p[1] * q[2] - p[2] * q[1];
            nrm[1] += p[2] * q[0] - p[0] * q[2];
            nrm[2] += p[0] * q[1] - p[1] * q[0];
        }
        if (nrm[0] * dir[0] + nrm[1] * dir[1] + nrm[2] * dir[2] < 0.0)
            for (int i = 0; i < k / 2; ++i) {
                const int t = loop[i];
                loop[i] = loop[k - 1 - i];
                loop[k - 1 - i] = t;
            }
        int lo = 0;
        for (int i = 1; i < k; ++i)
            if (loop[i] < loop[lo]) lo = i;
        w |= (unsigned long long)k << (48 + 4 * loops++);
        for (int i = 0; i < k; ++i) w |= (unsigned long long)loop[(lo + i) % k] << (4 * pos++);
        tris += k == 3 ? 1 : k;
    }
    *out = w;
    *ntri = (uint8_t)tris;
}

std::mutex g_case_mu;
bool g_case_ready[64] = {};

hipError_t ensure_cases(int device) {
    std::lock_guard<std::mutex> lk(g_case_mu);
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    if (g_case_ready[device]) return hipSuccess;
    static unsigned long long cases[256];
    static uint8_t ntri[256];
    for (int m = 0; m < 256; ++m) build_case(m, cases + m, ntri + m);
    hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_cases), cases, sizeof(cases));
    if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_case_tris), ntri, sizeof(ntri));
    if (e == hipSuccess) g_case_ready[device] = true;
    return e;
}

struct SesGrid {
    double o[3];
    double h;
    double inv_h;       // 1 / h (bounding boxes only)
    int nx, ny, nz;
    int W;              // distance window in grid steps
    double rp;
    // Margin of an atom's box in steps: slack0 + reach slack.  The box's ends
    // and the points' coordinates are rounded at the magnitude of the origin,
    // the points, the atom and its reach (eight roundings of 2^-53 at most in
    // all); an atom that reaches the grid is no further than the grid's
    // farthest point and its reach.  The product by 1 / h is rounded at the
    // magnitude of the grid coordinates (below 2^31, so by less than 2e-6).
    double slack0, slack;
};

__device__ inline size_t gidx(const SesGrid& G, int i, int j, int k) {
    return (size_t)i + (size_t)G.nx * ((size_t)j + (size_t)G.ny * k);
}

// The mark of a point is one bit: word (i / 4, j / 4, k / 4) of 64 bits holds
// a 4 x 4 x 4 cell of points, bit (k & 3) 16 + (j & 3) 4 + (i & 3).
struct MarkGrid {
    unsigned long long* bits;
    int nx, ny;          // cells along x and y
};
inline int mark_cells(int n) { return (n + 3) / 4; }

// Several atoms per wave (k_ses_mark), for grids with few points per atom,
// whose boxes of some eight cells leave most of a wave's lanes idle: the lanes
// take the cells of all its atoms in turn.  The wave's atoms lie a grid's width
// apart in the input, so neighbours in space, which often are neighbours there,
// do not meet in one wave.  1M atoms of reach 2.6 to 3.2, the whole call with a
// wave per atom and per 8: spacing 0.7 1,010 and 593 us, 1.4 845 and 214, 5 733
// and 150 (lanes by (x, y) columns of a byte grid: 2,727, 663 and 376).
constexpr int kMarkAtoms = 8;
constexpr uint64_t kManyPoints = 100;   // grid points per atom below which it is done

// An atom's box: centre, squared reach, first cell and cells.
struct AtomBox {
    double c[3], R2;
    int lo[3], nc[3];
};

// kAtoms atoms per wave: sets the bits of the grid points inside their
// solvent-accessible spheres (points no atom marks stay 0: exterior), one lane
// per 4 x 4 x 4 cell of an atom's box, one atomic per cell that has any.  The
// squared offsets and the two sums are rounded as the reading states; each
// rounding is monotone, so a cell whose nearest (farthest) corner fails
// (passes) the test is empty (full) without testing its points.  Bounded by
// the point tests' VALU instructions: 50,000 atoms of reach 2.6 to 3.2 at
// spacing 0.5 take 45 us, and took 90 with a byte per point (249 MB of
// write-backs for a 10 MB grid).  One atom's box stays in registers and the
// cell's test in the kernel itself: as functions of the box it was 1 to 3 us
// slower.
template <int kAtoms>
__global__ void __launch_bounds__(kSesMarkBlock) k_ses_mark(const float* __restrict__ pos,
                                                            const float* __restrict__ rad, uint32_t n, SesGrid G,
                                                            MarkGrid M) {
#pragma clang fp contract(off)
    constexpr bool kMany = kAtoms > 1;
    __shared__ AtomBox box[kMany ? kAtoms : 1];
    __shared__ uint32_t first[kAtoms + 1];   // where each box's cells start among the wave's
    const int lane = threadIdx.x;
    AtomBox B;
    uint32_t cells = 0;
    if (!kMany || lane < kAtoms) {
        const uint64_t a = blockIdx.x + (kMany ? (uint64_t)lane * gridDim.x : 0u);
        bool ok = a < n;
        if (ok) {
            for (int d = 0; d < 3; ++d) B.c[d] = pos[3 * a + d];
            const double R = (double)rad[a] + G.rp;
            ok = R > 0.0;
            B.R2 = R * R;
            const int nmax[3] = {G.nx - 1, G.ny - 1, G.nz - 1};
            // the box only has to hold every point the test can mark: see SesGrid::slack
            const double margin = fma(R, G.slack, G.slack0);
            for (int d = 0; d < 3; ++d) {
                const double from = fmax(0.0, ceil((B.c[d] - R - G.o[d]) * G.inv_h - margin));
                const double to = fmin((double)nmax[d], floor((B.c[d] + R - G.o[d]) * G.inv_h + margin));
                ok = ok && from <= to && B.c[d] - B.c[d] == 0.0;   // else beside the grid, or not a finite position
                const int l = (int)from, h = (int)to;
                B.lo[d] = l >> 2;
                B.nc[d] = (h >> 2) - B.lo[d] + 1;
            }
        }
        if (ok) cells = (uint32_t)B.nc[0] * (uint32_t)B.nc[1] * (uint32_t)B.nc[2];
        if (kMany) {
            box[kMany ? lane : 0] = B;
            uint32_t end = cells;
#pragma unroll
            for (int o = 1; o < kAtoms; o <<= 1) {
                const uint32_t u = (uint32_t)__shfl_up((int)end, o);
                if (lane >= o) end += u;
            }
            first[lane + 1] = end;
            if (lane == 0) first[0] = 0;
        }
    }
    if (kMany) {
        __syncthreads();
        cells = first[kAtoms];   // at most 2^27 of a box: fewer than 2^31 points, 2 or more a side
    }
    for (uint32_t q = (uint32_t)lane; q < cells; q += kSesMarkBlock) {
        int at = (int)q;
        if (kMany) {
            int a = 0;
#pragma unroll
            for (int k = 1; k < kAtoms; ++k) a = q >= first[k] ? k : a;
            B = box[kMany ? a : 0];
            at = (int)(q - first[a]);
        }
        const int qz = at / (B.nc[0] * B.nc[1]), qr = at - qz * (B.nc[0] * B.nc[1]), qy = qr / B.nc[0], qx = qr - qy * B.nc[0];
        const int cell[3] = {B.lo[0] + qx, B.lo[1] + qy, B.lo[2] + qz};
        double s[3][4], near[3], far[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double x = (G.o[d] + G.h * (4 * cell[d] + t)) - B.c[d];
                s[d][t] = x * x;
            }
            near[d] = fmin(fmin(s[d][0], s[d][1]), fmin(s[d][2], s[d][3]));
            far[d] = fmax(s[d][0], s[d][3]);
        }
        if (!((near[0] + near[1]) + near[2] < B.R2)) continue;
        unsigned long long m = ~0ull;
        if (!((far[0] + far[1]) + far[2] < B.R2)) {
            uint32_t w[2] = {0u, 0u};
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double sxy = s[0][i] + s[1][j];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        w[k >> 1] |= sxy + s[2][k] < B.R2 ? 1u << ((k & 1) * 16 + j * 4 + i) : 0u;
                }
            m = ((unsigned long long)w[1] << 32) | w[0];
        }
        if (m) atomicOr(&M.bits[((size_t)cell[2] * M.ny + cell[1]) * M.nx + cell[0]], m);
    }
}

// The mark words' nibble of row (j, k) (points 4 c to 4 c + 3 of it).
__device__ inline uint32_t mark_nibble(const MarkGrid& M, int c, int j, int k) {
    const uint32_t* half = reinterpret_cast<const uint32_t*>(M.bits + ((size_t)(k >> 2) * M.ny + (j >> 2)) * M.nx + c) + (k >> 1 & 1);
    return *half >> ((k & 1) * 16 + (j & 3) * 4) & 15u;
}

// The per-point passes below run one thread per point in x-fastest order;
// the grid holds fewer than 2^31 points, so the index and its decomposition
// stay in 32 bits.
__device__ inline bool flat_item(uint32_t n, int nx, int ny, int& i, int& j, int& k, uint32_t& p) {
    p = blockIdx.x * (uint32_t)kSesBlock + threadIdx.x;
    if (p >= n) return false;
    const uint32_t r = p / (uint32_t)nx;
    i = (int)(p - r * (uint32_t)nx);
    j = (int)(r % (uint32_t)ny);
    k = (int)(r / (uint32_t)ny);
    return true;
}

// Field of a squared grid distance g (exterior point farther than the
// window: any g > W^2).
__device__ inline float ses_field(const SesGrid& G, int g) {
    const double cap = G.W * G.h;
    const double D = g > G.W * G.W ? cap : fmin(G.h * sqrt((double)g), cap);
    return (float)(D - G.rp);
}

// The three distance passes of one brick of kBx x kBy x kBz points in LDS
// (window kW <= kMaxFusedW), the field and the sign bits (f >= 0) of its rows.
// The points within kW of the brick along y and z are recomputed by each
// brick that needs them; nothing goes through memory between the passes.
// Squared distances fit 16 bits (3 kW^2 at most, 127^2 for none on the row),
// two points to a register:
// x0 + t and x0 + 16 + t, so that stores of the field are consecutive.  (Three
// passes over int32 grids: 136 us for 9.75M points and kW = 5, now 36.)
constexpr int kBx = 32, kBy = 16, kBz = 16;
constexpr int kEdtBlock = 512;
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

// out[c] = the least over |d| <= kW of col[c + kW + d] + d^2.
template <int kW, int kN>
__device__ inline void window_min(const us2 (&col)[kN + 2 * kW], us2 (&out)[kN]) {
#pragma unroll
    for (int c = 0; c < kN; ++c) {
        us2 best = col[c + kW];
#pragma unroll
        for (int d = 1; d <= kW; ++d) {
            const unsigned short dd = (unsigned short)(d * d);
            best = __builtin_elementwise_min(best, (us2)(__builtin_elementwise_min(col[c + kW - d], col[c + kW + d]) + (us2){dd, dd}));
        }
        out[c] = best;
    }
}

template <int kW>
__global__ void __launch_bounds__(kEdtBlock) k_ses_edt(SesGrid G, MarkGrid M, uint32_t nbx, uint32_t nby,
                                                       float* __restrict__ field, uint32_t* __restrict__ sign, int nxw) {
    constexpr int kRows = kBy + 2 * kW, kPlanes = kBz + 2 * kW, kPairs = kBx / 2;
    constexpr int kLead = (kW + 3) / 4 * 4, kNibbles = (kLead + kBx + kW + 3) / 4;
    static_assert(kNibbles <= 16, "a row's window fits 64 bits");
    constexpr int kHalf = kBz / 2;
    static_assert(kEdtBlock == 2 * kBy * kPairs, "half a z column per thread");
    __shared__ us2 g[kPlanes][kRows | 1][kPairs];   // an odd row count: a wave's four planes lie in different banks
    __shared__ unsigned long long ext[kPlanes * kRows];   // bit p of a row: point x0 - kW + p is exterior
    __shared__ float tab[kW * kW + 2];                    // field by squared distance
    const int tid = threadIdx.x;
    const uint32_t b = blockIdx.x, bx = b % nbx, br = b / nbx;
    const int x0 = (int)bx * kBx, y0 = (int)(br % nby) * kBy, z0 = (int)(br / nby) * kBz;
    for (int r = tid; r < kPlanes * kRows; r += kEdtBlock) {
        const int j = y0 - kW + r % kRows, k = z0 - kW + r / kRows;
        // every load first, at cells clamped to the grid, so they overlap;
        // points outside the grid are no exterior points
        const int jc = min(max(j, 0), G.ny - 1), kc = min(max(k, 0), G.nz - 1);
        const int c0 = (x0 - kLead) / 4;   // exact: both are multiples of 4
        uint32_t nib[kNibbles], w[2] = {0u, 0u};
#pragma unroll
        for (int q = 0; q < kNibbles; ++q) nib[q] = mark_nibble(M, min(max(c0 + q, 0), M.nx - 1), jc, kc);
#pragma unroll
        for (int q = 0; q < kNibbles; ++q) w[q >> 3] |= (c0 + q >= 0 && c0 + q < M.nx ? nib[q] : 15u) << (4 * (q & 7));
        unsigned long long in = (unsigned long long)w[1] << 32 | w[0];
        const int end = G.nx - (x0 - kLead);   // first position past the row
        if (end < 64) in |= ~0ull << end;
        if (j != jc || k != kc) in = ~0ull;
        ext[r] = ~in >> (kLead - kW);
    }
    for (int q = tid; q < kW * kW + 2; q += kEdtBlock) tab[q] = ses_field(G, q);
    __syncthreads();
    // x: the nearest exterior point of the row
    const int t = tid % kPairs;
    for (int r = tid / kPairs; r < kPlanes * kRows; r += kEdtBlock / kPairs) {
        us2 v;
        const uint32_t lo = (uint32_t)ext[r], hi = (uint32_t)(ext[r] >> 32);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t w = __builtin_amdgcn_alignbit(hi, lo, t + 16 * h);   // bit kW: the point itself
            const uint32_t right = w >> kW, left = w << (31 - kW);
            const uint32_t d = min(right ? (uint32_t)__builtin_ctz(right) : ~0u, left ? (uint32_t)__builtin_clz(left) : ~0u);
            // a distance past the window squares to more than kW^2: far, whatever it is
            v[h] = (unsigned short)__umul24(min(d, 127u), min(d, 127u));
        }
        g[r / kRows][r % kRows][t] = v;
    }
    __syncthreads();
    // y, in place: a thread reads its whole column first
    for (int q = tid; q < kPlanes * kPairs; q += kEdtBlock) {
        const int p = q / kPairs;
        us2 col[kRows], out[kBy];
#pragma unroll
        for (int c = 0; c < kRows; ++c) col[c] = g[p][c][t];
        window_min<kW, kBy>(col, out);
#pragma unroll
        for (int c = 0; c < kBy; ++c) g[p][c][t] = out[c];
    }
    __syncthreads();
    // z, the field and the signs
    const int y = tid / kPairs % kBy, j = y0 + y, zh = tid / (kPairs * kBy) * kHalf;
    us2 col[kHalf + 2 * kW], out[kHalf];
#pragma unroll
    for (int c = 0; c < kHalf + 2 * kW; ++c) col[c] = g[zh + c][y][t];
    window_min<kW, kHalf>(col, out);
    const int lane = __lane_id();
#pragma unroll
    for (int c = 0; c < kHalf; ++c) {
        const int k = z0 + zh + c;
        if (k >= G.nz) break;   // the same for the whole wave
        bool pos[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float f = tab[min((int)out[c][h], kW * kW + 1)];
            const int x = x0 + t + 16 * h;
            pos[h] = f >= 0.0f;
            if (x < G.nx && j < G.ny) field[gidx(G, x, j, k)] = f;
        }
        const unsigned long long lo = __ballot(pos[0]), hi = __ballot(pos[1]);
        if (t == 0 && j < G.ny) {
            const int sh = lane & ~(kPairs - 1);   // this row's 16 lanes
            sign[((size_t)k * G.ny + j) * nxw + bx] = (uint32_t)(lo >> sh & 0xFFFFu) | (uint32_t)(hi >> sh & 0xFFFFu) << 16;
        }
    }
}

// The passes of larger windows (or grids of too many bricks), through memory.
// x pass: squared distance along the row to the nearest exterior point
// within W steps (kFar if none).  Cells of four points outwards from the
// point's own, so a load serves four steps (9.4M points, W = 33: 260 us with a
// byte per point and step, 312 with a cell per step, 97 so).
__global__ void __launch_bounds__(kSesBlock) k_ses_edt_x(SesGrid G, uint32_t np, MarkGrid M, int32_t* __restrict__ g) {
    int i, j, k;
    uint32_t p;
    if (!flat_item(np, G.nx, G.ny, i, j, k, p)) return;
    // exterior points of cell c of the row (points past the row's end are none)
    auto exterior = [&](int c) -> uint32_t {
        const int end = G.nx - 4 * c;
        return ~mark_nibble(M, c, j, k) & (end < 4 ? (1u << end) - 1u : 15u);
    };
    const int own = i >> 2, at = i & 3;
    const uint32_t e = exterior(own);
    int d = G.W + 1;
    const uint32_t right = e >> at, left = e << (31 - at);
    if (right) d = __builtin_ctz(right);
    if (left) d = min(d, __builtin_clz(left));
    // the nearest point of the cells c steps out is 4 c - at to the left at
    // most, 4 c + at - 3 to the right
    for (int c = 1; 4 * c - 3 <= min(d - 1, G.W) && (own + c < M.nx || own - c >= 0); ++c) {
        if (own + c < M.nx) {
            const uint32_t r = exterior(own + c);
            if (r) d = min(d, 4 * c - at + __builtin_ctz(r));
        }
        if (own - c >= 0) {
            const uint32_t l = exterior(own - c);
            if (l) d = min(d, 4 * c + at - 31 + __builtin_clz(l));
        }
    }
    g[p] = d <= G.W ? d * d : kFar;
}

constexpr int kEdtMaxW = 32;   // windows the passes through LDS take

// The x pass through LDS (W <= kEdtMaxW): work block b takes kSesBlock
// consecutive points of one row (x block b mod nxb of row b / nxb) and stages
// their exterior bits and a word of them more on each side; a point's nearest
// ones are the first and last bits of the words that start and end at it.
// 9.4M points: 28 us for W = 13 to 32; a point's marks one after another from
// memory 146 and 301, from bytes in LDS 105 and 219.
__global__ void __launch_bounds__(kSesBlock) k_ses_edt_x_lds(SesGrid G, uint32_t nxb, MarkGrid M, int32_t* __restrict__ g) {
    static_assert(kEdtMaxW == 32, "a word of bits on each side");
    constexpr int kWords = kSesBlock / 32 + 2;
    static_assert(kWords * 8 <= kSesBlock, "a thread per nibble");
    __shared__ uint32_t ext[kWords];
    const uint32_t r = blockIdx.x / nxb, xb = blockIdx.x - r * nxb;
    const int t = threadIdx.x, x0 = (int)xb * kSesBlock;
    const int j = (int)(r % (uint32_t)G.ny), k = (int)(r / (uint32_t)G.ny);
    const int c = x0 / 4 - 8 + t, end = G.nx - 4 * c;   // points of the row from cell c on
    uint32_t w = 0;
    if (t < kWords * 8 && c >= 0 && end > 0) w = ~mark_nibble(M, c, j, k) & (end < 4 ? (1u << end) - 1u : 15u);
    w <<= 4 * (t & 7);
    w |= (uint32_t)__shfl_xor((int)w, 1);
    w |= (uint32_t)__shfl_xor((int)w, 2);
    w |= (uint32_t)__shfl_xor((int)w, 4);
    if (t < kWords * 8 && (t & 7) == 0) ext[t >> 3] = w;
    __syncthreads();
    const int i = x0 + t;
    if (i >= G.nx) return;
    const int q = t >> 5, s = t & 31;   // the point is bit s of word q + 1
    const uint32_t right = __builtin_amdgcn_alignbit(ext[q + 2], ext[q + 1], s);   // bit 0: the point
    const uint32_t left = s == 31 ? ext[q + 1] : __builtin_amdgcn_alignbit(ext[q + 1], ext[q], s + 1);   // bit 31: the point
    uint32_t d = (ext[q + 2] | ext[q]) >> s & 1u ? 32u : ~0u;
    if (right) d = min(d, (uint32_t)__builtin_ctz(right));
    if (left) d = min(d, (uint32_t)__builtin_clz(left));
    g[(size_t)r * G.nx + i] = d <= (uint32_t)G.W ? (int32_t)(d * d) : kFar;
}

// y or z pass: the least of g(p + d e) + d^2 over |d| <= W along the axis.
// The z pass also writes the field.
template <bool kLast>
__global__ void __launch_bounds__(kSesBlock) k_ses_edt_yz(SesGrid G, uint32_t np, const int32_t* __restrict__ gin,
                                                          int32_t* __restrict__ gout, float* __restrict__ field) {
    int i, j, k;
    uint32_t p;
    if (!flat_item(np, G.nx, G.ny, i, j, k, p)) return;
    const int stride = kLast ? G.nx * G.ny : G.nx;
    const int len = kLast ? G.nz : G.ny;
    const int at = kLast ? k : j;
    int32_t best = kFar;
    for (int d = -G.W; d <= G.W; ++d) {
        const int q = at + d;
        if (q < 0 || q >= len) continue;
        const int32_t v = gin[(int)p + d * stride];
        if (v < kFar) best = min(best, v + d * d);
    }
    if (!kLast) {
        gout[p] = best;
        return;
    }
    field[p] = ses_field(G, best);
}

// The same passes through LDS (windows of W <= kEdtMaxW): work block b
// takes kEdtX consecutive x of one slice (z for the y pass, y for the z pass)
// and kEdtRows consecutive positions along the axis, stages those rows and
// W more on each side in LDS (one load per staged value), and each thread
// then takes the window minima of its column from LDS.
constexpr int kEdtX = 64, kEdtRows = 32;

template <bool kLast>
__global__ void __launch_bounds__(kSesBlock) k_ses_edt_yz_lds(SesGrid G, uint32_t nxb, uint32_t nrb,
                                                              const int32_t* __restrict__ gin,
                                                              int32_t* __restrict__ gout, float* __restrict__ field) {
    __shared__ int32_t tile[(kEdtRows + 2 * kEdtMaxW) * kEdtX];
    const uint32_t b = blockIdx.x, xb = b % nxb, rest = b / nxb, rb = rest % nrb, sl = rest / nrb;
    const int tx = threadIdx.x % kEdtX, ty = threadIdx.x / kEdtX;
    constexpr int kLanes = kSesBlock / kEdtX;
    const int x = (int)xb * kEdtX + tx, a0 = (int)rb * kEdtRows, W = G.W;
    const int len = kLast ? G.nz : G.ny;
    // element (x, axis position a) of this slice
    auto at = [&](int a) -> size_t {
        return kLast ? gidx(G, x, (int)sl, a) : gidx(G, x, a, (int)sl);
    };
    const int staged = kEdtRows + 2 * W;
    for (int r = ty; r < staged; r += kLanes) {
        const int a = a0 - W + r;
        tile[r * kEdtX + tx] = (x < G.nx && a >= 0 && a < len) ? gin[at(a)] : kFar;
    }
    __syncthreads();
    if (x >= G.nx) return;
    for (int o = ty; o < kEdtRows; o += kLanes) {
        const int a = a0 + o;
        if (a >= len) break;
        int32_t best = kFar;
        for (int d = -W; d <= W; ++d) {
            const int32_t v = tile[(o + W + d) * kEdtX + tx];
            if (v < kFar) best = min(best, v + d * d);
        }
        const size_t p = at(a);
        if (!kLast) {
            gout[p] = best;
        } else {
            field[p] = ses_field(G, best);
        }
    }
}

// Sign bits (f >= 0) of a field the passes through memory wrote: one thread
// per word of 32 points of a row.
__global__ void __launch_bounds__(kSesBlock) k_ses_sign(SesGrid G, const float* __restrict__ f, int nxw, uint32_t nw,
                                                        uint32_t* __restrict__ sign) {
    const uint32_t w = blockIdx.x * (uint32_t)kSesBlock + threadIdx.x;
    if (w >= nw) return;
    const uint32_t row = w / (uint32_t)nxw;
    const int x0 = (int)(w - row * (uint32_t)nxw) * 32;
    uint32_t m = 0;
    for (int q = 0; q < 32 && x0 + q < G.nx; ++q) m |= f[(size_t)row * G.nx + x0 + q] >= 0.0f ? 1u << q : 0u;
    sign[w] = m;
}

// The cubes of a word of sign bits: cube q of word wx of cube row (j, k) has
// its first corner at point (32 wx + q, j, k).  `corner[c]` holds the sign
// bits of corner c of every cube, `active` the cubes with triangles.
struct WordCubes {
    uint32_t corner[8];
    uint32_t active;
    int i0, j, k;
    __device__ uint32_t cube(int q) const {
        uint32_t m = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) m |= (corner[c] >> q & 1u) << c;
        return m;
    }
};

// Word w of the cube rows (nw of them), w in x-fastest order.
__device__ inline WordCubes word_cubes(const SesGrid& G, const uint32_t* __restrict__ sign, int nxw, uint32_t w, uint32_t nw) {
    WordCubes u;
    u.active = 0;
    if (w >= nw) return u;
    const uint32_t row = w / (uint32_t)nxw;
    const int wx = (int)(w - row * (uint32_t)nxw);
    u.i0 = 32 * wx;
    u.j = (int)(row % (uint32_t)(G.ny - 1));
    u.k = (int)(row / (uint32_t)(G.ny - 1));
    uint32_t any = 0, all = ~0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const size_t at = ((size_t)(u.k + (c >> 1)) * G.ny + (u.j + (c & 1))) * nxw + wx;
        const uint32_t a = sign[at], next = wx + 1 < nxw ? sign[at + 1] : 0u;
        u.corner[2 * c] = a;
        u.corner[2 * c + 1] = (a >> 1) | (next << 31);
        any |= u.corner[2 * c] | u.corner[2 * c + 1];
        all &= u.corner[2 * c] & u.corner[2 * c + 1];
    }
    const int cubes = min(32, G.nx - 1 - u.i0);   // the last word may hold none
    const uint32_t valid = cubes >= 32 ? ~0u : cubes > 0 ? (1u << cubes) - 1u : 0u;
    u.active = any & ~all & valid;
    return u;
}

// Triangles of each run of kSesRun words of cubes.
__global__ void __launch_bounds__(kSesRun) k_ses_count(SesGrid G, const uint32_t* __restrict__ sign, int nxw, uint32_t nw,
                                                       uint32_t* __restrict__ run_tris) {
    __shared__ uint8_t tris[256];
    __shared__ uint32_t sum;
    const int tid = threadIdx.x;
    for (int q = tid; q < 64; q += kSesRun) reinterpret_cast<uint32_t*>(tris)[q] = reinterpret_cast<const uint32_t*>(c_case_tris)[q];
    if (tid == 0) sum = 0;
    __syncthreads();
    const WordCubes u = word_cubes(G, sign, nxw, blockIdx.x * (uint32_t)kSesRun + tid, nw);
    uint32_t nt = 0;
    for (uint32_t m = u.active; m; m &= m - 1) nt += tris[u.cube(__builtin_ctz(m))];
    for (int o = 32; o > 0; o >>= 1) nt += (uint32_t)__shfl_xor((int)nt, o);
    if (__lane_id() == 0 && nt) atomicAdd(&sum, nt);
    __syncthreads();
    if (tid == 0) run_tris[blockIdx.x] = sum;
}

// The triangles of a run's cubes, from its offset on (those past the capacity
// are dropped).  One wave per run, 64 cubes with triangles a round, packed
// from the words: their case comes from the signs of the eight corner values
// they need anyway, a scan of the triangle counts places them, and the
// round's triangles are written from LDS in order: 30 us for 770k.  (A thread
// per cube writing its own triangles, from lists of 256 cubes: 58.)
__global__ void __launch_bounds__(kSesRun) k_ses_emit(SesGrid G, const uint32_t* __restrict__ sign, int nxw, uint32_t nw,
                                                      const float* __restrict__ f, const uint32_t* __restrict__ run_off,
                                                      float* __restrict__ tri, unsigned long long capacity) {
    static_assert(kSesRun == 64, "one wave");
    constexpr uint32_t kStage = 288;   // triangles staged at once: a round has 4 a cube or so (8 at most)
    __shared__ float stage[kStage * 9];
    __shared__ float corner[8][kSesRun];
    __shared__ uint16_t list[kSesRun];   // the round's cubes: word of the run * 32 + cube of the word
    const int lane = threadIdx.x;
    const uint32_t w0 = blockIdx.x * (uint32_t)kSesRun;
    uint32_t left = word_cubes(G, sign, nxw, w0 + lane, nw).active;   // this lane's cubes not yet taken
    const uint32_t mine = (uint32_t)__popc(left);
    uint32_t rank = mine;   // inclusive, then the rank of this lane's next cube
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)rank, o);
        if (lane >= o) rank += v;
    }
    const uint32_t cubes = (uint32_t)__shfl((int)rank, 63);
    rank -= mine;
    unsigned long long start = run_off[blockIdx.x];
    for (uint32_t done = 0; done < cubes; done += kSesRun) {
        for (; left && rank < done + kSesRun; ++rank, left &= left - 1)
            list[rank - done] = (uint16_t)(lane * 32 + __builtin_ctz(left));
        __syncthreads();
        const bool have = done + lane < cubes;
        int i = 0, j = 0, k = 0;
        uint32_t m = 0;
        if (have) {
            const uint32_t w = w0 + list[lane] / 32u;
            const uint32_t row = w / (uint32_t)nxw;
            i = 32 * (int)(w - row * (uint32_t)nxw) + (int)(list[lane] & 31u);
            j = (int)(row % (uint32_t)(G.ny - 1));
            k = (int)(row / (uint32_t)(G.ny - 1));
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float v = f[gidx(G, i + (c & 1), j + ((c >> 1) & 1), k + ((c >> 2) & 1))];
                corner[c][lane] = v;
                m |= (v >= 0.0f ? 1u : 0u) << c;
            }
        }
        const uint32_t nt = have ? c_case_tris[m] : 0u;
        uint32_t at = nt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)at, o);
            if (lane >= o) at += v;
        }
        const uint32_t n_tris = (uint32_t)__shfl((int)at, 63);
        // as many cubes at once as the staging holds (the usual round: all)
        for (uint32_t from = 0; from < n_tris;) {
            const bool now = nt && at - nt >= from && at - from <= kStage;
            const uint32_t to = (uint32_t)__shfl((int)at, 63 - __clzll((long long)__ballot(now)));
            if (now) {
                const float ox = (float)G.o[0], oy = (float)G.o[1], oz = (float)G.o[2], h = (float)G.h;
                float* t = stage + 9 * (at - nt - from);
                unsigned long long edges = c_cases[m];
                for (uint32_t lens = (uint32_t)(edges >> 48); lens; lens >>= 4) {
                    // vertex e of a fan is the second vertex of its triangle e and
                    // the third of triangle e - 1; the mean is the first of each
                    const int len = (int)(lens & 15u);
                    float sx = 0.f, sy = 0.f, sz = 0.f;
                    for (int e = 0; e < len; ++e) {
                        // edge ed: the (ed & 3)-th along axis ed >> 2, from corner a
                        const int ed = (int)edges & 15, axis = ed >> 2, r = ed & 3;
                        edges >>= 4;
                        const int a = axis == 0 ? 2 * r : axis == 1 ? (r & 1) | (r & 2) << 1 : r;
                        const float va = corner[a][lane], vb = corner[a + (1 << axis)][lane];
                        const float tt = va / (va - vb);
                        const float fx = axis == 0 ? tt : (float)(a & 1);
                        const float fy = axis == 1 ? tt : (float)((a >> 1) & 1);
                        const float fz = axis == 2 ? tt : (float)((a >> 2) & 1);
                        const float px = ox + h * ((float)i + fx);
                        const float py = oy + h * ((float)j + fy);
                        const float pz = oz + h * ((float)k + fz);
                        auto put = [&](float* o) {
                            o[0] = px;
                            o[1] = py;
                            o[2] = pz;
                        };
                        if (len == 3) {
                            put(t + 3 * e);
                        } else {
                            put(t + 9 * e + 3);
                            put(t + 9 * (e ? e - 1 : len - 1) + 6);
                        }
                        sx += px;
                        sy += py;
                        sz += pz;
                    }
                    if (len > 3) {
                        const float inv = 1.0f / (float)len;
                        for (int e = 0; e < len; ++e) {
                            t[9 * e] = sx * inv;
                            t[9 * e + 1] = sy * inv;
                            t[9 * e + 2] = sz * inv;
                        }
                    }
                    t += 9 * (len == 3 ? 1 : len);
                }
            }
            __syncthreads();
            const uint32_t room = start < capacity ? (uint32_t)min((unsigned long long)(to - from), capacity - start) : 0u;
            for (uint32_t q = (uint32_t)lane; q < 9u * room; q += kSesRun) tri[9 * start + q] = stage[q];
            start += to - from;
            from = to;
            __syncthreads();   // the staging, the list and the corners are rewritten next
        }
    }
}

template <int kW>
hipError_t launch_edt(int W, unsigned blocks, const SesGrid& G, const MarkGrid& M, uint32_t nbx, uint32_t nby, float* field,
                      uint32_t* sign, int nxw, hipStream_t stream) {
    if constexpr (kW > kMaxFusedW) return hipErrorInvalidValue;
    else
        return W == kW ? dispatch(k_ses_edt<kW>, blocks, kEdtBlock, 0, stream, G, M, nbx, nby, field, sign, nxw)
                       : launch_edt<kW + 1>(W, blocks, G, M, nbx, nby, field, sign, nxw, stream);
}

int ses_window(float probe, float spacing) { return (int)ceil((double)probe / (double)spacing) + 2; }
uint64_t ses_bricks(const int dims[3]) {
    return ((uint64_t)dims[0] + kBx - 1) / kBx * (((uint64_t)dims[1] + kBy - 1) / kBy) * (((uint64_t)dims[2] + kBz - 1) / kBz);
}
// Small windows (and bricks that fit one launch) take the passes in LDS.
bool ses_fused(float probe, float spacing, const int dims[3]) {
    return ses_window(probe, spacing) <= kMaxFusedW && ses_bricks(dims) * kEdtBlock < (1ull << 31);
}
}  // namespace

hipError_t ses_run(const float* pos, const float* rad, uint64_t n, float probe, const float origin[3], float spacing,
                   const int dims[3], float* field, float* tri, uint64_t capacity, unsigned long long* n_tri,
                   SesScratch& s, hipStream_t stream) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if ((e = ensure_cases(dev)) != hipSuccess) return e;
    SesGrid G;
    for (int d = 0; d < 3; ++d) G.o[d] = (double)origin[d];
    G.h = (double)spacing;
    G.inv_h = 1.0 / G.h;
    G.nx = dims[0];
    G.ny = dims[1];
    G.nz = dims[2];
    G.rp = (double)probe;
    G.W = ses_window(probe, spacing);
    double far = 0.0;   // the grid's largest coordinate
    for (int d = 0; d < 3; ++d) far = fmax(far, fmax(fabs(G.o[d]), fabs(G.o[d] + G.h * (dims[d] - 1))));
    G.slack = G.inv_h * 0x1p-48;
    G.slack0 = 1e-3 + far * G.inv_h * 0x1p-48;
    const size_t np = (size_t)G.nx * G.ny * G.nz;
    MarkGrid M;
    M.bits = s.mark;
    M.nx = mark_cells(G.nx);
    M.ny = mark_cells(G.ny);
    const size_t mark_words = 2 * (size_t)M.nx * M.ny * mark_cells(G.nz);
    if ((e = launch_zero(reinterpret_cast<uint32_t*>(s.mark), mark_words, stream)) != hipSuccess) return e;
    // Few points per atom: several atoms per wave.  The whole call at 50,000
    // atoms, one and eight: 28 points per atom 88 and 63 us, 75 92 and 77, 200
    // 124 and 126, 900 374 and 391; 2,000: 50 41 and 41, 130 44 and 46, 330 46
    // and 52; 200 atoms of 300,000 220 and 843.
    if (np < kManyPoints * n) {
        const unsigned waves = (unsigned)((n + kMarkAtoms - 1) / kMarkAtoms);
        if ((e = dispatch(k_ses_mark<kMarkAtoms>, waves, kSesMarkBlock, 0, stream, pos, rad, (uint32_t)n, G, M))) return e;
    } else if (n && (e = dispatch(k_ses_mark<1>, (unsigned)n, kSesMarkBlock, 0, stream, pos, rad, (uint32_t)n, G, M))) {
        return e;
    }
    const int nxw = (G.nx + 31) / 32;
    const uint32_t sign_words = (uint32_t)((size_t)nxw * G.ny * G.nz);
    if (ses_fused(probe, spacing, dims)) {
        const uint32_t nbx = (uint32_t)nxw, nby = (uint32_t)((G.ny + kBy - 1) / kBy);
        static_assert(kBx == 32, "a brick row is a word of sign bits");
        if ((e = launch_edt<2>(G.W, (unsigned)ses_bricks(dims), G, M, nbx, nby, field, s.sign, nxw, stream))) return e;
    } else {
        const unsigned gp = (unsigned)((np + kSesBlock - 1) / kSesBlock);
        const uint64_t nxr = (uint64_t)(G.nx + kSesBlock - 1) / kSesBlock, gx = nxr * (uint64_t)G.ny * (uint64_t)G.nz;
        if (G.W <= kEdtMaxW && gx * kSesBlock < (1ull << 31)) {
            if ((e = dispatch(k_ses_edt_x_lds, (uint32_t)gx, kSesBlock, 0, stream, G, (uint32_t)nxr, M, s.ga))) return e;
        } else if ((e = dispatch(k_ses_edt_x, gp, kSesBlock, 0, stream, G, (uint32_t)np, M, s.ga))) {
            return e;
        }
        const uint64_t nxb = (uint64_t)(G.nx + kEdtX - 1) / kEdtX;
        const uint64_t gy = nxb * (uint64_t)((G.ny + kEdtRows - 1) / kEdtRows) * (uint64_t)G.nz;
        const uint64_t gz = nxb * (uint64_t)((G.nz + kEdtRows - 1) / kEdtRows) * (uint64_t)G.ny;
        if (G.W <= kEdtMaxW && gy * kSesBlock < (1ull << 31) && gz * kSesBlock < (1ull << 31)) {
            if ((e = dispatch(k_ses_edt_yz_lds<false>, (uint32_t)gy, kSesBlock, 0, stream, G, (uint32_t)nxb,
                              (uint32_t)((G.ny + kEdtRows - 1) / kEdtRows), (const int32_t*)s.ga, s.gb, (float*)nullptr)))
                return e;
            if ((e = dispatch(k_ses_edt_yz_lds<true>, (uint32_t)gz, kSesBlock, 0, stream, G, (uint32_t)nxb,
                              (uint32_t)((G.nz + kEdtRows - 1) / kEdtRows), (const int32_t*)s.gb, s.ga, field)))
                return e;
        } else {
            if ((e = dispatch(k_ses_edt_yz<false>, gp, kSesBlock, 0, stream, G, (uint32_t)np, (const int32_t*)s.ga, s.gb,
                              (float*)nullptr)))
                return e;
            if ((e = dispatch(k_ses_edt_yz<true>, gp, kSesBlock, 0, stream, G, (uint32_t)np, (const int32_t*)s.gb, s.ga,
                              field)))
                return e;
        }
        if ((e = dispatch(k_ses_sign, (sign_words + kSesBlock - 1) / kSesBlock, kSesBlock, 0, stream, G, (const float*)field,
                          nxw, sign_words, s.sign)))
            return e;
    }
    const uint32_t nw = (uint32_t)((size_t)nxw * (G.ny - 1) * (G.nz - 1));
    const uint32_t runs = (nw + kSesRun - 1) / kSesRun;
    if ((e = dispatch(k_ses_count, runs, kSesRun, 0, stream, G, (const uint32_t*)s.sign, nxw, nw, s.cnt))) return e;
    if ((e = exclusive_scan(s.cnt, runs, s.bsum, n_tri, stream))) return e;
    return dispatch(k_ses_emit, runs, kSesRun, 0, stream, G, (const uint32_t*)s.sign, nxw, nw, (const float*)field,
                    (const uint32_t*)s.cnt, tri, (unsigned long long)capacity);
}

SesWords ses_scratch_words(float probe, float spacing, const int dims[3]) {
    const size_t np = (size_t)dims[0] * dims[1] * dims[2], nxw = ((size_t)dims[0] + 31) / 32;
    SesWords w;
    w.mark = 2 * (size_t)mark_cells(dims[0]) * mark_cells(dims[1]) * mark_cells(dims[2]);
    w.g = ses_fused(probe, spacing, dims) ? 0 : np;
    w.sign = nxw * dims[1] * dims[2];
    w.cnt = (nxw * (dims[1] - 1) * (dims[2] - 1) + kSesRun - 1) / kSesRun;
    w.bsum = scan_scratch_words(w.cnt);
    return w;
}

}  // namespace vtx
