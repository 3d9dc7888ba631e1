// Box-clipped Voronoi grid of the sites on the device, with Lloyd iterations
// (Sec. II-A: the grid is initialised with its generating sites at the
// particle positions and relaxed by Lloyd iterations).
//
// Sites are sorted by Morton key and grouped 8 per leaf of a box tree (heap
// order, internal boxes bottom-up).  One wavefront builds one cell (the box
// cut by bisector planes, nearest sites first, until no farther site can
// reach it; em_voronoi_core.h) into a per-cell record in device memory;
// its face, face-vertex and vertex counts are scanned into offsets in input
// order, and a second pass writes the cells in the library's cell format
// (faces counter-clockwise about outward unit normals, vertices per cell),
// the site or wall across each face, the volumes and the centroids.  A Lloyd
// step moves every site to its cell's centroid and builds the grid again.
#include <algorithm>
#include <cmath>

#include "em_internal.h"
#include "em_voronoi_core.h"
#include "em_wave.h"

namespace em {

namespace {

__device__ __forceinline__ uint64_t spread3v(uint64_t v)
{
    v &= 0x1fffffULL;
    v = (v | (v << 32)) & 0x1f00000000ffffULL;
    v = (v | (v << 16)) & 0x1f0000ff0000ffULL;
    v = (v | (v << 8)) & 0x100f00f00f00f00fULL;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ULL;
    v = (v | (v << 2)) & 0x1249249249249249ULL;
    return v;
}

__device__ __forceinline__ uint64_t axis21v(double x, double lo, double ext)
{
    const double t = ((x - lo) / ext) * 2097152.0;
    if (!(t > 0.0)) return 0;
    if (t >= 2097151.0) return 2097151ULL;
    return (uint64_t)floor(t);
}

struct VBox {
    double lo[3], hi[3];
};

// flags: bit 0 a site outside the box or not finite
__global__ void k_vor_keys(int64_t n, const double *__restrict__ s, VBox B, uint64_t *__restrict__ key,
                           uint32_t *__restrict__ idx, unsigned *flags)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint64_t k[3];
    bool bad = false;
    for (int d = 0; d < 3; d++) {
        const double x = s[3 * i + d];
        if (!(x >= B.lo[d] && x <= B.hi[d])) bad = true;
        k[d] = axis21v(x, B.lo[d], B.hi[d] - B.lo[d]);
    }
    if (bad) atomicOr(flags, 1u);
    key[i] = (spread3v(k[0]) << 2) | (spread3v(k[1]) << 1) | spread3v(k[2]);
    idx[i] = (uint32_t)i;
}

// sorted positions, input index of each sorted site, rank of each input site;
// flags bit 1: two sites coincide (neighbours in Morton order share the key)
__global__ void k_vor_sorted(int64_t n, const uint32_t *__restrict__ perm, const double *__restrict__ s,
                             double *__restrict__ ps, int32_t *__restrict__ orig, int64_t *__restrict__ rank,
                             unsigned *flags)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int64_t i = perm[r];
    ps[3 * r] = s[3 * i];
    ps[3 * r + 1] = s[3 * i + 1];
    ps[3 * r + 2] = s[3 * i + 2];
    orig[r] = (int32_t)i;
    rank[i] = r;
    if (r > 0) {
        const int64_t j = perm[r - 1];
        if (s[3 * i] == s[3 * j] && s[3 * i + 1] == s[3 * j + 1] && s[3 * i + 2] == s[3 * j + 2]) atomicOr(flags, 2u);
    }
}

__global__ void k_vor_leaf_boxes(int64_t n, int64_t NL, const double *__restrict__ ps, double *__restrict__ bx)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= NL) return;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t q = vor::kLeaf * j; q < vor::kLeaf * (j + 1) && q < n; q++)
        for (int d = 0; d < 3; d++) {
            lo[d] = fmin(lo[d], ps[3 * q + d]);
            hi[d] = fmax(hi[d], ps[3 * q + d]);
        }
    for (int d = 0; d < 3; d++) {
        bx[6 * (NL + j) + d] = lo[d];
        bx[6 * (NL + j) + 3 + d] = hi[d];
    }
}

// ---------------------------------------------------------------- one wavefront per cell
// The working cell of each wavefront is in LDS: the lanes own the cell's
// triangles (lane l: triangles l and l + 64), so a cut tests every vertex at
// once, finds the boundary of the removed triangles through a bit set of the
// kept triangles' directed edges (each dual edge is in exactly one triangle,
// so the reverse of a removed triangle's edge is kept exactly when it is in
// no removed triangle), and compacts kept and new triangles with prefix
// counts.  The candidate sites of a pass come from a walk of the site tree by
// the whole wavefront (pending nodes in LDS, 64 tests at a time) and are held
// by the lanes.  A cell built by one lane in private memory instead reads its
// arrays with a different index on every lane, so that each access fetches a
// cache line per lane.
//
// Bound by vector issue and latency together (9,600 vector instructions per
// cell, 0.16 per SIMD and clock at 4 wavefronts per SIMD): 6.3 ms for 262,144
// clumpy sites.  It was 18.7 ms with 26,300 instructions per cell: each leaf's 8
// sites by one lane, the candidate list sorted and every candidate's plane
// taken in turn, the reductions of every cut through the LDS crossbar, the
// new vertices of a cut by the lanes that lost one.
constexpr int kWCand = 192;   // candidates of one pass (wavefront walk), three per lane; the serial walk uses the first 64
constexpr int kWStack = 384;  // tree nodes pending in the wavefront walk
static_assert(kWCand >= vor::kMaxCand && kWCand <= 192, "the serial walk's candidates live in the same array");

struct WCell {
    vor::Plane pl[vor::kMaxPlanes];
    double vx[vor::kMaxTris], vy[vor::kMaxTris], vz[vor::kMaxTris];
    uint32_t tri[vor::kMaxTris];
    int32_t src[vor::kMaxPlanes];
    int32_t cand[kWCand];
    union {  // (never live at the same time)
        int32_t nodes[kWStack];  // the wavefront walk's pending nodes: inner ones from the front, leaves from the back
        struct {                 // the serial walk's stack and keys
            int64_t stack[64];
            double cd2[vor::kMaxCand];
        };
        uint32_t bits[vor::kMaxPlanes * vor::kMaxPlanes / 32];  // a cut's directed edges (x, y) of kept triangles: bit 64 x + y
    };
    int32_t status, cnt, more, pad;
};

__device__ __forceinline__ double wave_max_d(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ double wave_min_d(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}

// Largest of the lanes' values, wave-uniform, by data-parallel primitives (one
// vector instruction a step; a step through the LDS crossbar takes a
// hundred clocks and the reductions are on the path of every cut).
__device__ __forceinline__ unsigned wave_umax(unsigned v)
{
#define EM_DPP_MAX(ctrl, rows)                                                                              \
    {                                                                                                       \
        const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, true);          \
        v = v > o ? v : o;                                                                                  \
    }
    EM_DPP_MAX(0xB1, 0xf)   // quad_perm 1,0,3,2
    EM_DPP_MAX(0x4E, 0xf)   // quad_perm 2,3,0,1
    EM_DPP_MAX(0x141, 0xf)  // row_half_mirror
    EM_DPP_MAX(0x140, 0xf)  // row_mirror: every row of 16 has its largest value
    EM_DPP_MAX(0x142, 0xa)  // row_bcast15 into rows 1 and 3
    EM_DPP_MAX(0x143, 0xc)  // row_bcast31 into rows 2 and 3
#undef EM_DPP_MAX
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

__device__ __forceinline__ double lane_value(double v, int l)
{
    const uint64_t b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}

// This lane's triangles (lane, lane + 64) of the wavefront's cell, held in
// registers between cuts.
struct MyTris {
    uint32_t q[2];
    double x[2], y[2], z[2];
};

__device__ __forceinline__ void load_tris(const WCell &W, int nt, int lane, MyTris &T)
{
#pragma unroll
    for (int u = 0; u < 2; u++) {
        const int t = lane + 64 * u;
        if (t < nt) {
            T.q[u] = W.tri[t];
            T.x[u] = W.vx[t];
            T.y[u] = W.vy[t];
            T.z[u] = W.vz[t];
        }
    }
}

// Upper bounds of the cell about its site, wave-uniform: how far it reaches
// along the six axis directions and the squared distance of its farthest
// vertex.  (The site lies in its cell, so all are >= 0.)  They only decide
// which sites need no cut, so a bound that is a little too large changes
// nothing: the reduction takes the upper words of the doubles, 20 bits of
// mantissa and the whole range of exponents, and rounds up.  (With FP32 bounds
// and distances, cells were wrong where squared lengths leave FP32's range:
// neighbours 2e19 units apart or more were never cut.)
struct Bounds {
    double lo[3], hi[3];  // reach along -x, -y, -z and +x, +y, +z
    double m2;
};

// Upper word of a double >= 0 (-0 counts as 0): orders like the value.
__device__ __forceinline__ uint32_t upper_word(double v) { return (uint32_t)__double2hiint(v) & 0x7fffffffu; }

// The lanes' largest value (all >= 0), rounded up to its upper word.
__device__ __forceinline__ double wave_bound(double v)
{
    const uint32_t w = wave_umax(upper_word(v)) + 1u, inf = 0x7ff00000u;
    return __hiloint2double((int)(w < inf ? w : inf), 0);
}

__device__ __forceinline__ void bounds_of(const MyTris &T, int nt, int lane, Bounds &B)
{
    double l[3] = {0.0, 0.0, 0.0}, h[3] = {0.0, 0.0, 0.0}, m = 0.0;
#pragma unroll
    for (int u = 0; u < 2; u++)
        if (lane + 64 * u < nt) {
            const double f[3] = {T.x[u], T.y[u], T.z[u]};
            for (int d = 0; d < 3; d++) {
                l[d] = fmax(l[d], -f[d]);
                h[d] = fmax(h[d], f[d]);
            }
            m = fmax(m, f[0] * f[0] + f[1] * f[1] + f[2] * f[2]);
        }
    for (int d = 0; d < 3; d++) {
        B.lo[d] = wave_bound(l[d]);
        B.hi[d] = wave_bound(h[d]);
    }
    B.m2 = wave_bound(m);
}

// A site at offset w reaches the cell only if some vertex v has w.v > |w|^2 /
// 2; w.v is at most the box's reach along w (all of whose terms are >= 0).
// With a margin above the rounding.
__device__ __forceinline__ bool may_cut(const Bounds &B, double dx, double dy, double dz, double d2)
{
    const double r = fmax(-dx * B.lo[0], dx * B.hi[0]) + fmax(-dy * B.lo[1], dy * B.hi[1]) +
                     fmax(-dz * B.lo[2], dz * B.hi[2]);
    return d2 < r * (2.0 + 1e-12);
}

// The candidate sites of one pass with the whole wavefront: each step takes 16
// pending inner nodes of the site tree and tests their 64 grandchildren, one
// per lane, or the 64 sites of 8 pending leaves, with the tests of the serial
// walk (vor::collect).  The walk starts from the (at most 64) nodes of the
// tree's level 6.  The list of candidates holds kWCand: when it fills up, it
// is cut to its nearer half, and the distance of the nearest one dropped
// becomes the walk's radius, and *more is set.  So the result is the sites of
// the ball whose key follows (lo2, lo_q) and whose bisector can reach the
// cell's box, all of them unless *more.  Returns the count, or -1 when the
// pending nodes do not fit or a cut list keeps nothing (the caller then takes
// the serial walk).
__device__ int collect_wave(WCell &W, const double *__restrict__ ps, int64_t n, const double *__restrict__ bx,
                            int64_t NL, int64_t self, double sx, double sy, double sz, double lo2, int64_t lo_q,
                            double hi2, const double *blo, const double *bhi, int lane, bool *more)
{
    double h2 = hi2;
    *more = false;
    auto visit = [&](int64_t node) {
        const double *b = bx + 6 * node;
        const double g2 = vor::box_gap2(b, sx, sy, sz);
        const double ax = b[0] - sx, bxx = b[3] - sx, ay = b[1] - sy, by = b[4] - sy, az = b[2] - sz, bz = b[5] - sz;
        const double gm = fmax(fmax(ax * blo[0], ax * bhi[0]), fmax(bxx * blo[0], bxx * bhi[0])) +
                          fmax(fmax(ay * blo[1], ay * bhi[1]), fmax(by * blo[1], by * bhi[1])) +
                          fmax(fmax(az * blo[2], az * bhi[2]), fmax(bz * blo[2], bz * bhi[2]));
        return g2 < h2 && 0.5 * g2 < gm;
    };
    // the site's squared distance
    auto dist2 = [&](int64_t q, double &dx, double &dy, double &dz) {
        dx = ps[3 * q] - sx;
        dy = ps[3 * q + 1] - sy;
        dz = ps[3 * q + 2] - sz;
        return vor::length2(dx, dy, dz);
    };
    int sp = 0, nl = 0, cnt = 0;  // inner nodes, leaves, candidates
    auto push = [&](bool v, int64_t node) {  // false: no room
        const uint64_t leaf = __ballot(v && node >= NL), inner = __ballot(v && node < NL);
        if (sp + nl + __popcll(leaf) + __popcll(inner) > kWStack) return false;
        if (v) W.nodes[node < NL ? sp + lanes_below(inner) : kWStack - 1 - (nl + lanes_below(leaf))] = (int32_t)node;
        sp += __popcll(inner);
        nl += __popcll(leaf);
        return true;
    };
    {
        const int64_t first = NL < 64 ? NL : 64;  // NL is a power of two
        push(lane < first && visit(first + lane), first + lane);
    }
    lds_sync_wave();
    while (sp > 0 || nl > 0) {
        if (nl >= 8 || sp == 0) {
            if (cnt > kWCand - 64) {
                // full: keep the nearer half
                double d[3], dx, dy, dz;
                int32_t q[3];
                uint32_t key[3];
#pragma unroll
                for (int u = 0; u < 3; u++) {
                    const bool in = lane + 64 * u < cnt;
                    q[u] = in ? W.cand[lane + 64 * u] : 0;
                    d[u] = in ? dist2(q[u], dx, dy, dz) : INFINITY;
                    key[u] = upper_word(d[u]);
                }
                auto upto = [&](uint32_t k) {
                    return __popcll(__ballot(key[0] <= k)) + __popcll(__ballot(key[1] <= k)) +
                           __popcll(__ballot(key[2] <= k));
                };
                uint32_t ka = 0, kb = upper_word(INFINITY);  // at most half are <= ka, more than half <= kb
                while (kb - ka > 1) {
                    const uint32_t km = ka + (kb - ka) / 2;
                    if (upto(km) <= kWCand / 2) ka = km;
                    else kb = km;
                }
                double first_out = INFINITY;
#pragma unroll
                for (int u = 0; u < 3; u++)
                    if (key[u] > ka) first_out = fmin(first_out, d[u]);
                h2 = wave_min_d(first_out);
                lds_sync_wave();  // every entry read before the list is rewritten
                cnt = 0;
#pragma unroll
                for (int u = 0; u < 3; u++) {
                    const bool keep = key[u] <= ka;
                    const int at = wave_push(keep, cnt);
                    if (keep) W.cand[at] = q[u];
                }
                *more = true;
                if (cnt == 0) return -1;  // ties: the serial walk orders them by index
                lds_sync_wave();
            }
            const int k = nl < 8 ? nl : 8;
            const bool act = (lane >> 3) < k;
            const int64_t j = act ? (int64_t)W.nodes[kWStack - nl + (lane >> 3)] - NL : 0;
            nl -= k;
            const int64_t q = vor::kLeaf * j + (lane & 7);
            const bool ok = act && q < n && q != self;
            double dx, dy, dz;
            const double d2 = dist2(ok ? q : 0, dx, dy, dz);
            const bool take = ok && d2 < h2 && vor::key_less(lo2, lo_q, d2, q) && 0.5 * d2 < vor::reach(blo, bhi, dx, dy, dz);
            const int at = wave_push(take, cnt);
            if (take) W.cand[at] = (int32_t)q;
            lds_sync_wave();
            continue;
        }
        const int k = sp < 16 ? sp : 16;
        const bool act = (lane >> 2) < k;
        const int64_t node = act ? (int64_t)W.nodes[sp - k + (lane >> 2)] : 1;
        sp -= k;
        const bool two = 2 * node < NL;  // the grandchildren, or the children above the leaves
        const int64_t child = two ? 4 * node + (lane & 3) : 2 * node + (lane & 1);
        const bool v = act && (two || (lane & 3) < 2) && visit(child);
        lds_sync_wave();  // every node read before the pushes overwrite them
        if (!push(v, child)) return -1;
        lds_sync_wave();
    }
    return cnt;
}

// Cut by P (n.x <= d) in wave-uniform control flow; np, nt, status are
// wave-uniform copies of the cell's counts, T this lane's triangles (reloaded
// after a cut).  Returns true when P removed a vertex.
__device__ bool wclip(WCell &W, int &np, int &nt, int &status, const vor::Plane &P, int32_t src, int lane, MyTris &T)
{
    const double nn = sqrt(P.nx * P.nx + P.ny * P.ny + P.nz * P.nz);
    const double tol = vor::kEps * nn;
    const bool two = nt > 64;  // some lanes own a second triangle
    bool h[2] = {lane < nt, lane + 64 < nt}, o[2] = {false, false};
    uint64_t out[2] = {0, 0};
#pragma unroll
    for (int u = 0; u < 2; u++) {
        if (u == 1 && !two) break;
        o[u] = h[u] && P.nx * T.x[u] + P.ny * T.y[u] + P.nz * T.z[u] - P.d > tol;
        out[u] = __ballot(o[u]);
    }
    if ((out[0] | out[1]) == 0) return false;
    if (np >= vor::kMaxPlanes) {
        status = vor::ST_PLANES;
        return false;
    }
    const int p = np;
    if (lane == 0) {
        W.pl[p] = P;
        W.src[p] = src;
    }
    np++;
    // directed edges of the kept triangles
    W.bits[lane] = 0u;
    W.bits[lane + 64] = 0u;
    lds_sync_wave();
#pragma unroll
    for (int u = 0; u < 2; u++) {
        if (u == 1 && !two) break;
        if (h[u] && !o[u]) {
            const int a = vor::tri_a(T.q[u]), b = vor::tri_b(T.q[u]), c = vor::tri_c(T.q[u]);
            const int e0 = 64 * a + b, e1 = 64 * b + c, e2 = 64 * c + a;
            atomicOr(&W.bits[e0 >> 5], 1u << (e0 & 31));
            atomicOr(&W.bits[e1 >> 5], 1u << (e1 & 31));
            atomicOr(&W.bits[e2 >> 5], 1u << (e2 & 31));
        }
    }
    lds_sync_wave();
    // new triangles (x, y, p) on the boundary edges (x, y) of the removed
    // ones, in the serial order: by removed triangle, then edge
    bool on[2][3] = {{false, false, false}, {false, false, false}};  // edge e of triangle u is on the boundary
    int before[2] = {0, 0}, total[2] = {0, 0}, kept = 0, kept_below[2] = {0, 0};
#pragma unroll
    for (int u = 0; u < 2; u++) {
        if (u == 1 && !two) break;
        if (o[u]) {
            const int v[3] = {vor::tri_a(T.q[u]), vor::tri_b(T.q[u]), vor::tri_c(T.q[u])};
#pragma unroll
            for (int e = 0; e < 3; e++) {
                const int r = 64 * v[(e + 1) % 3] + v[e];
                on[u][e] = ((W.bits[r >> 5] >> (r & 31)) & 1u) != 0;
            }
        }
#pragma unroll
        for (int e = 0; e < 3; e++) {
            const uint64_t m = __ballot(on[u][e]);
            before[u] += lanes_below(m);
            total[u] += __popcll(m);
        }
        const uint64_t k = __ballot(h[u] && !o[u]);
        kept_below[u] = kept + lanes_below(k);
        kept += __popcll(k);
    }
    const int n_new = total[0] + total[1];
    if (kept + n_new > vor::kMaxTris) {
        status = vor::ST_TRIS;
        return false;
    }
    // every lane holds its triangles in registers: compact in place, the new ones after the kept ones
#pragma unroll
    for (int u = 0; u < 2; u++) {
        if (u == 1 && !two) break;
        if (h[u] && !o[u]) {
            const int k = kept_below[u];
            W.tri[k] = T.q[u];
            W.vx[k] = T.x[u];
            W.vy[k] = T.y[u];
            W.vz[k] = T.z[u];
        }
        if (o[u]) {
            const int v[3] = {vor::tri_a(T.q[u]), vor::tri_b(T.q[u]), vor::tri_c(T.q[u])};
            int k = kept + (u == 1 ? total[0] : 0) + before[u];
#pragma unroll
            for (int e = 0; e < 3; e++)
                if (on[u][e]) W.tri[k++] = vor::tri_pack(v[e], v[(e + 1) % 3], p);
        }
    }
    nt = kept + n_new;
    lds_sync_wave();
    for (int k = kept + lane; k < nt; k += 64) {  // the new vertices, one per lane
        const uint32_t q = W.tri[k];
        vor::meet(W.pl[vor::tri_a(q)], W.pl[vor::tri_b(q)], W.pl[vor::tri_c(q)], W.vx[k], W.vy[k], W.vz[k]);
    }
    lds_sync_wave();
    load_tris(W, nt, lane, T);
    return true;
}

// One wavefront per sorted site: its cell, the cell's record and its face,
// face-vertex slot and vertex counts (stored at the site's input index); flags
// bit 2: a cell needed more planes, vertices or passes than its record holds.
__global__ void __launch_bounds__(128, 4) k_vor_build_wave(int64_t n, const double *__restrict__ ps,
                                                        const int32_t *__restrict__ orig,
                                                        const double *__restrict__ bx, int64_t NL, VBox B,
                                                        char *__restrict__ recs, char *__restrict__ bigs,
                                                        unsigned n_big, unsigned *__restrict__ big_used,
                                                        int64_t *__restrict__ nfc, int64_t *__restrict__ nsc,
                                                        int64_t *__restrict__ nvc, unsigned *flags)
{
    __shared__ WCell cellbuf[2];
    const int lane = threadIdx.x & 63;
    WCell &W = cellbuf[threadIdx.x >> 6];
    const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (r >= n) return;  // whole wavefronts
    const double box[6] = {B.lo[0], B.lo[1], B.lo[2], B.hi[0], B.hi[1], B.hi[2]};
    const double sx = ps[3 * r], sy = ps[3 * r + 1], sz = ps[3 * r + 2];
    // the box: planes 0..5 = x-, x+, y-, y+, z-, z+ and its 8 corners (one lane each)
    if (lane < 6) {
        const int ax = lane >> 1, side = lane & 1;
        const double sg = side ? 1.0 : -1.0, sa = ax == 0 ? sx : (ax == 1 ? sy : sz);
        vor::Plane P;
        P.nx = ax == 0 ? sg : 0.0;
        P.ny = ax == 1 ? sg : 0.0;
        P.nz = ax == 2 ? sg : 0.0;
        const double lo = ax == 0 ? box[0] : (ax == 1 ? box[1] : box[2]), hi = ax == 0 ? box[3] : (ax == 1 ? box[4] : box[5]);
        P.d = side ? hi - sa : sa - lo;
        W.pl[lane] = P;
        W.src[lane] = -1 - lane;
    }
    if (lane < 8) {
        const int cx = lane & 1, cy = (lane >> 1) & 1, cz = (lane >> 2) & 1;
        const int a = cx, b = 2 + cy, c = 4 + cz;
        const bool pos = ((cx + cy + cz) & 1) != 0;  // det(n_a, n_b, n_c), the product of the three signs
        W.tri[lane] = pos ? vor::tri_pack(a, b, c) : vor::tri_pack(a, c, b);
        W.vx[lane] = cx ? box[3] - sx : -(sx - box[0]);
        W.vy[lane] = cy ? box[4] - sy : -(sy - box[1]);
        W.vz[lane] = cz ? box[5] - sz : -(sz - box[2]);
    }
    lds_sync_wave();
    int np = 6, nt = 8, status = vor::ST_OK;
    MyTris T = {};
    load_tris(W, nt, lane, T);
    // The first pass only looks within 0.87 times the diagonal of the site's
    // leaf box (about 110 sites when the leaf's 8 sites fill it: most cells
    // end within it), at least an eighth of the mean spacing (for a leaf of
    // very close sites); later passes look anywhere.  The cell does not depend
    // on this choice (see below).
    const double *lb = bx + 6 * (NL + r / vor::kLeaf);
    const double ex = box[3] - box[0], ey = box[4] - box[1], ez = box[5] - box[2];
    const double mean = cbrt(ex * ey * ez / (double)n);
    double hi2 = 0.75 * ((lb[3] - lb[0]) * (lb[3] - lb[0]) + (lb[4] - lb[1]) * (lb[4] - lb[1]) +
                         (lb[5] - lb[2]) * (lb[5] - lb[2]));
    if (hi2 < mean * mean / 64.0) hi2 = mean * mean / 64.0;
    double lo2 = -1.0;
    int64_t lo_q = -1;
    Bounds bd;
    bounds_of(T, nt, lane, bd);
    // Passes: the ball first, then everything that can still reach the cell;
    // each pass lists the sites whose key (squared distance, then index)
    // follows the last pass's.  The sites are cut in key order, skipping those
    // whose bisector cannot reach the vertices' current bounding box, until
    // one is at least twice as far as the farthest vertex: the sequence of
    // cuts, and so the cell, is the same however the passes split it.  The
    // lanes hold the candidates; the next one is the least key among those
    // that may still cut, so the list is not sorted and a site that cannot cut
    // costs nothing.
    bool done = false;
    int pass = 0;
    for (; pass < 4096 && !done && status == vor::ST_OK; pass++) {
        bool more = false;
        double blo[3], bhi[3];
        for (int d = 0; d < 3; d++) {
            blo[d] = -bd.lo[d];
            bhi[d] = bd.hi[d];
        }
        int cnt = collect_wave(W, ps, n, bx, NL, r, sx, sy, sz, lo2, lo_q, hi2, blo, bhi, lane, &more);
        if (cnt < 0) {  // the serial walk, 64 at a time
            lds_sync_wave();
            if (lane == 0) {
                bool m = false;
                W.status = vor::ST_OK;
                W.cnt = vor::collect(W, ps, n, bx, NL, r, sx, sy, sz, lo2, lo_q, hi2, blo, bhi, &m, W.stack);
                W.more = m ? 1 : 0;
            }
            lds_sync_wave();
            cnt = __builtin_amdgcn_readfirstlane(W.cnt);
            more = __builtin_amdgcn_readfirstlane(W.more) != 0;
            if (__builtin_amdgcn_readfirstlane(W.status) != vor::ST_OK) {
                status = vor::ST_PASSES;
                break;
            }
        }
        // candidates lane, lane + 64, lane + 128: offsets, squared distances (their upper words as the coarse key)
        double cx[3], cy[3], cz[3], cd[3];
        int32_t cq[3];
        bool left[3];
#pragma unroll
        for (int u = 0; u < 3; u++) {
            left[u] = lane + 64 * u < cnt;
            cq[u] = left[u] ? W.cand[lane + 64 * u] : 0;
            cx[u] = ps[3 * (int64_t)cq[u]] - sx;
            cy[u] = ps[3 * (int64_t)cq[u] + 1] - sy;
            cz[u] = ps[3 * (int64_t)cq[u] + 2] - sz;
            cd[u] = vor::length2(cx[u], cy[u], cz[u]);
        }
        bool fresh = true;  // the bounds have changed
        uint32_t key[3] = {~0u, ~0u, ~0u};
        while (status == vor::ST_OK) {
            if (fresh) {
#pragma unroll
                for (int u = 0; u < 3; u++) {
                    const bool cuts = left[u] && cd[u] < 4.0 * bd.m2 && cd[u] > 0.0 &&
                                      may_cut(bd, cx[u], cy[u], cz[u], cd[u]);
                    key[u] = cuts ? upper_word(cd[u]) : ~0u;
                }
                fresh = false;
            }
            const uint32_t mine = min(key[0], min(key[1], key[2]));
            const uint32_t least = ~wave_umax(~mine);
            if (least == ~0u) break;
            uint64_t at[3];
#pragma unroll
            for (int u = 0; u < 3; u++) at[u] = __ballot(key[u] == least);
            int bu = -1, bl = 0;
            double bd2 = 0.0;
            int32_t bq = 0;
            const bool tie = __popcll(at[0]) + __popcll(at[1]) + __popcll(at[2]) > 1;
#pragma unroll
            for (int u = 0; u < 3; u++)
                for (uint64_t m = at[u]; m != 0; m &= m - 1) {  // (one, but for equal upper words)
                    const int l = __builtin_ctzll(m);
                    if (tie) {
                        const double d = lane_value(cd[u], l);
                        const int32_t q = __builtin_amdgcn_readlane(cq[u], l);
                        if (bu >= 0 && !vor::key_less(d, q, bd2, bq)) continue;
                        bd2 = d;
                        bq = q;
                    }
                    bu = u;
                    bl = l;
                }
            vor::Plane P;
            int64_t q;
            auto take = [&](int u) {
                P.nx = lane_value(cx[u], bl);
                P.ny = lane_value(cy[u], bl);
                P.nz = lane_value(cz[u], bl);
                q = __builtin_amdgcn_readlane(cq[u], bl);
                if (lane == bl) {
                    left[u] = false;
                    key[u] = ~0u;
                }
            };
            if (bu == 0) take(0);
            else if (bu == 1) take(1);
            else take(2);
            P.d = 0.5 * vor::length2(P.nx, P.ny, P.nz);
            if (wclip(W, np, nt, status, P, orig[q], lane, T)) {
                bounds_of(T, nt, lane, bd);
                fresh = true;
            }
        }
        if (status != vor::ST_OK) break;
        // a listed site at least twice as far as the farthest vertex: it and every farther one miss the cell
        bool beyond = false;
#pragma unroll
        for (int u = 0; u < 3; u++) beyond = beyond || (lane + 64 * u < cnt && cd[u] >= 4.0 * bd.m2);
        if (__ballot(beyond) != 0) {
            done = true;
            break;
        }
        if (cnt > 0) {  // the next pass's keys follow the last of this one's
            double d = -1.0;
#pragma unroll
            for (int u = 0; u < 3; u++)
                if (lane + 64 * u < cnt) d = fmax(d, cd[u]);
            lo2 = wave_max_d(d);
            int32_t q = -1;
#pragma unroll
            for (int u = 0; u < 3; u++)
                if (lane + 64 * u < cnt && cd[u] == lo2) q = max(q, cq[u]);
            for (int o = 32; o > 0; o >>= 1) q = max(q, __shfl_xor(q, o, 64));
            lo_q = q;
        }
        if (!more) {
            if (hi2 == INFINITY) {
                done = true;
                break;
            }
            hi2 = INFINITY;
        }
        lds_sync_wave();  // the candidate list is rewritten by the next pass
    }
    if (!done && status == vor::ST_OK) status = vor::ST_PASSES;
    // the counts, and the record for the extraction pass: the planes that are left (a plane cut away by later ones
    // has no vertex), in order, and the triangles in terms of them
    int64_t f = 0, sl = 0;
    int c = 0;
    if (status == vor::ST_OK) {
        if (lane < np)
            for (int t = 0; t < nt; t++) {
                const uint32_t q = W.tri[t];
                c += (vor::tri_a(q) == lane || vor::tri_b(q) == lane || vor::tri_c(q) == lane) ? 1 : 0;
            }
        const bool face = c >= 3;
        f = __popcll(__ballot(face));
        int cs = face ? c : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cs += __shfl_xor(cs, o, 64);
        sl = cs;
    } else if (lane == 0) {
        atomicOr(flags, 4u);
    }
    const uint64_t used = __ballot(c > 0);
    const int nu = __popcll(used);
    char *base = recs + r * (int64_t)vor::kRecBytes;
    int big = -1;
    if (status == vor::ST_OK &&
        (vor::rec_bytes(nu, nt) > vor::kRecBytes || nu > vor::kRecPlanes || nt > vor::kRecTris)) {
        if (lane == 0) big = (int)atomicAdd(big_used, 1u);
        big = __builtin_amdgcn_readfirstlane(big);
    }
    if (lane == 0) *reinterpret_cast<vor::RecHead *>(base) = vor::RecHead{nu, nt, status, big, used};
    if (status == vor::ST_OK && (big < 0 || (unsigned)big < n_big)) {  // (too many big cells: the host builds again)
        char *at = big < 0 ? base : bigs + big * (int64_t)vor::kBigRecBytes;
        if (big >= 0 && lane == 0) *reinterpret_cast<int64_t *>(at) = r;  // whose it is, in the header's place
        const vor::Rec G = vor::rec_at(at, nu, nt);
        if (c > 0) {
            const int k = lanes_below(used);
            G.pl[k] = W.pl[lane];
            G.src[k] = W.src[lane];
        }
        auto now = [&](int p) { return __popcll(used & ((uint64_t(1) << p) - 1)); };
        for (int t = lane; t < nt; t += 64) {
            const uint32_t q = W.tri[t];
            G.tri[t] = vor::tri_pack(now(vor::tri_a(q)), now(vor::tri_b(q)), now(vor::tri_c(q)));
            G.vx[t] = W.vx[t];
            G.vy[t] = W.vy[t];
            G.vz[t] = W.vz[t];
        }
    }
    if (lane == 0) {
        const int64_t i = orig[r];
        nfc[i] = f;
        nsc[i] = sl;
        nvc[i] = status == vor::ST_OK ? nt : 0;
    }
}

struct VorOut {
    int64_t *cfo, *fvo, *fnb;
    int32_t *fv;
    double *plane, *verts, *vol, *cen;
};

// One wavefront per input site writes its cell at the scanned offsets: for
// each plane with at least 3 vertices (lane p: plane p), its vertices in
// order around it, counter-clockwise seen from outside (the triangle (p, a, b)
// is followed by the one holding the directed edge (p, b), found in a table of
// the cell's directed edges; the order is reversed if the polygon's vector
// area points inward), the outward unit normal and offset in box
// coordinates, and the site or wall across it; the cell's vertices (in box
// coordinates), volume and centroid (tetrahedra from the site over face fans,
// summed over the faces of each lane and then across the wavefront).  The
// record is read once into LDS.  flags bit 3: a face's vertices did not close
// into one loop.
template <int PLANES, int TRIS>
struct XCell {
    vor::Plane pl[PLANES];
    double vx[TRIS], vy[TRIS], vz[TRIS];
    uint32_t tri[TRIS];
    int32_t src[PLANES];
    uint8_t et[PLANES * PLANES];   // directed edge (x, y): its triangle at PLANES x + y, 0xff: none
    uint8_t ring[PLANES][PLANES];  // ring[k][p]: the k-th triangle around plane p
};
static_assert(vor::kMaxTris < 255 && vor::kMaxPlanes <= 64, "triangle ids in bytes, one plane per lane");

// BIG: one wavefront per big record (n of them); else one per input site, the
// big ones left out.  Bound by the latency of LDS and of the records: with 14 kB
// of LDS for every cell ten wavefronts fit a CU and 262,144 clumpy sites took
// 1.27 ms; with 5 kB, where registers allow 16, 0.86, and 24, 0.70 ms.
template <bool BIG>
__global__ void __launch_bounds__(128, BIG ? 1 : 6) k_vor_extract(int64_t n, const double *__restrict__ s,
                                                     const int64_t *__restrict__ rank,
                                                     const int32_t *__restrict__ orig,
                                                     char *__restrict__ recs, char *__restrict__ bigs,
                                                     const int64_t *__restrict__ foff, const int64_t *__restrict__ soff,
                                                     const int64_t *__restrict__ voff, VorOut O, unsigned *flags)
{
    constexpr int PLANES = BIG ? vor::kMaxPlanes : vor::kRecPlanes, TRIS = BIG ? vor::kMaxTris : vor::kRecTris;
    __shared__ XCell<PLANES, TRIS> xbuf[2];
    const int lane = threadIdx.x & 63;
    XCell<PLANES, TRIS> &X = xbuf[threadIdx.x >> 6];
    const int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (w >= n) return;  // whole wavefronts
    const int64_t r = BIG ? *reinterpret_cast<const int64_t *>(bigs + w * (int64_t)vor::kBigRecBytes) : rank[w];
    const int64_t i = BIG ? orig[r] : w;
    char *base = recs + r * (int64_t)vor::kRecBytes;
    const vor::RecHead H = *reinterpret_cast<const vor::RecHead *>(base);
    if (!BIG && lane == 0) {
        O.cfo[i] = foff[i];
        if (i == n - 1) O.cfo[n] = foff[n];
    }
    if (H.status != vor::ST_OK || (H.big >= 0) != BIG) return;
    const int np = H.np, nt = H.nt;
    const vor::Rec C = vor::rec_at(BIG ? bigs + w * (int64_t)vor::kBigRecBytes : base, np, nt);
    const double sx = s[3 * i], sy = s[3 * i + 1], sz = s[3 * i + 2];
    const int64_t vbase = voff[i], fbase = foff[i], sbase = soff[i];
    uint32_t *et32 = reinterpret_cast<uint32_t *>(X.et);
    for (int k = lane; k < PLANES * PLANES / 4; k += 64) et32[k] = 0xffffffffu;
    if (lane < np) {
        X.pl[lane] = C.pl[lane];
        X.src[lane] = C.src[lane];
    }
    for (int t = lane; t < nt; t += 64) {
        const double x = C.vx[t], y = C.vy[t], z = C.vz[t];
        X.tri[t] = C.tri[t];
        X.vx[t] = x;
        X.vy[t] = y;
        X.vz[t] = z;
        O.verts[3 * (vbase + t)] = x + sx;
        O.verts[3 * (vbase + t) + 1] = y + sy;
        O.verts[3 * (vbase + t) + 2] = z + sz;
    }
    lds_sync_wave();
    for (int t = lane; t < nt; t += 64) {
        const uint32_t q = X.tri[t];
        const int a = vor::tri_a(q), b = vor::tri_b(q), c = vor::tri_c(q);
        X.et[PLANES * a + b] = (uint8_t)t;
        X.et[PLANES * b + c] = (uint8_t)t;
        X.et[PLANES * c + a] = (uint8_t)t;
    }
    lds_sync_wave();
    // the ring of triangles around plane p = lane, from the first that holds it
    const int p = lane;
    int nr = 0, first = -1;
    for (int t = 0; t < nt; t++) {
        const uint32_t q = X.tri[t];
        if (vor::tri_a(q) == p || vor::tri_b(q) == p || vor::tri_c(q) == p) {
            nr++;
            if (first < 0) first = t;
        }
    }
    const bool face = p < np && nr >= 3;
    int len = 0;
    if (face) {
        int t = first;
        while (len < nr && len < PLANES) {  // (a valid cell has at most np - 1)
            X.ring[len][p] = (uint8_t)t;
            len++;
            const uint32_t q = X.tri[t];
            const int b = vor::tri_a(q) == p ? vor::tri_c(q) : (vor::tri_b(q) == p ? vor::tri_a(q) : vor::tri_b(q));
            const int nx = X.et[PLANES * p + b];  // the triangle holding the directed edge (p, b)
            if (nx == 0xff || nx == first) break;
            t = nx;
        }
    }
    if (__ballot(face && len != nr) != 0) {
        if (lane == 0) atomicOr(flags, 8u);
        return;
    }
    // face index and first slot: prefix counts over the lanes below
    const uint64_t fm = __ballot(face);
    const int nf = __popcll(fm);
    int incl = face ? len : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    const int total = __shfl(incl, 63, 64);
    double V = 0.0, M0 = 0.0, M1 = 0.0, M2 = 0.0;
    if (face) {
        const int64_t f = fbase + lanes_below(fm), slot = sbase + incl - len;
        const vor::Plane P = X.pl[p];
        const double nn = sqrt(P.nx * P.nx + P.ny * P.ny + P.nz * P.nz);
        const double ux = P.nx / nn, uy = P.ny / nn, uz = P.nz / nn;
        // vector area about the site (local coordinates)
        double ax = 0.0, ay = 0.0, az = 0.0;
        for (int k = 0; k < len; k++) {
            const int a = X.ring[k][p], b = X.ring[k + 1 < len ? k + 1 : 0][p];
            ax += X.vy[a] * X.vz[b] - X.vz[a] * X.vy[b];
            ay += X.vz[a] * X.vx[b] - X.vx[a] * X.vz[b];
            az += X.vx[a] * X.vy[b] - X.vy[a] * X.vx[b];
        }
        const bool rev = ax * ux + ay * uy + az * uz < 0.0;
        auto at = [&](int k) { return (int)X.ring[rev ? len - 1 - k : k][p]; };
        O.fvo[f] = slot;
        for (int k = 0; k < len; k++) O.fv[slot + k] = (int32_t)(vbase + at(k));
        O.plane[4 * f] = ux;
        O.plane[4 * f + 1] = uy;
        O.plane[4 * f + 2] = uz;
        O.plane[4 * f + 3] = P.d / nn + (ux * sx + uy * sy + uz * sz);
        O.fnb[f] = X.src[p];
        // tetrahedra (site, v0, vk, vk+1) in counter-clockwise order
        const int o0 = at(0);
        const double x0 = X.vx[o0], y0 = X.vy[o0], z0 = X.vz[o0];
        for (int k = 1; k + 1 < len; k++) {
            const int o1 = at(k), o2 = at(k + 1);
            const double x1 = X.vx[o1], y1 = X.vy[o1], z1 = X.vz[o1];
            const double x2 = X.vx[o2], y2 = X.vy[o2], z2 = X.vz[o2];
            const double tv = (x0 * (y1 * z2 - z1 * y2) + y0 * (z1 * x2 - x1 * z2) + z0 * (x1 * y2 - y1 * x2)) / 6.0;
            V += tv;
            M0 += tv * (x0 + x1 + x2) / 4.0;
            M1 += tv * (y0 + y1 + y2) / 4.0;
            M2 += tv * (z0 + z1 + z2) / 4.0;
        }
    }
    if (lane == 0) O.fvo[fbase + nf] = sbase + total;
    // summed as plane by plane in the order of the cuts: the rounding does not depend on which planes were dropped
    const int from = lanes_below(H.used);
    const bool left = (H.used >> lane) & 1;
    auto spread = [&](double v) {
        const double w = __shfl(v, from, 64);
        return left ? w : 0.0;
    };
    V = spread(V), M0 = spread(M0), M1 = spread(M1), M2 = spread(M2);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        V += __shfl_xor(V, o, 64);
        M0 += __shfl_xor(M0, o, 64);
        M1 += __shfl_xor(M1, o, 64);
        M2 += __shfl_xor(M2, o, 64);
    }
    if (lane == 0) {
        O.vol[i] = V;
        O.cen[3 * i] = sx + (V > 0.0 ? M0 / V : 0.0);
        O.cen[3 * i + 1] = sy + (V > 0.0 ? M1 / V : 0.0);
        O.cen[3 * i + 2] = sz + (V > 0.0 ? M2 / V : 0.0);
    }
}

// Merging of tightly packed sites: a site is dropped when a site of lower
// input index lies closer than sqrt(d2max) (one thread per sorted site, a walk
// of the site tree that stops at the first such site).
__global__ void k_vor_merge(int64_t n, const double *__restrict__ ps, const int32_t *__restrict__ orig,
                            const double *__restrict__ bx, int64_t NL, double d2max, int64_t *__restrict__ keep)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const double sx = ps[3 * r], sy = ps[3 * r + 1], sz = ps[3 * r + 2];
    const int32_t me = orig[r];
    bool found = false;
    int64_t i = 1;
    while (!found) {
        if (vor::box_gap2(bx + 6 * i, sx, sy, sz) < d2max) {
            if (i < NL) {
                i = 2 * i;
                continue;
            }
            const int64_t j = i - NL;
            for (int64_t q = vor::kLeaf * j; q < vor::kLeaf * (j + 1) && q < n && !found; q++) {
                if (orig[q] >= me) continue;
                const double dx = ps[3 * q] - sx, dy = ps[3 * q + 1] - sy, dz = ps[3 * q + 2] - sz;
                if (dx * dx + dy * dy + dz * dz < d2max) found = true;
            }
        }
        while (i & 1) i >>= 1;
        if (i == 0) break;
        i += 1;
    }
    keep[me] = found ? 0 : 1;
}

// the kept sites, in input order
__global__ void k_vor_gather(int64_t n, const double *__restrict__ s, const int64_t *__restrict__ keep,
                             const int64_t *__restrict__ koff, double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || !keep[i]) return;
    const int64_t k = koff[i];
    out[3 * k] = s[3 * i];
    out[3 * k + 1] = s[3 * i + 1];
    out[3 * k + 2] = s[3 * i + 2];
}

// The cell holding each input point by a walk over the grid's cells: from a
// start cell, move to the face neighbour whose site is nearest the point, as
// long as one is nearer than the current site.  Over the box-clipped Voronoi
// grid this ends at the cell that holds the point (the segment from a site to
// the point leaves the site's cell through a face whose neighbour is nearer;
// the cells fill the box).  A point with a face neighbour at the current
// distance or within a relative 1e-10 of it (a tie, or one that rounding could
// decide: a site tied at an edge or vertex of the cell is tied with a face
// neighbour too), or a walk longer than 4096 steps, is listed for the tree
// walk below instead, which breaks ties by the lower index.  Points take as
// start the cell of the same relative index (the point's own site after Lloyd
// steps; near it for points in a spatially coherent order).
__global__ void __launch_bounds__(128) k_vor_site_walk(int64_t n_in, const double *__restrict__ x, int64_t n,
                                                       const double *__restrict__ sites,
                                                       const int64_t *__restrict__ cfo,
                                                       const int64_t *__restrict__ fnb,
                                                       int64_t *__restrict__ site_cell, int64_t *__restrict__ list,
                                                       unsigned long long *__restrict__ n_list)
{
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n_in) return;
    const double px = x[3 * a], py = x[3 * a + 1], pz = x[3 * a + 2];
    auto dist2 = [&](int64_t q) {
        const double dx = sites[3 * q] - px, dy = sites[3 * q + 1] - py, dz = sites[3 * q + 2] - pz;
        return dx * dx + dy * dy + dz * dz;
    };
    int64_t c = n_in == n ? a : (int64_t)((double)a * (double)n / (double)n_in);
    if (c >= n) c = n - 1;
    double d = dist2(c);
    bool settled = false;
    for (int step = 0; step < 4096; step++) {
        int64_t best = -1;
        double bd = d;
        for (int64_t f = cfo[c]; f < cfo[c + 1]; f++) {
            const int64_t q = fnb[f];
            if (q < 0) continue;  // a wall
            const double dq = dist2(q);
            if (dq < bd) {
                bd = dq;
                best = q;
            }
        }
        if (best < 0) {
            settled = true;
            break;
        }
        c = best;
        d = bd;
    }
    bool tie = !settled;
    if (settled)
        for (int64_t f = cfo[c]; f < cfo[c + 1] && !tie; f++) {
            const int64_t q = fnb[f];
            tie = q >= 0 && dist2(q) <= d * (1.0 + 1e-10);
        }
    if (tie) {
        const unsigned long long k = atomicAdd(n_list, 1ull);
        list[k] = a;
    } else {
        site_cell[a] = c;
    }
}

// The cell holding each input point: its nearest site of the grid (ties to
// the lower index), by a walk of the grid's site tree, nearer child first,
// skipping boxes farther than the best so far.  Each thread's stack is a
// column of an LDS array (at most one pending sibling per level: 32 entries
// hold trees of up to 2^30 leaves).
constexpr int kSiteStack = 32;

__global__ void __launch_bounds__(128) k_vor_site_cell(int64_t n_in, const int64_t *__restrict__ list,
                                                       const double *__restrict__ x, int64_t n,
                                                       const double *__restrict__ ps, const int32_t *__restrict__ orig,
                                                       const double *__restrict__ bx, int64_t NL,
                                                       int64_t *__restrict__ site_cell)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_in) return;
    const int64_t a = list ? list[t] : t;  // the listed points, or every point
    const double px = x[3 * a], py = x[3 * a + 1], pz = x[3 * a + 2];
    double best = INFINITY;
    int32_t bi = -1;
    __shared__ int32_t stk[kSiteStack][128];
    int32_t *stack = &stk[0][threadIdx.x];  // entry k at stack[128 k]
    int sp = 0;
    stack[0] = 1;
    sp = 1;
    while (sp > 0) {
        const int64_t i = stack[128 * --sp];
        if (vor::box_gap2(bx + 6 * i, px, py, pz) > best) continue;
        if (i < NL) {
            if (sp + 2 > kSiteStack) break;  // cannot happen below 2^30 leaves
            const double gl = vor::box_gap2(bx + 6 * (2 * i), px, py, pz);
            const double gr = vor::box_gap2(bx + 6 * (2 * i + 1), px, py, pz);
            stack[128 * sp++] = (int32_t)(gl <= gr ? 2 * i + 1 : 2 * i);
            stack[128 * sp++] = (int32_t)(gl <= gr ? 2 * i : 2 * i + 1);
            continue;
        }
        const int64_t j = i - NL;
        for (int64_t q = vor::kLeaf * j; q < vor::kLeaf * (j + 1) && q < n; q++) {
            const double dx = ps[3 * q] - px, dy = ps[3 * q + 1] - py, dz = ps[3 * q + 2] - pz;
            const double d2 = dx * dx + dy * dy + dz * dz;
            if (d2 < best || (d2 == best && orig[q] < bi)) {
                best = d2;
                bi = orig[q];
            }
        }
    }
    site_cell[a] = bi;
}

unsigned vgrid(int64_t n, int block) { return (unsigned)((n + block - 1) / block > 0 ? (n + block - 1) / block : 1); }

template <typename T>
T *dev_alloc(T *&p, size_t &cap, size_t count)
{
    if (count > cap || !p) {
        if (p) EM_HIP(hipFree(p));
        p = nullptr;
        EM_HIP(hipMalloc(&p, sizeof(T) * (count > 0 ? count : 1)));
        cap = count;
    }
    return p;
}

struct SiteTree {
    const double *ps;
    const int32_t *orig;
    const int64_t *rank;
    double *bx;
    int64_t NL;
};

// Sites sorted by Morton key (positions, input index of each sorted site,
// rank of each input site) and the box tree over leaves of 8.  Rejects sites
// outside the box or not finite, and (when asked) coinciding sites.
SiteTree site_tree(Workspace &ws, int64_t n, const double *sites, const VBox &B, bool distinct, hipStream_t s)
{
    unsigned *flags = ws.get<unsigned>(S_FLAGS, 4);
    fill_zero_bytes(flags, sizeof(unsigned) * 4, s);
    uint64_t *key = ws.get<uint64_t>(S_VOR0, (size_t)n);
    uint64_t *key2 = ws.get<uint64_t>(S_VOR1, (size_t)n);
    uint32_t *perm = ws.get<uint32_t>(S_VOR2, (size_t)n);
    uint32_t *perm2 = ws.get<uint32_t>(S_VOR3, (size_t)n);
    hipLaunchKernelGGL(k_vor_keys, dim3(vgrid(n, 256)), dim3(256), 0, s, n, sites, B, key, perm, flags);
    EM_HIP(hipGetLastError());
    radix_sort_u64(ws, key, perm, key2, perm2, n, 63, s);
    double *ps = ws.get<double>(S_VOR4, (size_t)(3 * n));
    int32_t *orig = ws.get<int32_t>(S_VOR5, (size_t)n);
    int64_t *rank = ws.get<int64_t>(S_VOR6, (size_t)n);
    hipLaunchKernelGGL(k_vor_sorted, dim3(vgrid(n, 256)), dim3(256), 0, s, n, (const uint32_t *)perm, sites, ps, orig,
                       rank, flags);
    EM_HIP(hipGetLastError());
    unsigned hf = 0;
    read_back(ws, {{&hf, flags, sizeof(unsigned)}}, s);
    EM_CHECK(!(hf & 1u), MAP_EINVAL, "a site is not finite or lies outside the box");
    EM_CHECK(!distinct || !(hf & 2u), MAP_EINVAL, "two sites coincide (merge them first)");

    const int64_t nleaf = (n + vor::kLeaf - 1) / vor::kLeaf;
    int64_t NL = 1;
    while (NL < nleaf) NL <<= 1;
    double *bx = ws.get<double>(S_VOR7, (size_t)(12 * NL));
    hipLaunchKernelGGL(k_vor_leaf_boxes, dim3(vgrid(NL, 256)), dim3(256), 0, s, n, NL, (const double *)ps, bx);
    EM_HIP(hipGetLastError());
    tree_parent_boxes(bx, NL, s);
    return SiteTree{ps, orig, rank, bx, NL};
}

}  // namespace

// Builds the grid of n sites (device memory) into V; returns the counts.
void build_voronoi(Workspace &ws, VorGrid &V, int64_t n, const double *sites, const double box[6], hipStream_t s)
{
    VBox B;
    for (int d = 0; d < 3; d++) {
        B.lo[d] = box[d];
        B.hi[d] = box[3 + d];
    }
    const SiteTree T = site_tree(ws, n, sites, B, true, s);
    const double *ps = T.ps;
    const int32_t *orig = T.orig;
    const int64_t *rank = T.rank;
    const double *bx = T.bx;
    const int64_t NL = T.NL;
    unsigned *flags = ws.get<unsigned>(S_FLAGS, 4);
    unsigned hf = 0;
    int64_t *nfc = ws.get<int64_t>(S_VOR9, (size_t)n + 1);
    int64_t *nsc = ws.get<int64_t>(S_VOR10, (size_t)n + 1);
    int64_t *nvc = ws.get<int64_t>(S_VOR11, (size_t)n + 1);
    int64_t *foff = ws.get<int64_t>(S_VOR12, (size_t)n + 1);
    int64_t *soff = ws.get<int64_t>(S_VOR13, (size_t)n + 1);
    int64_t *voff = ws.get<int64_t>(S_VOR14, (size_t)n + 1);
    unsigned *big_used = flags + 1;
    // the cells' records, and big ones for one cell in 16, or as many as there is room for from the grid before; a
    // grid with more big cells is built again with as many as it asked for
    char *recs = static_cast<char *>(ws.get(S_VOR8, vor::kRecBytes * (size_t)n)), *bigs = nullptr;
    unsigned n_big = (unsigned)std::min<int64_t>(
        n, std::max<int64_t>(n / 16 + 16, (int64_t)(ws.held(S_VOR15) / vor::kBigRecBytes)));
    int64_t tot[3] = {0, 0, 0}, n_used = 0;
    for (;;) {
        bigs = static_cast<char *>(ws.get(S_VOR15, vor::kBigRecBytes * (size_t)n_big));
        hipLaunchKernelGGL(k_vor_build_wave, dim3(vgrid(64 * n, 128)), dim3(128), 0, s, n, (const double *)ps,
                           (const int32_t *)orig, (const double *)bx, NL, B, recs, bigs, n_big, big_used, nfc, nsc,
                           nvc, flags);
        EM_HIP(hipGetLastError());
        scan_counts(ws, nfc, foff, n, s);
        scan_counts(ws, nsc, soff, n, s);
        scan_counts(ws, nvc, voff, n, s);
        unsigned h2[2] = {0, 0};
        read_back(ws, {{&tot[0], foff + n, sizeof(int64_t)}, {&tot[1], soff + n, sizeof(int64_t)},
                       {&tot[2], voff + n, sizeof(int64_t)}, {h2, flags, sizeof(h2)}}, s);
        hf = h2[0];
        n_used = h2[1];
        if (h2[1] <= n_big) break;
        n_big = h2[1];
        fill_zero_bytes(flags, sizeof(unsigned) * 4, s);
    }
    EM_CHECK(!(hf & 4u), MAP_EDEVICE,
             "a Voronoi cell needs more than 64 faces or 128 vertices (or its neighbour search did not settle)");
    EM_CHECK(tot[2] < (int64_t)INT32_MAX, MAP_EINVAL, "too many Voronoi vertices for 32-bit vertex ids");
    V.n_faces = tot[0];
    V.n_slots = tot[1];
    V.n_verts = tot[2];
    VorOut O;
    O.cfo = dev_alloc(V.cfo, V.cap_cells, (size_t)n + 1);
    O.vol = dev_alloc(V.vol, V.cap_vol, (size_t)n);
    O.cen = dev_alloc(V.cen, V.cap_cen, (size_t)(3 * n));
    O.fvo = dev_alloc(V.fvo, V.cap_fvo, (size_t)tot[0] + 1);
    O.fnb = dev_alloc(V.fnb, V.cap_fnb, (size_t)tot[0]);
    O.plane = dev_alloc(V.plane, V.cap_plane, (size_t)(4 * tot[0]));
    O.fv = dev_alloc(V.fv, V.cap_fv, (size_t)tot[1]);
    O.verts = dev_alloc(V.verts, V.cap_verts, (size_t)(3 * tot[2]));
    hipLaunchKernelGGL(k_vor_extract<false>, dim3(vgrid(64 * n, 128)), dim3(128), 0, s, n, sites,
                       (const int64_t *)rank, orig, recs, bigs, (const int64_t *)foff, (const int64_t *)soff,
                       (const int64_t *)voff, O, flags);
    EM_HIP(hipGetLastError());
    if (n_used > 0) {
        hipLaunchKernelGGL(k_vor_extract<true>, dim3(vgrid(64 * n_used, 128)), dim3(128), 0, s, n_used, sites,
                           (const int64_t *)rank, orig, recs, bigs, (const int64_t *)foff, (const int64_t *)soff,
                           (const int64_t *)voff, O, flags);
        EM_HIP(hipGetLastError());
    }
    read_back(ws, {{&hf, flags, sizeof(unsigned)}}, s);
    EM_CHECK(!(hf & 8u), MAP_EDEVICE, "a Voronoi face did not close into one loop");
    V.n = n;
}

// Merging (d > 0): the n_in input sites less those with a lower-index site
// closer than d, in input order, into out (3 n_in doubles); returns the count.
int64_t merge_sites(Workspace &ws, int64_t n_in, const double *in, const double box[6], double d, double *out,
                    hipStream_t s)
{
    VBox B;
    for (int k = 0; k < 3; k++) {
        B.lo[k] = box[k];
        B.hi[k] = box[3 + k];
    }
    const SiteTree T = site_tree(ws, n_in, in, B, false, s);
    int64_t *keep = ws.get<int64_t>(S_VOR9, (size_t)n_in + 1);
    int64_t *koff = ws.get<int64_t>(S_VOR10, (size_t)n_in + 1);
    hipLaunchKernelGGL(k_vor_merge, dim3(vgrid(n_in, 128)), dim3(128), 0, s, n_in, T.ps, T.orig, (const double *)T.bx,
                       T.NL, d * d, keep);
    EM_HIP(hipGetLastError());
    scan_counts(ws, keep, koff, n_in, s);
    int64_t m = 0;
    hipLaunchKernelGGL(k_vor_gather, dim3(vgrid(n_in, 256)), dim3(256), 0, s, n_in, in, (const int64_t *)keep,
                       (const int64_t *)koff, out);
    EM_HIP(hipGetLastError());
    read_back(ws, {{&m, koff + n_in, sizeof(int64_t)}}, s);
    return m;
}

// The cell of the grid V that holds each of the n_in input points.
void site_cells(Workspace &ws, const VorGrid &V, int64_t n_in, const double *in, const double box[6],
                int64_t *site_cell, hipStream_t s)
{
    VBox B;
    for (int k = 0; k < 3; k++) {
        B.lo[k] = box[k];
        B.hi[k] = box[3 + k];
    }
    // the walk over the cells, then the tree walk for the points it lists
    int64_t *list = ws.get<int64_t>(S_VOR9, (size_t)n_in);
    unsigned long long *n_list = reinterpret_cast<unsigned long long *>(ws.get<int64_t>(S_VOR10, 1));
    fill_zero_bytes(n_list, sizeof(unsigned long long), s);
    hipLaunchKernelGGL(k_vor_site_walk, dim3(vgrid(n_in, 128)), dim3(128), 0, s, n_in, in, V.n,
                       (const double *)V.sites, (const int64_t *)V.cfo, (const int64_t *)V.fnb, site_cell, list,
                       n_list);
    EM_HIP(hipGetLastError());
    unsigned long long n_tree = 0;
    read_back(ws, {{&n_tree, n_list, sizeof(n_tree)}}, s);
    if (n_tree == 0) return;
    const SiteTree T = site_tree(ws, V.n, V.sites, B, true, s);
    hipLaunchKernelGGL(k_vor_site_cell, dim3(vgrid((int64_t)n_tree, 128)), dim3(128), 0, s, (int64_t)n_tree,
                       (const int64_t *)list, in, V.n, T.ps, T.orig, (const double *)T.bx, T.NL, site_cell);
    EM_HIP(hipGetLastError());
}

void free_voronoi(VorGrid &V)
{
    for (void *p : {(void *)V.cfo, (void *)V.vol, (void *)V.cen, (void *)V.fvo, (void *)V.fnb, (void *)V.plane,
                    (void *)V.fv, (void *)V.verts, (void *)V.sites, (void *)V.input, (void *)V.site_cell})
        if (p) (void)hipFree(p);
    V = VorGrid{};
}

}  // namespace em
