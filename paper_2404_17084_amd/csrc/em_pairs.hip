// Pair search: every (particle a, cell i) whose closed cell lies closer to r_a
// than 2 h_a, ordered by cell and then particle.
//
// The particles, in storage order, are grouped 8 per leaf of an implicit
// complete binary tree of the boxes their supports can reach.  Wavefronts walk
// the tree for a few cells each and list the particles whose support comes
// within a cell's bounding box (candidates), already in cell-major order with
// particles ascending.  Cheap ball and box tests settle most
// candidates, the rest take the exact distance test below, one wavefront per
// cell (FP32 screening with a rounding bound, then the exact IEEE arithmetic
// near the threshold), and a wavefront per cell compacts the pairs.
#include <cmath>

#include "em_internal.h"
#include "em_wave.h"

namespace em {

constexpr int64_t kLeaf = 8;  // particles per leaf of the bounding-volume tree

// Exact distance test.  Squared distance from p to the closed convex cell: 0
// inside; else the least squared distance to a wall polygon that p sees from
// outside (d_j < 0): d_j^2 if p projects inside the polygon, else the least
// squared distance to its edge segments.  Evaluated with plain IEEE adds,
// multiplies and divides in a fixed order, without fused multiply-adds, so
// that the decision dist^2 < (2h)^2 is reproducible on any IEEE machine.
// cell_meets decides dist^2 < r2 with that arithmetic, with two shortcuts
// that cannot change the decision.  (1) The cell lies inside every face's
// half-space, so its distance is at least max_j(-d_j); when that bound
// exceeds sqrt(r2) by a relative margin far above the rounding of the
// polygon distances, the pair is rejected.  (2) The first face or edge
// distance computed below r2 accepts the pair, since the minimum is no
// larger.
template <class G>
__device__ __forceinline__ bool meets_impl(double px, double py, double pz, double r2, const G &g)
{
#pragma clang fp contract(off)
    const int nf = g.n_faces();
    double far = 0.0;
    bool inside = true;
    for (int j = 0; j < nf; j++) {
        const double d = g.pl(j, 3) - (g.pl(j, 0) * px + g.pl(j, 1) * py + g.pl(j, 2) * pz);
        if (d < 0.0) {
            inside = false;
            if (-d > far) far = -d;
        }
    }
    if (inside) return true;
    if (far * far > r2 * (1.0 + 1e-9)) return false;
    for (int j = 0; j < nf; j++) {
        const double n0 = g.pl(j, 0), n1 = g.pl(j, 1), n2 = g.pl(j, 2), c = g.pl(j, 3);
        const double d = c - (n0 * px + n1 * py + n2 * pz);
        if (!(d < 0.0)) continue;
        const int k0 = g.slot0(j), nv = g.slot0(j + 1) - k0;
        bool left = true;
        for (int k = 0; k < nv; k++) {
            const int kb = k0 + (k + 1 == nv ? 0 : k + 1);
            const double ax = g.vx(k0 + k, 0), ay = g.vx(k0 + k, 1), az = g.vx(k0 + k, 2);
            const double ex = g.vx(kb, 0) - ax, ey = g.vx(kb, 1) - ay, ez = g.vx(kb, 2) - az;
            const double wx = px - ax, wy = py - ay, wz = pz - az;
            const double cr = (ey * wz - ez * wy) * n0 + (ez * wx - ex * wz) * n1 + (ex * wy - ey * wx) * n2;
            if (cr < 0.0) {
                left = false;
                break;
            }
        }
        if (left) {
            if (d * d < r2) return true;
            continue;
        }
        for (int k = 0; k < nv; k++) {
            const int kb = k0 + (k + 1 == nv ? 0 : k + 1);
            const double ax = g.vx(k0 + k, 0), ay = g.vx(k0 + k, 1), az = g.vx(k0 + k, 2);
            const double ex = g.vx(kb, 0) - ax, ey = g.vx(kb, 1) - ay, ez = g.vx(kb, 2) - az;
            const double wx = px - ax, wy = py - ay, wz = pz - az;
            const double ee = ex * ex + ey * ey + ez * ez;
            double t = 0.0;
            if (ee > 0.0) {
                t = (wx * ex + wy * ey + wz * ez) / ee;
                if (t < 0.0) t = 0.0;
                if (t > 1.0) t = 1.0;
            }
            const double qx = wx - t * ex, qy = wy - t * ey, qz = wz - t * ez;
            if (qx * qx + qy * qy + qz * qz < r2) return true;
        }
    }
    return false;
}

// One cell's walls read from the global tables (slots relative to the cell's first).
struct CellGlobal {
    const double *plane;  // at the cell's first wall
    const int64_t *fvo;   // at the cell's first wall
    const EdgeRec *edges;  // at the cell's first slot
    int nf;
    __device__ int n_faces() const { return nf; }
    __device__ double pl(int j, int q) const { return plane[4 * j + q]; }
    __device__ int slot0(int j) const { return (int)(fvo[j] - fvo[0]); }
    __device__ double vx(int k, int q) const { return q == 0 ? edges[k].vx : (q == 1 ? edges[k].vy : edges[k].vz); }
};

// One cell staged in LDS by a wavefront for the screened distance test:
// wall planes in FP64 (the exact test's plane pass) and, per slot, the edge
// start vertex relative to the cell centre g, the unit direction, the unit
// in-wall normal (pointing into the wall polygon) and the length, in FP32; the
// candidates that wait for the test, and the walls that undecided ones still
// have to look at.
constexpr int kExactMaxFaces = 40, kExactMaxSlots = 160;
constexpr int kExactQueue = 128;  // below 64 waiting before a push of at most 64
struct CellFast {
    double pl_[kExactMaxFaces][4];
    float p_[64][3];            // the tested particles, about g
    float4 a_[kExactMaxSlots];  // vertex - g (x, y, z), length
    float4 b_[kExactMaxSlots];  // e (x, y, z), m.x
    float2 c_[kExactMaxSlots];  // m.y, m.z
    unsigned dmin_[64];         // least squared distance of each tested particle (bits of a float >= 0)
    uint32_t wait_[kExactQueue], part_[kExactQueue];  // places in the candidate list, particles
    uint16_t task_[kExactQueue];                      // lane << 8 | wall
    uint16_t so_[66];
};

__device__ __noinline__ bool cell_meets(double px, double py, double pz, double r2, int64_t cell,
                                        const int64_t *cfo, const int64_t *fvo, const EdgeRec *edges,
                                        const double *plane)
{
    const int64_t j0 = cfo[cell];
    CellGlobal g{plane + 4 * j0, fvo + j0, edges + fvo[j0], (int)(cfo[cell + 1] - j0)};
    return meets_impl(px, py, pz, r2, g);
}


// Leaves of the implicit tree: heap nodes [NL, 2NL), leaf j holds the cells
// cperm[kLeaf*(j-NL) .. +kLeaf).  Empty leaves get an inverted box.
__global__ void k_leaf_boxes(int64_t n_items, int64_t NL, const uint32_t *perm, const double *aabb, double *nodes)
{
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= NL) return;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t t = kLeaf * j; t < kLeaf * (j + 1) && t < n_items; t++) {
        const double *bb = aabb + 6 * (perm ? (int64_t)perm[t] : t);
        for (int d = 0; d < 3; d++) {
            lo[d] = fmin(lo[d], bb[d]);
            hi[d] = fmax(hi[d], bb[3 + d]);
        }
    }
    double *o = nodes + 6 * (NL + j);
    for (int d = 0; d < 3; d++) {
        o[d] = lo[d];
        o[3 + d] = hi[d];
    }
}

// Box of every point a particle's support can reach: x +- 2h (1 + 1e-8), widened
// by 1e-15 (|x| + 2h) for the rounding of its ends, so that it meets every cell
// box that the candidate test below accepts.
__global__ void k_particle_boxes(int64_t n, const double *__restrict__ xyz, const double *__restrict__ h,
                                 double *__restrict__ pbox)
{
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n) return;
    const double R = 2.0 * h[a] * (1.0 + 1e-8);
    for (int d = 0; d < 3; d++) {
        const double x = xyz[3 * a + d];
        const double pad = 1e-15 * (fabs(x) + R);
        pbox[6 * a + d] = (x - R) - pad;
        pbox[6 * a + 3 + d] = (x + R) + pad;
    }
}

__device__ __forceinline__ double box_dist2(const double *bb, double px, double py, double pz)
{
    double dx = fmax(fmax(bb[0] - px, px - bb[3]), 0.0);
    double dy = fmax(fmax(bb[1] - py, py - bb[4]), 0.0);
    double dz = fmax(fmax(bb[2] - pz, pz - bb[5]), 0.0);
    return dx * dx + dy * dy + dz * dz;
}

// Candidates of every cell: the particles whose support ball (radius 2h, with
// a relative 1e-9 on its square) comes within the cell's bounding box.  The
// particles form an implicit complete binary tree (heap indices: children 2i,
// 2i+1) over leaves of 8 consecutive particles, each node holding the box of
// its particles' reach boxes.  A wavefront walks it for kCells consecutive
// cells: pending nodes lie on a stack in LDS, leftmost on top, and each step
// takes the top 16 and tests their 64 grandchildren, one per lane, against the
// cells' boxes; the nodes met go back in order.  Once 8 leaves are on top, the
// lanes take their 64 particles and test them against each cell.  Nodes are
// expanded left to right, so each cell lists its particles in ascending order:
// the candidate list comes out cell-major with particles ascending, with no
// sort.  Particles stored in a spatially coherent order (Morton, Hilbert, as
// SPH codes keep them) give tight boxes; any order gives the same candidates.
// The walk also settles what it can without the exact test: accepted when
// the cell's whole bounding box lies within (1 - 1e-6) 2h of the particle, or
// when the ball about the cell's interior point g (radius rin) comes closer
// than (1 - 1e-9) 2h; dropped when the ball about g that contains the cell
// (radius rc) stays (1 + 1e-9) 2h or more away; the balls' radii have a margin
// of 1e-14 of their own, for supports far smaller than the cell.  The margins
// exceed the rounding of every distance involved, so these decisions are the
// exact test's.  The rest are marked for the exact test.
// A cell has room for K candidates (particle index, bit 31 = marked), from c K
// on.  A cell with more has all of them in the overflow list, from ovf_off[c]
// on, which a second walk of those cells writes (SECOND).
//
// Bound by the dependent loads of a walk (about 25 per wavefront) and, on full
// chips, by the FP64 tests.  One lane per cell over a packet of 64 cells (the
// lanes walking together, one node at a time) was a chain of several hundred
// loads on 1/64 of the wavefronts: 0.57 -> 0.038 ms for 4,096 uniform particles,
// 1.38 -> 0.23 ms for 65,537 and 2.18 -> 0.74 ms for 262,144 clumpy ones.
// kCells = 4: more cells share a walk but test more particles that only the
// others need.
constexpr int kCells = 4;
// Stack entries: from the top down the pending nodes' levels never increase (6,
// 8, ..., the leaves' level, at most 28 for 2^31 particles), and a step takes
// the nodes of a level only when it takes all deeper inner ones too, so a level
// holds at most the 64 nodes that one step put there (the leaves' level 15
// more that waited).
constexpr int kCandStack = 13 * 64 + 16;

template <bool SECOND>
__global__ void __launch_bounds__(256) k_candidates(
    int64_t n_cells, const double *__restrict__ aabb, const double *__restrict__ centre,
    const double *__restrict__ radii, int64_t n, const double *__restrict__ xyz, const double *__restrict__ h,
    const double *__restrict__ nodes, int64_t NL, int64_t *__restrict__ ccount, uint32_t *__restrict__ buf, int K,
    const int64_t *__restrict__ ovf_off, unsigned *__restrict__ max_count)
{
    __shared__ int stacks[4][kCandStack];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int *S = stacks[wave];
    const int64_t c0 = ((int64_t)xcd_block(blockIdx.x, gridDim.x) * 4 + wave) * kCells;
    if (c0 >= n_cells) return;  // whole wavefronts
    const int ng = n_cells - c0 < kCells ? (int)(n_cells - c0) : kCells;
    double lo[kCells][3], hi[kCells][3];
    bool use[kCells], any_cell = false;
#pragma unroll
    for (int g = 0; g < kCells; g++) {
        const int64_t c = c0 + (g < ng ? g : 0);
        use[g] = g < ng && (!SECOND || ccount[c] > K);
        any_cell = any_cell || use[g];
        for (int d = 0; d < 3; d++) {  // an unused cell's inverted box meets nothing
            lo[g][d] = use[g] ? aabb[6 * c + d] : INFINITY;
            hi[g][d] = use[g] ? aabb[6 * c + 3 + d] : -INFINITY;
        }
    }
    if (!any_cell) return;
    int count[kCells];
#pragma unroll
    for (int g = 0; g < kCells; g++) count[g] = 0;
    auto meets = [&](int64_t node) {
        const double *b = nodes + 6 * node;
        const double b0 = b[0], b1 = b[1], b2 = b[2], b3 = b[3], b4 = b[4], b5 = b[5];
        bool m = false;
#pragma unroll
        for (int g = 0; g < kCells; g++)
            m = m || (b0 <= hi[g][0] && lo[g][0] <= b3 && b1 <= hi[g][1] && lo[g][1] <= b4 && b2 <= hi[g][2] &&
                      lo[g][2] <= b5);
        return m;
    };
    auto below = [&](unsigned long long m) {
        return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    };
    // level 6 of the tree (or the leaves of a smaller one)
    int sp;
    {
        const int64_t first = NL < 64 ? NL : 64;
        const bool v = lane < first && meets(first + lane);
        const unsigned long long m = __ballot(v);
        sp = __popcll(m);
        if (v) S[sp - 1 - below(m)] = (int)(first + lane);
    }
    lds_sync_wave();
    while (sp > 0) {
        const int k = sp < 16 ? sp : 16;
        const int e = lane >> 2, q = lane & 3;
        const int64_t node = e < k ? S[sp - 1 - e] : 0;
        const bool inner = e < k && node < NL;
        const unsigned long long im = __ballot(inner);
        const int lead = im ? __builtin_ctzll(im) >> 2 : k;  // leaves on top of the stack
        if (lead >= 8 || lead == k) {
            const int kk = lead < 8 ? lead : 8;
            const int64_t t = (lane >> 3) < kk ? kLeaf * ((int64_t)S[sp - 1 - (lane >> 3)] - NL) + (lane & 7) : n;
            sp -= kk;
            const bool valid = t < n;
            const int64_t a = valid ? t : 0;
            const double px = xyz[3 * a], py = xyz[3 * a + 1], pz = xyz[3 * a + 2], r = 2.0 * h[a], r2 = r * r;
#pragma unroll
            for (int g = 0; g < kCells; g++) {
                const double cb[6] = {lo[g][0], lo[g][1], lo[g][2], hi[g][0], hi[g][1], hi[g][2]};
                if (!use[g]) continue;
                const bool in_reach = valid && !(box_dist2(cb, px, py, pz) > r2 * (1.0 + 1e-9));
                if (__ballot(in_reach) == 0) continue;
                const int64_t c = c0 + g;
                const double fx = fmax(fabs(cb[0] - px), fabs(cb[3] - px));
                const double fy = fmax(fabs(cb[1] - py), fabs(cb[4] - py));
                const double fz = fmax(fabs(cb[2] - pz), fabs(cb[5] - pz));
                const double dx = centre[3 * c] - px, dy = centre[3 * c + 1] - py, dz = centre[3 * c + 2] - pz;
                const double dg2 = dx * dx + dy * dy + dz * dz;
                const double ri = r * (1.0 - 1e-9) + radii[2 * c] * (1.0 - 1e-14);
                const double ro = r * (1.0 + 1e-9) + radii[2 * c + 1] * (1.0 + 1e-14);
                const bool ok = fx * fx + fy * fy + fz * fz < r2 * 0.999998 || dg2 < ri * ri;
                const bool cand = in_reach && (ok || dg2 < ro * ro);
                const unsigned long long mc = __ballot(cand);
                const int at = count[g] + below(mc);
                if (cand && (SECOND || at < K))
                    buf[(SECOND ? ovf_off[c] : c * (int64_t)K) + at] = (uint32_t)t | (ok ? 0u : 0x80000000u);
                count[g] += __popcll(mc);
            }
            lds_sync_wave();  // the leaves are read before their places are written again
            continue;
        }
        // grandchildren (children above the leaves); a leaf below an inner node stays
        const bool two = 2 * node < NL;
        const int64_t child = inner ? (two ? 4 * node + q : 2 * node + q) : node;
        const bool exists = inner ? (two || q < 2) : (e < k && q == 0);
        const bool v = exists && (!inner || meets(child));
        const unsigned long long m = __ballot(v);
        sp += __popcll(m) - k;
        lds_sync_wave();  // every lane has its node before the places are written
        if (v) S[sp - 1 - below(m)] = (int)child;
        lds_sync_wave();
    }
    if (!SECOND && lane == 0) {
        int most = 0;
#pragma unroll
        for (int g = 0; g < kCells; g++)
            if (g < ng) {
                ccount[c0 + g] = count[g];
                most = most > count[g] ? most : count[g];
            }
        if (most > K) atomicMax(max_count, (unsigned)most);  // (asked for only where it is more than K)
    }
}

// The tested and accepted candidates of each cell, one wavefront per cell: the
// marked ones are collected 64 at a time and take the exact test, the rejected
// ones are struck from the list (kNoCand), and the cell's pairs are counted.
// The wavefront stages its cell in LDS.  Each lane then, for its particle, (1)
// runs the exact test's plane pass (inside: accept; a wall plane beyond the
// radius by the relative margin: reject), (2) takes the squared distance D to
// the wall polygon that is farthest beneath the particle, in FP32 about the
// cell centre: the wall's own distance when the foot point lies inside the
// polygon, which is then the distance to the cell, else the least distance to
// the wall's edge segments, an upper bound of it; accepted when below r^2; (3)
// the rest, whose nearest point may lie on another wall seen from outside,
// become tasks (lane, wall) that the lanes share, and D is the least of all.
// D decides when |D - r^2| exceeds a bound on its rounding, tol = 1e-6 (r + 2
// rc)^2 (every vector involved is shorter than r + 2 rc, FP32 rounding of D is
// below 10 u (r + 2 rc)^2, and the tasks' wall distance, taken from the rounded
// particle, below 4 u (r + 2 rc)^2 more: 14 u = 0.8e-6); (4) D within tol of r^2, and cells of more than 64
// walls, run the exact test.  Lengths are rounded to FP32 in a unit near the
// cell's size, a power of two, so that their squares stay in FP32's range
// whatever the caller's unit; a support 1e15 cells wide leaves it and takes
// the exact test.  Cells too large for the staging area are read
// from the global tables throughout.
//
// Bound by latency: 58 % of the wavefronts' time is waits (the cell's records,
// gathers from LDS), vector instructions at 0.12 per SIMD and clock with half
// of the lanes active.  With 64 list entries per wavefront (two or three cells
// each, staged one after the other, a third of the lanes each), every lane
// looping over all walls it sees, and the candidates gathered into lists of
// their own first, 262,144 clumpy particles took 2.22 ms here and 0.37 ms around
// it; 1.55 and 0.13 ms now.
constexpr uint32_t kNoCand = 0xffffffffu;

// One slot of the tested cell as the screened test takes it: edge start (about
// the cell centre) and length in the cell's unit, edge direction, in-wall normal.  From the staged
// cell, or for a cell too large for it from its records.
struct SlotF {
    float ax, ay, az, len, ex, ey, ez, mx, my, mz;
};

__device__ __forceinline__ SlotF slot_of(const EdgeRec &E, double gx, double gy, double gz, double per_unit)
{
    return SlotF{(float)((E.vx - gx) * per_unit), (float)((E.vy - gy) * per_unit), (float)((E.vz - gz) * per_unit),
                 (float)(E.L * per_unit), (float)E.ex, (float)E.ey, (float)E.ez, (float)E.mx, (float)E.my, (float)E.mz};
}

// squared FP32 distance from q (about the cell centre) to wall j of the cell: d2 (its plane's distance) when q's foot
// point lies inside the polygon
template <class Slots>
__device__ __forceinline__ float wall_dist2(const Slots &slot, int k0, int k1, float qx, float qy, float qz, float d2,
                                            bool &in_poly)
{
    in_poly = true;
    float D = INFINITY;
    for (int k = k0; k < k1; k++) {
        const SlotF E = slot(k);
        const float wx = qx - E.ax, wy = qy - E.ay, wz = qz - E.az;
        in_poly = in_poly && fmaf(E.mx, wx, fmaf(E.my, wy, E.mz * wz)) >= 0.0f;
        const float sp = fmaf(E.ex, wx, fmaf(E.ey, wy, E.ez * wz));
        const float tt = fminf(fmaxf(sp, 0.0f), E.len);
        const float ux = fmaf(-tt, E.ex, wx), uy = fmaf(-tt, E.ey, wy), uz = fmaf(-tt, E.ez, wz);
        D = fminf(D, fmaf(ux, ux, fmaf(uy, uy, uz * uz)));
    }
    return in_poly ? d2 : D;
}

constexpr int kExactWaves = 2;  // cells per workgroup: 20 KB of LDS, 4 wavefronts per SIMD

template <bool SECOND>
__global__ void __launch_bounds__(64 * kExactWaves) k_exact(
    int64_t n_cells, const int64_t *__restrict__ ccount, uint32_t *__restrict__ buf, int K,
    const int64_t *__restrict__ ovf_off, const double *__restrict__ xyz, const double *__restrict__ h,
    const int64_t *__restrict__ cfo, const int64_t *__restrict__ fvo, const EdgeRec *__restrict__ edges,
    const double *__restrict__ plane, const double *__restrict__ centre, const double *__restrict__ radii,
    int64_t *__restrict__ pcount, unsigned long long *__restrict__ n_tested)
{
#pragma clang fp contract(off)
    __shared__ CellFast stage[kExactWaves];
    __shared__ unsigned tested[kExactWaves];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    CellFast &L = stage[wave];
    const int64_t c = (int64_t)blockIdx.x * kExactWaves + wave;
    unsigned n_test = 0;
    const int64_t cnt = c < n_cells ? ccount[c] : 0;
    if (c < n_cells && (cnt > K) == SECOND) {
        uint32_t *mine = buf + (SECOND ? ovf_off[c] : c * (int64_t)K);
        const int64_t j0 = cfo[c], nf = cfo[c + 1] - j0;
        const int64_t s0 = fvo[j0], ns = fvo[j0 + nf] - s0;
        const bool screen = nf <= 64 && ns < 65536;  // (a bit per wall, 16-bit slot offsets)
        const bool fits = nf <= kExactMaxFaces && ns <= kExactMaxSlots;
        const double gx = centre[3 * c], gy = centre[3 * c + 1], gz = centre[3 * c + 2], rc2 = 2.0 * radii[2 * c + 1];
        const int ex = min(max(__builtin_amdgcn_frexp_exp(rc2), -1000), 1000);
        const double unit = __builtin_amdgcn_ldexp(1.0, ex), per_unit = __builtin_amdgcn_ldexp(1.0, -ex);
        int64_t pairs = 0;
        bool staged = false;
        int waiting = 0;
        auto test = [&](int n) {  // the first n (<= 64) of the waiting candidates
            if (screen && !staged) {
                for (int q = lane; q <= (int)nf; q += 64) L.so_[q] = (uint16_t)(fvo[j0 + q] - s0);
                if (fits) {
                    for (int q = lane; q < 4 * (int)nf; q += 64) L.pl_[q >> 2][q & 3] = plane[4 * j0 + q];
                    for (int q = lane; q < (int)ns; q += 64) {
                        const SlotF E = slot_of(edges[s0 + q], gx, gy, gz, per_unit);
                        L.a_[q] = make_float4(E.ax, E.ay, E.az, E.len);
                        L.b_[q] = make_float4(E.ex, E.ey, E.ez, E.mx);
                        L.c_[q] = make_float2(E.my, E.mz);
                    }
                }
                staged = true;
            }
            auto pl = [&](int j, int d) { return fits ? L.pl_[j][d] : plane[4 * (j0 + j) + d]; };
            auto wall = [&](int j, float qx, float qy, float qz, float d2, bool &in_poly) {
                auto lds = [&](int k) {
                    const float4 A = L.a_[k], B = L.b_[k];
                    const float2 C = L.c_[k];
                    return SlotF{A.x, A.y, A.z, A.w, B.x, B.y, B.z, B.w, C.x, C.y};
                };
                auto rec = [&](int k) { return slot_of(edges[s0 + k], gx, gy, gz, per_unit); };
                const int k0 = L.so_[j], k1 = L.so_[j + 1];
                return fits ? wall_dist2(lds, k0, k1, qx, qy, qz, d2, in_poly)
                            : wall_dist2(rec, k0, k1, qx, qy, qz, d2, in_poly);
            };
            lds_sync_wave();
            const bool valid = lane < n;
            const int64_t a = valid ? L.part_[lane] : 0;
            const double px = xyz[3 * a], py = xyz[3 * a + 1], pz = xyz[3 * a + 2], r = 2.0 * h[a], r2 = r * r;
            bool hit = false, exact = valid && !screen;
            if (screen) {
                bool inside = true;
                double far = 0.0;
                int jf = 0;
                unsigned long long seen = 0;  // walls seen from outside
                for (int j = 0; j < (int)nf; j++) {
                    const double d = pl(j, 3) - (pl(j, 0) * px + pl(j, 1) * py + pl(j, 2) * pz);
                    if (d < 0.0) {
                        inside = false;
                        seen |= 1ull << j;
                        if (-d > far) {
                            far = -d;
                            jf = j;
                        }
                    }
                }
                hit = valid && inside;
                bool open = valid && !inside && !(far * far > r2 * (1.0 + 1e-9));
                const double rs = r * per_unit, rs2 = rs * rs, rr = rs + rc2 * per_unit, tol = 1e-6 * rr * rr;
                if (open && !(rr < 1e15)) {
                    exact = true;
                    open = false;
                }
                const float qx = (float)((px - gx) * per_unit), qy = (float)((py - gy) * per_unit),
                            qz = (float)((pz - gz) * per_unit);
                const double fs = far * per_unit;
                float D = INFINITY;
                if (open) {
                    bool in_poly;
                    D = wall(jf, qx, qy, qz, (float)(fs * fs), in_poly);
                    seen &= in_poly ? 0ull : ~(1ull << jf);
                    if ((double)D < rs2 - tol) {
                        hit = true;
                        open = false;
                    }
                }
                unsigned long long sm = open ? seen : 0ull;
                if (__ballot(sm != 0) != 0) {
                    L.p_[lane][0] = qx;
                    L.p_[lane][1] = qy;
                    L.p_[lane][2] = qz;
                    L.dmin_[lane] = __float_as_uint(D);
                    int nt = 0;
                    auto run = [&](int at, int m) {
                        lds_sync_wave();
                        if (lane < m) {
                            const int o = L.task_[at + lane] >> 8, j = L.task_[at + lane] & 255;
                            const float x = L.p_[o][0], y = L.p_[o][1], z = L.p_[o][2];
                            const double d = (pl(j, 3) - (pl(j, 0) * (gx + x * unit) + pl(j, 1) * (gy + y * unit) +
                                                          pl(j, 2) * (gz + z * unit))) * per_unit;
                            bool in_poly;
                            const float Dj = wall(j, x, y, z, (float)(d * d), in_poly);
                            atomicMin(&L.dmin_[o], __float_as_uint(Dj));
                        }
                        lds_sync_wave();
                    };
                    while (__ballot(sm != 0) != 0) {
                        const bool want = sm != 0;
                        const int at = wave_push(want, nt);
                        if (want) L.task_[at] = (uint16_t)(lane << 8 | __builtin_ctzll(sm));
                        sm &= sm - 1;
                        if (nt >= 64) {
                            run(nt - 64, 64);
                            nt -= 64;
                        }
                    }
                    run(0, nt);
                    D = __uint_as_float(L.dmin_[lane]);
                }
                if (open) {
                    if ((double)D < rs2 - tol) hit = true;
                    else if (!((double)D > rs2 + tol)) exact = true;
                }
            }
            if (exact) hit = cell_meets(px, py, pz, r2, c, cfo, fvo, edges, plane);
            if (valid) mine[L.wait_[lane]] = hit ? (uint32_t)a : kNoCand;
            pairs += __popcll(__ballot(hit));
            n_test += (unsigned)n;
            // the others move up
            lds_sync_wave();
            const int left = waiting - n;
            const uint32_t w = lane < left ? L.wait_[n + lane] : 0u, q = lane < left ? L.part_[n + lane] : 0u;
            lds_sync_wave();
            if (lane < left) {
                L.wait_[lane] = w;
                L.part_[lane] = q;
            }
            waiting = left;
        };
        for (int64_t k0 = 0; k0 < cnt || waiting > 0;) {
            if (k0 < cnt && waiting < 64) {
                const int64_t k = k0 + lane;
                const uint32_t e = k < cnt ? mine[k] : 0u;
                const bool marked = k < cnt && (e >> 31) != 0;
                pairs += __popcll(__ballot(k < cnt && !marked));
                const int at = wave_push(marked, waiting);
                if (marked) {
                    L.wait_[at] = (uint32_t)k;
                    L.part_[at] = e & 0x7fffffffu;
                }
                k0 += 64;
            }
            if (waiting >= 64 || (k0 >= cnt && waiting > 0)) test(waiting < 64 ? waiting : 64);
        }
        if (lane == 0) pcount[c] = pairs;
    } else if (!SECOND && c < n_cells && lane == 0) {
        pcount[c] = 0;  // counted by the second pass
    }
    if (lane == 0) tested[wave] = n_test;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned all = 0;
        for (int w = 0; w < kExactWaves; w++) all += tested[w];
        if (all > 0) atomicAdd(counter_copy(n_tested), (unsigned long long)all);
    }
}

// Sizes of the overflow lists.
__global__ void k_overflow_sizes(int64_t n_cells, const int64_t *__restrict__ ccount, int K, int64_t *__restrict__ size)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n_cells) size[c] = ccount[c] > K ? ccount[c] : 0;
}

// The candidates left of each cell to the cell-major pair list (candidate
// order kept), one wavefront per cell.
__global__ void k_compact(int64_t n_cells, const int64_t *__restrict__ ccount, const uint32_t *__restrict__ buf, int K,
                          const uint32_t *__restrict__ ovf, const int64_t *__restrict__ ovf_off,
                          const int64_t *__restrict__ coff, uint32_t *__restrict__ pair_c,
                          uint32_t *__restrict__ pair_p)
{
    const int64_t c = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (c >= n_cells) return;
    const int64_t cnt = ccount[c];
    const uint32_t *mine = cnt > K ? ovf + ovf_off[c] : buf + c * (int64_t)K;
    int64_t o = coff[c];
    for (int64_t k0 = 0; k0 < cnt; k0 += 64) {
        const int64_t k = k0 + lane;
        const uint32_t e = k < cnt ? mine[k] : kNoCand;
        const bool take = e != kNoCand;
        const unsigned long long m = __ballot(take);
        if (take) {
            const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            pair_c[o + below] = (uint32_t)c;
            pair_p[o + below] = e;
        }
        o += __popcll(m);
    }
}

// Segment offsets of sorted keys: off[v] = first i with keys[i] >= v, v = 0..n_seg.
__global__ void k_seg_offsets(int64_t n_items, const uint32_t *__restrict__ keys, int64_t n_seg,
                              int64_t *__restrict__ off)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n_items) return;
    const int64_t prev = i == 0 ? -1 : (int64_t)keys[i - 1];
    const int64_t cur = i == n_items ? n_seg : (int64_t)keys[i];
    for (int64_t v = prev + 1; v <= cur; v++) off[v] = i;
}

void build_particle_view(Workspace &ws, const uint32_t *pair_p, int64_t n_pairs, int64_t n, uint32_t *perm,
                         int64_t *poff, hipStream_t s)
{
    if (n_pairs == 0) {
        fill_zero_bytes(poff, sizeof(int64_t) * (n + 1), s);
        return;
    }
    uint32_t *key = ws.get<uint32_t>(S_KEY2, (size_t)n_pairs);
    EM_HIP(hipMemcpyAsync(key, pair_p, sizeof(uint32_t) * n_pairs, hipMemcpyDeviceToDevice, s));
    fill_iota_u32(perm, n_pairs, s);
    int bits = 1;
    while (bits < 32 && ((uint64_t)(n - 1) >> bits) != 0) bits++;
    radix_sort_u32(ws, key, perm, ws.get<uint32_t>(S_IOTA, (size_t)n_pairs), ws.get<uint32_t>(S_PC_PM, (size_t)n_pairs),
                   n_pairs, bits, s);
    hipLaunchKernelGGL(k_seg_offsets, dim3((unsigned)((n_pairs + 1 + 255) / 256)), dim3(256), 0, s, n_pairs,
                       (const uint32_t *)key, n, poff);
    EM_HIP(hipGetLastError());
}

PairSet build_pairs(Workspace &ws, const DevInputs &in, const double *aabb, const EdgeRec *edges,
                    int64_t *counters, hipStream_t s)
{
    PairSet ps;
    const int64_t n = in.n, nc = in.n_cells;
    int64_t *coff = ws.get<int64_t>(S_COFF, (size_t)nc + 1);
    ps.coff = coff;
    if (n == 0 || nc == 0) {
        fill_zero_bytes(coff, sizeof(int64_t) * (nc + 1), s);
        return ps;
    }
    for (int d = 0; d < 3; d++) {
        const double ext = in.box[3 + d] - in.box[d];
        EM_CHECK(ext > 0.0 && std::isfinite(ext), MAP_EINVAL, "box has non-positive extent");
    }
    // bounding-volume tree over the particles' reach boxes, leaves of 8 particles in storage order
    double *pbox = ws.get<double>(S_PBOX, (size_t)(6 * n));
    hipLaunchKernelGGL(k_particle_boxes, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, in.xyz, in.h, pbox);
    EM_HIP(hipGetLastError());
    int64_t nleaf = (n + kLeaf - 1) / kLeaf, NL = 1;
    while (NL < nleaf) NL <<= 1;
    double *nodes = ws.get<double>(S_BINOFF_G, (size_t)(12 * NL));
    hipLaunchKernelGGL(k_leaf_boxes, dim3((unsigned)((NL + 255) / 256)), dim3(256), 0, s, n, NL,
                       (const uint32_t *)nullptr, (const double *)pbox, nodes);
    EM_HIP(hipGetLastError());
    tree_parent_boxes(nodes, NL, s);

    // candidates per cell (tree walk with the cheap tests, particles ascending),
    // the exact test of the marked ones, and the pairs per cell.  Each cell has
    // room for K candidates: at most 2^30 in all (4 GiB; 128 per cell at 8.4
    // million cells), and in arena mode at most a quarter of the free scratch.
    int64_t *ccount = ws.get<int64_t>(S_PCNT, (size_t)nc);
    int64_t *pcount = ws.get<int64_t>(S_PCNT2, (size_t)nc);
    const int64_t slot_cap = std::min<int64_t>(int64_t(1) << 30, (int64_t)std::min<size_t>(ws.arena_free() / 16, size_t(1) << 40));
    const int K = (int)std::max<int64_t>(32, std::min<int64_t>(512, slot_cap / nc));
    uint32_t *buf = ws.get<uint32_t>(S_CAND_BUF, (size_t)(nc * K)), *ovf = nullptr;
    int64_t *ovf_off = nullptr;
    unsigned *cmax = ws.get<unsigned>(S_CAND_MAX, 64);
    fill_zero_bytes(cmax, sizeof(unsigned), s);
    const double *centre = aabb + 6 * nc, *radii = aabb + 9 * nc;
    unsigned long long *tested = reinterpret_cast<unsigned long long *>(counters + C_CANDIDATES);
    const dim3 wg((unsigned)((nc + 4 * kCells - 1) / (4 * kCells))), eg((unsigned)((nc + kExactWaves - 1) / kExactWaves));
    hipLaunchKernelGGL(k_candidates<false>, wg, dim3(256), 0, s, nc, aabb, centre, radii, n, in.xyz, in.h,
                       (const double *)nodes, NL, ccount, buf, K, (const int64_t *)nullptr, cmax);
    EM_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_exact<false>, eg, dim3(64 * kExactWaves), 0, s, nc, (const int64_t *)ccount, buf, K,
                       (const int64_t *)nullptr, in.xyz, in.h, in.cfo, in.fvo, edges, in.plane, centre, radii, pcount,
                       tested);
    EM_HIP(hipGetLastError());
    scan_counts(ws, pcount, coff, nc, s);
    int64_t np = 0;
    unsigned max_cand = 0;
    read_back(ws, {{&np, coff + nc, sizeof(int64_t)}, {&max_cand, cmax, sizeof(unsigned)}}, s);
    if ((int64_t)max_cand > K) {
        // the cells with more candidates: their lists' places, the walk and the test again for them
        int64_t *size = ws.get<int64_t>(S_NCNT, (size_t)nc);
        ovf_off = ws.get<int64_t>(S_CCNT64, (size_t)(nc + 1));
        hipLaunchKernelGGL(k_overflow_sizes, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s, nc,
                           (const int64_t *)ccount, K, size);
        EM_HIP(hipGetLastError());
        scan_counts(ws, size, ovf_off, nc, s);
        int64_t n_ovf = 0;
        read_back(ws, {{&n_ovf, ovf_off + nc, sizeof(int64_t)}}, s);
        ovf = ws.get<uint32_t>(S_BINLIST, (size_t)n_ovf);
        hipLaunchKernelGGL(k_candidates<true>, wg, dim3(256), 0, s, nc, aabb, centre, radii, n, in.xyz, in.h,
                           (const double *)nodes, NL, ccount, ovf, K, (const int64_t *)ovf_off, cmax);
        EM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_exact<true>, eg, dim3(64 * kExactWaves), 0, s, nc, (const int64_t *)ccount, ovf, K,
                           (const int64_t *)ovf_off, in.xyz, in.h, in.cfo, in.fvo, edges, in.plane, centre, radii,
                           pcount, tested);
        EM_HIP(hipGetLastError());
        scan_counts(ws, pcount, coff, nc, s);
        read_back(ws, {{&np, coff + nc, sizeof(int64_t)}}, s);
    }
    EM_CHECK(np < (int64_t)UINT32_MAX, MAP_ENOMEM, "pair count exceeds 2^32-1");
    ps.n_pairs = np;
    if (np == 0) return ps;
    uint32_t *pair_c = ws.get<uint32_t>(S_PAIR_C, (size_t)np);
    uint32_t *pair_p = ws.get<uint32_t>(S_PAIR_P, (size_t)np);
    hipLaunchKernelGGL(k_compact, dim3((unsigned)((nc + 3) / 4)), dim3(256), 0, s, nc, (const int64_t *)ccount,
                       (const uint32_t *)buf, K, (const uint32_t *)ovf, (const int64_t *)ovf_off,
                       (const int64_t *)coff, pair_c, pair_p);
    EM_HIP(hipGetLastError());
    ps.pair_c = pair_c;
    ps.pair_p = pair_p;
    return ps;
}

}  // namespace em
