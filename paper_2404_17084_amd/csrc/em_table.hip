// Tabulated variant of the pair integral (Sec. II-B: the vertex-pyramid
// integral pre-computed on a grid and interpolated).
//
// The table holds I(r0, R0, phi) on a uniform n0 x n1 x n2 grid over
// r0, R0 in [0, 2] and phi in [0, pi/2] (FP32 node values of the FP64 closed
// form).  A pair is assembled in the far-field-subtracted form of the closed
// form: with D = Omega / (4 pi) - I, the mass of a pyramid's cone beyond its
// wall,
//     f = [p inside] - sum_walls sigma_j sum_edges sign(rho) [D~(l_b) - D~(l_a)],
//     D~(l) = sign(l) D(r0, R0, atan(|l| / R0)),
// because the solid angles of a cell's pyramids add up to its winding number
// about the particle.  D = 0 for walls with r0 >= 2 (skipped), and for R0 > 2
// D does not depend on R0 (the support's cross-section with the wall lies in
// the triangle's wedge), so it is read at R0 = 2 with the same angle.  Each D
// is one solid angle (FP32, one atan2) less a trilinear read of the table;
// geometry is FP64, sums are FP64.
//
// One lane per pair, cell-major pair order (neighbouring lanes share a cell, so
// wall and edge records are read once per wavefront from cache); the table
// stays in L2.  The lanes of a wavefront walk their cells' wall
// slots with one counter, so that an edge's two table reads run once for all
// lanes that have an edge.  Bound by the gathers: a read with its eight nodes in
// four places fetched four cache lines per lane, 40 TB/s from L2 on 2.8e6
// pairs, and took 6.5 ms however few instructions went with it; with the nodes
// of a read in 32 neighbouring bytes (a table of four times the size, 4 MiB at
// 64^3) it is 2.3 ms.
#include <cmath>

#include "em_boundary.h"
#include "em_internal.h"
#include "em_fmath.h"
#include "em_wave.h"

namespace em {

namespace {

struct TableView {
    const TabNode *__restrict__ t;  // per node (i, j, k), i < n0 - 1, j < n1 - 1: the values at (i, j), (i, j + 1), (i + 1, j), (i + 1, j + 1)
    int n0, n1, n2;
    float s0, s1, s2;  // grid coordinates per unit of r0, R0, phi
};

__device__ __forceinline__ void grid_cell(float x, int n, int &i, float &a)
{
    int k = (int)floorf(x);
    k = k < 0 ? 0 : (k > n - 2 ? n - 2 : k);
    i = k;
    a = x - (float)k;
}

__device__ __forceinline__ float table_I(const TableView &T, float r0, float R0, float phi)
{
    int i, j, k;
    float a, b, c;
    grid_cell(r0 * T.s0, T.n0, i, a);
    grid_cell(R0 * T.s1, T.n1, j, b);
    grid_cell(phi * T.s2, T.n2, k, c);
    const TabNode *p = T.t + ((int64_t)i * T.n1 + j) * T.n2 + k;
    const TabNode A = p[0], B = p[1];
    const float v00 = A.x + c * (B.x - A.x);
    const float v01 = A.y + c * (B.y - A.y);
    const float v10 = A.z + c * (B.z - A.z);
    const float v11 = A.w + c * (B.w - A.w);
    const float v0 = v00 + b * (v01 - v00);
    const float v1 = v10 + b * (v11 - v10);
    return v0 + a * (v1 - v0);
}

// D of the right triangle [0, |l|] at wall distance r0 < 2, odd in l
__device__ __forceinline__ float table_Dt(const TableView &T, float r0, float R0, float ls)
{
    const float l = fabsf(ls);
    const float phi = atan2_f32(l, R0);
    const bool far = R0 > 2.0f;  // same angle at R0 = 2
    const float Rc = far ? 2.0f : R0, lc = far ? l * (2.0f * rcp_f32(R0)) : l;
    const float R2 = Rc * Rc, l2 = lc * lc;
    const float S = sqrt_f32(fmaf(lc, lc, fmaf(Rc, Rc, r0 * r0)));
    const float om = atan2_f32(lc * Rc * fmaf(Rc, Rc, l2), (S + r0) * fmaf(l2, r0, R2 * S));
    const float D = fmaf(om, 0.0795774715459477f, -table_I(T, r0, Rc, phi));
    return l > 0.0f ? (ls < 0.0f ? -D : D) : 0.0f;
}

__global__ void __launch_bounds__(256) k_integrate_table(int64_t np, const uint32_t *__restrict__ pair_p,
                                                         const uint32_t *__restrict__ pair_c,
                                                         const double *__restrict__ xyz, const double *__restrict__ h,
                                                         const int64_t *__restrict__ cfo,
                                                         const int64_t *__restrict__ fvo,
                                                         const double *__restrict__ plane,
                                                         const EdgeRec *__restrict__ edges, TableView T,
                                                         double *__restrict__ f, unsigned long long *counters)
{
    const int64_t q = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const bool active = q < np;
    unsigned n_faces = 0, n_edges = 0, n_terms = 0;
    double px = 0.0, py = 0.0, pz = 0.0, invh = 1.0;
    int64_t cell = 0;
    int32_t j = 0, s = 0, s_end = 0;
    if (active) {
        const int64_t a = pair_p[q];
        cell = pair_c[q];
        px = xyz[3 * a];
        py = xyz[3 * a + 1];
        pz = xyz[3 * a + 2];
        invh = 1.0 / h[a];
        j = (int32_t)cfo[cell] - 1;
        s = (int32_t)fvo[cfo[cell]];
        s_end = (int32_t)fvo[cfo[cell + 1]];
    }
    int32_t face_end = s;  // first slot past the current wall: the first step opens the cell's first wall
    int n_steps = s_end - s;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n_steps = max(n_steps, __shfl_xor(n_steps, o, 64));
    bool inside = true, in_j = true, face_ok = false;
    int n_on = 0;
    double acc = 0.0, face = 0.0;
    float r0 = 0.0f;
    for (int it = 0; it < n_steps; it++, s++) {
        const bool valid = s < s_end;
        if (valid && s == face_end) {  // the next wall
            acc += in_j ? face : -face;
            face = 0.0;
            j++;
            face_end = (int32_t)fvo[j + 1];
            const double *pl = plane + plane_at(j);
            const double nx = pl[0], ny = pl[1], nz = pl[2], cj = pl[3];
            const double d = cj - (nx * px + ny * py + nz * pz);
            n_faces++;
            in_j = d >= 0.0;
            inside = inside && in_j;
            n_on += d == 0.0 ? 1 : 0;
            const double r0d = fabs(d) * invh;
            face_ok = r0d < 2.0;
            r0 = (float)r0d;
        }
        if (valid && face_ok) {
            const EdgeRec E = edges[s];
            const double wx = px - E.vx, wy = py - E.vy, wz = pz - E.vz;
            const double rho = E.mx * wx + E.my * wy + E.mz * wz;
            n_edges++;
            if (rho != 0.0) {
                const double la = -(E.ex * wx + E.ey * wy + E.ez * wz) * invh;
                const double lb = la + E.L * invh;
                const float R0 = (float)(fabs(rho) * invh);
                const float t = table_Dt(T, r0, R0, (float)lb) - table_Dt(T, r0, R0, (float)la);
                n_terms += 2;
                face += rho > 0.0 ? (double)t : -(double)t;
            }
        }
    }
    if (active) {
        acc += in_j ? face : -face;
        f[q] = winding_term(inside, n_on, px, py, pz, cell, cfo, fvo, plane, edges) - acc;
    }
    unsigned long long v[3] = {n_faces, n_edges, n_terms};
    for (int u = 0; u < 3; u++)
        for (int o = 32; o > 0; o >>= 1) v[u] += __shfl_xor(v[u], o, 64);
    // lane q brings the q-th (one atomic instruction on one cache line)
    const int lane = threadIdx.x & 63;
    if (lane < 3)
        atomicAdd(counter_copy(counters) + (lane == 0 ? C_FACES : (lane == 1 ? C_EDGES : C_EDGE_TERMS)),
                  lane == 0 ? v[0] : (lane == 1 ? v[1] : v[2]));
}

}  // namespace

void launch_integrate_table(const DevInputs &in, const EdgeRec *edges, const PairSet &ps, const TabNode *tab, int n0,
                            int n1, int n2, double *f, int64_t *counters, hipStream_t s)
{
    const int64_t np = ps.n_pairs;
    if (np <= 0) return;
    TableView T;
    T.t = tab;
    T.n0 = n0;
    T.n1 = n1;
    T.n2 = n2;
    T.s0 = (float)(n0 - 1) * 0.5f;
    T.s1 = (float)(n1 - 1) * 0.5f;
    T.s2 = (float)((double)(n2 - 1) / (0.5 * M_PI));
    hipLaunchKernelGGL(k_integrate_table, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, np, ps.pair_p,
                       ps.pair_c, in.xyz, in.h, in.cfo, in.fvo, in.plane, edges, T, f,
                       reinterpret_cast<unsigned long long *>(counters));
    EM_HIP(hipGetLastError());
}

}  // namespace em
