// Droplet surface (for D_LBM, Sec. 5 Eq. 17), droplet mass and mass reinjection
// (Sec. 2: the open boundary does not conserve mass; mass is put back into the
// droplet so that its density stays fixed).
#pragma once

#include "aux_kernels.hpp"
#include "wave.hpp"

namespace sclbm {

// Zero set of phi (linear inside the tetrahedron with corners p[0..3], values s[0..3]):
// adds its area and the volume of {phi > 0}.  The volume uses the edge fractions of the
// cut (barycentric closed forms); the tetrahedron's volume is 1/6 (one sixth of a cell).
__device__ __forceinline__ double tri_area2(const double *a, const double *b, const double *c) {
    const double ux = b[0] - a[0], uy = b[1] - a[1], uz = b[2] - a[2];
    const double vx = c[0] - a[0], vy = c[1] - a[1], vz = c[2] - a[2];
    const double wx = uy * vz - uz * vy, wy = uz * vx - ux * vz, wz = ux * vy - uy * vx;
    return sqrt(wx * wx + wy * wy + wz * wz);  // twice the area
}

__device__ __forceinline__ void cut_point(const double *p, const double *q, double t, double *x) {
    x[0] = p[0] + t * (q[0] - p[0]);
    x[1] = p[1] + t * (q[1] - p[1]);
    x[2] = p[2] + t * (q[2] - p[2]);
}

__device__ __forceinline__ void tet_cut(const double (&p)[4][3], const double (&s)[4], double &area, double &vol) {
    int ip[4], in[4], np = 0, nn = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (s[i] > 0.0) ip[np++] = i;
        else in[nn++] = i;
    }
    constexpr double V6 = 1.0 / 6.0;
    if (np == 0) return;
    if (np == 4) {
        vol += V6;
        return;
    }
    if (np == 1 || np == 3) {
        // one vertex v alone on its side; t_k = fraction from v along the edge to the others
        const int v = np == 1 ? ip[0] : in[0];
        const int o0 = np == 1 ? in[0] : ip[0], o1 = np == 1 ? in[1] : ip[1], o2 = np == 1 ? in[2] : ip[2];
        const double t0 = s[v] / (s[v] - s[o0]), t1 = s[v] / (s[v] - s[o1]), t2 = s[v] / (s[v] - s[o2]);
        double x0[3], x1[3], x2[3];
        cut_point(p[v], p[o0], t0, x0);
        cut_point(p[v], p[o1], t1, x1);
        cut_point(p[v], p[o2], t2, x2);
        area += 0.5 * tri_area2(x0, x1, x2);
        const double corner = V6 * t0 * t1 * t2;
        vol += np == 1 ? corner : V6 - corner;
        return;
    }
    // two and two: a, b positive, c, d not
    const int a = ip[0], b = ip[1], c = in[0], d = in[1];
    const double al = s[a] / (s[a] - s[c]), be = s[a] / (s[a] - s[d]);
    const double ga = s[b] / (s[b] - s[c]), de = s[b] / (s[b] - s[d]);
    double xac[3], xad[3], xbc[3], xbd[3];
    cut_point(p[a], p[c], al, xac);
    cut_point(p[a], p[d], be, xad);
    cut_point(p[b], p[c], ga, xbc);
    cut_point(p[b], p[d], de, xbd);
    // planar quadrilateral xac, xad, xbd, xbc: half the cross product of its diagonals
    const double ex = xbd[0] - xac[0], ey = xbd[1] - xac[1], ez = xbd[2] - xac[2];
    const double fx = xbc[0] - xad[0], fy = xbc[1] - xad[1], fz = xbc[2] - xad[2];
    const double cx = ey * fz - ez * fy, cy = ez * fx - ex * fz, cz = ex * fy - ey * fx;
    area += 0.5 * sqrt(cx * cx + cy * cy + cz * cz);
    // the positive part is a prism; its three tetrahedra have volume fractions
    // al be, al de (1 - be) and (1 - al) ga de of the whole
    vol += V6 * (al * be + al * de * (1.0 - be) + (1.0 - al) * ga * de);
}

// phi = rho_A - rho_B of every node, phi[box][node]; grid (blocks of 256 nodes, boxes).
template <int P>
__global__ __launch_bounds__(NRED_THREADS) void k_phi(const typename Prec<P>::S *f, const __half *ref, BoxGeom g,
                                                      double *phi) {
    const int box = blockIdx.y;
    const int64_t k = (int64_t)blockIdx.x * NRED_THREADS + threadIdx.x;
    if (k >= g.nnode) return;
    f += (int64_t)box * 2 * Q * g.nnode;
    if (Prec<P>::DEV) ref += (int64_t)box * 2 * g.nnode;
    double rho[2], j[2][3];
    node_moments<P>(f, ref, g, k, rho, j);
    phi[(int64_t)box * g.nnode + k] = rho[0] - rho[1];
}

// Area of {phi = 0} and volume of {phi > 0} over the cells of each box; grid (blocks, boxes),
// cell (x, y, z) to (x + 1, y + 1, z + 1) with its lowest corner's thread.
//
// The populations are read once, node by node, by k_phi (bound by that read: 53 us at 128^3
// FP32), and the cells take phi from an array that fits the caches: 8 B a node written and read
// against 152 of populations.  One kernel that marched 16 x 16 cells along z and summed the
// populations of its 17 x 17 nodes on the way had one workgroup per column of cells (64 at
// 128^3, a quarter of the CUs) and two barriers a plane: 1316 us.
// Thread t takes nodes t, t + stride, ... and carries (x, y, z) on, as k_stats does.  Few of
// the 64 cells a wavefront looks at are cut by the interface, so it only notes them, in a list
// of its own in lane order, and then gives each of its lanes one tetrahedron of one noted
// cell at a time (cutting the six of a cell in the cell's own lane left most lanes idle:
// 62 against 22 us at 128^3).  The sums' order is fixed.
constexpr int SURF_LIST = 256;  // cells a wavefront notes before it cuts them
__global__ __launch_bounds__(NRED_THREADS) void k_surface(const double *phi, BoxGeom g, double *partial) {
    __shared__ uint32_t list[NRED_THREADS / 64][SURF_LIST];
    phi += (int64_t)blockIdx.y * g.nnode;
    const int lane = threadIdx.x & 63;
    uint32_t *const mine = list[threadIdx.x >> 6];
    const uint32_t nn = uint32_t(g.nnode), nx = uint32_t(g.nx), ny = uint32_t(g.ny), nz = uint32_t(g.nz);
    const uint32_t nxy = nx * ny;
    const uint32_t stride = gridDim.x * NRED_THREADS;
    uint32_t k = blockIdx.x * NRED_THREADS + threadIdx.x;
    uint32_t x = k % nx, y = (k / nx) % ny, z = k / nx / ny;
    const uint32_t sx = stride % nx, sy = (stride / nx) % ny, sz = stride / nx / ny;
    double v[2] = {0.0, 0.0};
    int count = 0;  // noted cells, the same in every lane
    auto cut = [&]() {
        wave_lds_sync();  // the list's writes stand before its reads
        for (int e = lane; e < 6 * count; e += 64) {
            const uint32_t c = mine[e / 6];
            const int t = e % 6;
            // tetrahedron t: from the cell's lowest corner one step along each axis, in the t-th
            // order of (x, y, z); coordinates relative to that corner (the sums do not change)
            const int a0 = t >> 1, a1 = (t & 1) ? (a0 == 2 ? 1 : 2) : (a0 == 0 ? 1 : 0);
            const uint32_t off0 = a0 == 0 ? 1u : (a0 == 1 ? nx : nxy), off1 = a1 == 0 ? 1u : (a1 == 1 ? nx : nxy);
            double pp[4][3], ss[4];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                pp[0][d] = 0.0;
                pp[1][d] = d == a0 ? 1.0 : 0.0;
                pp[2][d] = d == a0 || d == a1 ? 1.0 : 0.0;
                pp[3][d] = 1.0;
            }
            ss[0] = phi[c];
            ss[1] = phi[c + off0];
            ss[2] = phi[c + off0 + off1];
            ss[3] = phi[c + 1u + nx + nxy];
            tet_cut(pp, ss, v[0], v[1]);
        }
        wave_lds_sync();  // and those before the next writes
        count = 0;
    };
    // every lane of a wavefront stays in the loop until its last one is done
    while (__any(k < nn)) {
        bool noted = false;
        if (k < nn && x + 1 < nx && y + 1 < ny && z + 1 < nz) {
            bool any_pos = false, any_neg = false;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double s = phi[k + uint32_t(q >> 2) * nxy + uint32_t((q >> 1) & 1) * nx + uint32_t(q & 1)];
                any_pos |= s > 0.0;
                any_neg |= !(s > 0.0);
            }
            noted = any_pos && any_neg;
            if (any_pos && !any_neg) v[1] += 1.0;  // a cell wholly inside
        }
        const uint64_t who = __ballot(noted);
        if (noted) mine[count + __popcll(who & ((1ull << lane) - 1ull))] = k;
        count += __popcll(who);
        if (count > SURF_LIST - 64) cut();
        k = k < nn ? k + stride : k;
        x += sx;
        const uint32_t carry_x = x >= nx ? 1u : 0u;
        x -= carry_x * nx;
        y += sy + carry_x;
        const uint32_t carry_y = y >= ny ? 1u : 0u;
        y -= carry_y * ny;
        z += sz + carry_y;
    }
    cut();
    block_reduce_store<2>(v, partial + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 2);
}

// Per-block partial sums of rho_A over the droplet nodes (rho_A > rho_B) and, with mark
// ([box][node]), which nodes those are; grid (blocks, boxes).
template <int P>
__global__ __launch_bounds__(NRED_THREADS) void k_drop_mass(const typename Prec<P>::S *f, const __half *ref,
                                                            BoxGeom g, int b0, double *partial, uint8_t *mark) {
    const int box = b0 + blockIdx.y;
    f += (int64_t)box * 2 * Q * g.nnode;
    if (Prec<P>::DEV) ref += (int64_t)box * 2 * g.nnode;
    double v[1] = {0.0};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < g.nnode; k += stride) {
        double rho[2], j[2][3];
        node_moments<P>(f, ref, g, k, rho, j);
        const bool in = rho[0] > rho[1];
        if (in) v[0] += rho[0];
        if (mark) mark[(int64_t)box * g.nnode + k] = in;
    }
    block_reduce_store<1>(v, partial + (int64_t)blockIdx.y * gridDim.x + blockIdx.x);
}

// Reinjection: at every marked node of box b0 + blockIdx.y, scale component A by
// target[box] / mass[box] (every population; for the deviation formats, whose
// populations are w_i rho_ref (1 + d_i), the node's reference density instead).
// The droplet is a few percent of a box: reading the marks of k_drop_mass and the
// populations of those nodes alone took the launch at 128^3 FP32 from 152 us (every
// population read again) to 8 us.
template <int P>
__global__ __launch_bounds__(256) void k_reinject(typename Prec<P>::S *f, __half *ref, BoxGeom g, int b0,
                                                  const uint8_t *mark, const double *mass, const double *target) {
    using R = typename Prec<P>::R;
    const int box = b0 + blockIdx.y;
    f += (int64_t)box * 2 * Q * g.nnode;
    if (Prec<P>::DEV) ref += (int64_t)box * 2 * g.nnode;
    mark += (int64_t)box * g.nnode;
    const double scale = target[box] / mass[box];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < g.nnode; k += stride) {
        if (!mark[k]) continue;
        if (Prec<P>::DEV) {
            ref_store(ref + ref_index(k, 0), float(double(ref_load(ref + ref_index(k, 0))) * scale));
        } else {
            typename Prec<P>::S *p = f + pop_base(g, k);
            R w[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) w[i] = Prec<P>::load(p + (int64_t)i * g.nx, R(0));
#pragma unroll
            for (int i = 0; i < Q; ++i) Prec<P>::store(p + (int64_t)i * g.nx, R(double(w[i]) * scale), R(0));
        }
    }
}

}  // namespace sclbm
