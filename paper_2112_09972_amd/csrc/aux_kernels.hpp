// Initialisation, observables and FP64 reductions (arXiv 2112.09972, Sec. 2
// Eqs. 6-8, Sec. 4 Eq. 16; droplet inertia tensor for Sec. 2 Eq. 4).
//
// Reductions are deterministic: a fixed grid of NRED_BLOCKS workgroups, each
// thread accumulating a fixed strided subset of nodes in FP64, a wavefront
// butterfly (64 lanes), a fixed-order pass over the wavefronts in LDS, one
// partial per workgroup, then one workgroup summing the partials in a fixed
// order.  No atomics anywhere, so repeated runs give identical bits.
#pragma once

#include "lattice.hpp"

namespace sclbm {

constexpr int NRED_BLOCKS = 512;        // workgroups of the single-box diagnostic reductions
constexpr int NRED_MAX_PER_BOX = 1024;  // workgroups per box of the statistics reduction
constexpr int NRED_THREADS = 256;
constexpr int NSTAT = 16;  // mass 2, momentum 3, S0, S1 3, S2 6, bad-node count

struct Mat3 {
    double a[9];  // row-major, a[3*i + j] = d u_i / d x_j
};

struct BoxGeom {
    int nx, ny, nz;
    int64_t nnode;
    double xc[3];
};

// Element offset of direction 0 of node k = (z ny + y) nx + x in one component's
// population block (row-blocked order [z][y][direction][x]); direction i adds i nx.
__device__ __forceinline__ int64_t pop_base(const BoxGeom &g, int64_t k) {
    const int64_t row = k / g.nx;
    return row * (int64_t)(Q * g.nx) + (k - row * g.nx);
}

__device__ __forceinline__ void node_xyz(const BoxGeom &g, int64_t k, int &x, int &y, int &z) {
    x = (int)(k % g.nx);
    int64_t t = k / g.nx;
    y = (int)(t % g.ny);
    z = (int)(t / g.ny);
}

struct DropletInit {
    double ctr[3], radius, width, rho_in, rho_out;
    Mat3 A0;
    double u0[3];  // mode 2: uniform velocity (densities rho_in for A, rho_out for B)
};

// mode 0: tanh droplet (DropletInit); mode 1: FP64 fields rho_a, rho_b, u;
// mode 2: uniform densities (rho_in, rho_out) moving with u0.
template <int P>
__global__ __launch_bounds__(256) void k_init(typename Prec<P>::S *f, __half *ref, BoxGeom g, int mode, DropletInit d,
                                              const double *rho_a, const double *rho_b, const double *u) {
    using R = typename Prec<P>::R;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= g.nnode) return;
    int x, y, z;
    node_xyz(g, k, x, y, z);
    double ra, rb, ux, uy, uz;
    if (mode == 0) {
        // tanh droplet, linear velocity about the box centre
        const double dx = x - d.ctr[0], dy = y - d.ctr[1], dz = z - d.ctr[2];
        const double r = sqrt(dx * dx + dy * dy + dz * dz);
        ra = 0.5 * (d.rho_in + d.rho_out) - 0.5 * (d.rho_in - d.rho_out) * tanh((r - d.radius) / d.width);
        rb = d.rho_in + d.rho_out - ra;
        const double ex = x - g.xc[0], ey = y - g.xc[1], ez = z - g.xc[2];
        const double *A = d.A0.a;
        ux = A[0] * ex + A[1] * ey + A[2] * ez;
        uy = A[3] * ex + A[4] * ey + A[5] * ez;
        uz = A[6] * ex + A[7] * ey + A[8] * ez;
    } else if (mode == 2) {
        ra = d.rho_in;
        rb = d.rho_out;
        ux = d.u0[0];
        uy = d.u0[1];
        uz = d.u0[2];
    } else {
        ra = rho_a[k];
        rb = rho_b[k];
        if (u) {
            ux = u[k];
            uy = u[g.nnode + k];
            uz = u[2 * g.nnode + k];
        } else {
            ux = uy = uz = 0.0;
        }
    }
    const double usq = ux * ux + uy * uy + uz * uz;
    const double rr[2] = {ra, rb};
    const int64_t e = pop_base(g, k);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        double rref = 0.0;
        if (Prec<P>::DEV) {
            ref_store(ref + ref_index(k, s), float(rr[s]));
            rref = ref_load(ref + ref_index(k, s));
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const double fe = equilibrium<double>(i, rr[s], ux, uy, uz, usq);
            Prec<P>::store(f + pop_index<P>(g.nnode, e + (int64_t)i * g.nx, s), R(fe), R(w_of<R>(i) * R(rref)));
        }
    }
}

template <int P>
__device__ __forceinline__ void node_moments(const typename Prec<P>::S *f, const __half *ref, const BoxGeom &g,
                                             int64_t k, double rho[2], double j[2][3]) {
    using R = typename Prec<P>::R;
    const int64_t N = g.nnode;
    const int64_t e = pop_base(g, k);
    // the populations as stored (decoded in the format's arithmetic type), summed in FP64
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        double r = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
        const R rref = Prec<P>::DEV ? R(ref_load(ref + ref_index(k, s))) : R(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const double v = double(Prec<P>::load(f + pop_index<P>(N, e + (int64_t)i * g.nx, s), w_of<R>(i) * rref));
            r += v;
            if (cx_of(i)) jx += double(cx_of(i)) * v;
            if (cy_of(i)) jy += double(cy_of(i)) * v;
            if (cz_of(i)) jz += double(cz_of(i)) * v;
        }
        rho[s] = r;
        j[s][0] = jx;
        j[s][1] = jy;
        j[s][2] = jz;
    }
}

// Densities of every node and, with j, the momentum j_A + j_B: one read of the populations
// (bound by it: 54 us at 128^3 FP32, 6.5 TB/s, 63 us with the momentum written too).
template <int P>
__global__ __launch_bounds__(256) void k_density(const typename Prec<P>::S *f, const __half *ref, BoxGeom g,
                                                 double *rho_a, double *rho_b, double *j) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= g.nnode) return;
    double rho[2], js[2][3];
    node_moments<P>(f, ref, g, k, rho, js);
    rho_a[k] = rho[0];
    rho_b[k] = rho[1];
    if (j) {
#pragma unroll
        for (int c = 0; c < 3; ++c) j[c * g.nnode + k] = js[0][c] + js[1][c];
    }
}

template <int K, int NT = NRED_THREADS>
__device__ __forceinline__ void block_reduce_store(double (&v)[K], double *out /* K values */) {
    // wavefront butterfly, fixed order
#pragma unroll
    for (int c = 0; c < K; ++c) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[c] += __shfl_down(v[c], off, 64);
    }
    __shared__ double part[NT / 64][K];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < K; ++c) part[wv][c] = v[c];
    __syncthreads();
    if (threadIdx.x < K) {
        double acc = 0.0;
        for (int w = 0; w < NT / 64; ++w) acc += part[w][threadIdx.x];
        out[threadIdx.x] = acc;
    }
}

// Barycentric velocity with the half-force term from the densities and momenta written by
// k_density (same neighbour rules as the step kernel): in place, u in the momentum's array,
// or with E0 the sums of |u - A d|^2 and |A d|^2 (Sec. 4 Eq. 16) per workgroup instead.
//
// The momentum costs 48 B a node of traffic where summing the populations again would read
// 152 (FP32).  Tiles of 64 x 8 nodes march along z with one plane of densities, ring
// included, in LDS (two buffers, one barrier a plane); the next plane's loads are under way
// meanwhile.  A plane enters the stencil of its own nodes and, through three sums per
// node, that of the planes on either side, so each is read from LDS once: 18 reads a node.
// 36 us at 128^3 and 202 us at 256^3 (5.3 TB/s); gathering the 36 neighbours from global
// memory instead 69 and 529 us, and summing the populations again as well 187 us (128^3
// FP32) and 1322 us (256^3 FP16).
// The items (x tile, y tile, z-chunk) of a workgroup are consecutive, and the workgroups of
// one XCD next to one another, so that rings and chunk ends hit in its L2.
// Boxes at most 8 nodes wide take tiles of 8 x 64 (TX = 8), or of 8 x 8 in one wavefront (NT = 64) where
// y is as short: 64 x 8 would leave most lanes idle (densities and velocity, FP32: 3 x 300 x 300 59 -> 28 us,
// 5 x 512 x 512 150 -> 71, 3 x 3 x 20000 62 -> 25; gathering from global memory 50, 163 and 34).
constexpr int VEL_BLOCKS = 2048;  // most workgroups of a launch
template <bool E0, int TX, int NT>
__global__ __launch_bounds__(NT) void k_velocity(BoxGeom g, const double *rho_a, const double *rho_b, int ghost,
                                                          double gab, double rb0, double rb1, double *u, int zchunk,
                                                          Mat3 A, double *partial) {
    constexpr int TY = NT / TX, RING = 2 * (TX + 2) + 2 * TY;
    static_assert(RING <= NT, "one ring node per thread");
    __shared__ double ld[2][2][TY + 2][TX + 2];
    const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY;
    const uint32_t nitem = uint32_t(ntx) * uint32_t(nty) * uint32_t((g.nz + zchunk - 1) / zchunk);
    const uint32_t q8 = gridDim.x / 8, r8 = gridDim.x % 8, xcd = blockIdx.x % 8, k8 = blockIdx.x / 8;
    const uint32_t blk = xcd < r8 ? xcd * (q8 + 1) + k8 : r8 * (q8 + 1) + (xcd - r8) * q8 + k8;
    const uint32_t first = uint32_t(uint64_t(blk) * nitem / gridDim.x);
    const uint32_t last = uint32_t(uint64_t(blk + 1) * nitem / gridDim.x);
    const uint32_t nxy = uint32_t(g.nx) * uint32_t(g.ny);
    const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
    const double rbnd[2] = {rb0, rb1};
    double v[2] = {0.0, 0.0};
    for (uint32_t item = first; item < last; ++item) {
        const int x0 = int(item % uint32_t(ntx)) * TX, y0 = int(item / uint32_t(ntx) % uint32_t(nty)) * TY;
        const int zs = int(item / uint32_t(ntx) / uint32_t(nty)) * zchunk, ze = min(zs + zchunk, g.nz);
        const int x = x0 + lx, y = y0 + ly;
        const bool valid = x < g.nx && y < g.ny;
        // the ring node of this thread: rows y0 - 1 and y0 + TY, then columns x0 - 1 and x0 + TX
        const bool ring_on = tid < RING;
        int rx, ry;
        if (tid < 2 * (TX + 2)) {
            ry = tid < TX + 2 ? 0 : TY + 1;
            rx = tid < TX + 2 ? tid : tid - (TX + 2);
        } else {
            const int r = tid - 2 * (TX + 2);
            rx = r < TY ? 0 : TX + 1;
            ry = 1 + (r < TY ? r : r - TY);
        }
        // offset of a (x, y) in its plane after the wrap; false where it is a ghost or lies beyond
        // the one node past the box that a valid node's stencil reaches
        auto place = [&](int px, int py, uint32_t &off) {
            const bool in = px >= 0 && px < g.nx && py >= 0 && py < g.ny;
            const bool reach = px <= g.nx && py <= g.ny;
            if (!ghost) {
                px = px < 0 ? px + g.nx : (px >= g.nx ? px - g.nx : px);
                py = py < 0 ? py + g.ny : (py >= g.ny ? py - g.ny : py);
            }
            off = uint32_t(py) * uint32_t(g.nx) + uint32_t(px);
            return ghost ? in : reach;
        };
        uint32_t own_off, ring_off;
        const bool own_in = place(x, y, own_off);
        const bool ring_in = ring_on && place(x0 - 1 + rx, y0 - 1 + ry, ring_off);
        double own[2], ring[2];
        auto load = [&](int z) {
            const bool zin = z >= 0 && z < g.nz;
            const int zz = zin ? z : (z < 0 ? z + g.nz : z - g.nz);
            const bool live = zin || !ghost;
            const uint32_t base = uint32_t(zz) * nxy;
            own[0] = rbnd[0];
            own[1] = rbnd[1];
            if (own_in && live) {
                own[0] = rho_a[base + own_off];
                own[1] = rho_b[base + own_off];
            }
            ring[0] = rbnd[0];
            ring[1] = rbnd[1];
            if (ring_in && live) {
                ring[0] = rho_a[base + ring_off];
                ring[1] = rho_b[base + ring_off];
            }
        };
        // per component: stencil sums of the node's own plane (sx, sy) and the terms (c, dx, dy)
        // it adds to the planes beside it: c to sz, with the sign of the step, dx and dy to sx and sy
        struct Plane {
            double sx[2], sy[2], c[2], dx[2], dy[2], rho[2];
        };
        Plane p0{}, p1{};  // planes z - 2 and z - 1
        load(zs - 1);
        for (int z = zs - 1; z <= ze; ++z) {
            double(*const pl)[TY + 2][TX + 2] = ld[(z - zs + 1) & 1];
            pl[0][ly + 1][lx + 1] = own[0];
            pl[1][ly + 1][lx + 1] = own[1];
            if (ring_on) {
                pl[0][ry][rx] = ring[0];
                pl[1][ry][rx] = ring[1];
            }
            __syncthreads();
            Plane p2;
            p2.rho[0] = own[0];
            p2.rho[1] = own[1];
            if (z < ze) load(z + 1);
            const int zc = z - 1;
            const uint32_t k = uint32_t(zc) * nxy + own_off;
            const bool emit = zc >= zs && valid;
            double jm[3] = {0.0, 0.0, 0.0};
            if (emit) {
#pragma unroll
                for (int c = 0; c < 3; ++c) jm[c] = u[c * g.nnode + k];
            }
            constexpr double w1 = 1.0 / 18.0, w2 = 1.0 / 36.0;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                auto at = [&](int cx, int cy) { return pl[s][ly + 1 + cy][lx + 1 + cx]; };
                const double xp = at(1, 0), xm = at(-1, 0), yp = at(0, 1), ym = at(0, -1);
                const double pp = at(1, 1), mm = at(-1, -1), pm = at(1, -1), mp = at(-1, 1);
                p2.sx[s] = w1 * (xp - xm) + w2 * ((pp - mm) + (pm - mp));
                p2.sy[s] = w1 * (yp - ym) + w2 * ((pp - mm) - (pm - mp));
                p2.c[s] = w1 * p2.rho[s] + w2 * ((xp + xm) + (yp + ym));
                p2.dx[s] = w2 * (xp - xm);
                p2.dy[s] = w2 * (yp - ym);
            }
            if (emit) {
                double F[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int o = 1 - s;
                    const double pre = -gab * p1.rho[s];
                    F[0] += pre * (p1.sx[o] + (p0.dx[o] + p2.dx[o]));
                    F[1] += pre * (p1.sy[o] + (p0.dy[o] + p2.dy[o]));
                    F[2] += pre * (p2.c[o] - p0.c[o]);
                }
                const double rt = p1.rho[0] + p1.rho[1];
                double vel[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) vel[c] = (jm[c] + 0.5 * F[c]) / rt;
                if constexpr (E0) {
                    const double dx = x - g.xc[0], dy = y - g.xc[1], dz = zc - g.xc[2];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const double lin = A.a[3 * c] * dx + A.a[3 * c + 1] * dy + A.a[3 * c + 2] * dz;
                        const double e = vel[c] - lin;
                        v[0] += e * e;
                        v[1] += lin * lin;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 3; ++c) u[c * g.nnode + k] = vel[c];
                }
            }
            p0 = p1;
            p1 = p2;
        }
        __syncthreads();  // the next item writes the buffer the last plane was read from
    }
    if constexpr (E0) block_reduce_store<2, NT>(v, partial + (int64_t)blk * 2);
}

// Per-workgroup partials of: mass A, mass B, momentum (3), indicator moments
// S0, S1 (3), S2 (6) about the box centre, and the count of bad nodes.
// Grid (blocks per box, boxes): box b0 + blockIdx.y, partials [box][block][NSTAT].
template <int P>
__global__ __launch_bounds__(NRED_THREADS) void k_stats(const typename Prec<P>::S *f, const __half *ref, BoxGeom g,
                                                        int b0, double *partial) {
    using S = typename Prec<P>::S;
    using R = typename Prec<P>::R;
    const int box = b0 + blockIdx.y;
    f += (int64_t)box * 2 * Q * g.nnode;
    if (Prec<P>::DEV) ref += (int64_t)box * 2 * g.nnode;
    double v[NSTAT];
#pragma unroll
    for (int c = 0; c < NSTAT; ++c) v[c] = 0.0;
    // Thread t takes nodes k = t, t + stride, ... (k = (z ny + y) nx + x), carrying (x, y, z) from
    // one to the next, so that the loop does no integer division; a box holds fewer than 2^31 nodes.
    const uint32_t nn = uint32_t(g.nnode), nx = uint32_t(g.nx), ny = uint32_t(g.ny);
    const uint32_t stride = gridDim.x * blockDim.x;
    uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t x = k % nx, y = (k / nx) % ny, z = k / nx / ny;
    const uint32_t sx = stride % nx, sy = (stride / nx) % ny, sz = stride / nx / ny;
    // FP64 and FP32 storage: raw buffer loads, one byte offset per node and a uniform one per
    // direction (the 16-bit formats take the decoding loads of node_moments)
    constexpr uint32_t EB = sizeof(S);
    const uint32_t comp_bytes = uint32_t(Q) * nn * EB, plane_bytes = nx * EB;
    const rsrc_t rs[2] = {make_rsrc(f, comp_bytes), make_rsrc(f + (int64_t)Q * g.nnode, comp_bytes)};
    // the node's contributions, in a fixed order (one node after the other)
    auto accumulate = [&](const double (&rho)[2], const double (&j)[2][3], uint32_t xx, uint32_t yy, uint32_t zz) {
        v[0] += rho[0];
        v[1] += rho[1];
        v[2] += j[0][0] + j[1][0];
        v[3] += j[0][1] + j[1][1];
        v[4] += j[0][2] + j[1][2];
        if (!(rho[0] > 0.0) || !(rho[1] > 0.0) || !isfinite(rho[0]) || !isfinite(rho[1])) v[15] += 1.0;
        if (rho[0] > rho[1]) {
            const double dx = double(xx) - g.xc[0], dy = double(yy) - g.xc[1], dz = double(zz) - g.xc[2];
            v[5] += 1.0;
            v[6] += dx;
            v[7] += dy;
            v[8] += dz;
            v[9] += dx * dx;
            v[10] += dx * dy;
            v[11] += dx * dz;
            v[12] += dy * dy;
            v[13] += dy * dz;
            v[14] += dz * dz;
        }
    };
    // the next node's coordinates: add (sx, sy, sz) with carries (sx < nx, sy < ny)
    auto advance = [&](uint32_t &xx, uint32_t &yy, uint32_t &zz) {
        xx += sx;
        const uint32_t carry_x = xx >= nx ? 1u : 0u;
        xx -= carry_x * nx;
        yy += sy + carry_x;
        const uint32_t carry_y = yy >= ny ? 1u : 0u;
        yy -= carry_y * ny;
        zz += sz + carry_y;
    };
    // density and momentum of a node from its 2 x 19 populations, summed in FP64
    auto moments = [&](const auto &w, double (&rho)[2], double (&j)[2][3]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            double r = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const double wi = double(w[s][i]);
                r += wi;
                if (cx_of(i)) jx += double(cx_of(i)) * wi;
                if (cy_of(i)) jy += double(cy_of(i)) * wi;
                if (cz_of(i)) jz += double(cz_of(i)) * wi;
            }
            rho[s] = r;
            j[s][0] = jx;
            j[s][1] = jy;
            j[s][2] = jz;
        }
    };
    auto node_vo = [&](uint32_t xx, uint32_t yy, uint32_t zz) { return ((zz * ny + yy) * uint32_t(Q) * nx + xx) * EB; };
    if constexpr (Prec<P>::DEV) {
        for (; k < nn; k += stride) {
            double rho[2], j[2][3];
            node_moments<P>(f, ref, g, k, rho, j);
            accumulate(rho, j, x, y, z);
            advance(x, y, z);
        }
    } else if constexpr (sizeof(S) == 4) {
        // FP32 storage: the loads of node k + stride go out while node k is summed
        float wn[2][Q];
        auto load = [&](uint32_t vo) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < Q; ++i) wn[s][i] = Prec<P>::bload(rs[s], vo, uint32_t(i) * plane_bytes, R(0));
        };
        if (k < nn) load(node_vo(x, y, z));
        for (; k < nn; k += stride) {
            float w[2][Q];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < Q; ++i) w[s][i] = wn[s][i];
            uint32_t xn = x, yn = y, zn = z;
            advance(xn, yn, zn);
            if (k + stride < nn) load(node_vo(xn, yn, zn));
            double rho[2], j[2][3];
            moments(w, rho, j);
            accumulate(rho, j, x, y, z);
            x = xn;
            y = yn;
            z = zn;
        }
    } else {
        for (; k < nn; k += stride) {
            S w[2][Q];
            const uint32_t vo = node_vo(x, y, z);
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < Q; ++i) w[s][i] = Prec<P>::bload(rs[s], vo, uint32_t(i) * plane_bytes, R(0));
            double rho[2], j[2][3];
            moments(w, rho, j);
            accumulate(rho, j, x, y, z);
            advance(x, y, z);
        }
    }
    block_reduce_store<NSTAT>(v, partial + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * NSTAT);
}

// Fixed-order sum of nblk partials of K values each; workgroup b handles the
// partials of box b ([b][nblk][K] -> out[b][K]).
template <int K>
__global__ __launch_bounds__(NRED_THREADS) void k_final(const double *partial, int nblk, double *out) {
    partial += (int64_t)blockIdx.x * nblk * K;
    out += (int64_t)blockIdx.x * K;
    double v[K];
#pragma unroll
    for (int c = 0; c < K; ++c) v[c] = 0.0;
    for (int b = threadIdx.x; b < nblk; b += NRED_THREADS)
#pragma unroll
        for (int c = 0; c < K; ++c) v[c] += partial[(int64_t)b * K + c];
    block_reduce_store<K>(v, out);
}

}  // namespace sclbm
