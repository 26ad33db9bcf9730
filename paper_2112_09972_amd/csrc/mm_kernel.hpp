// Maffettone-Minale droplet model (arXiv 2112.09972, Sec. 2 Eqs. 1, 2, 5) for
// many trajectories at once: FP64, classical RK4 with `substeps` steps per row
// of the velocity-gradient table, A(t) linear between rows.  In the table's time
// unit the model reads
//   dM/dt = f2(Ca) (S M + M S) + W M - M W - (f1/tau_d) (M - 3 det(M)/II_M I),
// S, W the symmetric / antisymmetric parts of A, Ca = tau_d max|A_ij|,
// II_M = (tr(M)^2 - M:M)/2, f1, f2 of Eq. 5; tau_d = eta_s R / sigma.  With
//   L = f2 S + W - (f1 / 2 tau_d) I
// the same equation is dM/dt = L M + M L^T + 3 (f1/tau_d) det(M)/II_M I, and L
// depends on the table alone.
//
// The trajectory is a serial chain of RK4 stages, so a launch of few trajectories
// lasts as long as one of them: rows times the instructions a stage issues in the
// wavefront that carries the chain.  Three things shorten it against one thread
// doing all the work (64 trajectories of 20,001 rows: 46.8 ms, 2.3 us a row).
//  - Folding f1 into L halves the products of a stage.
//  - k_mm_quad: three wavefronts beside the chain's compute the matrices L of the coming
//    substeps (table loads, Ca, f2) into LDS while the chain runs the present ones; one
//    barrier a chunk.
//  - A start from M = I keeps M symmetric, and in k_mm_quad three lanes of a quad share
//    a trajectory.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sclbm {

struct MmArgs {
    const double *A;   // [ntraj][nrows][9]
    int64_t ntraj, nrows;
    double tau_d, chi;
    int substeps, record_every;
    const double *M0;  // [ntraj][9] or null: the identity
    double *out;       // [ntraj][nrec][9], nrec = 1 + (nrows - 1) / record_every, record r at time r * record_every
};

constexpr int MM_THREADS = 256;       // k_mm_quad: wavefront 0 carries the chains, 1 .. 3 prepare L
constexpr int MM_QUAD_TRAJ = 16;      // trajectories of a workgroup, three lanes each
constexpr int MM_LANE_TRAJ = 64;      // and one lane each

// f1 / tau_d.  The same rounded value enters L and the det(M) / II_M term: where the two
// differ by a rounding, det M (which the model conserves) drifts by that fraction of
// f1 / tau_d every step (2.7e-14 against 1.5e-15 after 20,000 rows).
__device__ __forceinline__ double mm_relax(const MmArgs &a) {
    return 40.0 * (a.chi + 1.0) / ((3.0 + 2.0 * a.chi) * (16.0 + 19.0 * a.chi)) / a.tau_d;
}

// L at the fraction t of the way from row G0 to row G1.
__device__ __forceinline__ void mm_matrix(const MmArgs &a, const double *G0, const double *G1, double t, double (&L)[9]) {
    double G[9], gmax = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        G[k] = G0[k] + (G1[k] - G0[k]) * t;
        gmax = fmax(gmax, fabs(G[k]));
    }
    const double ca = a.tau_d * gmax;
    const double f2 = 5.0 / (3.0 + 2.0 * a.chi) + 3.0 * ca * ca / (2.0 + 6.0 * ca * ca);
    const double half_relax = 0.5 * mm_relax(a);
    // f2 (G + G^T)/2 + (G - G^T)/2
    const double cp = 0.5 * (f2 + 1.0), cm = 0.5 * (f2 - 1.0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            L[3 * i + j] = i == j ? f2 * G[4 * i] - half_relax : cp * G[3 * i + j] + cm * G[3 * j + i];
}

// Value of v one (C = 0xC9) or two (0xD2) places on in the cyclic order of a quad's first three lanes.
template <int CTRL>
__device__ __forceinline__ double quad_rot(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_mov_dpp(int(uint32_t(u)), CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_mov_dpp(int(uint32_t(u >> 32)), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, uint64_t(lo) | (uint64_t(hi) << 32));
}

// Start from M = I: symmetric for all times.  Lane j of a quad holds a = M_jj and
// b = M_j,j+1 (indices mod 3); the other four entries come from its neighbours.
// A stage is 61 instructions (8 of them lane moves) and bound by the latency of the
// dependent FP64 chain through det / II.  64 trajectories: 0.54 us a row (one lane a
// trajectory, L in the chain: 1.07); 8192: 0.71 against 1.11.
__global__ __launch_bounds__(MM_THREADS) void k_mm_quad(MmArgs a) {
    constexpr int CH = 8;              // substeps of a chunk
    constexpr int NS = 2 * CH + 1;     // half substeps whose L it needs
    // per half substep, trajectory and lane j: L_jj, L_j,j+1, L_j,j+2, L_j+1,j, L_jj + L_j+1,j+1, L_j+1,j+2
    __shared__ __attribute__((aligned(16))) double Ls[2][NS][MM_QUAD_TRAJ][3][6];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t t0 = (int64_t)blockIdx.x * MM_QUAD_TRAJ;
    const int64_t nsub = (a.nrows - 1) * a.substeps;
    const int64_t nchunk = (nsub + CH - 1) / CH;
    auto produce = [&](int64_t c, int first, int step) {
        const int64_t n0 = c * CH / a.substeps;
        const int s0 = int(c * CH % a.substeps);
        for (int e = first; e < NS * MM_QUAD_TRAJ; e += step) {
            const int tr = e / NS, m = e % NS;
            const int64_t t = min(t0 + tr, a.ntraj - 1);
            // row n and fraction f / (2 substeps) of the m-th half substep (past the table: its end).  At
            // f = 0 the matrix is row n's alone: a record depends on no row after its own, which may
            // hold anything (tables of several lengths are padded, with NaN for one)
            const uint32_t sub = uint32_t(s0) + uint32_t(m >> 1);
            int64_t n = n0 + sub / uint32_t(a.substeps);
            uint32_t f = 2u * (sub % uint32_t(a.substeps)) + uint32_t(m & 1);
            if (n >= a.nrows - 1) {
                n = a.nrows - 1;
                f = 0;
            }
            const double *p = a.A + (t * a.nrows + n) * 9;
            double L[9];
            mm_matrix(a, p, f ? p + 9 : p, double(f) * (0.5 / double(a.substeps)), L);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int j1 = (j + 1) % 3, j2 = (j + 2) % 3;
                double *d = Ls[c & 1][m][tr][j];
                d[0] = L[4 * j];
                d[1] = L[3 * j + j1];
                d[2] = L[3 * j + j2];
                d[3] = L[3 * j1 + j];
                d[4] = L[4 * j] + L[4 * j1];
                d[5] = L[3 * j1 + j2];
            }
        }
    };
    if (nchunk > 0) produce(0, tid, MM_THREADS);
    __syncthreads();
    const int tr = lane >> 2, j = min(lane & 3, 2);
    const int64_t t = t0 + tr;
    const bool live = tid < 64 && (lane & 3) < 3 && t < a.ntraj;
    double *Ot = a.out + t * (1 + (a.nrows - 1) / a.record_every) * 9;
    const int j1 = (j + 1) % 3;
    double ma = 1.0, mb = 0.0;
    auto record = [&](int64_t r) {
        if (!live) return;
        Ot[r * 9 + 4 * j] = ma;
        Ot[r * 9 + 3 * j + j1] = mb;
        Ot[r * 9 + 3 * j1 + j] = mb;
    };
    record(0);
    const double relax = mm_relax(a), h = 1.0 / a.substeps;
    struct Coef {
        double v[6];
    };
    auto fetch = [&](int buf, int m) {
        Coef q;
        const double2 *p = reinterpret_cast<const double2 *>(Ls[buf][m][tr][j]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double2 v = p[k];
            q.v[2 * k] = v.x;
            q.v[2 * k + 1] = v.y;
        }
        return q;
    };
    auto rhs = [&](const Coef &q, double va, double vb, double &da, double &db) {
        const double a1 = quad_rot<0xC9>(va), a2 = quad_rot<0xD2>(va);
        const double b1 = quad_rot<0xC9>(vb), b2 = quad_rot<0xD2>(vb);
        const double t01 = va * a1 - vb * vb, t12 = a1 * a2 - b1 * b1, t20 = a2 * va - b2 * b2;
        const double II = t01 + t12 + t20;
        const double det = va * t12 + b2 * (vb * b1 - a1 * b2) + vb * (b1 * b2 - a2 * vb);
        const double p = q.v[0] * va + q.v[1] * vb + q.v[2] * b2;
        db = q.v[4] * vb + q.v[3] * va + q.v[1] * a1 + q.v[2] * b1 + q.v[5] * b2;
        da = (p + p) + relax * ((3.0 * det) / II);
    };
    int sub = 0, rec_in = a.record_every;
    int64_t rec = 1;
    // the chain's wavefront first where the producers beside it compete for issue (64 trajectories of
    // 2001 rows 1091 -> 1063 us, 1000 of them 1135 -> 1102)
    if (tid < 64) __builtin_amdgcn_s_setprio(3);
    for (int64_t c = 0; c < nchunk; ++c) {
        if (tid < 64) {
            const int buf = int(c & 1), len = int(min<int64_t>(CH, nsub - c * CH));
            Coef La = fetch(buf, 0), Lm = fetch(buf, 1), Lb = fetch(buf, 2);
            for (int s = 0; s < len; ++s) {
                // the next substep's matrices (within the chunk's NS; unused after the last)
                const Coef Lm2 = fetch(buf, min(2 * s + 3, NS - 1)), Lb2 = fetch(buf, min(2 * s + 4, NS - 1));
                double ka, kb, sa, sb;
                rhs(La, ma, mb, ka, kb);
                sa = ka;
                sb = kb;
                rhs(Lm, ma + 0.5 * h * ka, mb + 0.5 * h * kb, ka, kb);
                sa += 2.0 * ka;
                sb += 2.0 * kb;
                rhs(Lm, ma + 0.5 * h * ka, mb + 0.5 * h * kb, ka, kb);
                sa += 2.0 * ka;
                sb += 2.0 * kb;
                rhs(Lb, ma + h * ka, mb + h * kb, ka, kb);
                sa += ka;
                sb += kb;
                ma += (h / 6.0) * sa;
                mb += (h / 6.0) * sb;
                La = Lb;
                Lm = Lm2;
                Lb = Lb2;
                if (++sub == a.substeps) {
                    sub = 0;
                    if (--rec_in == 0) {
                        rec_in = a.record_every;
                        record(rec++);
                    }
                }
            }
        } else if (c + 1 < nchunk) {
            produce(c + 1, tid - 64, MM_THREADS - 64);
        }
        __syncthreads();
    }
}

// Any M0 (M need not be symmetric), and launches of many trajectories: one lane a
// trajectory, which computes L itself (twice a substep: the middle and the end; the end's
// serves the next substep's start) and loads the next row while it integrates the
// present one.  The issue rate binds once the device is full, so nothing is computed twice
// here and no wavefront waits at a barrier.  65,536 trajectories: 1.43 us a row (one
// thread with the unfolded equation 3.0; L prepared by other wavefronts 3.4).
__global__ __launch_bounds__(MM_LANE_TRAJ) void k_mm_lane(MmArgs a) {
    const int64_t t = (int64_t)blockIdx.x * MM_LANE_TRAJ + threadIdx.x;
    if (t >= a.ntraj) return;
    const double *At = a.A + t * a.nrows * 9;
    double *Ot = a.out + t * (1 + (a.nrows - 1) / a.record_every) * 9;
    double M[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) M[k] = a.M0 ? a.M0[t * 9 + k] : ((k % 4) == 0 ? 1.0 : 0.0);
    auto record = [&](int64_t r) {
#pragma unroll
        for (int k = 0; k < 9; ++k) Ot[r * 9 + k] = M[k];
    };
    record(0);
    if (a.nrows < 2) return;
    const double relax = mm_relax(a), h = 1.0 / a.substeps;
    auto rhs = [&](const double (&L)[9], const double (&Y)[9], double (&out)[9]) {
        const double tr = Y[0] + Y[4] + Y[8];
        double mm = 0.0;
#pragma unroll
        for (int k = 0; k < 9; ++k) mm += Y[k] * Y[k];
        const double II = 0.5 * (tr * tr - mm);
        const double det = Y[0] * (Y[4] * Y[8] - Y[5] * Y[7]) - Y[1] * (Y[3] * Y[8] - Y[5] * Y[6]) +
                           Y[2] * (Y[3] * Y[7] - Y[4] * Y[6]);
        const double c = (3.0 * det) / II;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                double s = 0.0;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    s += L[3 * i + k] * Y[3 * k + j];
                    s += Y[3 * i + k] * L[3 * j + k];
                }
                out[3 * i + j] = i == j ? s + relax * c : s;
            }
    };
    double G0[9], G1[9], G2[9], La[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        G0[k] = At[k];
        G1[k] = At[9 + k];
    }
    mm_matrix(a, G0, G1, 0.0, La);
    int rec_in = a.record_every;
    int64_t rec = 1;
    for (int64_t n = 0; n + 1 < a.nrows; ++n) {
        const double *next = At + min(n + 2, a.nrows - 1) * 9;
#pragma unroll
        for (int k = 0; k < 9; ++k) G2[k] = next[k];
        for (int s = 0; s < a.substeps; ++s) {
            double k[9], sum[9], Y[9], L[9];
            rhs(La, M, k);
            mm_matrix(a, G0, G1, (s + 0.5) * h, L);
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                sum[e] = k[e];
                Y[e] = M[e] + 0.5 * h * k[e];
            }
            rhs(L, Y, k);
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                sum[e] += 2.0 * k[e];
                Y[e] = M[e] + 0.5 * h * k[e];
            }
            rhs(L, Y, k);
            mm_matrix(a, G0, G1, (s + 1) * h, La);
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                sum[e] += 2.0 * k[e];
                Y[e] = M[e] + h * k[e];
            }
            rhs(La, Y, k);
#pragma unroll
            for (int e = 0; e < 9; ++e) M[e] += (h / 6.0) * (sum[e] + k[e]);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            G0[k] = G1[k];
            G1[k] = G2[k];
        }
        if (--rec_in == 0) {
            rec_in = a.record_every;
            record(rec++);
        }
    }
}

}  // namespace sclbm
