// Kernels of the droplet-shape surrogate: a 576 -> 512 -> 512 -> 512 -> 3 ReLU
// perceptron from a window of the velocity-gradient history (64 samples of A(t),
// Sec. 3) to the droplet's three semi-axes (Sec. 2 Eq. 4 takes D from them).
//
// Arithmetic: BF16 operands, FP32 accumulation on the gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16), FP32 biases, FP32 master weights and Adam moments.
// Every product is "NT": C[m][n] = sum_k A[m][k] B[n][k].
//
// Operands live in memory in the order the matrix instructions take them (fragment order,
// frag_index): for a tile of 32 rows and a k-step of 16, lane l's 16 bytes hold row l % 32,
// k = 8 (l / 32) .. + 7, and the 64 lanes' follow one another, 1 KB a fragment.  A wavefront then
// reads each fragment with one fully coalesced 16-byte load straight into the registers the
// instruction reads; no product stages anything in LDS or waits at a barrier.  The writers
// pay for it: an accumulator lane holds one column and groups of four consecutive rows, so the
// copy whose contraction runs over the rows (the batch, for the weight gradients) goes out as
// 8-byte stores from registers, and the copy whose contraction runs over the columns (the
// next layer's input) passes through a wavefront's own 2.5 KB of LDS.
//
// One training step of up to 2048 rows is eight launches: input, three layers, output layer with
// its loss and input gradient, two hidden input gradients, and all parameter gradients with
// Adam.  At 256 rows each lasts as long as its chain of memory latencies (launch, arguments,
// operands from the other XCDs' side of the cache, stores), 3.5 to 7 us, 11 us the last, which
// moves 23 MB of parameters and moments: 39.5 us a step, 107 with seventeen launches of
// LDS-staged products and separate transposes, sums and Adam.  At 8192 rows 108 us against 411.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "wave.hpp"

namespace sclmlp {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NIN = 576;    // 64 samples x 9 gradient entries
constexpr int NHID = 512;
constexpr int NOUT = 3;
constexpr int NLAYER = 4;
constexpr int ROW_ALIGN = 128;  // the batch is padded to this many rows inside the library

// flat FP32 parameter vector: W1 [512][576], b1, W2 [512][512], b2, W3, b3, W4 [3][512], b4
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + NHID * NIN;
constexpr int OFF_W2 = OFF_B1 + NHID;
constexpr int OFF_B2 = OFF_W2 + NHID * NHID;
constexpr int OFF_W3 = OFF_B2 + NHID;
constexpr int OFF_B3 = OFF_W3 + NHID * NHID;
constexpr int OFF_W4 = OFF_B3 + NHID;
constexpr int OFF_B4 = OFF_W4 + NOUT * NHID;
constexpr int NPARAM = OFF_B4 + NOUT;
static_assert(NPARAM == 822275, "parameter count");

// Position of X[n][k] (K = the contraction's length, a multiple of 16; n and k non-negative) in
// fragment order: [tile n / 32][k-step k / 16][lane n % 32 + 32 ((k % 16) / 8)][k % 8].
__host__ __device__ __forceinline__ size_t frag_index(size_t n, size_t k, size_t K) {
    return (((n >> 5) * (K >> 4) + (k >> 4)) * 64 + (n & 31) + 32 * ((k & 15) >> 3)) * 8 + (k & 7);
}
constexpr size_t FRAG = 512;  // elements of a fragment

// 16 bytes of bf16 (loaded as a vector of them: as the elements were stored)
__device__ __forceinline__ uint4 ld16(const bf16 *p) { return __builtin_bit_cast(uint4, *reinterpret_cast<const bf16x8 *>(p)); }
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// acc += A B^T over nk k-steps for RT x CT tiles of 32 x 32: A and B point at this lane's 16
// bytes of the first fragments; as and bs are the distances of consecutive tiles.  D k-steps of
// fragments are under way in registers.  The k-steps accumulate in order.
template <int RT, int CT, int D, typename NK>
__device__ __forceinline__ void tile_product(const bf16 *A, size_t as, const bf16 *B, size_t bs, NK nk,
                                             f32x16 (&acc)[RT][CT]) {
    uint4 a[D][RT], b[D][CT];
    auto load = [&](int d, int k) {
#pragma unroll
        for (int i = 0; i < RT; ++i) a[d][i] = ld16(A + i * as + (size_t)k * FRAG);
#pragma unroll
        for (int j = 0; j < CT; ++j) b[d][j] = ld16(B + j * bs + (size_t)k * FRAG);
    };
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < nk) load(d, d);
    // (the scheduling barriers keep each load where it stands: moved down to its use to save
    // registers, it would leave the product waiting for memory at every k-step)
    __builtin_amdgcn_sched_barrier(0);
    auto round = [&](int k0) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (k0 + d < nk) {
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int j = 0; j < CT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[d][i]),
                                                                            __builtin_bit_cast(bf16x8, b[d][j]),
                                                                            acc[i][j], 0, 0, 0);
                if (k0 + d + D < nk) load(d, k0 + d + D);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    if constexpr (std::is_same_v<NK, int>) {
        for (int k0 = 0; k0 < nk; k0 += D) round(k0);
    } else {
#pragma unroll
        for (int k0 = 0; k0 < NK::value; k0 += D) round(k0);
    }
}

// ---------------------------------------------------------------------------------------------
// Input preparation: gather (optional index), optional cubic symmetry of the box, normalise,
// round to BF16; rows >= n are zero.  A workgroup takes PREP_ROWS rows of all 576 features
// through LDS, three features a thread with all its rows' loads under way, and writes both
// fragment orders: X (contraction over the features) and XT (over the rows).  Grid Mpad / PREP_ROWS.
// A row whose index (or symmetry id) is out of range is treated as padding and counted in *bad.
//
// Symmetry id s in [0, 48): P = signed permutation with P[i][perm(i)] = sign(i), perm the
// (s / 8)-th permutation of (0, 1, 2) in lexicographic order, sign(i) = -1 where bit i of s % 8
// is set.  Every sample A of the window becomes P A P^T:  A'_ij = sign(i) sign(j) A_{perm(i) perm(j)}.
__device__ __forceinline__ int sym_source(int s, int e, float &sgn) {
    // e = 3 i + j within one 3 x 3 sample
    const int i = e / 3, j = e - 3 * i;
    const int pi = s >> 3;                       // 012 021 102 120 201 210
    const int p0 = pi < 2 ? 0 : (pi < 4 ? 1 : 2);
    const int p1 = (pi == 0 || pi == 5) ? 1 : ((pi == 1 || pi == 3) ? 2 : 0);
    const int p2 = 3 - p0 - p1;
    const int qi = i == 0 ? p0 : (i == 1 ? p1 : p2);
    const int qj = j == 0 ? p0 : (j == 1 ? p1 : p2);
    sgn = (((s >> i) ^ (s >> j)) & 1) ? -1.0f : 1.0f;
    return 3 * qi + qj;
}


constexpr int PREP_ROWS = 8;
constexpr int PREP_T = NIN / 3;  // threads, three features each
__global__ __launch_bounds__(PREP_T) void k_prep(const float *win, const int32_t *index, const int32_t *sym, int n,
                                              int ndata, const float *shift, const float *scale, bf16 *X, bf16 *XT,
                                              int Mpad, unsigned *bad) {
    constexpr int LD = NIN + 8;
    __shared__ __attribute__((aligned(16))) bf16 tile[PREP_ROWS][LD];
    const int m0 = blockIdx.x * PREP_ROWS, tid = threadIdx.x;
    // the rows' sources, the same for the whole workgroup (-1: zero)
    int64_t src[PREP_ROWS];
    int sy[PREP_ROWS];
#pragma unroll
    for (int r = 0; r < PREP_ROWS; ++r) {
        const int m = min(m0 + r, n - 1);
        src[r] = index ? (int64_t)index[m] : (int64_t)m;
        sy[r] = sym ? sym[m] : 0;
    }
#pragma unroll
    for (int r = 0; r < PREP_ROWS; ++r) {
        const bool bad_row = src[r] < 0 || src[r] >= ndata || sy[r] < 0 || sy[r] >= 48;
        if (m0 + r >= n || bad_row) src[r] = -1;
        if (m0 + r < n && bad_row && tid == 0) atomicAdd(bad, 1u);
    }
    float v[3][PREP_ROWS], sgn[3][PREP_ROWS];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int f0 = tid + k * PREP_T, t9 = f0 / 9, e = f0 - 9 * t9;
#pragma unroll
        for (int r = 0; r < PREP_ROWS; ++r) {
            sgn[k][r] = 1.0f;
            const int f = sy[r] ? 9 * t9 + sym_source(sy[r], e, sgn[k][r]) : f0;
            v[k][r] = src[r] >= 0 ? win[src[r] * NIN + f] : 0.0f;
        }
    }
    static_assert(PREP_ROWS == 8, "16-byte pieces of XT and X, one each per feature");
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int f = tid + k * PREP_T;
        const float sh = shift[f], sc = scale[f];
        bf16x8 h;
#pragma unroll
        for (int r = 0; r < PREP_ROWS; ++r) {
            h[r] = (bf16)(src[r] >= 0 ? (v[k][r] * sgn[k][r] - sh) * sc : 0.0f);
            tile[r][f] = h[r];
        }
        *reinterpret_cast<bf16x8 *>(XT + frag_index(f, m0, Mpad)) = h;  // the 8 rows of a feature
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int i = tid + k * PREP_T, r = i % 8, c = i / 8 * 8;       // 8 features of a row
        *reinterpret_cast<uint4 *>(X + frag_index(m0 + r, c, NIN)) = ld16(&tile[r][c]);
    }
}

// ---------------------------------------------------------------------------------------------
// One hidden layer over the batch.  Forward: H = relu(X W^T + b).  MASK: the gradient of the layer
// below, dZ_prev = (dZ W) * (H_prev > 0).  C (may be null) is written with the contraction over
// the units, CT over the rows; the mask is read in CT's order.
//
// A wavefront computes RT x CT tiles of 32 x 32; W x W wavefronts a workgroup.
struct LayerArgs {
    const bf16 *A;      // rows of the batch, contraction over K
    const bf16 *B;      // units (W, or its transpose), contraction over K
    const float *bias;  // forward
    const bf16 *mask;   // MASK: H_prev in CT's order
    bf16 *C, *CT;
    int Mpad;
};

template <int K, int RT, int CT, bool MASK, int W>
__global__ __launch_bounds__(64 * W * W) void k_layer(LayerArgs g) {
    constexpr int WC = W, WR = W;                      // wavefronts of a workgroup: columns, rows
    constexpr int NCB = NHID / (32 * CT * WC);         // workgroups across the units
    constexpr int D = RT * CT == 1 ? (K == NHID ? 32 : 18) : 8;
    constexpr int LDC = 40;                            // 32 columns and a 16-byte pad
    __shared__ __attribute__((aligned(16))) bf16 smem[W * W][32 * LDC];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c31 = lane & 31, hi = lane >> 5;
    // the workgroups of one block of rows go to one XCD
    const int total = gridDim.x;
    int lin = blockIdx.x;
    if ((total & 7) == 0) lin = (lin & 7) * (total >> 3) + (lin >> 3);
    const int rt = (lin / NCB * WR + wave / WC) * RT, ct = (lin % NCB * WC + wave % WC) * CT;
    // what the epilogue reads, loaded ahead of the product
    const int kst = g.Mpad / 16;
    auto at = [&](int i, int j, int q) {  // rows 32 (rt + i) + 8q + 4 hi .. + 3 of this lane's column, in CT's order
        return (((size_t)(ct + j) * kst + (rt + i) * 2 + (q >> 1)) * 64 + c31 + 32 * (q & 1)) * 8 + 4 * hi;
    };
    uint2 mk[RT][CT][4];
    float bias[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) bias[j] = MASK ? 0.0f : g.bias[(ct + j) * 32 + c31];
    if (MASK) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) mk[i][j][q] = *reinterpret_cast<const uint2 *>(g.mask + at(i, j, q));
    }
    f32x16 acc[RT][CT];
    tile_product<RT, CT, D>(g.A + (size_t)rt * (K / 16) * FRAG + lane * 8, (size_t)(K / 16) * FRAG,
                            g.B + (size_t)ct * (K / 16) * FRAG + lane * 8, (size_t)(K / 16) * FRAG,
                            std::integral_constant<int, K / 16>{}, acc);
    // accumulator element 4q + e of a 32x32 fragment sits at row 8q + 4 hi + e, column lane % 32
    bf16 *const Cs = smem[wave];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16x4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = acc[i][j][4 * q + e];
                    if (MASK) v = (float)__builtin_bit_cast(bf16x4, mk[i][j][q])[e] > 0.0f ? v : 0.0f;
                    else v = fmaxf(v + bias[j], 0.0f);
                    h[e] = (bf16)v;
                    if (g.C) Cs[(8 * q + 4 * hi + e) * LDC + c31] = h[e];
                }
                *reinterpret_cast<bf16x4 *>(g.CT + at(i, j, q)) = h;
            }
            if (g.C) {
                sclbm::wave_lds_sync();  // the wavefront's own tile
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    *reinterpret_cast<uint4 *>(g.C + ((size_t)(rt + i) * (NHID / 16) + (ct + j) * 2 + t) * FRAG + lane * 8) =
                        ld16(Cs + c31 * LDC + t * 16 + hi * 8);
                sclbm::wave_lds_sync();
            }
        }
}

// ---------------------------------------------------------------------------------------------
// Output layer (3 units, no activation), its loss and the gradient of its input: one wavefront
// per row, each lane 8 of the 512 inputs.  Writes dY = 2 (y - t) / (3 n) (zero on padding rows),
// per-block sums of (y - t)^2 and of dY, and dZ3[m][k] = (sum_j dY[m][j] W4[j][k]) * (H3[m][k] > 0)
// with the contraction over the units (dZ) and over the rows (dZT).  OUT_ROWS rows per block
// (two per wave), grid Mpad / OUT_ROWS.
constexpr int OUT_ROWS = 8;
__global__ __launch_bounds__(256) void k_out(const bf16 *H, const bf16 *W4, const float *b4, int n, const float *oshift,
                                             const float *oscale, const float *targets, const int32_t *index,
                                             const int32_t *sym, int ndata, float *dY, double *partial, bf16 *dZ,
                                             bf16 *dZT, int Mpad) {
    constexpr int LD = NHID + 8;
    __shared__ double red[4][4];
    __shared__ __attribute__((aligned(16))) bf16 tile[OUT_ROWS][LD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = blockIdx.x * OUT_ROWS;
    constexpr int WROWS = OUT_ROWS / 4;  // rows of a wavefront
    // every load first: the rows' activations, the weights, and the targets behind the index
    bf16x8 hrow[WROWS];
    bool valid[WROWS];
    float tgt[WROWS][NOUT];
#pragma unroll
    for (int r = 0; r < WROWS; ++r)
        hrow[r] = *reinterpret_cast<const bf16x8 *>(H + frag_index(m0 + wave * WROWS + r, lane * 8, NHID));
    float w[NOUT][8];
#pragma unroll
    for (int j = 0; j < NOUT; ++j) {
        const bf16x8 v = *reinterpret_cast<const bf16x8 *>(W4 + j * NHID + lane * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) w[j][e] = (float)v[e];
    }
#pragma unroll
    for (int r = 0; r < WROWS; ++r) {
        const int m = __builtin_amdgcn_readfirstlane(m0 + wave * WROWS + r);
        valid[r] = m < n;
        int64_t src = 0;
        if (valid[r]) {
            src = index ? (int64_t)index[m] : (int64_t)m;
            const int sv = sym ? sym[m] : 0;
            valid[r] = src >= 0 && src < ndata && sv >= 0 && sv < 48;
        }
#pragma unroll
        for (int j = 0; j < NOUT; ++j) tgt[r][j] = valid[r] ? targets[src * NOUT + j] - oshift[j] : 0.0f;
    }
    double loss = 0.0, db[NOUT] = {0.0, 0.0, 0.0};
    const float inv = n > 0 ? 2.0f / (3.0f * (float)n) : 0.0f;
#pragma unroll
    for (int r = 0; r < WROWS; ++r) {
        const int rl = wave * WROWS + r, m = m0 + rl;
        const size_t at = frag_index(m, lane * 8, NHID);
        const bf16x8 h = hrow[r];
        float s[NOUT] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float hv = (float)h[e];
#pragma unroll
            for (int j = 0; j < NOUT; ++j) s[j] = fmaf(hv, w[j][e], s[j]);
        }
#pragma unroll
        for (int j = 0; j < NOUT; ++j) s[j] = wave_sum(s[j]) + b4[j];
        float d[NOUT];
#pragma unroll
        for (int j = 0; j < NOUT; ++j) {
            const float dj = valid[r] ? fmaf(-tgt[r][j], oscale[j], s[j]) : 0.0f;
            const float g = dj * inv;
            if (lane == j) dY[(size_t)m * NOUT + j] = g;
            loss += (double)dj * (double)dj;
            db[j] += (double)g;
            d[j] = g;
        }
        bf16x8 z;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = fmaf(d[2], w[2][e], fmaf(d[0], w[0][e], d[1] * w[1][e]));
            z[e] = (bf16)((float)h[e] > 0.0f ? v : 0.0f);
        }
        *reinterpret_cast<bf16x8 *>(dZ + at) = z;
        *reinterpret_cast<bf16x8 *>(&tile[rl][lane * 8]) = z;
    }
    if (lane == 0) {
        red[wave][0] = loss;
        for (int j = 0; j < NOUT; ++j) red[wave][1 + j] = db[j];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        double t = 0.0;
        for (int q = 0; q < 4; ++q) t += red[q][threadIdx.x];
        partial[blockIdx.x * 4 + threadIdx.x] = t;
    }
    static_assert(OUT_ROWS == 8, "a 16-byte piece of dZT");
    for (int u = threadIdx.x; u < NHID; u += 256) {
        bf16x8 h;
#pragma unroll
        for (int r = 0; r < 8; ++r) h[r] = tile[r][u];
        *reinterpret_cast<bf16x8 *>(dZT + frag_index(u, m0, Mpad)) = h;
    }
}

// ---------------------------------------------------------------------------------------------
// Inference in one launch: the four layers for FW_M rows per workgroup, the hidden activations
// kept in LDS.  The first layer reads the FP32 windows (ALIGNED: 16-byte aligned, else float by
// float) and normalises them; the products, the epilogue and the output layer round as k_layer
// and k_out do.  Wavefront w of the 8 computes output units
// 64 w .. 64 w + 63 of all FW_M rows (two 32 x 32 accumulator tiles) from its own weight rows,
// loaded FW_K columns at a time.  Grid Mpad / FW_M.
constexpr int FW_M = 32;
constexpr int FW_K = 32;
constexpr int FW_LDX = NIN + 8;   // 16-byte row pad: fragment reads spread over the banks
constexpr int FW_LDH = NHID + 8;
constexpr int FW_T = 512;         // threads
constexpr int FW_D = 4;           // weight stages in flight per wavefront (register buffers)

struct ForwardArgs {
    const float *win;             // [n][NIN]
    int n;
    const float *ashift, *ascale; // input normalisation
    const bf16 *W[3];             // hidden weights in fragment order (frag_index)
    const float *bias[3];
    const bf16 *W4;               // [NOUT][NHID]
    const float *b4, *oshift, *oscale;
    float *out;                   // [n][NOUT]
};

template <bool ALIGNED>
__global__ __launch_bounds__(FW_T) void k_forward(ForwardArgs f) {
    __shared__ __attribute__((aligned(16))) bf16 hx[FW_M * FW_LDX];          // input, then layer 2's output
    __shared__ __attribute__((aligned(16))) bf16 ha[FW_M * FW_LDH];          // layers 1 and 3's outputs
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.x * FW_M;

    // input rows: (a - shift) * scale rounded to BF16, rows >= n zero
    for (int c = tid; c < FW_M * NIN / 8; c += FW_T) {
        const int r = c / (NIN / 8), kc = (c % (NIN / 8)) * 8;
        const bool live = m0 + r < f.n;
        float4 a0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), a1 = a0;
        if (live) {
            const float *src = f.win + (size_t)(m0 + r) * NIN + kc;
            if (ALIGNED) {
                a0 = reinterpret_cast<const float4 *>(src)[0];
                a1 = reinterpret_cast<const float4 *>(src)[1];
            } else {
                a0 = make_float4(src[0], src[1], src[2], src[3]);
                a1 = make_float4(src[4], src[5], src[6], src[7]);
            }
        }
        const float4 sa = *reinterpret_cast<const float4 *>(f.ashift + kc);
        const float4 sb = *reinterpret_cast<const float4 *>(f.ashift + kc + 4);
        const float4 ca = *reinterpret_cast<const float4 *>(f.ascale + kc);
        const float4 cb = *reinterpret_cast<const float4 *>(f.ascale + kc + 4);
        bf16x8 h;
        h[0] = (bf16)((a0.x - sa.x) * ca.x);
        h[1] = (bf16)((a0.y - sa.y) * ca.y);
        h[2] = (bf16)((a0.z - sa.z) * ca.z);
        h[3] = (bf16)((a0.w - sa.w) * ca.w);
        h[4] = (bf16)((a1.x - sb.x) * cb.x);
        h[5] = (bf16)((a1.y - sb.y) * cb.y);
        h[6] = (bf16)((a1.z - sb.z) * cb.z);
        h[7] = (bf16)((a1.w - sb.w) * cb.w);
        if (!live) h = bf16x8{};
        *reinterpret_cast<bf16x8 *>(hx + r * FW_LDX + kc) = h;
    }

    // one hidden layer: Hout = relu(Hin W^T + b), K = NIN or NHID.  Every weight fragment is used
    // by one wavefront only (the one owning its output units), so each wavefront loads its own
    // fragments, 1 KB of consecutive bytes each in the fragment-ordered copy, into a ring of FW_D
    // register stages, FW_D - 1 stages of products ahead of their use (the loop is unrolled: buffer
    // indices are constants); only the activations, which all wavefronts read, go through LDS.
    auto layer = [&](auto kconst, const bf16 *Hin, int ldin, const bf16 *W, const float *bias, bf16 *Hout) {
        constexpr int K = decltype(kconst)::value;
        constexpr int nk = K / FW_K;
        uint4 bq[FW_D][FW_K / 16][2];  // [stage][k-step][tile]
        // this wavefront's tiles 2 wave, 2 wave + 1 of K / 16 fragments of 1 KB each
        const bf16 *wtile = W + ((size_t)(2 * wave) * (K / 16) * 64 + lane) * 8;
        auto gload = [&](int st, uint4 (&q)[FW_K / 16][2]) {
#pragma unroll
            for (int s = 0; s < FW_K / 16; ++s)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    q[s][j] = ld16(wtile + ((size_t)j * (K / 16) + st * (FW_K / 16) + s) * 512);
        };
        f32x16 acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
#pragma unroll
        for (int d = 0; d < FW_D; ++d)
            if (d < nk) gload(d, bq[d]);
#pragma unroll
        for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
            for (int s = 0; s < FW_K / 16; ++s) {
                const int kk = s * 16 + (lane >> 5) * 8;
                const bf16x8 av = *reinterpret_cast<const bf16x8 *>(Hin + (lane & 31) * ldin + kt * FW_K + kk);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        av, __builtin_bit_cast(bf16x8, bq[kt % FW_D][s][j]), acc[j], 0, 0, 0);
            }
            if (kt + FW_D < nk) gload(kt + FW_D, bq[kt % FW_D]);
        }
        // accumulator element 4q + e of a 32x32 tile sits at row 8q + 4 (lane / 32) + e, column lane % 32
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = wave * 64 + j * 32 + (lane & 31);
            const float bb = bias[col];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    Hout[(8 * q + 4 * (lane >> 5) + e) * FW_LDH + col] = (bf16)fmaxf(acc[j][4 * q + e] + bb, 0.0f);
        }
        __syncthreads();
    };
    __syncthreads();
    layer(std::integral_constant<int, NIN>{}, hx, FW_LDX, f.W[0], f.bias[0], ha);
    layer(std::integral_constant<int, NHID>{}, ha, FW_LDH, f.W[1], f.bias[1], hx);
    layer(std::integral_constant<int, NHID>{}, hx, FW_LDH, f.W[2], f.bias[2], ha);

    // output layer (k_out's arithmetic): each wavefront FW_M / 8 rows, lane l the inputs 8 l .. 8 l + 7
    float w[NOUT][8];
#pragma unroll
    for (int j = 0; j < NOUT; ++j) {
        const bf16x8 v = *reinterpret_cast<const bf16x8 *>(f.W4 + j * NHID + lane * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) w[j][e] = (float)v[e];
    }
    for (int r = 0; r < FW_M / 8; ++r) {
        const int rl = wave * (FW_M / 8) + r, m = m0 + rl;
        const bf16x8 h = *reinterpret_cast<const bf16x8 *>(ha + rl * FW_LDH + lane * 8);
        float s[NOUT] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float hv = (float)h[e];
#pragma unroll
            for (int j = 0; j < NOUT; ++j) s[j] = fmaf(hv, w[j][e], s[j]);
        }
#pragma unroll
        for (int j = 0; j < NOUT; ++j) s[j] = wave_sum(s[j]) + f.b4[j];
        if (m < f.n && lane < NOUT) {
            const float y = lane == 0 ? s[0] : (lane == 1 ? s[1] : s[2]);
            f.out[(size_t)m * NOUT + lane] = y / f.oscale[lane] + f.oshift[lane];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Adam on the FP32 master parameters, then the BF16 copies the products read: the hidden weights
// in fragment order (w: contraction over the inputs; wt, layers 2 and 3: over the units) and W4.
struct AdamArgs {
    float *p, *g, *m, *v;
    const float *part;  // the weights' gradients are the sums of `slices` of these (OFF_W4 apart), written
    int slices;         // to g on the way; null: they stand in g
    int update;         // 0: only refresh the BF16 copies
    float lr, beta1, beta2, eps, bc1, bc2;  // bc = 1 - beta^step
    bf16 *w[3], *wt[3], *w4;
};
__device__ __forceinline__ void adam_step(const AdamArgs &a, float &p, float g, float &m, float &v) {
    // (the multiply-adds are spelled out so that every kernel that updates rounds alike)
    m = fmaf(1.0f - a.beta1, g, a.beta1 * m);
    v = fmaf(a.beta2, v, ((1.0f - a.beta2) * g) * g);
    p -= a.lr * (m / a.bc1) / (sqrtf(v / a.bc2) + a.eps);
}

// The gradient g of parameter i (a bias, or an entry of W4) is final: into G, and with ADAM the update.
template <bool ADAM>
__device__ __forceinline__ void small_param(const AdamArgs &a, int i, float g) {
    a.g[i] = g;
    if (!ADAM) return;
    float p = a.p[i], m = a.m[i], v = a.v[i];
    adam_step(a, p, g, m, v);
    a.m[i] = m;
    a.v[i] = v;
    a.p[i] = p;
    if (i >= OFF_W4 && i < OFF_B4) a.w4[i - OFF_W4] = (bf16)p;
}

// Sum of the per-block partials in a fixed order (thread t takes blocks t, t + 256, ...; then a
// fixed tree): loss = sum (y - t)^2 / (3 n), db4 = sum dY.  256 threads; red in LDS.
template <bool ADAM>
__device__ __forceinline__ void loss_final(double (*red)[4], const double *partial, int nblocks, int n, double *loss,
                                           const AdamArgs &a) {
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nblocks; b += 256)
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] += partial[b * 4 + j];
#pragma unroll
    for (int j = 0; j < 4; ++j) red[threadIdx.x][j] = t[j];
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[threadIdx.x][j] += red[threadIdx.x + h][j];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (loss) *loss = n > 0 ? red[0][0] / (3.0 * (double)n) : 0.0;
        for (int j = 0; j < NOUT; ++j) small_param<ADAM>(a, OFF_B4 + j, (float)red[0][1 + j]);
    }
}

// Row sums over the batch of 8 units' entries of a [unit][row] matrix in fragment order, by one
// workgroup: J = 1, sum_m T[u][m]; J = 3, sum_m T[u][m] V[m][j].  Wavefront w takes the rows with
// m / 64 % 4 = w, its lane 8 c + i rows 8 c .. 8 c + 7 (mod 64) of unit u0 + i, so that 8 lanes read 128
// consecutive bytes.  The sum of a unit has a fixed order: rows m, m + 256, ... first, then
// the tree over m % 64, then the four groups of 64.
template <int J, bool ADAM>
__device__ __forceinline__ void unit_sums(float (*red)[8][4], const bf16 *T, int u0, int Mpad, const float *V,
                                          const AdamArgs &a, int off) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, u = u0 + (lane & 7), c = lane >> 3;
    float s[J][8];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[j][e] = 0.0f;
    const bf16 *p = T + frag_index(u, 64 * wave + 8 * c, Mpad);
    const float *pv = V + (size_t)(64 * wave + 8 * c) * J;
    // 256 rows on, the same place 16 fragments on
#pragma unroll 4
    for (int m = 64 * wave; m < Mpad; m += 256, p += 16 * FRAG, pv += 256 * J) {
        const bf16x8 x = *reinterpret_cast<const bf16x8 *>(p);
        float v[8 * J];
        if (J > 1) {
#pragma unroll
            for (int k = 0; k < 2 * J; ++k) {
                const float4 f = *reinterpret_cast<const float4 *>(pv + 4 * k);
                v[4 * k] = f.x, v[4 * k + 1] = f.y, v[4 * k + 2] = f.z, v[4 * k + 3] = f.w;
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int j = 0; j < J; ++j) s[j][e] = J > 1 ? fmaf((float)x[e], v[e * J + j], s[j][e]) : s[j][e] + (float)x[e];
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        float (&v)[8] = s[j];
#pragma unroll
        for (int o = 32; o >= 8; o >>= 1)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += __shfl_xor(v[e], o, 64);
        if (c == 0) red[j][lane & 7][wave] = ((v[0] + v[4]) + (v[2] + v[6])) + ((v[1] + v[5]) + (v[3] + v[7]));
    }
    __syncthreads();
    if (threadIdx.x < 8 * J) {
        const int j = threadIdx.x >> 3, i = threadIdx.x & 7;
        small_param<ADAM>(a, off + u0 + i + j * NHID, red[j][i][0] + red[j][i][1] + red[j][i][2] + red[j][i][3]);
    }
}

// All parameter gradients in one launch: dW_l = dZ_l^T H_{l-1} for the three hidden layers (tiles),
// the bias gradients and dW4 (unit_sums), the loss and db4 (one workgroup).  They depend on one
// another in nothing, and one after the other each would leave most of the device idle.
// The contraction runs over the batch: kst k-steps, `slices` workgroups of `per` k-steps each share
// a tile; with one slice the sums go to G, else to part[slice][OFF_W4], added in order by k_sum
// or k_adam.  Slice s sits on XCD s % 8 where there are 8, whose L2 then reads an eighth of the
// operands.
// ADAM (one slice): every workgroup also updates the parameters whose gradients it holds; no launch
// of the chain reads them any more.
struct GradArgs {
    const bf16 *dzT[3], *prevT[3];  // [unit][row] in fragment order
    const bf16 *hT3;                // the third layer's output
    const float *dY;
    const double *partial;          // k_out's per-block sums
    int npartial, n, Mpad, slices, per;
    float *part;
    double *loss;
    AdamArgs ad;                    // with its g, where the gradients go
};
constexpr int GRAD_SUMS = 4 * (NHID / 8);  // workgroups of the row sums (8 units each)

template <int RT, int CT, bool ADAM>
__global__ __launch_bounds__(256) void k_grad(GradArgs g) {
    // wavefronts of a workgroup: 2 x 2 of 32 x 32 tiles, or 4 x 1 of 64 x 64
    constexpr int WC = CT == 1 ? 2 : 1, WR = 4 / WC;
    constexpr int NR = NHID / (32 * RT * WR), TC = 32 * CT * WC;
    constexpr int N0 = NR * (NIN / TC), N1 = NR * (NHID / TC), NT = N0 + 2 * N1;
    constexpr int D = RT * CT == 1 ? 16 : 4;
    __shared__ union {
        double loss[256][4];
        float sums[NOUT][8][4];
        __attribute__((aligned(16))) bf16 cols[4][32 * 40];
    } red;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int b = blockIdx.x;
    if (b < NT * g.slices) {
        const int slice = b % g.slices;
        b /= g.slices;
        const int l = b < N0 ? 0 : (b < N0 + N1 ? 1 : 2);
        b -= l == 0 ? 0 : (l == 1 ? N0 : N0 + N1);
        const int K = l == 0 ? NIN : NHID, off = l == 0 ? OFF_W1 : (l == 1 ? OFF_W2 : OFF_W3);
        const bf16 *dz = l == 0 ? g.dzT[0] : (l == 1 ? g.dzT[1] : g.dzT[2]);
        const bf16 *pv = l == 0 ? g.prevT[0] : (l == 1 ? g.prevT[1] : g.prevT[2]);
        const int rt = (b % NR * WR + wave / WC) * RT, ct = (b / NR * WC + wave % WC) * CT;
        const size_t ts = (size_t)(g.Mpad / 16) * FRAG;
        const int k0 = slice * g.per, nk = min(g.per, g.Mpad / 16 - k0);
        float *out = (RT == 1 ? g.ad.g : (g.slices > 1 ? g.part + (size_t)slice * OFF_W4 : g.ad.g)) + off;
        auto at = [&](int i, int j, int e) {  // of accumulator element e = 4q + (row in the group)
            return ((rt + i) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * K + (ct + j) * 32 + (lane & 31);
        };
        f32x16 acc[RT][CT];
        if constexpr (ADAM && RT == 1) {
            // the parameters and moments, loaded ahead of the product
            float p[16], m[16], v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                p[e] = g.ad.p[off + at(0, 0, e)];
                m[e] = g.ad.m[off + at(0, 0, e)];
                v[e] = g.ad.v[off + at(0, 0, e)];
            }
            tile_product<1, 1, D>(dz + rt * ts + lane * 8, ts, pv + ct * ts + lane * 8, ts, nk, acc);
            // BF16 copies: over the inputs through the wavefront's LDS, over the units from registers
            constexpr int LDC = 40;
            bf16 *const Cs = red.cols[wave];
            bf16 *const w = l == 0 ? g.ad.w[0] : (l == 1 ? g.ad.w[1] : g.ad.w[2]);
            bf16 *const wt = l == 0 ? nullptr : (l == 1 ? g.ad.wt[1] : g.ad.wt[2]);
            const int c31 = lane & 31, hi = lane >> 5;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16x4 h;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int e = 4 * q + r;
                    adam_step(g.ad, p[e], acc[0][0][e], m[e], v[e]);
                    out[at(0, 0, e)] = acc[0][0][e];
                    g.ad.p[off + at(0, 0, e)] = p[e];
                    g.ad.m[off + at(0, 0, e)] = m[e];
                    g.ad.v[off + at(0, 0, e)] = v[e];
                    h[r] = (bf16)p[e];
                    Cs[(8 * q + 4 * hi + r) * LDC + c31] = h[r];
                }
                if (wt)
                    *reinterpret_cast<bf16x4 *>(wt + ((size_t)(ct * (NHID / 16) + rt * 2 + (q >> 1)) * 64 + c31 + 32 * (q & 1)) * 8 +
                                                4 * hi) = h;
            }
            sclbm::wave_lds_sync();
#pragma unroll
            for (int t = 0; t < 2; ++t)
                *reinterpret_cast<uint4 *>(w + ((size_t)rt * (K / 16) + ct * 2 + t) * FRAG + lane * 8) =
                    ld16(Cs + c31 * LDC + t * 16 + hi * 8);
            return;
        }
        tile_product<RT, CT, D>(dz + rt * ts + k0 * FRAG + lane * 8, ts, pv + ct * ts + k0 * FRAG + lane * 8, ts, nk, acc);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) out[at(i, j, e)] = acc[i][j][e];
        return;
    }
    b -= NT * g.slices;
    if (b < GRAD_SUMS) {
        const int v = b / (NHID / 8), u0 = b % (NHID / 8) * 8;
        if (v == 0) unit_sums<1, ADAM>(red.sums, g.dzT[0], u0, g.Mpad, nullptr, g.ad, OFF_B1);
        else if (v == 1) unit_sums<1, ADAM>(red.sums, g.dzT[1], u0, g.Mpad, nullptr, g.ad, OFF_B2);
        else if (v == 2) unit_sums<1, ADAM>(red.sums, g.dzT[2], u0, g.Mpad, nullptr, g.ad, OFF_B3);
        else unit_sums<NOUT, ADAM>(red.sums, g.hT3, u0, g.Mpad, g.dY, g.ad, OFF_W4);
        return;
    }
    loss_final<ADAM>(red.loss, g.partial, g.npartial, g.n, g.loss, g.ad);
}

// G = the sum over the slices of the weights' partial gradients, in order.
__global__ __launch_bounds__(256) void k_sum(const float *part, int slices, float *G) {
    const int i = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= OFF_W4 || (i >= OFF_B1 && i < OFF_W2) || (i >= OFF_B2 && i < OFF_W3) || i >= OFF_B3) return;
    float4 s = *reinterpret_cast<const float4 *>(part + i);
    for (int k = 1; k < slices; ++k) {
        const float4 p = *reinterpret_cast<const float4 *>(part + (size_t)k * OFF_W4 + i);
        s.x += p.x;
        s.y += p.y;
        s.z += p.z;
        s.w += p.w;
    }
    *reinterpret_cast<float4 *>(G + i) = s;
}

// A wavefront takes 8 rows of 64 columns of a hidden weight, lane 8 r + c eight columns of
// row r: 16-byte pieces of w, and through its own LDS 16-byte pieces of wt.  ADAM_TILES wavefronts' worth of those, then
// the biases, W4 and b4, one parameter a thread.
constexpr int ADAM_TILES = (NHID / 8) * (NIN / 64 + 2 * (NHID / 64));
constexpr int ADAM_REST = 3 * NHID + NOUT * NHID + NOUT;
constexpr int ADAM_BLOCKS = ADAM_TILES / 4 + (ADAM_REST + 255) / 256;
static_assert(ADAM_TILES % 4 == 0, "whole workgroups of tiles");
__global__ __launch_bounds__(256) void k_adam(AdamArgs a) {
    __shared__ __attribute__((aligned(16))) bf16 tile[4][8][72];
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t < ADAM_TILES) {
        constexpr int T0 = (NHID / 8) * (NIN / 64), T1 = (NHID / 8) * (NHID / 64);
        const int l = t < T0 ? 0 : (t < T0 + T1 ? 1 : 2);
        const int tl = t - (l == 0 ? 0 : (l == 1 ? T0 : T0 + T1));
        const int K = l == 0 ? NIN : NHID, off = l == 0 ? OFF_W1 : (l == 1 ? OFF_W2 : OFF_W3);
        bf16 *const w = l == 0 ? a.w[0] : (l == 1 ? a.w[1] : a.w[2]);
        bf16 *const wt = l == 0 ? nullptr : (l == 1 ? a.wt[1] : a.wt[2]);
        const int n = tl % (NHID / 8) * 8 + (lane >> 3), k = tl / (NHID / 8) * 64 + (lane & 7) * 8;
        const int at = off + n * K + k;
        float p[8];
        auto load8 = [&](const float *src, float (&x)[8]) {
            const float4 lo = *reinterpret_cast<const float4 *>(src + at), hi = *reinterpret_cast<const float4 *>(src + at + 4);
            x[0] = lo.x, x[1] = lo.y, x[2] = lo.z, x[3] = lo.w, x[4] = hi.x, x[5] = hi.y, x[6] = hi.z, x[7] = hi.w;
        };
        auto store8 = [&](float *dst, const float (&x)[8]) {
            *reinterpret_cast<float4 *>(dst + at) = make_float4(x[0], x[1], x[2], x[3]);
            *reinterpret_cast<float4 *>(dst + at + 4) = make_float4(x[4], x[5], x[6], x[7]);
        };
        load8(a.p, p);
        if (a.update) {
            float g[8], m[8], v[8];
            if (a.part) {
                load8(a.part, g);
                for (int k = 1; k < a.slices; ++k) {
                    float x[8];
                    load8(a.part + (size_t)k * OFF_W4, x);
#pragma unroll
                    for (int e = 0; e < 8; ++e) g[e] += x[e];
                }
                store8(a.g, g);
            } else {
                load8(a.g, g);
            }
            load8(a.m, m);
            load8(a.v, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) adam_step(a, p[e], g[e], m[e], v[e]);
            store8(a.m, m);
            store8(a.v, v);
            store8(a.p, p);
        }
        bf16x8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = (bf16)p[e];
        *reinterpret_cast<bf16x8 *>(w + frag_index(n, k, K)) = h;
        if (wt) {
            // lane l: the 8 rows of column l
            bf16(*const T)[72] = tile[threadIdx.x >> 6];
            *reinterpret_cast<bf16x8 *>(&T[lane >> 3][(lane & 7) * 8]) = h;
            sclbm::wave_lds_sync();
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = T[e][lane];
            *reinterpret_cast<bf16x8 *>(wt + frag_index(k - (lane & 7) * 8 + lane, n - (lane >> 3), NHID)) = h;
        }
        return;
    }
    const int i = (blockIdx.x - ADAM_TILES / 4) * 256 + threadIdx.x;
    if (i >= ADAM_REST) return;
    const int off = i < NHID ? OFF_B1 + i : (i < 2 * NHID ? OFF_B2 + i - NHID : OFF_B3 + i - 2 * NHID);
    float p = a.p[off];
    if (a.update) {
        float m = a.m[off], v = a.v[off];
        adam_step(a, p, a.g[off], m, v);
        a.m[off] = m;
        a.v[off] = v;
        a.p[off] = p;
    }
    if (off >= OFF_W4 && off < OFF_B4) a.w4[off - OFF_W4] = (bf16)p;
}

}  // namespace sclmlp
