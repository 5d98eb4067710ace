// Spectral corrector for gfx950 (paper Sec. 3.2; Alg. 1; App. E).
//
// sc_build_prior: anchor EMA, then the top-r SVD of the EMA by randomised
// block subspace iteration (MFMA tall-skinny passes over M, CholeskyQR2 with an
// fp64 Gram and an fp64 Cholesky in LDS), Rayleigh-Ritz by one-sided Jacobi in
// LDS, and the soft filter.
// sc_correct: T = G V (MFMA, split-K), X = U^T T, X_f = d X d, P = U X_f, then
// one fused pass G_proj = alpha G + (1 - alpha) P V^T.
#include "common.h"

#include <cstdlib>
#include <cstring>
#include "sc_status.h"
#include "sc_pass.h"
#include "sc_blend.h"
#include "sc_chol.h"
#include "sc_orth.h"
#include "sc_f32.h"

#include <algorithm>
#include <utility>
#include <vector>

namespace acsc {
namespace {

typedef float nf4 __attribute__((ext_vector_type(4)));
typedef unsigned int nu4 __attribute__((ext_vector_type(4)));

constexpr int kKMax = SC_KMAX;
// Singular values of the prior at or below this fraction of the largest are
// returned as zero (numerical rank of an fp32 subspace iteration).
constexpr double kRankCutoff = 1e-5;
// Largest k whose Rayleigh-Ritz Jacobi runs in fp64 (beyond it: fp32, whose
// columns take half the LDS)
constexpr int kJacobiF64MaxK = 128;

__host__ __device__ inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

// A launch works on up to kMaxBatch matrices: blockIdx.z selects the job,
// whose pointers and sizes travel by value in the kernel arguments.
constexpr int kMaxBatch = 16;
template <class Job>
struct Batch {
    int count;
    Job j[kMaxBatch];
};
__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// Element conversion helpers.  "CT" is the compute element type of the matrix
// cores: uint16_t (bf16 bits) or float.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ float to_f32(T v);
template <>
__device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float to_f32<uint16_t>(uint16_t v) { return bf16_to_f32(v); }

template <typename T>
__device__ __forceinline__ T from_f32(float v);
template <>
__device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ uint16_t from_f32<uint16_t>(float v) { return f32_to_bf16(v); }

// Anchor EMA with a bf16 shadow for the streaming passes (one thread per 8
// consecutive elements of a row; 16-byte accesses when rows are aligned):
//   M <- beta * M + (1 - beta) * G;  M16 <- bf16(M).   With G == NULL only the
// shadow is written.  The shadow is stored in 64 x 64 tiles (ntc tiles per
// tile row; see sc_pass.h).
struct EmaJob {
    float *M;
    const uint16_t *G;
    int m, n, vec;
    uint16_t *M16;
    int64_t ntc;
};

__device__ __forceinline__ int64_t tile_at(int64_t i, int64_t j, int64_t ntc)
{
    return ((i >> 6) * ntc + (j >> 6)) * 4096 + (i & 63) * 64 + (j & 63);
}

__global__ __launch_bounds__(256) void ema_shadow_kernel(const Batch<EmaJob> jb, float beta, float omb)
{
    const EmaJob &J = jb.j[blockIdx.z];
    float *M = J.M;
    const uint16_t *G = J.G;
    const int m = J.m, n = J.n;
    const bool VEC = J.vec != 0;
    uint16_t *M16 = J.M16;
    const int64_t ntc = J.ntc;
    const int nch = (n + 7) / 8;
    const int64_t total = static_cast<int64_t>(m) * nch;
    for (int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; q < total;
         q += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t i = q / nch;
        const int j0 = static_cast<int>(q - i * nch) * 8;
        float *mr = M + i * n + j0;
        const uint16_t *gr = G ? G + i * n + j0 : nullptr;
        float v[8];
        if (j0 + 8 <= n) {
            if (VEC) {
                const nf4 m0 = __builtin_nontemporal_load(reinterpret_cast<const nf4 *>(mr));
                const nf4 m1 = __builtin_nontemporal_load(reinterpret_cast<const nf4 *>(mr + 4));
                v[0] = m0.x; v[1] = m0.y; v[2] = m0.z; v[3] = m0.w;
                v[4] = m1.x; v[5] = m1.y; v[6] = m1.z; v[7] = m1.w;
            } else {
                // rows of other widths: the same accesses, not 16-byte aligned
                const F4Any m0 = *reinterpret_cast<const F4Any *>(mr), m1 = *reinterpret_cast<const F4Any *>(mr + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = m0.v[e];
                    v[4 + e] = m1.v[e];
                }
            }
            if (gr) {
                float g[8];
                uint32_t w4[4];
                if (VEC) {
                    const nu4 gb = __builtin_nontemporal_load(reinterpret_cast<const nu4 *>(gr));
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w4[e] = gb[e];
                } else {
                    const Bf8Any gb = *reinterpret_cast<const Bf8Any *>(gr);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w4[e] = gb.w[e];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    g[2 * e] = __uint_as_float(w4[e] << 16);
                    g[2 * e + 1] = __uint_as_float(w4[e] & 0xFFFF0000u);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = ema_step(v[e], g[e], beta, omb);
                if (VEC) {
                    __builtin_nontemporal_store(nf4{v[0], v[1], v[2], v[3]}, reinterpret_cast<nf4 *>(mr));
                    __builtin_nontemporal_store(nf4{v[4], v[5], v[6], v[7]}, reinterpret_cast<nf4 *>(mr + 4));
                } else {
                    *reinterpret_cast<F4Any *>(mr) = F4Any{{v[0], v[1], v[2], v[3]}};
                    *reinterpret_cast<F4Any *>(mr + 4) = F4Any{{v[4], v[5], v[6], v[7]}};
                }
            }
            uint16_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                h[e] = f32_to_bf16(v[e]);
            uint4 hv;
            __builtin_memcpy(&hv, h, sizeof(hv));
            *reinterpret_cast<uint4 *>(M16 + tile_at(i, j0, ntc)) = hv;
        } else {
            for (int e = 0; e < 8 && j0 + e < n; ++e) {
                float x = mr[e];
                if (gr) {
                    x = ema_step(x, bf16_to_f32(gr[e]), beta, omb);
                    mr[e] = x;
                }
                M16[tile_at(i, j0 + e, ntc)] = f32_to_bf16(x);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// fp64 Gram matrix of the first KP columns of A (rows x lda, fp32), on
// v_mfma_f64_16x16x4_f64: one workgroup per block of rows computes every
// upper 16 x 16 tile (ti <= tj) of that block's partial Gram; the partials
// are summed by gram_reduce_kernel, which also mirrors the lower triangle.
// The rows pass through LDS in 32-row chunks, converted to fp64 once and
// double-buffered (one barrier per chunk).  Operands (one fp64 per lane):
// A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k, so both come from the
// same read of a chunk row group: lane l takes row k0 + l / 16, column
// 16 b + l % 16, and every wave reads the KP / 16 column blocks once per
// 4-row step.  The result D[i][j] sits in lane j + 16 (i % 4), element i / 4.
// ---------------------------------------------------------------------------
constexpr int kGT = 16;
constexpr int kGRows = 32;
constexpr int kGWaves = 8;                         // waves per Gram workgroup
typedef double v4d __attribute__((ext_vector_type(4)));

struct GramJob {
    float *A;
    int64_t lda;
    int rows, rows_per_block, blocks;
    double *part;
    // > 1: A is still in that many partials of a pass (row stride KP, stride
    // rows * KP), which are added in order as they are read, and stored to A:
    // each row is read by one workgroup only, so a launch that would only add
    // them up (4 to 7 us) is saved
    const float *src;
    int splits;
};

// Staged row pitch in doubles: an odd multiple of 128 bytes, so that the two
// rows of a 32-lane half of an operand read fall in different bank halves.
__host__ __device__ constexpr int gram_pitch(int NB) { return NB * kGT + ((NB & 1) ? 0 : kGT); }

// Upper tiles in row-major order: tile t of an NB x NB block grid.
__host__ __device__ constexpr int gram_tile_row(int t, int NB)
{
    int ti = 0;
    while (t >= NB - ti) {
        t -= NB - ti;
        ++ti;
    }
    return ti;
}
__host__ __device__ constexpr int gram_tile_col(int t, int NB)
{
    int ti = 0;
    while (t >= NB - ti) {
        t -= NB - ti;
        ++ti;
    }
    return ti + t;
}

// One 4-row step of wave W's tiles: tile T = W + kGWaves U takes block rows
// ti(T) and tj(T) of the step's operands (indices fixed at compile time).
template <int NB, int T>
__device__ __forceinline__ v4d gram_mfma(const double (&op)[NB], v4d acc)
{
    constexpr int ti = gram_tile_row(T, NB), tj = gram_tile_col(T, NB);
    return __builtin_amdgcn_mfma_f64_16x16x4f64(op[ti], op[tj], acc, 0, 0, 0);
}
template <int NB, int W, int... U>
__device__ __forceinline__ void gram_mfmas(v4d *acc, const double (&op)[NB], std::integer_sequence<int, U...>)
{
    ((acc[U] = gram_mfma<NB, W + kGWaves * U>(op, acc[U])), ...);
}

// Wave W's share of the upper tiles: t = W, W + kGWaves, ...  (compile-time, so
// that the operand registers are indexed by constants).
template <int NB, int W, bool PARTS>
__device__ __forceinline__ void gram_wave(double *Ys0, double *Ys1, int lane, int nchunks,
                                          const GramJob &J, int r0, int r1, int KP, double *pb, int tid)
{
    float *A = J.A;
    const int64_t lda = J.lda;
    const int splits = J.splits;
    const int64_t ss = static_cast<int64_t>(J.rows) * KP;
    constexpr int NTILES = NB * (NB + 1) / 2;
    constexpr int TPW = NTILES > W ? (NTILES - W + kGWaves - 1) / kGWaves : 0;
    constexpr int NTH = 64 * kGWaves;              // threads
    constexpr int PITCH = gram_pitch(NB);          // doubles per staged row
    constexpr int q4 = NB * kGT / 4;               // float4 per staged row
    constexpr int PF = (kGRows * q4 + NTH - 1) / NTH;  // float4 per thread and chunk
    v4d acc[TPW > 0 ? TPW : 1];
#pragma unroll
    for (int u = 0; u < TPW; ++u)
        acc[u] = v4d{0.0, 0.0, 0.0, 0.0};
    float4 pf[PF];
    auto load = [&](int rb) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int idx = tid + NTH * u;
            const int rr = idx / q4, c4 = (idx % q4) * 4;
            const int gr = rb + rr;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (idx < kGRows * q4 && gr < r1 && c4 < KP) {
                if constexpr (PARTS) {
                    v = sum_partials(J.src + static_cast<int64_t>(gr) * KP + c4, ss, splits);
                    *reinterpret_cast<float4 *>(A + static_cast<int64_t>(gr) * lda + c4) = v;
                } else {
                    v = *reinterpret_cast<const float4 *>(A + static_cast<int64_t>(gr) * lda + c4);
                }
            }
            pf[u] = v;
        }
    };
    load(r0);
    for (int c = 0; c < nchunks; ++c) {
        double *Ys = (c & 1) ? Ys1 : Ys0;
        // stage this chunk (loaded during the previous one) as fp64; the
        // buffer was last read two chunks ago, before the previous barrier
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int idx = tid + NTH * u;
            if (idx < kGRows * q4) {
                double *d = Ys + (idx / q4) * PITCH + (idx % q4) * 4;
                *reinterpret_cast<double2 *>(d) = make_double2(pf[u].x, pf[u].y);
                *reinterpret_cast<double2 *>(d + 2) = make_double2(pf[u].z, pf[u].w);
            }
        }
        __syncthreads();
        if (c + 1 < nchunks)
            load(r0 + (c + 1) * kGRows);
        if constexpr (TPW > 0) {
            // the next step's operands are read before this step's products
            // are issued, so their latency hides under the MFMAs
            const double *yr = Ys + (lane >> 4) * PITCH + (lane & 15);
            double opA[NB], opB[NB];
            auto read = [&](double (&o)[NB], int k0) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    o[b] = yr[k0 * PITCH + b * kGT];
            };
            // (scheduling barriers keep each read ahead of the products before
            // it: left alone, the compiler sinks the reads to just before
            // their use and waits for them there)
            read(opA, 0);
#pragma unroll
            for (int k0 = 0; k0 < kGRows; k0 += 8) {
                read(opB, k0 + 4);
                __builtin_amdgcn_sched_barrier(0);
                gram_mfmas<NB, W>(acc, opA, std::make_integer_sequence<int, TPW>{});
                __builtin_amdgcn_sched_barrier(0);
                if (k0 + 8 < kGRows)
                    read(opA, k0 + 8);
                __builtin_amdgcn_sched_barrier(0);
                gram_mfmas<NB, W>(acc, opB, std::make_integer_sequence<int, TPW>{});
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
        const int t = W + kGWaves * u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = gram_tile_row(t, NB) * kGT + (lane >> 4) + 4 * e;
            const int j = gram_tile_col(t, NB) * kGT + (lane & 15);
            if (i < KP && j < KP)
                pb[static_cast<int64_t>(i) * KP + j] = acc[u][e];
        }
    }
}

template <int NB, bool PARTS>
__global__ __launch_bounds__(64 * kGWaves) void gram_partial_kernel(const Batch<GramJob> jb, int KP)
{
    const GramJob &J = jb.j[blockIdx.z];
    if (static_cast<int>(blockIdx.x) >= J.blocks)
        return;
    constexpr int PITCH = gram_pitch(NB);
    __shared__ __attribute__((aligned(16))) double Ys[2][kGRows * PITCH];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = blockIdx.x * J.rows_per_block;
    const int r1 = min(J.rows, r0 + J.rows_per_block);
    const int nchunks = (r1 - r0 + kGRows - 1) / kGRows;
    double *pb = J.part + static_cast<int64_t>(blockIdx.x) * KP * KP;
    switch (wave) {
    case 0: gram_wave<NB, 0, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    case 1: gram_wave<NB, 1, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    case 2: gram_wave<NB, 2, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    case 3: gram_wave<NB, 3, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    case 4: gram_wave<NB, 4, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    case 5: gram_wave<NB, 5, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    case 6: gram_wave<NB, 6, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    default: gram_wave<NB, 7, PARTS>(Ys[0], Ys[1], lane, nchunks, J, r0, r1, KP, pb, tid); break;
    }
}

struct GramRedJob {
    const double *part;
    int blocks;
    double *G;
};

__global__ __launch_bounds__(256) void gram_reduce_kernel(const Batch<GramRedJob> jb, int KP)
{
    // 32 consecutive elements x 8 groups of blocks per workgroup; only the
    // upper tiles are read (coalesced) and each is also written mirrored
    const GramRedJob &J = jb.j[blockIdx.z];
    __shared__ double red[8][32];
    const int e = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int idx = blockIdx.x * 32 + e;
    const int i = idx / KP, j = idx - (idx / KP) * KP;
    const bool live = idx < KP * KP && i / kGT <= j / kGT;
    double s = 0.0;
    if (live) {
        const int64_t stride = static_cast<int64_t>(KP) * KP;
        const double *p = J.part + idx;
        double s0 = 0.0, s1 = 0.0;
        int b = g;
        for (; b + 8 < J.blocks; b += 16) {
            s0 += p[b * stride];
            s1 += p[(b + 8) * stride];
        }
        if (b < J.blocks)
            s0 += p[b * stride];
        s = s0 + s1;
    }
    red[g][e] = s;
    __syncthreads();
    if (g == 0 && live) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            t += red[q][e];
        J.G[idx] = t;
        if (i / kGT < j / kGT)
            J.G[static_cast<int64_t>(j) * KP + i] = t;
    }
}

// Lane permutes within a row of 16 lanes (DPP: VALU, no LDS).
template <int CTRL>
__device__ __forceinline__ float dpp(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;        // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;                  // lane i of each 8 takes lane 7 - i
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;      // lane i takes lane i - 4 (i - 8) of its row
constexpr int kDppBcast = 0x150;                       // + L: every lane takes lane L of its row

// Sum over each group of 8 lanes; every lane of the group ends with it.
__device__ __forceinline__ float group8_sum(float x)
{
    x += dpp<kDppXor1>(x);
    x += dpp<kDppXor2>(x);
    x += dpp<kDppHalfMirror>(x);
    return x;
}

// Four sums over the 16 lanes of a row at once: quad q of the row ends with
// the sum of p[q] in its four lanes.  Each step halves the values a lane
// carries as it halves the lanes that are still apart, so four sums cost
// five exchanges instead of sixteen.
template <typename T>
__device__ __forceinline__ T row_sum4(const T (&p)[4], bool hi8, bool hi4)
{
    T a = (hi8 ? p[2] : p[0]) + dpp<kDppRor8>(hi8 ? p[0] : p[2]);
    T b = (hi8 ? p[3] : p[1]) + dpp<kDppRor8>(hi8 ? p[1] : p[3]);
    T s = (hi4 ? b : a) + dpp<kDppHalfMirror>(hi4 ? a : b);
    s += dpp<kDppXor1>(s);
    s += dpp<kDppXor2>(s);
    return s;
}

// Tangent t of the rotation that makes two columns of squared norms al, be and
// inner product ga orthogonal (0 where they already are to `tol`), and
// c = 1 / sqrt(1 + t^2), ic = sqrt(1 + t^2); `worst` takes the pair's
// |ga| / sqrt(al be).  A rotation has to be orthogonal to working precision,
// but its angle need not be exact: one that is off by 1e-7 leaves 1e-7 of
// the pair's inner product for the next sweep, which is less than a sweep
// leaves anyway.  So the angle comes from the hardware estimates and fp32,
// and only c from a refined reciprocal square root, which the columns do not
// wait for.  |zeta| past 1e18 is clamped: an angle below 1e-18 does not move a
// column.
__device__ __forceinline__ void rotation(double al, double be, double ga, double tol, float &worst, double &t,
                                         double &c, double &ic)
{
    const double prod = al * be;
    const double ratio = prod > 0.0 ? fabs(ga) * __builtin_amdgcn_rsq(prod) : (prod < 0.0 ? 1.0 : 0.0);
    worst = fmaxf(worst, static_cast<float>(ratio));
    const double zd = (be - al) * __builtin_amdgcn_rcp(2.0 * ga);
    const float z = static_cast<float>(fmin(fmax(zd, -1e18), 1e18));
    const float z2 = fmaf(z, z, 1.f);
    const float tt = copysignf(__builtin_amdgcn_rcpf(fabsf(z) + z2 * __builtin_amdgcn_rsqf(z2)), z);
    t = prod > 0.0 && ratio > tol ? static_cast<double>(tt) : 0.0;
    const double q = __builtin_fma(t, t, 1.0);
    c = __builtin_amdgcn_rsq(q);
    const double hq = 0.5 * q;
    c = __builtin_fma(c, __builtin_fma(-hq * c, c, 0.5), c);   // c + c (1 - q c^2) / 2
    c = __builtin_fma(c, __builtin_fma(-hq * c, c, 0.5), c);
    ic = q * c;
}

// ---------------------------------------------------------------------------
// One-sided (Hestenes) Jacobi SVD of the k x k factor L, one workgroup:
// rotate column pairs until every pair is orthogonal to `tol`.  Then
// sigma_c = ||a_c||, u_c = a_c / sigma_c, sorted descending, and the right
// factors of the final products are written:  Bu[:, t] = u_(t),
// Bv[:, t] = u_(t) / sigma_(t), s[t] = sigma_(t), d[t] = s / (s + tau), t < r.
//
// What bounds it is the chain of rounds (k - 1 per sweep, 6 or 7 sweeps), each
// a few hundred cycles of dependent work on one CU.  The columns sit in LDS
// in blocks of four; a row of 16 lanes holds a pair of blocks in registers
// (R rows of 8 columns per lane) and makes all 16 cross pairs orthogonal in
// four rounds of four rotations before it stores them: one LDS round trip
// and one barrier for four rounds, and the four rotations of a round share
// one reduction and one evaluation of the angle (quad q of the row has
// rotation q).  In between a column is held as x / d with its scale d apart
// (x' = c (x - t y), y' = c (y + t x): the factors c go to the scales), so a
// rotation is two multiply-adds per element and waits for t only.  Block pairs follow a round-robin tournament; the pairs
// within a block go before the first of a sweep, together with the exact
// squared norms, which the rotations then update.
// Measured (six 48 x 48, four 80 x 80 factors): 190 and 400 us with a barrier
// and an LDS round trip per round, 145 and 310 us so; one factor of a 1024 x 1024
// matrix, from a random start: 46 and 43 us at k = 16, 69 and 59 at 24, 95 and
// 74 at 32, 409 and 174 at 64, 723 and 396 at 96, 872 and 517 at 112, 4077
// and 759 at 128.  Warm-started, also with no new gradient, where the
// form before could leave out the pairs that were orthogonal already: 46 and
// 43, 72 and 58, 93 and 74, 311 and 174, 544 and 336, 615 and 441, 2642 and
// 545.  Sweeps: 6 to 8 then, one fewer now (the inner-product check).
// ---------------------------------------------------------------------------
struct JacJob {
    const double *Lf;
    float *Bu, *Bv, *s_out, *d_out;
    int *info;
};

constexpr int kJacobiMaxSweeps = 40;

// Column pitch of the fp64 kernel in LDS: past the padded rows, so that the
// lanes that read or write one row of many columns fall on different banks.
// (The fp32 kernel's 16-byte accesses run best unpadded: 600 us against 850
// with four more rows at k = 144.)
__host__ __device__ constexpr int jacobi_pitch_f64(int rows) { return rows + 1; }

constexpr int kJacBlk = 4;   // columns per block

// blocks of the tournament: an even number
__host__ __device__ constexpr int jacobi_blocks(int k) { return ((k + kJacBlk - 1) / kJacBlk + 1) & ~1; }

// The columns of the factor into LDS (column c at A[c * kp]), rows and columns
// past k as zeros.  Rows of the factor are read whole, and eight loads go
// out before the first is stored.
template <typename T, int kp>
__device__ __forceinline__ void jacobi_load(T *A, int cols, const double *Lf, int k, int KP)
{
    const int nth = blockDim.x, total = cols * kp;
    for (int i0 = threadIdx.x; i0 < total; i0 += 8 * nth) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = min(i0 + u * nth, total - 1);
            const int i = idx / cols, c = idx - i * cols;
            v[u] = Lf[static_cast<int64_t>(min(i, k - 1)) * KP + min(c, k - 1)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = i0 + u * nth;
            const int i = idx / cols, c = idx - i * cols;
            if (idx < total)
                A[c * kp + i] = i < k && c < k ? static_cast<T>(v[u]) : T(0);
        }
    }
}

// What follows the sweeps: the status words, then singular values, their order,
// the right factors of the final products and the filter.  Column c of the
// orthogonal factor is A[c * kp] in LDS.
template <typename T, int kp>
__device__ __forceinline__ void jacobi_finish(const JacJob &J, const T *A, int k, int KP, int r, int RP, float tau,
                                              float tol, int sweeps_used, float last_off, int stamp)
{
    float *Bu = J.Bu, *Bv = J.Bv, *s_out = J.s_out, *d_out = J.d_out;
    int *info = J.info;
    __shared__ double sh_cut;
    __shared__ double sig[kKMax], inv[kKMax];
    __shared__ int rank_of[kKMax], col_of[kKMax];
    const int tid = threadIdx.x, nth = blockDim.x, grp = tid >> 4, gl = tid & 15;
    if (tid == 0 && info) {
        info[kInfoSweeps] = sweeps_used;
        info[kInfoResidual] = __float_as_int(last_off);
        info[kInfoTol] = __float_as_int(tol);
        info[kInfoStatus] = (last_off > tol ? kStatusNoConv : 0) |
                            (stamp != kSubspaceStamp && stamp != kSubspaceStalledStamp ? kStatusNoSubspace : 0) |
                            (stamp == kSubspaceStalledStamp ? kStatusStalled : 0);
        info[kInfoStamp] = 0;
    }
    // norms, one row of 16 lanes per column
    for (int c = grp; c < k; c += nth >> 4) {
        double ss = 0.0;
        for (int i = gl; i < k; i += 16) {
            const double x = A[c * kp + i];
            ss += x * x;
        }
        ss += dpp<kDppRor8>(ss);
        ss += dpp<kDppHalfMirror>(ss);
        ss += dpp<kDppXor1>(ss);
        ss += dpp<kDppXor2>(ss);
        if (gl == 0)
            sig[c] = sqrt(ss);
    }
    __syncthreads();
    for (int c = tid; c < k; c += nth) {
        int rk = 0;
        for (int c2 = 0; c2 < k; ++c2)
            rk += (sig[c2] > sig[c]) || (sig[c2] == sig[c] && c2 < c);
        rank_of[c] = rk;
        col_of[c] = c;   // a factor with NaNs has equal ranks and leaves places of col_of unset below
    }
    __syncthreads();
    // numerical rank: singular values at the fp32 rounding floor of the
    // largest one are zero (their vectors are noise, and 1/sigma would blow up)
    for (int c = tid; c < k; c += nth) {
        col_of[rank_of[c]] = c;
        if (rank_of[c] == 0)
            sh_cut = kRankCutoff * sig[c];
    }
    __syncthreads();
    for (int c = tid; c < k; c += nth)
        if (sig[c] <= sh_cut)
            sig[c] = 0.0;
    __syncthreads();
    for (int c = tid; c < k; c += nth)
        inv[c] = sig[c] > 0.0 ? 1.0 / sig[c] : 0.0;
    __syncthreads();
#pragma unroll 4
    for (int idx = tid; idx < KP * RP; idx += nth) {
        const int i = idx / RP, t = idx - i * RP;
        const int c = col_of[min(t, k - 1)];
        const double ud = i < k && t < r ? static_cast<double>(A[c * kp + min(i, k - 1)]) * inv[c] : 0.0;
        Bu[idx] = static_cast<float>(ud);
        Bv[idx] = static_cast<float>(ud * inv[c]);
    }
    for (int t = tid; t < r; t += nth) {
        const float sg = static_cast<float>(sig[col_of[t]]);
        s_out[t] = sg;
        const float den = sg + tau;
        d_out[t] = den != 0.f ? sg / den : 0.f;
    }
}

// fp32 (beyond the orders whose fp64 columns fit LDS): column pairs of a
// round-robin tournament, 8 lanes per pair, one round per barrier.  At 72
// pairs of 160 rows a round is bound by the instructions that one CU can
// issue, which the wider rows of the blocked form below do not cut: 144 x 144
// takes 600 to 630 us so and 890 us in blocks.
template <int R>
__global__ __launch_bounds__(1024) void jacobi_pairs_kernel(const Batch<JacJob> jb, int k, int KP, int r, int RP,
                                                            float tau, float tol, int max_sweeps)
{
    const JacJob &J = jb.j[blockIdx.z];
    const double *Lf = J.Lf;
    int *info = J.info;
    extern __shared__ __attribute__((aligned(16))) unsigned char jsm[];
    // column c at A[c * kp], rows k..kp-1 are zero.  Lane gl of a pair's 8
    // lanes holds the R consecutive rows gl R .. gl R + R - 1 of both columns
    // (R a multiple of 4: 16-byte LDS accesses).
    using T = float;
    constexpr int V = 4, kp = 8 * R;
    T *A = reinterpret_cast<T *>(jsm);
    T *nrm = A + static_cast<size_t>(k) * kp;   // squared column norms
    __shared__ unsigned int sh_off;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwave = blockDim.x >> 6;
    jacobi_load<T, kp>(A, k, Lf, k, KP);
    const int n2 = k + (k & 1);
    const int npairs = n2 / 2;
    // eight column pairs per wave, 8 lanes each
    const int grp = lane >> 3, gl = lane & 7;
    const int slots = nwave * 8;
    static_assert(R % V == 0, "rows per lane");
    int sweeps_used = 0;
    float last_off = 0.f;
    // the subspace phase that produced Lf stamps the workspace (read before
    // this kernel clears the stamp, by the same thread)
    const int stamp = (tid == 0 && info) ? info[kInfoStamp] : 0;
    __syncthreads();
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
        // exact squared norms at the start of every sweep (the rotations
        // update them incrementally within it)
        for (int c = wave * 8 + grp; c < k; c += slots) {
            const T *ac = A + c * kp + gl * R;
            T ss = 0;
#pragma unroll
            for (int e = 0; e < R; ++e)
                ss += ac[e] * ac[e];
            ss = group8_sum(ss);
            if (gl == 0)
                nrm[c] = ss;
        }
        if (tid == 0)
            sh_off = 0u;
        __syncthreads();
        float wmax = 0.f;
        for (int round = 0; round < n2 - 1; ++round) {
            for (int p = wave * 8 + grp; p < npairs; p += slots) {
                auto pos = [&](int x) {
                    if (x == 0)
                        return 0;
                    int t = x - 1 + round;
                    if (t >= n2 - 1)
                        t -= n2 - 1;
                    return t + 1;
                };
                int cp = pos(p), cq = pos(n2 - 1 - p);
                if (cp >= k || cq >= k)
                    continue;
                if (cp > cq) {
                    const int t = cp;
                    cp = cq;
                    cq = t;
                }
                T *ap = A + cp * kp + gl * R;
                T *aq = A + cq * kp + gl * R;
                T xv[R], yv[R];
#pragma unroll
                for (int e = 0; e < R; e += V) {
                    const uint4 ux = *reinterpret_cast<const uint4 *>(ap + e);
                    const uint4 uy = *reinterpret_cast<const uint4 *>(aq + e);
                    __builtin_memcpy(&xv[e], &ux, 16);
                    __builtin_memcpy(&yv[e], &uy, 16);
                }
                const T al = nrm[cp], be = nrm[cq];
                T gp[4] = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < R; ++e)
                    gp[e & 3] += xv[e] * yv[e];
                const T ga = group8_sum((gp[0] + gp[1]) + (gp[2] + gp[3]));
                const T prod = al * be;
                if (ga == T(0) || prod == T(0))
                    continue;
                const T ratio = fabs(ga) * __builtin_amdgcn_rsqf(prod);
                wmax = fmaxf(wmax, static_cast<float>(ratio));
                if (ratio <= tol)
                    continue;
                const T zeta = (be - al) * __builtin_amdgcn_rcpf(T(2) * ga);
                const T z2 = T(1) + zeta * zeta;
                const T t = (zeta >= T(0) ? T(1) : T(-1)) * __builtin_amdgcn_rcpf(fabs(zeta) + z2 * __builtin_amdgcn_rsqf(z2));
                const T c = __builtin_amdgcn_rsqf(T(1) + t * t);
                const T sn = c * t;
#pragma unroll
                for (int e = 0; e < R; e += V) {
                    T xo[V], yo[V];
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        xo[v] = c * xv[e + v] - sn * yv[e + v];
                        yo[v] = sn * xv[e + v] + c * yv[e + v];
                    }
                    uint4 ux, uy;
                    __builtin_memcpy(&ux, xo, 16);
                    __builtin_memcpy(&uy, yo, 16);
                    *reinterpret_cast<uint4 *>(ap + e) = ux;
                    *reinterpret_cast<uint4 *>(aq + e) = uy;
                }
                // the rotation zeroes the pair's inner product: the norms move by t gamma
                if (gl == 0) {
                    nrm[cp] = al - t * ga;
                    nrm[cq] = be + t * ga;
                }
            }
            __syncthreads();
        }
        // reduce the sweep's largest off-diagonal ratio over the workgroup
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            wmax = fmaxf(wmax, __shfl_xor(wmax, off, 64));
        if (lane == 0)
            atomicMax(&sh_off, __float_as_uint(wmax));
        __syncthreads();
        const float off = __uint_as_float(sh_off);
        __syncthreads();
        sweeps_used = sweep + 1;
        last_off = off;
        if (off <= static_cast<float>(tol))
            break;
    }
    jacobi_finish<T, kp>(J, A, k, KP, r, RP, tau, static_cast<float>(tol), sweeps_used, last_off, stamp);
}

// fp64: see above.  At an order of 16 to 80 a round takes 0.45 to 0.58 us (0.67
// to 0.72 with a barrier and an LDS round trip per round).
constexpr float kJacCheck = 1e-6f;   // a sweep that met less than this may be the last

template <int R>
__global__ __launch_bounds__(256) void jacobi_blocks_kernel(const Batch<JacJob> jb, int k, int KP, int r, int RP,
                                                            float tau, double tol, int max_sweeps)
{
    using T = double;
    const JacJob &J = jb.j[blockIdx.z];
    const double *Lf = J.Lf;
    int *info = J.info;
    extern __shared__ __attribute__((aligned(16))) unsigned char jsm[];
    constexpr int kp = jacobi_pitch_f64(16 * R);   // rows k .. are zero
    const int nb = jacobi_blocks(k), cols = nb * kJacBlk;   // columns k .. cols - 1 are zero
    T *A = reinterpret_cast<T *>(jsm);         // column c at A[c * kp]
    T *nrm = A + static_cast<size_t>(cols) * kp;   // squared column norms
    __shared__ unsigned int sh_off;
    const int tid = threadIdx.x, lane = tid & 63;
    const int nth = blockDim.x;
    jacobi_load<T, kp>(A, cols, Lf, k, KP);
    const int grp = tid >> 4, gl = tid & 15, quad = gl >> 2;
    const bool hi8 = gl & 8, hi4 = gl & 4;
    const bool live = grp < nb / 2;            // whole rows of 16 lanes
    int sweeps_used = 0;
    float last_off = 0.f;
    // the subspace phase that produced Lf stamps the workspace (read before
    // this kernel clears the stamp, by the same thread)
    const int stamp = (tid == 0 && info) ? info[kInfoStamp] : 0;
    __syncthreads();
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
        if (tid == 0)
            sh_off = 0u;
        float worst = 0.f;
        for (int round = 0; round < nb - 1; ++round) {
            if (live) {
                auto pos = [&](int x) {
                    if (x == 0)
                        return 0;
                    int t = x - 1 + round;
                    if (t >= nb - 1)
                        t -= nb - 1;
                    return t + 1;
                };
                const int b0 = pos(grp), b1 = pos(nb - 1 - grp);
                const int c0 = min(b0, b1) * kJacBlk, c1 = max(b0, b1) * kJacBlk;
                // lane gl holds rows gl, gl + 16, ... of columns c0 .. c0 + 3 and c1 .. c1 + 3
                T x[2 * kJacBlk][R];
                T *pa = A + c0 * kp + gl, *pb = A + c1 * kp + gl;
#pragma unroll
                for (int j = 0; j < kJacBlk; ++j)
#pragma unroll
                    for (int e = 0; e < R; ++e) {
                        x[j][e] = pa[j * kp + 16 * e];
                        x[kJacBlk + j][e] = pb[j * kp + 16 * e];
                    }
                // the four pairs (u[q], v[q]) at once: quad q has its two
                // columns' squared norms n, scales d and 1 / d
                struct Col {
                    T n, d, id;
                };
                auto rotate = [&](const int (&u)[4], const int (&v)[4], Col &a, Col &b) {
                    T p[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        p[q] = x[u[q]][0] * x[v[q]][0];
#pragma unroll
                        for (int e = 1; e < R; ++e)
                            p[q] += x[u[q]][e] * x[v[q]][e];
                    }
                    const T ga = row_sum4(p, hi8, hi4) * (a.d * b.d);
                    T t, c, ic;
                    rotation(a.n, b.n, ga, tol, worst, t, c, ic);
                    const T fu = t * (b.d * a.id), fv = t * (a.d * b.id);
                    const T uu[4] = {dpp<kDppBcast>(fu), dpp<kDppBcast + 4>(fu), dpp<kDppBcast + 8>(fu),
                                     dpp<kDppBcast + 12>(fu)};
                    const T vv[4] = {dpp<kDppBcast>(fv), dpp<kDppBcast + 4>(fv), dpp<kDppBcast + 8>(fv),
                                     dpp<kDppBcast + 12>(fv)};
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int e = 0; e < R; ++e) {
                            const T xa = x[u[q]][e], xb = x[v[q]][e];
                            x[u[q]][e] = xa - uu[q] * xb;
                            x[v[q]][e] = xb + vv[q] * xa;
                        }
                    const T c2 = c * c, tg = T(2) * t * ga, t2 = t * t;
                    const T na = c2 * (a.n - tg + t2 * b.n), nb2 = c2 * (b.n + tg + t2 * a.n);
                    a = Col{na, a.d * c, a.id * ic};
                    b = Col{nb2, b.d * c, b.id * ic};
                };
                Col ca{T(0), T(1), T(1)}, cb = ca;
                if (round == 0) {
                    // exact squared norms, then the pairs within the two blocks:
                    // quads 0, 1 take block c0's, quads 2, 3 block c1's
                    T p[4], n0, n1;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            p[q] = x[4 * h + q][0] * x[4 * h + q][0];
#pragma unroll
                            for (int e = 1; e < R; ++e)
                                p[q] += x[4 * h + q][e] * x[4 * h + q][e];
                        }
                        (h ? n1 : n0) = row_sum4(p, hi8, hi4);
                    }
                    // a column's norm, scale and its reciprocal go through LDS from
                    // pair to pair (scl: two words per column after the norms)
                    T *scl = nrm + cols;
                    auto at = [&](int a) { return (a < 4 ? c0 : c1 - 4) + a; };
                    auto put = [&](int a, const Col &v) {
                        if ((gl & 3) == 0) {
                            nrm[at(a)] = v.n;
                            scl[2 * at(a)] = v.d;
                            scl[2 * at(a) + 1] = v.id;
                        }
                    };
                    auto get = [&](int a) { return Col{nrm[at(a)], scl[2 * at(a)], scl[2 * at(a) + 1]}; };
                    auto wave_sync = [&]() {
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    };
                    put(quad, Col{n0, T(1), T(1)});
                    put(4 + quad, Col{n1, T(1), T(1)});
                    auto step = [&](const int (&u)[4], const int (&v)[4]) {
                        wave_sync();
                        const int a = quad == 0 ? u[0] : quad == 1 ? u[1] : quad == 2 ? u[2] : u[3];
                        const int b = quad == 0 ? v[0] : quad == 1 ? v[1] : quad == 2 ? v[2] : v[3];
                        Col va = get(a), vb = get(b);
                        rotate(u, v, va, vb);
                        wave_sync();
                        put(a, va);
                        put(b, vb);
                    };
                    step({0, 2, 4, 6}, {1, 3, 5, 7});
                    step({0, 1, 4, 5}, {2, 3, 6, 7});
                    step({0, 1, 4, 5}, {3, 2, 7, 6});
                    wave_sync();
                    ca = get(quad);
                    cb = get(4 + quad);
                } else {
                    ca.n = nrm[c0 + quad];
                    cb.n = nrm[c1 + quad];
                }
                // round s: column q of c0 with column (q - s) % 4 of c1; the
                // scalars of c1's columns move on by one quad per round
                auto next = [&]() { cb = Col{dpp<kDppRor4>(cb.n), dpp<kDppRor4>(cb.d), dpp<kDppRor4>(cb.id)}; };
                rotate({0, 1, 2, 3}, {4, 5, 6, 7}, ca, cb);
                next();
                rotate({0, 1, 2, 3}, {7, 4, 5, 6}, ca, cb);
                next();
                rotate({0, 1, 2, 3}, {6, 7, 4, 5}, ca, cb);
                next();
                rotate({0, 1, 2, 3}, {5, 6, 7, 4}, ca, cb);
                next();
                const T da[4] = {dpp<kDppBcast>(ca.d), dpp<kDppBcast + 4>(ca.d), dpp<kDppBcast + 8>(ca.d),
                                 dpp<kDppBcast + 12>(ca.d)};
                const T db[4] = {dpp<kDppBcast>(cb.d), dpp<kDppBcast + 4>(cb.d), dpp<kDppBcast + 8>(cb.d),
                                 dpp<kDppBcast + 12>(cb.d)};
                if ((gl & 3) == 0) {
                    nrm[c0 + quad] = ca.n;
                    nrm[c1 + quad] = cb.n;
                }
#pragma unroll
                for (int j = 0; j < kJacBlk; ++j)
#pragma unroll
                    for (int e = 0; e < R; ++e) {
                        pa[j * kp + 16 * e] = da[j] * x[j][e];
                        pb[j * kp + 16 * e] = db[j] * x[kJacBlk + j][e];
                    }
            }
            __syncthreads();
        }
        // reduce the sweep's largest off-diagonal ratio over the workgroup
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            worst = fmaxf(worst, __shfl_xor(worst, off, 64));
        if (lane == 0)
            atomicMax(&sh_off, __float_as_uint(worst));
        __syncthreads();
        const float off = __uint_as_float(sh_off);
        __syncthreads();
        sweeps_used = sweep + 1;
        last_off = off;
        if (off <= static_cast<float>(tol))
            break;
        if (off < kJacCheck) {
            // a sweep leaves about the square of what it met: the inner
            // products themselves (matrix cores, about 2 us) tell whether
            // this one was the last, instead of one more sweep
            if (tid == 0)
                sh_off = 0u;
            __syncthreads();
            const int nt = cols / 16 + (cols % 16 ? 1 : 0);
            float w = 0.f;
            for (int t = tid >> 6; t < nt * nt; t += nth >> 6) {
                const int ti = t / nt, tj = t - ti * nt;
                if (ti > tj)
                    continue;
                const int ci = ti * 16 + (lane & 15), cj = tj * 16 + (lane & 15);
                const T *ai = A + min(ci, cols - 1) * kp + (lane >> 4), *aj = A + min(cj, cols - 1) * kp + (lane >> 4);
                v4d g = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < 16 * R; e += 4)
                    g = __builtin_amdgcn_mfma_f64_16x16x4f64(ai[e], aj[e], g, 0, 0, 0);
                // D[i][j] in lane j + 16 (i % 4), element i / 4
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = ti * 16 + 4 * e + (lane >> 4);
                    if (i < cj && cj < k) {
                        const double prod = nrm[i] * nrm[cj];
                        if (prod > 0.0)
                            w = fmaxf(w, static_cast<float>(fabs(g[e]) * __builtin_amdgcn_rsq(prod)));
                    }
                }
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1)
                w = fmaxf(w, __shfl_xor(w, o, 64));
            if (lane == 0)
                atomicMax(&sh_off, __float_as_uint(w));
            __syncthreads();
            const float left = __uint_as_float(sh_off);
            __syncthreads();
            if (left <= static_cast<float>(tol)) {
                last_off = left;
                break;
            }
        }
    }
    jacobi_finish<T, kp>(J, A, k, KP, r, RP, tau, static_cast<float>(tol), sweeps_used, last_off, stamp);
}

// ---------------------------------------------------------------------------
// Elementwise kernels.
// ---------------------------------------------------------------------------
// M <- beta * M + (1 - beta) * G  (fp32 state)
struct Ema32Job {
    float *M;
    const float *G;
    int64_t count;
};

__global__ __launch_bounds__(256) void ema_kernel(const Batch<Ema32Job> jb, float beta, float omb)
{
    float *M = jb.j[blockIdx.z].M;
    const float *G = jb.j[blockIdx.z].G;
    const int64_t count = jb.j[blockIdx.z].count;
    if (!G)
        return;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x * 4;
    for (int64_t i = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) * 4; i < count;
         i += stride) {
        if (i + 4 <= count) {
            float4 m = *reinterpret_cast<const float4 *>(M + i);
            const float4 g = *reinterpret_cast<const float4 *>(G + i);
            m.x = ema_step(m.x, g.x, beta, omb);
            m.y = ema_step(m.y, g.y, beta, omb);
            m.z = ema_step(m.z, g.z, beta, omb);
            m.w = ema_step(m.w, g.w, beta, omb);
            *reinterpret_cast<float4 *>(M + i) = m;
        } else {
            for (int64_t j = i; j < count; ++j)
                M[j] = ema_step(M[j], G[j], beta, omb);
        }
    }
}

// Starting block Z0 [n, KP]: V_warm columns first (if given), then uniform
// random values in [-1, 1) from a counter-based hash of (seed, i, c); zero
// beyond k.
// Entry (i, c) of the seeded starting block: the low 32 bits of the seed
// added to a Weyl combination of row and column, then C. Wellons's lowbias32
// integer hash (two 32-bit multiplies), the top 24 bits mapped to [-1, 1).
// The subspace iteration only needs a seeded block of full rank with no
// preferred direction; a 64-bit mixer here made the start block the most
// expensive step of a cold build after the passes.
__device__ __forceinline__ float start_uniform(uint64_t seed, int64_t i, int c)
{
    uint32_t h = static_cast<uint32_t>(i) * 0x9E3779B1u + static_cast<uint32_t>(c) * 0x632BE5ABu +
                 static_cast<uint32_t>(seed) + static_cast<uint32_t>(seed >> 32) * 0x85EBCA6Bu;
    h ^= h >> 16;
    h *= 0x7FEB352Du;
    h ^= h >> 15;
    h *= 0x846CA68Bu;
    h ^= h >> 16;
    return static_cast<float>(h >> 8) * (2.0f / 16777216.0f) - 1.0f;
}

struct InitJob {
    float *Z;
    int n;
    const float *Vw;
    uint64_t seed;
};

__global__ __launch_bounds__(256) void init_block_kernel(const Batch<InitJob> jb, int k, int KP, int r)
{
    float *Z = jb.j[blockIdx.z].Z;
    const int n = jb.j[blockIdx.z].n;
    const float *Vw = jb.j[blockIdx.z].Vw;
    const int rw = Vw ? r : 0;
    const uint64_t seed = jb.j[blockIdx.z].seed;
    const int64_t total = static_cast<int64_t>(n) * KP;
    for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < total;
         idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t i = idx / KP;
        const int c = static_cast<int>(idx - i * KP);
        float v = 0.f;
        if (c < k) {
            if (Vw && c < rw)
                v = Vw[i * rw + c];
            else
                v = start_uniform(seed, i, c);
        }
        Z[idx] = v;
    }
}

// 64-row tiles of a thin fp32 block [rows, cols] to bf16, zero-padded to CP
// columns, through LDS: the transposed copy Xt[c][i] (row stride ldt, 16-byte
// stores along i) and/or the row-major copy Xc[i][c] (row stride CP).  With
// X == nullptr the block is the starting block of the subspace iteration
// (V_warm columns, then seeded uniform draws, for c < cols).
struct TileJob {
    const float *X;
    int64_t ldx;
    int rows, cols, CP;
    uint16_t *Xt;
    int64_t ldt;
    uint16_t *Xc;
    const float *Vw;
    int rw;
    uint64_t seed;
    int blk0;   // first workgroup of this job in the launch (set by launch_tiles)
};

constexpr int kTileRows = 64;

__global__ __launch_bounds__(256) void tile_bf16_kernel(const Batch<TileJob> jb)
{
    // one workgroup per 64-row tile of every job of the batch, jobs one after
    // another along x
    int ji = 0;
    while (ji + 1 < jb.count && static_cast<int>(blockIdx.x) >= jb.j[ji + 1].blk0)
        ++ji;
    const TileJob &J = jb.j[ji];
    const int row0 = (static_cast<int>(blockIdx.x) - J.blk0) * kTileRows;
    if (row0 >= J.rows)
        return;
    // The tile is staged already rounded to bf16 (both copies take bf16 of the
    // same values): 25 KiB, six workgroups per CU.  Staged rows are 97 words
    // apart, so the eight rows a transposed 16-byte store gathers sit in
    // distinct banks.
    constexpr int kPitch = kKMax + 2;
    __shared__ __attribute__((aligned(16))) uint16_t Ts[kTileRows * kPitch];
    const int CP = J.CP;
    // wave w fills rows w, w + 4, ..., its lanes 64 consecutive columns; a
    // lane's 16 values of a column leave memory together (one at a time, each
    // waits for its own load: 13.7 us for the V of an 8B-class layer at rank
    // 64, 7.7 us so)
    const int cl = threadIdx.x & 63, rg = threadIdx.x >> 6;
    constexpr int RPT = kTileRows / 4;
    for (int c = cl; c < CP; c += 64) {
        float v[RPT];
        const float *src = J.X ? J.X : J.Vw && c < J.rw ? J.Vw : nullptr;
        const int64_t ld = J.X ? J.ldx : J.rw;
        if (src && c < J.cols) {
#pragma unroll
            for (int u = 0; u < RPT; ++u)
                v[u] = src[static_cast<int64_t>(min(row0 + rg + 4 * u, J.rows - 1)) * ld + c];
        } else {
#pragma unroll
            for (int u = 0; u < RPT; ++u)
                v[u] = c < J.cols ? start_uniform(J.seed, row0 + rg + 4 * u, c) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < RPT; ++u)
            Ts[(rg + 4 * u) * kPitch + c] = f32_to_bf16(row0 + rg + 4 * u < J.rows ? v[u] : 0.f);
    }
    __syncthreads();
    if (J.Xc) {
        // 32 lanes per row, lane q copies the 16-byte chunk q of the row (CP / 8 <= 24 chunks)
        const int q = threadIdx.x & 31;
        if (q < CP / 8)
            for (int r = threadIdx.x >> 5; r < kTileRows && row0 + r < J.rows; r += 8) {
                const uint32_t *src = reinterpret_cast<const uint32_t *>(&Ts[r * kPitch + 8 * q]);
                *reinterpret_cast<uint4 *>(J.Xc + static_cast<int64_t>(row0 + r) * CP + 8 * q) =
                    make_uint4(src[0], src[1], src[2], src[3]);
            }
    }
    if (J.Xt) {
        for (int idx = threadIdx.x; idx < CP * (kTileRows / 8); idx += 256) {
            const int c = idx / (kTileRows / 8), r8 = (idx % (kTileRows / 8)) * 8;
            if (row0 + r8 >= J.rows)
                continue;
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                w[e] = static_cast<uint32_t>(Ts[(r8 + 2 * e) * kPitch + c]) |
                       (static_cast<uint32_t>(Ts[(r8 + 2 * e + 1) * kPitch + c]) << 16);
            *reinterpret_cast<uint4 *>(J.Xt + static_cast<int64_t>(c) * J.ldt + row0 + r8) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
}

// ---------------------------------------------------------------------------
// Global-norm clipping of the corrected AdamW step without a pass over
// G_proj: with U and V orthonormal, X = U^T G V and X_f = d X d,
//   ||alpha G + (1 - alpha) U X_f V^T||^2
//     = alpha^2 ||G||^2 + 2 alpha (1 - alpha) <X, X_f> + (1 - alpha)^2 ||X_f||^2.
// ||G||^2 is summed by sumsq_kernel (kSumBlocks fp64 partials per matrix, a
// grid and order that never depend on the device), the rest by
// clip_norm_kernel in one workgroup, matrix by matrix in call order.
// ---------------------------------------------------------------------------
constexpr int kSumBlocks = 512;

struct SumJob {
    const void *G;
    int64_t count;    // elements of G (contiguous)
    int vec;          // 16-byte aligned G: 16-byte loads but for the last elements
    int chunk32;      // whole 16-byte chunks only: a chunk's squares are added in fp32
    double *part;     // [kSumBlocks]
};

__device__ __forceinline__ double block_sum(double v, double *red)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w)
            red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    const double t = red[0];
    __syncthreads();
    return t;
}

template <typename GT>
__global__ __launch_bounds__(256) void sumsq_kernel(const Batch<SumJob> jb)
{
    __shared__ double red[256];
    const SumJob &J = jb.j[blockIdx.z];
    const GT *G = static_cast<const GT *>(J.G);
    double acc = 0.0;
    constexpr int V = 16 / sizeof(GT);
    const int64_t stride = static_cast<int64_t>(kSumBlocks) * 256;
    const int64_t start = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (J.vec) {
        // squares of bf16 are exact in fp32; with chunk32 the V of one chunk are
        // added in fp32, otherwise every square is formed and added in fp64
        for (int64_t c = start; c < J.count / V; c += stride) {
            const uint4 raw = reinterpret_cast<const uint4 *>(G)[c];
            GT e[V];
            __builtin_memcpy(e, &raw, sizeof(e));
            if (J.chunk32) {
                float s = 0.f;
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float g = to_f32<GT>(e[i]);
                    s += g * g;
                }
                acc += s;
            } else {
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const double g = to_f32<GT>(e[i]);
                    acc += g * g;
                }
            }
        }
        const int64_t i = J.count / V * V + start;
        if (i < J.count) {
            const double g = to_f32<GT>(G[i]);
            acc += g * g;
        }
    } else {
        for (int64_t i = start; i < J.count; i += stride) {
            const double g = to_f32<GT>(G[i]);
            acc += g * g;
        }
    }
    const double t = block_sum(acc, red);
    if (threadIdx.x == 0)
        J.part[blockIdx.x] = t;
}

constexpr int kTermBlocks = 16;   // partial terms per matrix
static_assert(kSumBlocks % kTermBlocks == 0, "term slices");

struct NormJob {
    const double *part;   // ||G||^2 partials [kSumBlocks]
    const float *X;       // [r, RP]
    const float *Xf;      // [RP, RP] (rows >= r are zero)
    int r, RP;
    double *terms;        // [kTermBlocks]
};

// Block b of matrix z: its share of alpha^2 ||G||^2 + 2 alpha (1 - alpha)
// <X, X_f> + (1 - alpha)^2 ||X_f||^2, from fixed slices (grid kTermBlocks).
__global__ __launch_bounds__(256) void norm_terms_kernel(const Batch<NormJob> jb, float alpha)
{
    __shared__ double red[256];
    const NormJob &J = jb.j[blockIdx.z];
    const int b = blockIdx.x;
    const double a = alpha, c = 1.0 - static_cast<double>(alpha);
    double gg = 0.0, xx = 0.0, ff = 0.0;
    constexpr int PB = kSumBlocks / kTermBlocks;
    for (int p = threadIdx.x; p < PB; p += 256)
        gg += J.part[b * PB + p];
    const int n = J.r * J.RP;
    const int per = (n + kTermBlocks - 1) / kTermBlocks;
    const int q0 = b * per, q1 = min(n, q0 + per);
    for (int q = q0 + static_cast<int>(threadIdx.x); q < q1; q += 256) {
        const double x = J.X[q], f = J.Xf[q];
        xx += x * f;
        ff += f * f;
    }
    const double t = block_sum(a * a * gg + 2.0 * a * c * xx + c * c * ff, red);
    if (threadIdx.x == 0)
        J.terms[b] = t;
}

// One workgroup.  acc (fp64) carries the squared norm over the launches of
// one call (first: start at zero; last: write the clip coefficient and the
// norm).  Terms are added matrix by matrix in call order.
__global__ __launch_bounds__(64) void clip_norm_kernel(const Batch<NormJob> jb, float max_norm, double *acc,
                                                       float *coef, float *norm_out, int first, int last)
{
    if (threadIdx.x != 0)
        return;
    double total = first ? 0.0 : *acc;
    for (int i = 0; i < jb.count; ++i)
        for (int b = 0; b < kTermBlocks; ++b)
            total += jb.j[i].terms[b];
    *acc = total;
    if (last) {
        const double N = sqrt(total > 0.0 ? total : 0.0);
        float c = 1.0f;
        if (max_norm > 0.f) {
            const double q = static_cast<double>(max_norm) / (N + 1e-6);
            if (q < 1.0)
                c = static_cast<float>(q);
        }
        *coef = c;
        if (norm_out)
            *norm_out = static_cast<float>(N);
    }
}

// Vc[i][c] = V[i][c] for c < r, zero up to RP, converted to the compute type.
template <typename CT>
struct PadJob {
    const float *V;
    int n;
    CT *Vc;
};

template <typename CT>
__global__ __launch_bounds__(256) void pad_convert_kernel(const Batch<PadJob<CT>> jb, int r, int RP)
{
    const float *V = jb.j[blockIdx.z].V;
    const int n = jb.j[blockIdx.z].n;
    CT *Vc = jb.j[blockIdx.z].Vc;
    const int64_t total = static_cast<int64_t>(n) * RP;
    for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < total;
         idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t i = idx / RP;
        const int c = static_cast<int>(idx - i * RP);
        Vc[idx] = from_f32<CT>(c < r ? V[i * r + c] : 0.f);
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
struct Carve {
    char *base;
    size_t off = 0;
    explicit Carve(void *b) : base(static_cast<char *>(b)) {}
    template <typename T>
    T *take(size_t count)
    {
        off = static_cast<size_t>(round_up(static_cast<int64_t>(off), 256));
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

// Most k pieces of an fp32 product with M rows (two 64-row workgroups per CU,
// 256 deep at least): what the workspaces have room for.
int split_count(int64_t Mdim, int64_t Kdim)
{
    const int64_t mb = cdiv(Mdim, 64);
    int64_t s = cdiv(512, mb);
    s = std::min<int64_t>(s, std::max<int64_t>(1, Kdim / 256));
    return static_cast<int>(std::max<int64_t>(1, s));
}

// Most Gram partial blocks a matrix of this many rows may be split into.
int gram_blocks_max(int64_t rows) { return static_cast<int>(std::min<int64_t>(128, cdiv(rows, kGRows))); }

struct Dims {
    int m, n, r, k, KP, RP;
};

Dims dims_of(int m, int n, int r, int oversample)
{
    Dims d;
    d.m = m;
    d.n = n;
    d.r = r;
    d.k = std::min(std::min(r + oversample, std::min(m, n)), kKMax);
    d.KP = static_cast<int>(round_up(d.k, 16));
    d.RP = static_cast<int>(round_up(r, 32));
    return d;
}

// Buffers of sc_build_prior (carved in this order).
struct PriorWs {
    int *info;   // status words (kInfo*): Jacobi sweeps, residual, tolerance, status, phase stamp
    float *Y, *Z, *part, *T, *Bu, *Bv;
    double *gpart, *gram;
    uint16_t *M16, *Yt16, *Zt16;   // bf16 path: shadow of M (64 x 64 tiles), transposed thin factors
    int64_t ntc16, ldy16, ldz16;
};

size_t carve_prior(const Dims &d, bool use16, void *base, PriorWs *w)
{
    Carve c(base);
    const int64_t mx = std::max(d.m, d.n);
    int64_t s1 = split_count(d.m, d.n), s2 = split_count(d.n, d.m);
    if (use16) {
        s1 = std::max<int64_t>(s1, pass::max_splits(d.m, d.n));
        s2 = std::max<int64_t>(s2, pass::max_splits(d.n, d.m));
    }
    const int64_t part = std::max<int64_t>(s1 * d.m, s2 * d.n) * d.KP;
    PriorWs t;
    t.info = c.take<int>(64);
    t.ntc16 = pass::tiles_per_row(d.n);
    t.ldy16 = round_up(d.m, 8);
    t.ldz16 = round_up(d.n, 8);
    t.M16 = use16 ? c.take<uint16_t>(static_cast<size_t>(pass::tiled_elems(d.m, d.n))) : nullptr;
    t.Yt16 = use16 ? c.take<uint16_t>(static_cast<size_t>(d.KP) * t.ldy16) : nullptr;
    t.Zt16 = use16 ? c.take<uint16_t>(static_cast<size_t>(d.KP) * t.ldz16) : nullptr;
    t.Y = c.take<float>(static_cast<size_t>(d.m) * d.KP);
    t.Z = c.take<float>(static_cast<size_t>(d.n) * d.KP);
    t.part = c.take<float>(static_cast<size_t>(part));
    t.T = c.take<float>(static_cast<size_t>(d.KP) * d.KP);
    t.Bu = c.take<float>(static_cast<size_t>(d.KP) * d.RP);
    t.Bv = c.take<float>(static_cast<size_t>(d.KP) * d.RP);
    t.gpart = c.take<double>(static_cast<size_t>(gram_blocks_max(mx)) * d.KP * d.KP);
    t.gram = c.take<double>(static_cast<size_t>(d.KP) * d.KP);
    if (w)
        *w = t;
    return c.off;
}

// Buffers of sc_correct.
struct CorrWs {
    float *Tm, *part, *xpart, *X, *Xf;
    void *Pc, *Vc;
    uint16_t *Vt16;
    int64_t ldv16;
    double *sq, *terms, *acc;
    float *coef;
};

size_t carve_correct(const Dims &d, size_t esize, void *base, CorrWs *w)
{
    Carve c(base);
    const int s1 = std::max(split_count(d.m, d.n), esize == 2 ? pass::max_splits(d.m, d.n) : 1);
    const int s2 = split_count(d.r, d.m);
    CorrWs t;
    t.ldv16 = round_up(d.n, 8);
    t.Vt16 = esize == 2 ? c.take<uint16_t>(static_cast<size_t>(d.RP) * t.ldv16) : nullptr;
    t.Tm = c.take<float>(static_cast<size_t>(d.m) * d.RP);
    t.part = c.take<float>(static_cast<size_t>(s1) * d.m * d.RP);
    t.xpart = c.take<float>(static_cast<size_t>(s2) * d.r * d.RP);
    t.X = c.take<float>(static_cast<size_t>(d.r) * d.RP);
    t.Xf = c.take<float>(static_cast<size_t>(d.RP) * d.RP);
    t.Pc = c.take<unsigned char>(static_cast<size_t>(d.m) * d.RP * esize);
    t.Vc = c.take<unsigned char>(static_cast<size_t>(d.n) * d.RP * esize);
    // corrected AdamW: ||G||^2 partials, the norm accumulator, the clip coefficient
    t.sq = c.take<double>(kSumBlocks);
    t.terms = c.take<double>(kTermBlocks);
    t.acc = c.take<double>(1);
    t.coef = c.take<float>(1);
    if (w)
        *w = t;
    return c.off;
}

unsigned grid1d(int64_t total, int per = 256)
{
    return static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(cdiv(total, per), 65536)));
}

// Enqueue `kernel` over `jobs`, kMaxBatch jobs per launch (grid.z = job).
template <class Job, class K, class... Args>
void launch_jobs(const char *tag, K kernel, const std::vector<Job> &jobs, dim3 grid, dim3 block, size_t lds,
                 hipStream_t st, Args... args)
{
    for (size_t c0 = 0; c0 < jobs.size(); c0 += kMaxBatch) {
        Batch<Job> b{};
        b.count = static_cast<int>(std::min<size_t>(kMaxBatch, jobs.size() - c0));
        for (int i = 0; i < b.count; ++i)
            b.j[i] = jobs[c0 + i];
        ACSC_LAUNCH(tag, kernel, dim3(grid.x, grid.y, b.count), block, lds, st, b, args...);
    }
}

// tile_bf16_kernel over a list of jobs: each launch takes up to kMaxBatch jobs
// and exactly as many workgroups as they have 64-row tiles.
void launch_tiles(const char *tag, std::vector<TileJob> jobs, hipStream_t st)
{
    for (size_t c0 = 0; c0 < jobs.size(); c0 += kMaxBatch) {
        Batch<TileJob> b{};
        b.count = static_cast<int>(std::min<size_t>(kMaxBatch, jobs.size() - c0));
        int blocks = 0;
        for (int i = 0; i < b.count; ++i) {
            b.j[i] = jobs[c0 + i];
            b.j[i].blk0 = blocks;
            blocks += static_cast<int>(cdiv(b.j[i].rows, kTileRows));
        }
        if (blocks > 0)
            ACSC_LAUNCH(tag, tile_bf16_kernel, dim3(blocks), dim3(256), 0, st, b);
    }
}

using JacobiF64 = void (*)(const Batch<JacJob>, int, int, int, int, float, double, int);
using JacobiF32 = void (*)(const Batch<JacJob>, int, int, int, int, float, float, int);

// fp64, k <= kJacobiF64MaxK: rows per lane of a row of 16
JacobiF64 jacobi_f64(int k)
{
    switch ((k + 15) / 16) {
    case 1: return jacobi_blocks_kernel<1>;
    case 2: return jacobi_blocks_kernel<2>;
    case 3: return jacobi_blocks_kernel<3>;
    case 4: return jacobi_blocks_kernel<4>;
    case 5: return jacobi_blocks_kernel<5>;
    case 6: return jacobi_blocks_kernel<6>;
    case 7: return jacobi_blocks_kernel<7>;
    default: return jacobi_blocks_kernel<8>;
    }
}

// fp32, beyond: rows per lane of a group of 8 (a multiple of 4)
JacobiF32 jacobi_f32(int k) { return k <= 160 ? jacobi_pairs_kernel<20> : jacobi_pairs_kernel<24>; }

// fp64: one row of 16 lanes per pair of blocks (16 pairs at most); four waves,
// for what is not rounds.  fp32: one 8-lane group per column pair of a round.
unsigned jacobi_threads(int k)
{
    static_assert(kJacobiF64MaxK / kJacBlk / 2 * 16 <= 256, "a row of lanes per pair of blocks");
    return k <= kJacobiF64MaxK ? 256u : 64u * static_cast<unsigned>(std::min<int64_t>(16, cdiv((k + 1) / 2, 8)));
}

// fp64: every block's columns, padded to 16 rows, and each column's squared
// norm, scale and reciprocal scale; fp32: columns padded to 32 rows, and the
// squared norms
size_t jacobi_lds(int k)
{
    return k <= kJacobiF64MaxK ? static_cast<size_t>(jacobi_blocks(k) * kJacBlk) * (jacobi_pitch_f64(round_up(k, 16)) + 3) *
                                     sizeof(double)
                               : static_cast<size_t>(k) * (round_up(k, 32) + 1) * sizeof(float);
}

int jacobi_prepare(int k)
{
    return k <= kJacobiF64MaxK ? allow_lds(jacobi_f64(k), jacobi_lds(k)) : allow_lds(jacobi_f32(k), jacobi_lds(k));
}

// Per-matrix state of a batched call.
struct Mat {
    const sc_matrix *in;
    Dims D;
    PriorWs pw;
    CorrWs cw;
    uint64_t seed;
    const sc_adamw_state *ad = nullptr;   // corrected AdamW: this matrix's optimiser state
    float *q32 = nullptr;                 // PowerSGD: the final basis goes here (r columns) and not over Y
};

// Corrected AdamW: the epilogue constants and the call's norm accumulator.
struct AdamCtx {
    blend::AdamArgs args;   // args.coef: the clip coefficient (workspace of the call's first matrix)
    double *acc;            // squared-norm accumulator (same workspace)
    float max_norm;
    float *norm_out;        // device or NULL
};

template <int NB>
void gram_launch_nb(bool parts, const std::vector<GramJob> &gj, dim3 grid, int KP, hipStream_t st)
{
    if (parts)
        launch_jobs("sc_gram", gram_partial_kernel<NB, true>, gj, grid, dim3(64 * kGWaves), 0, st, KP);
    else
        launch_jobs("sc_gram", gram_partial_kernel<NB, false>, gj, grid, dim3(64 * kGWaves), 0, st, KP);
}

void gram_launch(int nt, bool parts, const std::vector<GramJob> &gj, dim3 grid, int KP, hipStream_t st)
{
    switch (nt) {
    case 1: gram_launch_nb<1>(parts, gj, grid, KP, st); break;
    case 2: gram_launch_nb<2>(parts, gj, grid, KP, st); break;
    case 3: gram_launch_nb<3>(parts, gj, grid, KP, st); break;
    case 4: gram_launch_nb<4>(parts, gj, grid, KP, st); break;
    case 5: gram_launch_nb<5>(parts, gj, grid, KP, st); break;
    case 6: gram_launch_nb<6>(parts, gj, grid, KP, st); break;
    case 7: gram_launch_nb<7>(parts, gj, grid, KP, st); break;
    case 8: gram_launch_nb<8>(parts, gj, grid, KP, st); break;
    case 9: gram_launch_nb<9>(parts, gj, grid, KP, st); break;
    case 10: gram_launch_nb<10>(parts, gj, grid, KP, st); break;
    case 11: gram_launch_nb<11>(parts, gj, grid, KP, st); break;
    default: gram_launch_nb<12>(parts, gj, grid, KP, st); break;
    }
}

// Gram matrices (fp64) of the first KP columns of one block per matrix.
// `splits`: the partials (in pw.part) that each block still lies in, or 1.
// Returns the partials per matrix that are left for the factorisation to add
// (see chol::adds_partials), or zeros with pw.gram formed.
std::vector<int> gram(const std::vector<Mat> &ms, const std::vector<float *> &A, const std::vector<int> &rows,
          const std::vector<int> &splits, hipStream_t st)
{
    const int KP = ms[0].D.KP;
    const int nt = static_cast<int>(cdiv(KP, kGT));
    std::vector<GramJob> gj;
    std::vector<GramRedJob> rj;
    int gy = 1;
    // one row count per block across the batch, so that the blocks of all
    // matrices (one workgroup each) come to at most two per CU
    int64_t total = 0;
    for (int r : rows)
        total += r;
    auto rpb_of = [&](size_t i, int64_t rpb_batch) {
        return std::max<int64_t>(rpb_batch, round_up(cdiv(rows[i], gram_blocks_max(rows[i])), kGRows));
    };
    int64_t rpb_batch = round_up(std::max<int64_t>(1, cdiv(total, 512)), kGRows);
    for (;;) {
        int64_t nb = 0;
        for (size_t i = 0; i < ms.size(); ++i)
            nb += cdiv(rows[i], rpb_of(i, rpb_batch));
        if (nb <= 512 || rpb_batch >= total)
            break;
        rpb_batch += kGRows;
    }
    for (size_t i = 0; i < ms.size(); ++i) {
        const int rpb = static_cast<int>(rpb_of(i, rpb_batch));
        const int gb = static_cast<int>(cdiv(rows[i], rpb));
        gj.push_back(GramJob{A[i], KP, rows[i], rpb, gb, ms[i].pw.gpart, ms[i].pw.part, splits[i]});
        rj.push_back(GramRedJob{ms[i].pw.gpart, gb, ms[i].pw.gram});
        gy = std::max(gy, gb);
    }
    bool parts = false;
    for (int sp : splits)
        parts = parts || sp > 1;
    for (size_t i = 0; i < ms.size() && parts; ++i)
        if (splits[i] <= 1)
            gj[i].src = A[i];   // a whole product among cut ones: one "partial", added to nothing
    gram_launch(nt, parts, gj, dim3(gy), KP, st);
    std::vector<int> left;
    int most = 0;
    for (const GramJob &j : gj) {
        left.push_back(j.blocks);
        most = std::max(most, j.blocks);
    }
    if (chol::adds_partials(KP, most))
        return left;
    launch_jobs("sc_gram_reduce", gram_reduce_kernel, rj, dim3(static_cast<unsigned>(cdiv(int64_t(KP) * KP, 32))),
                dim3(256), 0, st, KP);
    return std::vector<int>(ms.size(), 0);
}

// Q <- Y L^{-T}, `passes` times (CholeskyQR; two passes = CholeskyQR2), for
// one block Y [rows, KP] per matrix (first k columns live; `which` selects
// the Y or the Z block).  The Gram matrix is accumulated in fp64 from the
// fp32 block, so one pass already leaves the columns orthonormal to about
// 1e-7 * cond(Y); the iteration only needs a well-conditioned basis, and the
// final basis gets the second pass.  The last pass also writes the bf16
// transposed copy that the next streaming pass reads.
// `splits`: as for gram().  `last`: this is the last basis of a subspace phase,
// whose kernel also stamps the workspace.
int orthonormalise(std::vector<Mat> &ms, bool onY, int passes, bool use16, std::vector<int> splits, bool last,
                   hipStream_t st)
{
    const Dims &d0 = ms[0].D;
    std::vector<float *> A;
    std::vector<int> rows;
    for (auto &m : ms) {
        A.push_back(onY ? m.pw.Y : m.pw.Z);
        rows.push_back(onY ? m.D.m : m.D.n);
    }
    for (int pass = 0; pass < passes; ++pass) {
        const std::vector<int> left = gram(ms, A, rows, splits, st);
        splits.assign(ms.size(), 1);   // added up by the Gram kernel
        std::vector<chol::Req> cj;
        for (size_t i = 0; i < ms.size(); ++i)
            cj.push_back(chol::Req{ms[i].pw.gram, ms[i].pw.T, ms[i].pw.gpart, left[i]});
        if (int rc = chol::run("sc_chol_inv", cj, d0.k, d0.KP, true, st))
            return rc;
        // fp32 Q is read by the second Gram of CholeskyQR2 and by the final
        // basis; otherwise (bf16 passes) only its bf16 transposed copy is
        std::vector<orth::Req> g;
        for (size_t i = 0; i < ms.size(); ++i) {
            float *Y = A[i];
            uint16_t *t16 = (use16 && pass + 1 == passes) ? (onY ? ms[i].pw.Yt16 : ms[i].pw.Zt16) : nullptr;
            const int64_t ldt = onY ? ms[i].pw.ldy16 : ms[i].pw.ldz16;
            float *out = pass + 1 == passes ? ms[i].q32 : nullptr;
            g.push_back(orth::Req{Y, rows[i], ms[i].pw.T, t16, ldt, !use16 || passes == 2, out, ms[i].D.r, ms[i].D.r,
                                  last && pass + 1 == passes ? ms[i].pw.info : nullptr});
        }
        if (int rc = orth::run("sc_orth_apply", g, d0.KP, st))
            return rc;
    }
    return ACSC_OK;
}

// EMA + top-r SVD + filter for a group of matrices with the same k.
// Phases of the build: the subspace iteration (EMA, power passes, the final
// Z = M^T Q) and the Rayleigh-Ritz step on Z (Gram, Cholesky, Jacobi, basis,
// filter).  The second reads only what the first left in the workspace.
constexpr int kPhaseSubspace = 1, kPhaseRitz = 2;

int build_group(std::vector<Mat> &ms, acsc_dtype dt, float beta, int r, int power_iters, float tau,
                int phases, hipStream_t st)
{
    const Dims &d0 = ms[0].D;
    const int k = d0.k, KP = d0.KP, RP = d0.RP;
    const bool use16 = dt == ACSC_BF16;
    const float omb = 1.0f - beta;
    // with a bf16 shadow and a large enough batch, the EMA runs fused with the
    // first pass Y = M16 Z (after the starting block exists)
    std::vector<pass::EmaReq> er;
    for (auto &m : ms)
        er.push_back(pass::EmaReq{m.in->M, static_cast<const uint16_t *>(m.in->G), m.pw.M16, m.pw.Zt16, m.pw.ldz16,
                                  m.pw.Y, KP, m.D.m, m.D.n, KP, m.pw.part, m.pw.info + kInfoStall});
    const bool fused = use16 && pass::ema_fusable(er);
    if ((phases & kPhaseSubspace) && !fused) {
        if (use16) {
            std::vector<EmaJob> j;
            int64_t tot = 1;
            for (auto &m : ms) {
                j.push_back(EmaJob{m.in->M, static_cast<const uint16_t *>(m.in->G), m.D.m, m.D.n,
                                             (m.D.n % 8) == 0 ? 1 : 0, m.pw.M16, m.pw.ntc16});
                tot = std::max<int64_t>(tot, static_cast<int64_t>(m.D.m) * cdiv(m.D.n, 8));
            }
            launch_jobs("sc_ema", ema_shadow_kernel, j, dim3(grid1d(tot)), dim3(256), 0, st, beta, omb);
        } else {
            std::vector<Ema32Job> j;
            int64_t tot = 1;
            for (auto &m : ms) {
                const int64_t c = static_cast<int64_t>(m.D.m) * m.D.n;
                j.push_back(Ema32Job{m.in->M, static_cast<const float *>(m.in->G), c});
                tot = std::max(tot, cdiv(c, 4));
            }
            bool any = false;
            for (auto &m : ms)
                any = any || m.in->G;
            if (any)
                launch_jobs("sc_ema", ema_kernel, j, dim3(grid1d(tot)), dim3(256), 0, st, beta, omb);
        }
    }
    if (phases & kPhaseSubspace) {
        std::vector<InitJob> j;
        int64_t tot = 1;
        for (auto &m : ms) {
            j.push_back(InitJob{m.pw.Z, m.D.n, m.in->V_warm, m.seed});
            tot = std::max<int64_t>(tot, static_cast<int64_t>(m.D.n) * KP);
        }
        if (use16) {
            // the bf16 passes read only the transposed copy of the starting block
            std::vector<TileJob> tj;
            for (auto &m : ms)
                tj.push_back(TileJob{nullptr, 0, m.D.n, k, KP, m.pw.Zt16, m.pw.ldz16, nullptr, m.in->V_warm,
                                     m.in->V_warm ? r : 0, m.seed});
            launch_tiles("sc_init", tj, st);
        } else {
            launch_jobs("sc_init", init_block_kernel, j, dim3(grid1d(tot)), dim3(256), 0, st, k, KP, r);
        }
    }
    // one pass Y = M Z  /  Z = M^T Y over every EMA (bf16 shadow on matrix cores, or fp32);
    // `splits` takes the partials that the products are left in
    auto reqs16 = [&](bool mz) {
        std::vector<pass::Req> q;
        for (auto &m : ms) {
            if (mz)
                q.push_back(pass::Req{m.pw.M16, 0, true, m.pw.Zt16, m.pw.ldz16, m.pw.Y, KP, m.D.m, m.D.n,
                                    KP, m.pw.part, static_cast<int>(m.pw.ntc16)});
            else
                q.push_back(pass::Req{m.pw.M16, 0, true, m.pw.Yt16, m.pw.ldy16, m.pw.Z, KP, m.D.n, m.D.m,
                                    KP, m.pw.part, static_cast<int>(m.pw.ntc16)});
        }
        return q;
    };
    auto reqs32 = [&](bool mz) {
        std::vector<f32::PassReq> q;
        for (auto &m : ms) {
            const int M = mz ? m.D.m : m.D.n, K = mz ? m.D.n : m.D.m;
            q.push_back(f32::PassReq{m.in->M, m.D.n, mz ? m.pw.Z : m.pw.Y, KP, mz ? m.pw.Y : m.pw.Z, KP, M, K, k, KP,
                                     m.pw.part, split_count(M, K)});
        }
        return q;
    };
    std::vector<int> splits(ms.size(), 1);
    auto pass = [&](bool mz, bool whole = false) {
        const char *tag = mz ? "sc_pass_mz" : "sc_pass_mtq";
        int *left = whole ? nullptr : splits.data();
        return use16 ? pass::run(tag, !mz, reqs16(mz), st, left) : f32::pass(tag, !mz, reqs32(mz), st, left);
    };
    int rc = ACSC_OK;
    if (phases & kPhaseSubspace) {
        rc = fused ? pass::ema_run("sc_ema", er, beta, omb, st) : pass(true);
        if (rc)
            return rc;
        if ((rc = orthonormalise(ms, true, power_iters == 0 ? 2 : 1, use16, splits, power_iters == 0, st)))
            return rc;
        for (int it = 0; it < power_iters; ++it) {
            if ((rc = pass(false)))
                return rc;
            if ((rc = orthonormalise(ms, false, 1, use16, splits, false, st)))
                return rc;
            if ((rc = pass(true)))
                return rc;
            if ((rc = orthonormalise(ms, true, it + 1 == power_iters ? 2 : 1, use16, splits, it + 1 == power_iters, st)))
                return rc;
        }
        // Z = M^T Q (= B^T) for the Rayleigh-Ritz step: B B^T = Z^T Z = L L^T, SVD of L by Jacobi.
        // A subspace call of its own leaves Z whole: how a product is cut
        // depends on its batch, and the Rayleigh-Ritz call may come in another one.
        const bool whole = !(phases & kPhaseRitz);
        if ((rc = pass(false, whole)))
            return rc;
    }
    if (!(phases & kPhaseRitz))
        return ACSC_OK;
    {
        std::vector<float *> A;
        std::vector<int> rows;
        std::vector<chol::Req> cj;
        std::vector<JacJob> jj;
        for (auto &m : ms) {
            A.push_back(m.pw.Z);
            rows.push_back(m.D.n);
            jj.push_back(JacJob{m.pw.gram, m.pw.Bu, m.pw.Bv, m.in->s, m.in->d, m.pw.info});
        }
        const std::vector<int> left = gram(ms, A, rows, splits, st);
        for (size_t i = 0; i < ms.size(); ++i)
            cj.push_back(chol::Req{ms[i].pw.gram, nullptr, ms[i].pw.gpart, left[i]});
        if ((rc = chol::run("sc_chol", cj, k, KP, false, st)))
            return rc;
        // the sweep cap can be lowered (not raised) through the environment, so
        // that the non-convergence report can be exercised
        int max_sweeps = kJacobiMaxSweeps;
        if (const char *e = std::getenv("ACSC_JACOBI_MAX_SWEEPS"))
            max_sweeps = std::max(1, std::min(kJacobiMaxSweeps, std::atoi(e)));
        if (k <= kJacobiF64MaxK)
            launch_jobs("sc_jacobi", jacobi_f64(k), jj, dim3(1), dim3(jacobi_threads(k)), jacobi_lds(k), st, k, KP, r,
                        RP, tau, 1e-13, max_sweeps);
        else
            launch_jobs("sc_jacobi", jacobi_f32(k), jj, dim3(1), dim3(jacobi_threads(k)), jacobi_lds(k), st, k, KP, r,
                        RP, tau, 1e-5f, max_sweeps);
    }
    // U = Q Bu, V = Z Bv (first r columns)
    std::vector<orth::GemmReq> og;
    for (auto &m : ms) {
        og.push_back(orth::GemmReq{m.pw.Y, KP, m.D.m, KP, m.pw.Bu, RP, RP, m.in->U, nullptr, r, r});
        og.push_back(orth::GemmReq{m.pw.Z, KP, m.D.n, KP, m.pw.Bv, RP, RP, m.in->V, nullptr, r, r});
    }
    return orth::gemm("sc_basis", og, st);
}

// Squared global norm of the call's G_proj and the clip coefficient (see
// clip_norm_kernel), from ||G||^2 and the filtered projections X, X_f.
template <typename GT>
void clip_norm(const std::vector<Mat> &ms, int r, float alpha, const AdamCtx &ad, hipStream_t st)
{
    std::vector<SumJob> sj;
    for (const Mat &m : ms) {
        const int64_t cnt = static_cast<int64_t>(m.D.m) * m.D.n;
        sj.push_back(SumJob{m.in->G, cnt, aligned(m.in->G, 16) ? 1 : 0,
                            cnt % static_cast<int64_t>(16 / sizeof(GT)) == 0 ? 1 : 0, m.cw.sq});
    }
    launch_jobs("sc_sumsq", sumsq_kernel<GT>, sj, dim3(kSumBlocks), dim3(256), 0, st);
    for (size_t c0 = 0; c0 < ms.size(); c0 += kMaxBatch) {
        Batch<NormJob> b{};
        b.count = static_cast<int>(std::min<size_t>(kMaxBatch, ms.size() - c0));
        for (int i = 0; i < b.count; ++i) {
            const Mat &m = ms[c0 + i];
            b.j[i] = NormJob{m.cw.sq, m.cw.X, m.cw.Xf, r, m.D.RP, m.cw.terms};
        }
        const int first = c0 == 0, last = c0 + b.count == ms.size();
        ACSC_LAUNCH("sc_norm_terms", norm_terms_kernel, dim3(kTermBlocks, 1, b.count), dim3(256), 0, st, b, alpha);
        ACSC_LAUNCH("sc_clip_norm", clip_norm_kernel, dim3(1), dim3(64), 0, st, b, ad.max_norm, ad.acc,
                    const_cast<float *>(ad.args.coef), ad.norm_out, first, last);
    }
}

// X = U^T G V, X_f = d X d, P = U X_f, then G_proj = alpha G + (1 - alpha) P V^T,
// stored, or (adam) taken as the gradient of the AdamW step of each matrix.
template <typename GT>
int correct_group(std::vector<Mat> &ms, int r, float alpha, hipStream_t st, const AdamCtx *adam = nullptr)
{
    const int RP = ms[0].D.RP;
    const bool b16 = sizeof(GT) == 2;
    // T = G V   [m, RP]
    if (b16) {
        // V to bf16 once: transposed for T = G V, row-major for the blend
        std::vector<TileJob> t;
        std::vector<pass::Req> q;
        for (auto &m : ms) {
            t.push_back(TileJob{m.in->V, r, m.D.n, r, RP, m.cw.Vt16, m.cw.ldv16, static_cast<uint16_t *>(m.cw.Vc),
                                nullptr, 0, 0});
            const bool avec = aligned(m.in->G, 16) && (m.D.n % 8) == 0;
            q.push_back(pass::Req{static_cast<const uint16_t *>(m.in->G), m.D.n, avec, m.cw.Vt16, m.cw.ldv16, m.cw.Tm,
                                RP, m.D.m, m.D.n, RP, m.cw.part});
        }
        launch_tiles("sc_vconvert", t, st);
        const int rc = pass::run("sc_gv", false, q, st, nullptr, "sc_gv_reduce");
        if (rc)
            return rc;
    } else {
        std::vector<f32::PassReq> q;
        for (auto &m : ms)
            q.push_back(f32::PassReq{static_cast<const float *>(static_cast<const void *>(m.in->G)), m.D.n, m.in->V, r,
                                     m.cw.Tm, RP, m.D.m, m.D.n, r, RP, m.cw.part, split_count(m.D.m, m.D.n)});
        if (int rc = f32::pass("sc_gv", false, q, st, nullptr, "sc_gv_reduce"))
            return rc;
    }
    // X = U^T T   [r, RP], and X_f = d X d   [RP, RP], zero-padded
    {
        std::vector<orth::InnerReq> iq;
        for (auto &m : ms)
            iq.push_back(orth::InnerReq{m.in->U, r, m.cw.Tm, RP, m.D.m, r, RP, m.cw.X, RP, m.cw.xpart,
                                        split_count(m.D.r, m.D.m), m.in->d, m.cw.Xf});
        if (int rc = orth::inner("sc_utt", iq, st))
            return rc;
    }
    // P = U X_f  [m, RP] in the compute type; V in the compute type [n, RP]
    {
        std::vector<PadJob<GT>> pj;
        std::vector<orth::GemmReq> og;
        int64_t tot = 1;
        for (auto &m : ms) {
            pj.push_back(PadJob<GT>{m.in->V, m.D.n, static_cast<GT *>(m.cw.Vc)});
            tot = std::max<int64_t>(tot, static_cast<int64_t>(m.D.n) * RP);
            og.push_back(orth::GemmReq{m.in->U, r, m.D.m, r, m.cw.Xf, RP, RP,
                                       b16 ? nullptr : static_cast<float *>(m.cw.Pc),
                                       b16 ? static_cast<uint16_t *>(m.cw.Pc) : nullptr, RP, RP});
        }
        if (int rc = orth::gemm("sc_ux", og, st))
            return rc;
        if (!b16)   // the bf16 copy was made with the transposed one
            launch_jobs("sc_vconvert", pad_convert_kernel<GT>, pj, dim3(grid1d(tot)), dim3(256), 0, st, r, RP);
    }
    if (adam)
        clip_norm<GT>(ms, r, alpha, *adam, st);
    const blend::AdamArgs ad = adam ? adam->args : blend::AdamArgs{};
    const char *btag = adam ? "sc_blend_adamw" : "sc_blend";
    {
        if constexpr (sizeof(GT) == 2) {
            std::vector<blend::Req> q;
            for (auto &m : ms)
                q.push_back(blend::Req{static_cast<const uint16_t *>(m.in->G), static_cast<uint16_t *>(m.in->G_proj),
                                       m.D.m, m.D.n, static_cast<const uint16_t *>(m.cw.Pc),
                                       static_cast<const uint16_t *>(m.cw.Vc), m.ad ? m.ad->W : nullptr,
                                       m.ad ? m.ad->m1 : nullptr, m.ad ? m.ad->m2 : nullptr, nullptr});
            return blend::run(btag, q, RP, alpha, st, adam ? &ad : nullptr);
        } else {
            std::vector<f32::BlendReq> q;
            for (auto &m : ms)
                q.push_back(f32::BlendReq{static_cast<const float *>(static_cast<const void *>(m.in->G)),
                                          static_cast<float *>(m.in->G_proj), m.D.m, m.D.n,
                                          static_cast<const float *>(m.cw.Pc), static_cast<const float *>(m.cw.Vc),
                                          m.ad ? m.ad->W : nullptr, m.ad ? m.ad->m1 : nullptr,
                                          m.ad ? m.ad->m2 : nullptr, nullptr});
            return f32::blend(btag, q, RP, alpha, st, adam ? &ad : nullptr, false);
        }
    }
    return ACSC_OK;
}

int check_matrix(const sc_matrix &a, int r, int oversample, acsc_dtype dt, bool build, size_t *need,
                 bool need_gproj = true)
{
    ACSC_CHECK_ARG(a.m >= 1 && a.n >= 1, ACSC_EINVAL, "m=%d, n=%d must be >= 1", a.m, a.n);
    ACSC_CHECK_ARG(r >= 1 && r <= std::min(std::min(a.m, a.n), kKMax), ACSC_EINVAL,
                   "r=%d outside [1, min(m, n, %d)] for a %d x %d matrix", r, kKMax, a.m, a.n);
    const Dims d = dims_of(a.m, a.n, r, oversample);
    *need = build ? carve_prior(d, dt == ACSC_BF16, nullptr, nullptr) : carve_correct(d, dtype_size(dt), nullptr, nullptr);
    ACSC_CHECK_ARG(a.ws != nullptr && a.U && a.s && a.V && a.d, ACSC_EINVAL, "null pointer argument");
    ACSC_CHECK_ARG(a.ws_bytes >= *need, ACSC_ENOSPC, "workspace %zu bytes < %zu needed", a.ws_bytes, *need);
    ACSC_CHECK_ARG(aligned(a.ws, 256), ACSC_EALIGN, "workspace must be 256-byte aligned");
    ACSC_CHECK_ARG(aligned(a.U, 4) && aligned(a.V, 4) && aligned(a.s, 4) && aligned(a.d, 4), ACSC_EALIGN,
                   "U, s, V, d must be 4-byte aligned");
    const size_t es = dtype_size(dt);
    if (build) {
        ACSC_CHECK_ARG(a.M != nullptr, ACSC_EINVAL, "M is NULL");
        ACSC_CHECK_ARG(aligned(a.M, 16), ACSC_EALIGN, "M must be 16-byte aligned");
        ACSC_CHECK_ARG(!a.G || aligned(a.G, 16), ACSC_EALIGN, "G_anc must be 16-byte aligned");
    } else {
        ACSC_CHECK_ARG(a.G && (a.G_proj || !need_gproj), ACSC_EINVAL, "G or G_proj is NULL");
        ACSC_CHECK_ARG(aligned(a.G, es) && (!need_gproj || aligned(a.G_proj, es)), ACSC_EALIGN,
                       "G, G_proj must be element-aligned");
    }
    return ACSC_OK;
}

// ---------------------------------------------------------------------------
// PowerSGD compressor with error feedback (the data-parallel compressor the
// method is paired with; rank-r step of Vogels et al. 2019):
//   project:        M = G + E (into E) and P = M Q, one sweep over M (the
//                   fused EMA pass with coefficients 1, 1, which also writes
//                   the bf16 copy of M the second projection reads)
//   orthogonalize:  P_hat = CholeskyQR2(P), Q' = M^T P_hat
//   decompress:     out = P_hat Q'^T and E = M - out, one sweep over E (the
//                   streamed-tile product with the feedback epilogue)
// The phases meet through the caller's P [m, r] and Q [n, r], so that a
// data-parallel caller can average them between the phases.
// ---------------------------------------------------------------------------

// dst [rows, cols] (row stride cols) = the first cols columns of src (row stride lds).
struct CropJob {
    const float *src;
    int64_t lds;
    float *dst;
    int rows, cols;
    int splits;      // > 1: src is the first of that many partials, ss apart, added in order
    int64_t ss;
};

__global__ __launch_bounds__(256) void crop_kernel(const Batch<CropJob> jb)
{
    const CropJob &J = jb.j[blockIdx.z];
    const int64_t total = static_cast<int64_t>(J.rows) * J.cols;
    for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < total;
         idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t i = idx / J.cols;
        const int c = static_cast<int>(idx - i * J.cols);
        float v = J.src[i * J.lds + c];
#pragma unroll 4
        for (int p = 1; p < J.splits; ++p)
            v += J.src[p * J.ss + i * J.lds + c];
        J.dst[idx] = v;
    }
}

struct PsgdWs {
    PriorWs pw;     // M16, Zt16 (Q^T bf16), Y (P, P_hat), Yt16 (P_hat^T bf16), Z (Q'), part, T, gram
    void *Pc, *Vc;  // decompression factors [m, RPd], [n, RPd] in the compute type
    int RPd;
};

size_t carve_psgd(const Dims &d, acsc_dtype dt, void *base, PsgdWs *w)
{
    const bool use16 = dt == ACSC_BF16;
    PsgdWs t;
    Carve c(base);
    c.off = carve_prior(d, use16, base, &t.pw);
    t.RPd = d.RP;
    const size_t es = dtype_size(dt);
    t.Pc = c.take<unsigned char>(static_cast<size_t>(d.m) * t.RPd * es);
    t.Vc = c.take<unsigned char>(static_cast<size_t>(d.n) * t.RPd * es);
    if (w)
        *w = t;
    return c.off;
}

struct PsgdItem {
    const psgd_matrix *in;
    Mat mat;   // dims and the CholeskyQR2 buffers (mat.pw == w.pw)
    PsgdWs w;
};

void crop(const char *tag, const std::vector<CropJob> &jobs, hipStream_t st)
{
    int64_t tot = 1;
    for (const CropJob &j : jobs)
        tot = std::max<int64_t>(tot, static_cast<int64_t>(j.rows) * j.cols);
    launch_jobs(tag, crop_kernel, jobs, dim3(grid1d(tot)), dim3(256), 0, st);
}

// The first r columns of a product [rows, KP] into the caller's factor; a bf16
// pass cut along k is still in the workspace's partials.
CropJob crop_of(const PsgdItem &x, const float *src, int rows, float *dst, int r, int splits)
{
    const int KP = x.mat.D.KP;
    return CropJob{splits > 1 ? x.w.pw.part : src, KP, dst, rows, r, splits, static_cast<int64_t>(rows) * KP};
}

// With `left` (the whole step) P stays in the workspace: in Y, or in the
// partials that `left` counts; otherwise it goes to the caller's factor.
int psgd_project_phase(std::vector<PsgdItem> &it, bool use16, int r, std::vector<int> *left, hipStream_t st)
{
    const int KP = it[0].mat.D.KP;
    std::vector<int> splits(it.size(), 1);
    if (use16) {
        // Q^T in bf16, rows r .. KP-1 zero: the thin factor of the pass
        std::vector<TileJob> tj;
        for (auto &x : it)
            tj.push_back(TileJob{x.in->Q, r, x.in->n, r, KP, x.w.pw.Zt16, x.w.pw.ldz16, nullptr, nullptr, 0, 0});
        launch_tiles("psgd_qconvert", tj, st);
        std::vector<pass::EmaReq> er;
        for (auto &x : it)
            er.push_back(pass::EmaReq{x.in->E, static_cast<const uint16_t *>(x.in->G), x.w.pw.M16, x.w.pw.Zt16,
                                      x.w.pw.ldz16, x.w.pw.Y, KP, x.in->m, x.in->n, KP, x.w.pw.part});
        if (pass::ema_fusable(er)) {
            if (int rc = pass::ema_run("psgd_feedback_mq", er, 1.0f, 1.0f, st))
                return rc;
        } else {
            std::vector<EmaJob> j;
            std::vector<pass::Req> q;
            int64_t tot = 1;
            for (auto &x : it) {
                j.push_back(EmaJob{x.in->E, static_cast<const uint16_t *>(x.in->G), x.in->m, x.in->n,
                                             (x.in->n % 8) == 0 ? 1 : 0, x.w.pw.M16, x.w.pw.ntc16});
                tot = std::max<int64_t>(tot, static_cast<int64_t>(x.in->m) * cdiv(x.in->n, 8));
                q.push_back(pass::Req{x.w.pw.M16, 0, true, x.w.pw.Zt16, x.w.pw.ldz16, x.w.pw.Y, KP,
                                      x.in->m, x.in->n, KP, x.w.pw.part, static_cast<int>(x.w.pw.ntc16)});
            }
            launch_jobs("psgd_feedback", ema_shadow_kernel, j, dim3(grid1d(tot)), dim3(256), 0, st, 1.0f,
                        1.0f);
            if (int rc = pass::run("psgd_pass_mq", false, q, st, splits.data()))
                return rc;
        }
    } else {
        std::vector<PadJob<float>> pj;
        std::vector<Ema32Job> ej;
        std::vector<f32::PassReq> q;
        int64_t tp = 1, te = 1;
        for (auto &x : it) {
            pj.push_back(PadJob<float>{x.in->Q, x.in->n, x.w.pw.Z});
            tp = std::max<int64_t>(tp, static_cast<int64_t>(x.in->n) * KP);
            const int64_t c = static_cast<int64_t>(x.in->m) * x.in->n;
            ej.push_back(Ema32Job{x.in->E, static_cast<const float *>(x.in->G), c});
            te = std::max(te, cdiv(c, 4));
            q.push_back(f32::PassReq{x.in->E, x.in->n, x.w.pw.Z, KP, x.w.pw.Y, KP, x.in->m, x.in->n, r, KP,
                                     x.w.pw.part, split_count(x.in->m, x.in->n)});
        }
        launch_jobs("psgd_qconvert", pad_convert_kernel<float>, pj, dim3(grid1d(tp)), dim3(256), 0, st, r, KP);
        launch_jobs("psgd_feedback", ema_kernel, ej, dim3(grid1d(te)), dim3(256), 0, st, 1.0f, 1.0f);
        if (int rc = f32::pass("psgd_pass_mq", false, q, st, splits.data()))
            return rc;
    }
    if (left) {
        *left = splits;
        return ACSC_OK;
    }
    std::vector<CropJob> cj;
    for (size_t i = 0; i < it.size(); ++i)
        cj.push_back(crop_of(it[i], it[i].w.pw.Y, it[i].in->m, it[i].in->P, r, splits[i]));
    crop("psgd_crop", cj, st);
    return ACSC_OK;
}

// `left`: what psgd_project_phase left of P; nullptr: P is the caller's.
int psgd_orthogonalize_phase(std::vector<PsgdItem> &it, bool use16, int r, const std::vector<int> *left,
                             hipStream_t st)
{
    const int KP = it[0].mat.D.KP;
    if (!left) {
        std::vector<PadJob<float>> pj;
        int64_t tp = 1;
        for (auto &x : it) {
            pj.push_back(PadJob<float>{x.in->P, x.in->m, x.w.pw.Y});
            tp = std::max<int64_t>(tp, static_cast<int64_t>(x.in->m) * KP);
        }
        launch_jobs("psgd_pconvert", pad_convert_kernel<float>, pj, dim3(grid1d(tp)), dim3(256), 0, st, r, KP);
    }
    std::vector<Mat> ms;
    for (auto &x : it) {
        ms.push_back(x.mat);
        if (use16)
            ms.back().q32 = x.in->P;   // the pass below reads the bf16 copy only
    }
    // CholeskyQR2: P_hat (fp32), and its bf16 transposed copy for the pass
    if (int rc = orthonormalise(ms, true, 2, use16, left ? *left : std::vector<int>(ms.size(), 1), false, st))
        return rc;
    std::vector<CropJob> cj;
    if (!use16) {
        for (auto &x : it)
            cj.push_back(crop_of(x, x.w.pw.Y, x.in->m, x.in->P, r, 1));
        crop("psgd_crop", cj, st);
        cj.clear();
    }
    std::vector<int> splits(it.size(), 1);
    if (use16) {
        std::vector<pass::Req> q;
        for (auto &x : it)
            q.push_back(pass::Req{x.w.pw.M16, 0, true, x.w.pw.Yt16, x.w.pw.ldy16, x.w.pw.Z, KP, x.in->n,
                                  x.in->m, KP, x.w.pw.part, static_cast<int>(x.w.pw.ntc16)});
        if (int rc = pass::run("psgd_pass_mtp", true, q, st, splits.data()))
            return rc;
    } else {
        std::vector<f32::PassReq> q;
        for (auto &x : it)
            q.push_back(f32::PassReq{x.in->E, x.in->n, x.w.pw.Y, KP, x.w.pw.Z, KP, x.in->n, x.in->m, r, KP,
                                     x.w.pw.part, split_count(x.in->n, x.in->m)});
        if (int rc = f32::pass("psgd_pass_mtp", true, q, st, splits.data()))
            return rc;
    }
    for (size_t i = 0; i < it.size(); ++i)
        cj.push_back(crop_of(it[i], it[i].w.pw.Z, it[i].in->n, it[i].in->Q, r, splits[i]));
    crop("psgd_crop", cj, st);
    return ACSC_OK;
}

int psgd_decompress_phase(std::vector<PsgdItem> &it, bool use16, int r, hipStream_t st)
{
    const int RPd = it[0].w.RPd;
    if (use16) {
        std::vector<TileJob> tj;
        std::vector<blend::Req> q;
        for (auto &x : it) {
            tj.push_back(TileJob{x.in->P, r, x.in->m, r, RPd, nullptr, 0, static_cast<uint16_t *>(x.w.Pc), nullptr, 0,
                                 0});
            tj.push_back(TileJob{x.in->Q, r, x.in->n, r, RPd, nullptr, 0, static_cast<uint16_t *>(x.w.Vc), nullptr, 0,
                                 0});
            q.push_back(blend::Req{nullptr, static_cast<uint16_t *>(x.in->out), x.in->m, x.in->n,
                                   static_cast<const uint16_t *>(x.w.Pc), static_cast<const uint16_t *>(x.w.Vc),
                                   nullptr, nullptr, nullptr, x.in->E});
        }
        launch_tiles("psgd_fconvert", tj, st);
        return blend::run_feedback("psgd_decompress", q, RPd, st);
    }
    std::vector<PadJob<float>> pj;
    std::vector<f32::BlendReq> bj;
    int64_t tp = 1;
    for (auto &x : it) {
        pj.push_back(PadJob<float>{x.in->P, x.in->m, static_cast<float *>(x.w.Pc)});
        pj.push_back(PadJob<float>{x.in->Q, x.in->n, static_cast<float *>(x.w.Vc)});
        tp = std::max<int64_t>(tp, static_cast<int64_t>(std::max(x.in->m, x.in->n)) * RPd);
        bj.push_back(f32::BlendReq{nullptr, static_cast<float *>(x.in->out), x.in->m, x.in->n,
                                   static_cast<const float *>(x.w.Pc), static_cast<const float *>(x.w.Vc), nullptr,
                                   nullptr, nullptr, x.in->E});
    }
    launch_jobs("psgd_fconvert", pad_convert_kernel<float>, pj, dim3(grid1d(tp)), dim3(256), 0, st, r, RPd);
    return f32::blend("psgd_decompress", bj, RPd, 0.0f, st, nullptr, true);
}

int check_psgd(const psgd_matrix &a, int i, int r, acsc_dtype dt, int phase)
{
    ACSC_CHECK_ARG(a.m >= 1 && a.n >= 1, ACSC_EINVAL, "matrix %d: m=%d, n=%d must be >= 1", i, a.m, a.n);
    ACSC_CHECK_ARG(r >= 1 && r <= std::min(std::min(a.m, a.n), kKMax), ACSC_EINVAL,
                   "matrix %d: r=%d outside [1, min(m, n, %d)] for a %d x %d matrix", i, r, kKMax, a.m, a.n);
    const Dims d = dims_of(a.m, a.n, r, 0);
    const size_t need = carve_psgd(d, dt, nullptr, nullptr);
    ACSC_CHECK_ARG(a.ws != nullptr && a.E && a.P && a.Q, ACSC_EINVAL, "matrix %d: null ws, E, P or Q", i);
    ACSC_CHECK_ARG(a.ws_bytes >= need, ACSC_ENOSPC, "matrix %d: workspace %zu bytes < %zu needed", i, a.ws_bytes,
                   need);
    ACSC_CHECK_ARG(aligned(a.ws, 256), ACSC_EALIGN, "matrix %d: workspace must be 256-byte aligned", i);
    ACSC_CHECK_ARG(aligned(a.E, 16), ACSC_EALIGN, "matrix %d: E must be 16-byte aligned", i);
    ACSC_CHECK_ARG(aligned(a.P, 4) && aligned(a.Q, 4), ACSC_EALIGN, "matrix %d: P, Q must be 4-byte aligned", i);
    if (phase == 0 || phase == 3) {
        ACSC_CHECK_ARG(a.G != nullptr, ACSC_EINVAL, "matrix %d: G is NULL", i);
        ACSC_CHECK_ARG(aligned(a.G, 16), ACSC_EALIGN, "matrix %d: G must be 16-byte aligned", i);
    }
    if (phase == 2 || phase == 3) {
        ACSC_CHECK_ARG(a.out != nullptr, ACSC_EINVAL, "matrix %d: out is NULL", i);
        ACSC_CHECK_ARG(aligned(a.out, dtype_size(dt)), ACSC_EALIGN, "matrix %d: out must be element-aligned", i);
    }
    return ACSC_OK;
}

// phase 0 project, 1 orthogonalize, 2 decompress, 3 all three
int psgd_run(int count, const psgd_matrix *mats, acsc_dtype dt, int r, int phase, hipStream_t st)
{
    clear_error();
    ACSC_CHECK_ARG(count >= 0, ACSC_EINVAL, "count=%d < 0", count);
    ACSC_CHECK_ARG(count == 0 || mats != nullptr, ACSC_EINVAL, "mats is NULL");
    ACSC_CHECK_ARG(dt == ACSC_F32 || dt == ACSC_BF16, ACSC_EDTYPE, "unknown dtype %d", (int)dt);
    std::vector<PsgdItem> it;
    for (int i = 0; i < count; ++i) {
        if (int rc = check_psgd(mats[i], i, r, dt, phase))
            return rc;
        PsgdItem x;
        x.in = &mats[i];
        x.mat.in = nullptr;
        x.mat.D = dims_of(mats[i].m, mats[i].n, r, 0);
        carve_psgd(x.mat.D, dt, mats[i].ws, &x.w);
        x.mat.pw = x.w.pw;
        x.mat.seed = 0;
        it.push_back(x);
    }
    if (it.empty())
        return ACSC_OK;
    const bool use16 = dt == ACSC_BF16;
    if (int rc = chol::prepare(it[0].mat.D.KP))
        return rc;
    // within one step nothing else reads P = M Q: it need not go through the
    // caller's factor (two launches of about 4.5 us per group of equal rank)
    int rc = ACSC_OK;
    std::vector<int> left;
    if (phase == 0 || phase == 3)
        rc = psgd_project_phase(it, use16, r, phase == 3 ? &left : nullptr, st);
    if (!rc && (phase == 1 || phase == 3))
        rc = psgd_orthogonalize_phase(it, use16, r, phase == 3 ? &left : nullptr, st);
    if (!rc && (phase == 2 || phase == 3))
        rc = psgd_decompress_phase(it, use16, r, st);
    if (rc)
        return rc;
    return check_launch("psgd");
}

}  // namespace
}  // namespace acsc

using namespace acsc;

extern "C" int sc_workspace_size(int m, int n, int r, int oversample, acsc_dtype dt, size_t *bytes)
{
    clear_error();
    ACSC_CHECK_ARG(bytes != nullptr, ACSC_EINVAL, "bytes is NULL");
    ACSC_CHECK_ARG(dt == ACSC_F32 || dt == ACSC_BF16, ACSC_EDTYPE, "unknown dtype %d", (int)dt);
    ACSC_CHECK_ARG(m >= 1 && n >= 1, ACSC_EINVAL, "m=%d, n=%d must be >= 1", m, n);
    ACSC_CHECK_ARG(r >= 1 && r <= std::min(std::min(m, n), kKMax), ACSC_EINVAL,
                   "r=%d outside [1, min(m, n, %d)]", r, kKMax);
    ACSC_CHECK_ARG(oversample >= 0, ACSC_EINVAL, "oversample=%d < 0", oversample);
    const Dims d = dims_of(m, n, r, oversample);
    *bytes = std::max(carve_prior(d, dt == ACSC_BF16, nullptr, nullptr),
                      carve_correct(d, dtype_size(dt), nullptr, nullptr));
    return ACSC_OK;
}

namespace {

int build_batched(int count, const sc_matrix *mats, acsc_dtype dt, float beta, int r, int oversample,
                  int power_iters, float tau, uint64_t seed, int phases, hipStream_t stream)
{
    clear_error();
    ACSC_CHECK_ARG(count >= 0, ACSC_EINVAL, "count=%d < 0", count);
    ACSC_CHECK_ARG(count == 0 || mats != nullptr, ACSC_EINVAL, "mats is NULL");
    ACSC_CHECK_ARG(dt == ACSC_F32 || dt == ACSC_BF16, ACSC_EDTYPE, "unknown dtype %d", (int)dt);
    ACSC_CHECK_ARG(beta >= 0.f && beta <= 1.f, ACSC_EINVAL, "beta=%g outside [0, 1]", beta);
    ACSC_CHECK_ARG(tau >= 0.f && std::isfinite(tau), ACSC_EINVAL, "tau=%g must be finite, >= 0", tau);
    ACSC_CHECK_ARG(power_iters >= 0 && power_iters <= 64, ACSC_EINVAL, "power_iters=%d outside [0, 64]",
                   power_iters);
    ACSC_CHECK_ARG(oversample >= 0, ACSC_EINVAL, "oversample=%d < 0", oversample);
    std::vector<Mat> all;
    for (int i = 0; i < count; ++i) {
        size_t need = 0;
        int rc = check_matrix(mats[i], r, oversample, dt, true, &need);
        if (rc)
            return rc;
        Mat m;
        m.in = &mats[i];
        m.D = dims_of(mats[i].m, mats[i].n, r, oversample);
        carve_prior(m.D, dt == ACSC_BF16, mats[i].ws, &m.pw);
        m.seed = seed + static_cast<uint64_t>(i);
        all.push_back(m);
    }
    if (all.empty())
        return ACSC_OK;
    // LDS of the one-workgroup kernels, for every k in the batch
    for (const Mat &m : all) {
        int rc = chol::prepare(m.D.KP);
        if (!rc)
            rc = jacobi_prepare(m.D.k);
        if (rc)
            return rc;
    }
    // matrices with the same k (= min(r + oversample, m, n)) share every launch
    std::vector<bool> done(all.size(), false);
    for (size_t i = 0; i < all.size(); ++i) {
        if (done[i])
            continue;
        std::vector<Mat> group;
        for (size_t j = i; j < all.size(); ++j)
            if (!done[j] && all[j].D.k == all[i].D.k) {
                group.push_back(all[j]);
                done[j] = true;
            }
        const int rc = build_group(group, dt, beta, r, power_iters, tau, phases, stream);
        if (rc)
            return rc;
    }
    return check_launch("sc_build_prior");
}

}  // namespace

extern "C" int sc_build_prior_batched(int count, const sc_matrix *mats, acsc_dtype dt, float beta, int r,
                                      int oversample, int power_iters, float tau, uint64_t seed,
                                      hipStream_t stream)
{
    return build_batched(count, mats, dt, beta, r, oversample, power_iters, tau, seed,
                         kPhaseSubspace | kPhaseRitz, stream);
}

extern "C" int sc_build_subspace_batched(int count, const sc_matrix *mats, acsc_dtype dt, float beta, int r,
                                         int oversample, int power_iters, float tau, uint64_t seed,
                                         hipStream_t stream)
{
    return build_batched(count, mats, dt, beta, r, oversample, power_iters, tau, seed, kPhaseSubspace, stream);
}

extern "C" int sc_build_ritz_batched(int count, const sc_matrix *mats, acsc_dtype dt, float beta, int r,
                                     int oversample, int power_iters, float tau, uint64_t seed,
                                     hipStream_t stream)
{
    return build_batched(count, mats, dt, beta, r, oversample, power_iters, tau, seed, kPhaseRitz, stream);
}

extern "C" int sc_build_status(int count, const sc_matrix *mats, int *sweeps, float *residual, hipStream_t stream)
{
    clear_error();
    ACSC_CHECK_ARG(count >= 0, ACSC_EINVAL, "count=%d < 0", count);
    ACSC_CHECK_ARG(count == 0 || mats != nullptr, ACSC_EINVAL, "mats is NULL");
    for (int i = 0; i < count; ++i) {
        ACSC_CHECK_ARG(mats[i].ws != nullptr, ACSC_EINVAL, "matrix %d: workspace is NULL", i);
        ACSC_CHECK_ARG(aligned(mats[i].ws, 256), ACSC_EALIGN, "matrix %d: workspace must be 256-byte aligned", i);
        ACSC_CHECK_ARG(mats[i].ws_bytes >= 5 * sizeof(int), ACSC_ENOSPC, "matrix %d: workspace too small", i);
    }
    std::vector<int> words(static_cast<size_t>(count) * 5, 0);
    for (int i = 0; i < count; ++i) {
        const hipError_t e = hipMemcpyAsync(words.data() + 5 * i, mats[i].ws, 5 * sizeof(int), hipMemcpyDeviceToHost,
                                            stream);
        if (e != hipSuccess)
            return set_error(ACSC_EHIP, "reading the status of matrix %d: %s", i, hipGetErrorString(e));
    }
    const hipError_t e = hipStreamSynchronize(stream);
    if (e != hipSuccess)
        return set_error(ACSC_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
    int rc = ACSC_OK;
    for (int i = 0; i < count; ++i) {
        const int *w = words.data() + 5 * i;
        float res, tol;
        std::memcpy(&res, &w[kInfoResidual], sizeof(float));
        std::memcpy(&tol, &w[kInfoTol], sizeof(float));
        if (sweeps)
            sweeps[i] = w[kInfoSweeps];
        if (residual)
            residual[i] = res;
        if (rc)
            continue;   // report the first failing matrix
        if (w[kInfoStatus] & kStatusNoSubspace)
            rc = set_error(ACSC_ENOCONV, "matrix %d: the Rayleigh-Ritz phase ran without a subspace phase on its "
                                         "workspace before it", i);
        else if (w[kInfoStatus] & kStatusStalled)
            rc = set_error(ACSC_ENOCONV, "matrix %d: a wait of the fused EMA pass ran out of polls (its "
                                         "subspace and prior are not to be trusted)", i);
        else if (w[kInfoStatus] & kStatusNoConv)
            rc = set_error(ACSC_ENOCONV, "matrix %d: the Rayleigh-Ritz Jacobi stopped after %d sweeps with an "
                                         "off-diagonal ratio %g above its tolerance %g", i, w[kInfoSweeps], res, tol);
        else if (w[kInfoStatus] != 0)
            rc = set_error(ACSC_ENOCONV, "matrix %d: no status of a build (word %d)", i, w[kInfoStatus]);
    }
    return rc;
}

extern "C" int sc_correct_batched(int count, const sc_matrix *mats, acsc_dtype dt, int r, float alpha,
                                  hipStream_t stream)
{
    clear_error();
    ACSC_CHECK_ARG(count >= 0, ACSC_EINVAL, "count=%d < 0", count);
    ACSC_CHECK_ARG(count == 0 || mats != nullptr, ACSC_EINVAL, "mats is NULL");
    ACSC_CHECK_ARG(dt == ACSC_F32 || dt == ACSC_BF16, ACSC_EDTYPE, "unknown dtype %d", (int)dt);
    ACSC_CHECK_ARG(std::isfinite(alpha), ACSC_EINVAL, "alpha must be finite");
    std::vector<Mat> all;
    for (int i = 0; i < count; ++i) {
        size_t need = 0;
        int rc = check_matrix(mats[i], r, 0, dt, false, &need);
        if (rc)
            return rc;
        Mat m;
        m.in = &mats[i];
        m.D = dims_of(mats[i].m, mats[i].n, r, 0);
        carve_correct(m.D, dtype_size(dt), mats[i].ws, &m.cw);
        m.seed = 0;
        all.push_back(m);
    }
    if (all.empty())
        return ACSC_OK;
    int rc = ACSC_OK;
    if (dt == ACSC_BF16)
        rc = correct_group<uint16_t>(all, r, alpha, stream);
    else
        rc = correct_group<float>(all, r, alpha, stream);
    if (rc)
        return rc;
    return check_launch("sc_correct");
}

extern "C" int sc_adamw_workspace_size(int m, int n, int r, acsc_dtype dt, size_t *bytes)
{
    clear_error();
    ACSC_CHECK_ARG(bytes != nullptr, ACSC_EINVAL, "bytes is NULL");
    ACSC_CHECK_ARG(dt == ACSC_F32 || dt == ACSC_BF16, ACSC_EDTYPE, "unknown dtype %d", (int)dt);
    ACSC_CHECK_ARG(m >= 1 && n >= 1, ACSC_EINVAL, "m=%d, n=%d must be >= 1", m, n);
    ACSC_CHECK_ARG(r >= 1 && r <= std::min(std::min(m, n), kKMax), ACSC_EINVAL,
                   "r=%d outside [1, min(m, n, %d)]", r, kKMax);
    *bytes = carve_correct(dims_of(m, n, r, 0), dtype_size(dt), nullptr, nullptr);
    return ACSC_OK;
}

extern "C" int sc_correct_adamw_batched(int count, const sc_matrix *mats, const sc_adamw_state *states,
                                        acsc_dtype dt, int r, float alpha, const sc_adamw_hparams *hp,
                                        float *norm_out, hipStream_t stream)
{
    clear_error();
    ACSC_CHECK_ARG(count >= 0, ACSC_EINVAL, "count=%d < 0", count);
    ACSC_CHECK_ARG(count == 0 || (mats != nullptr && states != nullptr), ACSC_EINVAL, "mats or states is NULL");
    ACSC_CHECK_ARG(hp != nullptr, ACSC_EINVAL, "hp is NULL");
    ACSC_CHECK_ARG(dt == ACSC_F32 || dt == ACSC_BF16, ACSC_EDTYPE, "unknown dtype %d", (int)dt);
    ACSC_CHECK_ARG(std::isfinite(alpha), ACSC_EINVAL, "alpha must be finite");
    ACSC_CHECK_ARG(std::isfinite(hp->lr) && hp->lr >= 0.f, ACSC_EINVAL, "lr=%g must be finite, >= 0", hp->lr);
    ACSC_CHECK_ARG(hp->beta1 >= 0.f && hp->beta1 < 1.f && hp->beta2 >= 0.f && hp->beta2 < 1.f, ACSC_EINVAL,
                   "betas (%g, %g) must lie in [0, 1)", hp->beta1, hp->beta2);
    ACSC_CHECK_ARG(std::isfinite(hp->eps) && hp->eps > 0.f, ACSC_EINVAL, "eps=%g must be finite, > 0", hp->eps);
    ACSC_CHECK_ARG(std::isfinite(hp->weight_decay) && hp->weight_decay >= 0.f, ACSC_EINVAL,
                   "weight_decay=%g must be finite, >= 0", hp->weight_decay);
    ACSC_CHECK_ARG(hp->step >= 1, ACSC_EINVAL, "step=%lld must be >= 1", (long long)hp->step);
    ACSC_CHECK_ARG(std::isfinite(hp->max_norm), ACSC_EINVAL, "max_norm must be finite");
    ACSC_CHECK_ARG(!norm_out || aligned(norm_out, 4), ACSC_EALIGN, "norm_out must be 4-byte aligned");
    std::vector<Mat> all;
    for (int i = 0; i < count; ++i) {
        size_t need = 0;
        int rc = check_matrix(mats[i], r, 0, dt, false, &need, false);
        if (rc)
            return rc;
        const sc_adamw_state &a = states[i];
        ACSC_CHECK_ARG(a.W && a.m1 && a.m2, ACSC_EINVAL, "state %d: W, m1 or m2 is NULL", i);
        ACSC_CHECK_ARG(aligned(a.W, 4) && aligned(a.m1, 4) && aligned(a.m2, 4), ACSC_EALIGN,
                       "state %d: W, m1, m2 must be 4-byte aligned", i);
        Mat m;
        m.in = &mats[i];
        m.D = dims_of(mats[i].m, mats[i].n, r, 0);
        carve_correct(m.D, dtype_size(dt), mats[i].ws, &m.cw);
        m.seed = 0;
        m.ad = &a;
        all.push_back(m);
    }
    if (all.empty())
        return ACSC_OK;
    int rc = ACSC_OK;
    // bias corrections and the step size in double on the host, then fp32
    const double t = static_cast<double>(hp->step);
    const double bc1 = 1.0 - std::pow(static_cast<double>(hp->beta1), t);
    const double bc2 = 1.0 - std::pow(static_cast<double>(hp->beta2), t);
    AdamCtx ctx{};
    ctx.args.beta1 = hp->beta1;
    ctx.args.beta2 = hp->beta2;
    ctx.args.omb1 = static_cast<float>(1.0 - hp->beta1);
    ctx.args.omb2 = static_cast<float>(1.0 - hp->beta2);
    ctx.args.wdf = static_cast<float>(1.0 - static_cast<double>(hp->lr) * hp->weight_decay);
    ctx.args.step = static_cast<float>(hp->lr / bc1);
    ctx.args.isbc2 = static_cast<float>(1.0 / std::sqrt(bc2));
    ctx.args.eps = hp->eps;
    ctx.args.coef = all[0].cw.coef;
    ctx.acc = all[0].cw.acc;
    ctx.max_norm = hp->max_norm;
    ctx.norm_out = norm_out;
    if (dt == ACSC_BF16)
        rc = correct_group<uint16_t>(all, r, alpha, stream, &ctx);
    else
        rc = correct_group<float>(all, r, alpha, stream, &ctx);
    if (rc)
        return rc;
    return check_launch("sc_correct_adamw");
}

extern "C" int sc_build_prior(const void *G_anc, acsc_dtype dt, float *M, int m, int n, float beta, int r,
                              int oversample, int power_iters, float tau, const float *V_warm, uint64_t seed,
                              float *U, float *s, float *V, float *d, void *ws, size_t ws_bytes,
                              hipStream_t stream)
{
    sc_matrix a{};
    a.G = G_anc;
    a.M = M;
    a.m = m;
    a.n = n;
    a.U = U;
    a.s = s;
    a.V = V;
    a.d = d;
    a.V_warm = V_warm;
    a.ws = ws;
    a.ws_bytes = ws_bytes;
    return sc_build_prior_batched(1, &a, dt, beta, r, oversample, power_iters, tau, seed, stream);
}

extern "C" int sc_correct(const void *G, acsc_dtype dt, int m, int n, const float *U, const float *d,
                          const float *V, int r, float alpha, void *G_proj, void *ws, size_t ws_bytes,
                          hipStream_t stream)
{
    sc_matrix a{};
    a.G = G;
    a.m = m;
    a.n = n;
    a.U = const_cast<float *>(U);
    a.s = const_cast<float *>(d);   // unused by the correction; only checked non-null
    a.V = const_cast<float *>(V);
    a.d = const_cast<float *>(d);
    a.G_proj = G_proj;
    a.ws = ws;
    a.ws_bytes = ws_bytes;
    return sc_correct_batched(1, &a, dt, r, alpha, stream);
}

extern "C" int psgd_workspace_size(int m, int n, int r, acsc_dtype dt, size_t *bytes)
{
    clear_error();
    ACSC_CHECK_ARG(bytes != nullptr, ACSC_EINVAL, "bytes is NULL");
    ACSC_CHECK_ARG(dt == ACSC_F32 || dt == ACSC_BF16, ACSC_EDTYPE, "unknown dtype %d", (int)dt);
    ACSC_CHECK_ARG(m >= 1 && n >= 1, ACSC_EINVAL, "m=%d, n=%d must be >= 1", m, n);
    ACSC_CHECK_ARG(r >= 1 && r <= std::min(std::min(m, n), kKMax), ACSC_EINVAL,
                   "r=%d outside [1, min(m, n, %d)]", r, kKMax);
    *bytes = carve_psgd(dims_of(m, n, r, 0), dt, nullptr, nullptr);
    return ACSC_OK;
}

extern "C" int psgd_project(int count, const psgd_matrix *mats, acsc_dtype dt, int r, hipStream_t stream)
{
    return psgd_run(count, mats, dt, r, 0, stream);
}

extern "C" int psgd_orthogonalize(int count, const psgd_matrix *mats, acsc_dtype dt, int r, hipStream_t stream)
{
    return psgd_run(count, mats, dt, r, 1, stream);
}

extern "C" int psgd_decompress(int count, const psgd_matrix *mats, acsc_dtype dt, int r, hipStream_t stream)
{
    return psgd_run(count, mats, dt, r, 2, stream);
}

extern "C" int psgd_step(int count, const psgd_matrix *mats, acsc_dtype dt, int r, hipStream_t stream)
{
    return psgd_run(count, mats, dt, r, 3, stream);
}
