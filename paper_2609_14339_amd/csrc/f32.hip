// fp32 products for gfx950 (see sc_f32.h), on v_mfma_f32_16x16x4f32.
//
// The thin products C = A B and C = A^T B.  A is streamed once; the thin
// factor B comes from L2.  A workgroup owns 16 RT rows of C, and its waves
// cut k among themselves: small matrices, which have few rows, then still
// keep many loads in flight, and the waves meet once, in LDS, at the end.
// Operands go from memory straight into the lanes that multiply them, with
// no staging and no barrier in the loop.  A product over k may take k in any
// order as long as both operands do: with lane i + 16 q of step s holding
// k = k0 + 4 q + s, four consecutive k of a row of A are one 16-byte load.
// Measured when each 32-deep step went through LDS with element loads and two
// barriers, and so: 256 x 256 by 16 columns 24 and 5 us; 8448 x 9088 and 2944 x
// 4608 by 96 560-640 and 200-230 us (83 TFLOP/s of 153 that a large matrix
// product reaches); 4096 x 8192 by 144 340 and 102-117 us.
#include "common.h"
#include "sc_f32.h"
#include "sc_pass.h"

#include <algorithm>
#include <type_traits>

namespace acsc {
namespace f32 {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
using F4 = F4Any;

constexpr int kMaxJobs = 16;

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct Job {
    const float *A;
    int64_t lda;
    const float *B;
    int64_t ldb;
    float *C;
    int64_t ldc, split_stride;
    int M, K, nvalid, kchunk, splits, nblocks;
};
struct Batch {
    int count;
    Job j[kMaxJobs];
};

// Row tiles of a wide workgroup: four while their sums and the operands of two
// steps fit the registers.
constexpr int wide_tiles(int NT) { return NT <= 9 ? 4 : 2; }

// RT > 1: 16 RT rows and four waves; RT = 1: 16 rows and eight waves.
template <bool TRANS, int RT, int NT>
__global__ __launch_bounds__(RT > 1 ? 256 : 512) void pass_kernel(const Batch jb)
{
    constexpr int WK = RT > 1 ? 4 : 8;
    constexpr int NP = NT * 16;
    constexpr int KU = RT == 1 && NT <= 4 ? 2 : 1;   // 16-deep groups per loop step
    const Job &J = jb.j[blockIdx.z];
    if (static_cast<int>(blockIdx.x) >= J.nblocks)
        return;
    __shared__ __attribute__((aligned(16))) float red[WK][16][NP];
    const float *__restrict__ A = J.A;
    const float *__restrict__ B = J.B;
    const int64_t lda = J.lda, ldb = J.ldb;
    const int M = J.M, nvalid = J.nvalid;
    const int split = static_cast<int>(blockIdx.x) % J.splits;
    const int row0 = static_cast<int>(blockIdx.x) / J.splits * 16 * RT;
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sbeg = split * J.kchunk, send = min(J.K, sbeg + J.kchunk);
    const int per = ((send - sbeg + WK - 1) / WK + 15) & ~15;
    const int kb = sbeg + wave * per, ke = min(send, kb + per);

    f32x4 acc[RT][NT];
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            acc[a][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    struct Step {
        float a[KU][RT][4], b[KU][4][NT];
    };
    const bool rows_whole = row0 + 16 * RT <= M;
    // the 16 KU k from k0 on.  A whole step's values go to the products as they
    // come, with nothing between that would wait for them: columns past
    // nvalid repeat the last one and are stored as zeros, rows past M repeat
    // the last one and are not stored.  Only a tail step masks k past ke.
    auto load = [&](Step &S, int k0, auto tail) {
        constexpr bool TAIL = decltype(tail)::value;
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int kq = k0 + 16 * u + 4 * q;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float *br = B + static_cast<int64_t>(TAIL ? min(kq + s, ke - 1) : kq + s) * ldb;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const float v = br[min(16 * t + i, nvalid - 1)];
                    S.b[u][s][t] = !TAIL || kq + s < ke ? v : 0.f;
                }
            }
            if constexpr (!TRANS) {
#pragma unroll
                for (int a = 0; a < RT; ++a) {
                    const float *ar = A + static_cast<int64_t>(min(row0 + 16 * a + i, M - 1)) * lda;
                    if constexpr (!TAIL) {
                        const F4 v = *reinterpret_cast<const F4 *>(ar + kq);
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            S.a[u][a][s] = v.v[s];
                    } else {
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const float v = ar[min(kq + s, ke - 1)];
                            S.a[u][a][s] = kq + s < ke ? v : 0.f;
                        }
                    }
                }
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float *ar = A + static_cast<int64_t>(TAIL ? min(kq + s, ke - 1) : kq + s) * lda;
                    float v[RT];
                    // lane i holds rows row0 + RT i + a, one of each tile a
                    if (RT == 4 && rows_whole) {
                        const F4 x = *reinterpret_cast<const F4 *>(ar + row0 + 4 * i);
#pragma unroll
                        for (int a = 0; a < RT; ++a)
                            v[a] = x.v[a];
                    } else {
#pragma unroll
                        for (int a = 0; a < RT; ++a)
                            v[a] = ar[min(row0 + RT * i + a, M - 1)];
                    }
#pragma unroll
                    for (int a = 0; a < RT; ++a)
                        S.a[u][a][s] = !TAIL || kq + s < ke ? v[a] : 0.f;
                }
            }
        }
    };
    auto mul = [&](const Step &S) {
#pragma unroll
        for (int u = 0; u < KU; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int a = 0; a < RT; ++a)
                        acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(S.a[u][a][s], S.b[u][s][t], acc[a][t], 0, 0, 0);
    };
    if (kb < ke) {
        // the next step's loads leave before this step's products
        constexpr std::false_type whole{};
        constexpr std::true_type tail{};
        constexpr int KS = 16 * KU;
        const int full = (ke - kb) / KS;
        Step S0, S1;
        if (full > 0) {
            load(S0, kb, whole);
            int s = 0;
            for (; s + 2 < full; s += 2) {
                load(S1, kb + (s + 1) * KS, whole);
                mul(S0);
                load(S0, kb + (s + 2) * KS, whole);
                mul(S1);
            }
            if (s + 1 < full) {
                load(S1, kb + (s + 1) * KS, whole);
                mul(S0);
                mul(S1);
            } else {
                mul(S0);
            }
        }
        if (kb + full * KS < ke) {
            load(S0, kb + full * KS, tail);
            mul(S0);
        }
    }
    // D[i][j] of a tile: lane j + 16 (i / 4), element i % 4.  The waves' sums
    // are added in wave order, one row tile at a time.
    float *C = J.C + static_cast<int64_t>(split) * J.split_stride;
    const int64_t ldc = J.ldc;
#pragma unroll
    for (int a = 0; a < RT; ++a) {
        if (a)
            __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                red[wave][4 * q + e][16 * t + i] = acc[a][t][e];
        __syncthreads();
        for (int idx = tid; idx < 16 * NP / 4; idx += 64 * WK) {
            const int r = idx / (NP / 4), c = idx % (NP / 4) * 4;
            f32x4 v = *reinterpret_cast<const f32x4 *>(&red[0][r][c]);
#pragma unroll
            for (int w = 1; w < WK; ++w)
                v += *reinterpret_cast<const f32x4 *>(&red[w][r][c]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = c + e < nvalid ? v[e] : 0.f;
            const int row = TRANS ? row0 + RT * r + a : row0 + 16 * a + r;
            if (row < M)
                *reinterpret_cast<f32x4 *>(C + static_cast<int64_t>(row) * ldc + c) = v;
        }
    }
}

struct Plan {
    int rows;                  // per workgroup: 16, or those of a wide one
    std::vector<int> splits;
};

// Wide workgroups (64 rows, 32 beyond 144 columns) once they fill the GPU (two
// per CU, cut along k as far as the partials' room goes), else 16-row ones,
// which read the thin factor more often but are as many times more; a wave
// gets at least 32 deep.
Plan plan(const std::vector<PassReq> &reqs)
{
    auto cut = [&](int rows, int waves, std::vector<int> *out) {
        int64_t blocks = 0, total = 0;
        for (const PassReq &q : reqs)
            blocks += cdiv(q.M, rows);
        const int64_t want = cdiv(512, std::max<int64_t>(1, blocks));
        for (const PassReq &q : reqs) {
            const int64_t s = std::max<int64_t>(
                1, std::min<int64_t>({want, q.part ? q.cap : 1, static_cast<int64_t>(q.K) / (32 * waves)}));
            const int64_t chunk = (cdiv(q.K, s) + 15) / 16 * 16;
            out->push_back(static_cast<int>(cdiv(q.K, chunk)));
            total += cdiv(q.M, rows) * out->back();
        }
        return total;
    };
    Plan p;
    p.rows = 16 * wide_tiles(reqs[0].NP / 16);
    if (cut(p.rows, 4, &p.splits) < 256) {
        p.rows = 16;
        p.splits.clear();
        cut(16, 8, &p.splits);
    }
    return p;
}

template <bool TRANS, int NT>
void launch_nt(const char *tag, bool wide, const Batch &b, int gx, hipStream_t st)
{
    if (wide)
        ACSC_LAUNCH(tag, (pass_kernel<TRANS, wide_tiles(NT), NT>), dim3(gx, 1, b.count), dim3(256), 0, st, b);
    else
        ACSC_LAUNCH(tag, (pass_kernel<TRANS, 1, NT>), dim3(gx, 1, b.count), dim3(512), 0, st, b);
}

template <bool TRANS>
void launch(const char *tag, int NP, bool wide, const Batch &b, int gx, hipStream_t st)
{
    switch (NP / 16) {
    case 1: launch_nt<TRANS, 1>(tag, wide, b, gx, st); break;
    case 2: launch_nt<TRANS, 2>(tag, wide, b, gx, st); break;
    case 3: launch_nt<TRANS, 3>(tag, wide, b, gx, st); break;
    case 4: launch_nt<TRANS, 4>(tag, wide, b, gx, st); break;
    case 5: launch_nt<TRANS, 5>(tag, wide, b, gx, st); break;
    case 6: launch_nt<TRANS, 6>(tag, wide, b, gx, st); break;
    case 7: launch_nt<TRANS, 7>(tag, wide, b, gx, st); break;
    case 8: launch_nt<TRANS, 8>(tag, wide, b, gx, st); break;
    case 9: launch_nt<TRANS, 9>(tag, wide, b, gx, st); break;
    case 10: launch_nt<TRANS, 10>(tag, wide, b, gx, st); break;
    case 11: launch_nt<TRANS, 11>(tag, wide, b, gx, st); break;
    default: launch_nt<TRANS, 12>(tag, wide, b, gx, st); break;
    }
}

// Blend: a workgroup's tile is 64 rows by 128 columns of G, a wave's 32 by 64.
// The product is formed as V P^T, so that a lane's four accumulators are four
// consecutive columns of a row; its G (or E) is loaded before the products.
// Up to 128 padded columns P and V come from L2 in less time than G streams.
struct BJob {
    const float *G;
    float *out;
    int m, n;
    const float *P, *V;
    float *W, *m1, *m2, *E;
};
struct BBatch {
    int count;
    BJob j[kMaxJobs];
};

template <int MODE>
__global__ __launch_bounds__(256) void blend_kernel(const BBatch jb, int RP, float alpha, const blend::AdamArgs ad)
{
    constexpr bool ADAM = MODE == blend::kAdam, EF = MODE == blend::kFeedback;
    const BJob &J = jb.j[blockIdx.z];
    const int m = J.m, n = J.n;
    if (static_cast<int>(blockIdx.x) * 128 >= n || static_cast<int>(blockIdx.y) * 64 >= m)
        return;
    const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = blockIdx.y * 64 + (wave >> 1) * 32, col0 = blockIdx.x * 128 + (wave & 1) * 64;
    const bool whole = row0 + 32 <= m && col0 + 64 <= n;
    const float *src = EF ? J.E : J.G;
    auto at = [&](int a, int c) {
        return static_cast<int64_t>(row0 + 16 * a + i) * n + col0 + 16 * c + 4 * q;
    };
    auto get = [&](const float *p, int a, int c) {
        F4 v;
        if (whole) {
            v = *reinterpret_cast<const F4 *>(p + at(a, c));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v.v[e] = row0 + 16 * a + i < m && col0 + 16 * c + 4 * q + e < n ? p[at(a, c) + e] : 0.f;
        }
        return v;
    };
    auto put = [&](float *p, int a, int c, const F4 &v) {
        if (whole) {
            *reinterpret_cast<F4 *>(p + at(a, c)) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (row0 + 16 * a + i < m && col0 + 16 * c + 4 * q + e < n)
                    p[at(a, c) + e] = v.v[e];
        }
    };
    F4 g[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            g[a][c] = get(src, a, c);
    f32x4 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            acc[a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // lane x + 16 q of step s: k = k0 + 4 q + s of row x
    const float *pr[2], *vr[4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
        pr[a] = J.P + static_cast<int64_t>(min(row0 + 16 * a + i, m - 1)) * RP + 4 * q;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        vr[c] = J.V + static_cast<int64_t>(min(col0 + 16 * c + i, n - 1)) * RP + 4 * q;
    // 32 deep per step (RP is a multiple of 32), the next one's operands ahead
    struct Step {
        f32x4 p[2][2], v[2][4];
    };
    auto load = [&](Step &S, int k0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
                S.p[u][a] = *reinterpret_cast<const f32x4 *>(pr[a] + k0 + 16 * u);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                S.v[u][c] = *reinterpret_cast<const f32x4 *>(vr[c] + k0 + 16 * u);
        }
    };
    auto mul = [&](const Step &S) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[a][c] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(S.v[u][c][s], S.p[u][a][s], acc[a][c], 0, 0, 0);
    };
    {
        Step S0, S1;
        load(S0, 0);
        int k0 = 0;
        for (; k0 + 64 < RP; k0 += 64) {
            load(S1, k0 + 32);
            mul(S0);
            load(S0, k0 + 64);
            mul(S1);
        }
        if (k0 + 32 < RP) {
            load(S1, k0 + 32);
            mul(S0);
            mul(S1);
        } else {
            mul(S0);
        }
    }
    const float oma = 1.0f - alpha;
    const float cf = ADAM ? *ad.coef : 1.0f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if constexpr (EF) {
                F4 o, d;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o.v[e] = acc[a][c][e];
                    d.v[e] = g[a][c].v[e] - o.v[e];
                }
                put(J.out, a, c, o);
                put(J.E, a, c, d);
            } else if constexpr (ADAM) {
                F4 w = get(J.W, a, c), x = get(J.m1, a, c), y = get(J.m2, a, c);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    blend::adamw_elem(cf * blend_step(g[a][c].v[e], acc[a][c][e], alpha, oma), w.v[e], x.v[e], y.v[e],
                                      ad);
                put(J.W, a, c, w);
                put(J.m1, a, c, x);
                put(J.m2, a, c, y);
            } else {
                F4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    o.v[e] = blend_step(g[a][c].v[e], acc[a][c][e], alpha, oma);
                put(J.out, a, c, o);
            }
        }
}

template <int MODE>
void launch_blend(const char *tag, const std::vector<BlendReq> &reqs, int RP, float alpha, const blend::AdamArgs &ad,
                  hipStream_t st)
{
    for (size_t c0 = 0; c0 < reqs.size(); c0 += kMaxJobs) {
        BBatch b{};
        b.count = static_cast<int>(std::min<size_t>(kMaxJobs, reqs.size() - c0));
        int64_t gx = 1, gy = 1;
        for (int i = 0; i < b.count; ++i) {
            const BlendReq &q = reqs[c0 + i];
            b.j[i] = BJob{q.G, q.out, q.m, q.n, q.P, q.V, q.W, q.m1, q.m2, q.E};
            gx = std::max(gx, cdiv(q.n, 128));
            gy = std::max(gy, cdiv(q.m, 64));
        }
        // y is limited to 65535 blocks: 4 million rows
        auto kern = blend_kernel<MODE>;
        ACSC_LAUNCH(tag, kern, dim3(static_cast<unsigned>(gx), static_cast<unsigned>(gy), b.count), dim3(256), 0, st, b,
                    RP, alpha, ad);
    }
}

}  // namespace

int pass(const char *tag, bool trans, const std::vector<PassReq> &reqs, hipStream_t st, int *splits,
         const char *red_tag)
{
    if (reqs.empty())
        return ACSC_OK;
    const int NP = reqs[0].NP;
    for (const PassReq &q : reqs)
        if (q.NP != NP || NP < 16 || NP % 16 != 0 || NP > SC_KMAX || q.nvalid < 1 || q.nvalid > NP || q.ldc % 4 != 0 ||
            !aligned(q.C, 16) || !aligned(q.part, 16))
            return set_error(ACSC_EINVAL, "fp32 product with %d thin-factor columns", q.NP);
    const Plan p = plan(reqs);
    std::vector<pass::Partials> red;
    for (size_t c0 = 0; c0 < reqs.size(); c0 += kMaxJobs) {
        Batch b{};
        b.count = static_cast<int>(std::min<size_t>(kMaxJobs, reqs.size() - c0));
        int gx = 1;
        for (int i = 0; i < b.count; ++i) {
            const PassReq &q = reqs[c0 + i];
            const int s = p.splits[c0 + i];
            const int chunk = static_cast<int>((cdiv(q.K, s) + 15) / 16 * 16);
            const int64_t ss = static_cast<int64_t>(q.M) * NP;
            const int nb = static_cast<int>(cdiv(q.M, p.rows)) * s;
            gx = std::max(gx, nb);
            b.j[i] = Job{q.A, q.lda, q.B, q.ldb, s > 1 ? q.part : q.C, s > 1 ? NP : q.ldc, ss, q.M, q.K, q.nvalid,
                         chunk, s, nb};
            if (splits)
                splits[c0 + i] = s;
            else if (s > 1)
                red.push_back(pass::Partials{q.part, ss, q.C, q.ldc, q.M, NP, s});
        }
        if (trans)
            launch<true>(tag, NP, p.rows > 16, b, gx, st);
        else
            launch<false>(tag, NP, p.rows > 16, b, gx, st);
    }
    pass::add_partials(red_tag, red, st);
    return ACSC_OK;
}

int blend(const char *tag, const std::vector<BlendReq> &reqs, int RP, float alpha, hipStream_t st,
          const blend::AdamArgs *adam, bool feedback)
{
    if (RP < 32 || RP % 32 != 0)
        return set_error(ACSC_EINVAL, "fp32 blend: padded rank %d", RP);
    const blend::AdamArgs none{};
    if (feedback)
        launch_blend<blend::kFeedback>(tag, reqs, RP, alpha, none, st);
    else if (adam)
        launch_blend<blend::kAdam>(tag, reqs, RP, alpha, *adam, st);
    else
        launch_blend<blend::kPlain>(tag, reqs, RP, alpha, none, st);
    return ACSC_OK;
}

}  // namespace f32
}  // namespace acsc
