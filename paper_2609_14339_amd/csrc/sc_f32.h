// fp32 products of the spectral corrector and of PowerSGD (internal; not part
// of the ABI): the thin products with a large fp32 matrix, and the blend of
// an fp32 gradient.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "sc_blend.h"

namespace acsc {
namespace f32 {

// C = A B or A^T B: A [M, K] row-major with row stride lda (or stored [K, M]),
// B [K, ldb] of which columns >= nvalid read as zero, C [M, NP] with row
// stride ldc, NP a multiple of 16 up to SC_KMAX.
struct PassReq {
    const float *A;
    int64_t lda;
    const float *B;
    int64_t ldb;
    float *C;
    int64_t ldc;
    int M, K, nvalid, NP;
    float *part;     // room for `cap` partials of M * NP floats
    int cap;
};

// Enqueue the products (one NP per call).  With `splits` a product that was
// cut along k is left in its partials (stride M * NP, row stride NP), as by
// pass::run; without it C always holds the product.
int pass(const char *tag, bool trans, const std::vector<PassReq> &reqs, hipStream_t st, int *splits = nullptr,
         const char *red_tag = "sc_split_reduce");

// out = alpha G + (1 - alpha) P V^T with P [m, RP] and V [n, RP] zero-padded to
// RP (a multiple of 32); with `adam` the blended values are the gradient of
// the AdamW step of W, m1, m2; with `feedback` out = P V^T and E takes
// E - out.
struct BlendReq {
    const float *G;
    float *out;
    int m, n;
    const float *P, *V;
    float *W, *m1, *m2;
    float *E;
};
int blend(const char *tag, const std::vector<BlendReq> &reqs, int RP, float alpha, hipStream_t st,
          const blend::AdamArgs *adam, bool feedback);

}  // namespace f32
}  // namespace acsc
