// Expert FFN: X_e[i] = act(X_in[i].W1[i]).W2[i] for every expert i (Sec. 3.2, Eq. 3).
//
// Two grouped (one launch covers all experts) GEMMs: A = X_in.W1 with the
// activation fused into the epilogue, then X_e = H.W2.
//  * bf16: matrix cores (v_mfma_f32_32x32x16_bf16), fp32 accumulation, LDS-staged
//    tiles (gemm_bf16.h).  Both products are "row-major x row-major": the left
//    operand is contraction-contiguous and read from LDS as 16-byte fragments;
//    the right operand (the weights) keeps its own [k][columns] form in LDS and
//    its fragments come from transposing LDS reads.
//  * fp32: matrix cores too (v_mfma_f32_32x32x2_f32, gemm_f32.h).
#include <cmath>

#include "ec_common.h"
#include "gemm_bf16.h"
#include "gemm_f32.h"

namespace ecmoe {

// True when the matrix-core kernel covers the product (with rows gathered from a [gather_rows, K] matrix if asked).
// The left operand is contraction-contiguous, the right one keeps k as its row index: past K (any multiple of 8) the
// buffer range check hands out zeros for both (the left operand's offsets are moved out of range for the last stage).
static bool gemm_bf16_fast_ok(int64_t M, int64_t N, int64_t K, bool gather, int64_t gather_rows) {
    constexpr int64_t most = ((int64_t)1 << 32) - (1 << 20);  // bytes of a group's matrix: 32-bit unsigned offsets
    return (K % 8) == 0 && (N % 8) == 0 && M * K * 2 < most && (K + 128) * N * 2 < most && M * N < (int64_t)1 << 31 &&
           (!gather || gather_rows * K * 2 < ((int64_t)1 << 31) - 65536);
}

template <int BM, int BN, int STAGES, int OCC>
static int launch_gemm_bf16(const bf16_t* A, const bf16_t* B, bf16_t* C, bf16_t* Cpre, int G, int M, int N, int K,
                            int act, const int32_t* gather, int gather_rows, hipStream_t stream, bf16_t* Clo) {
#define EC_GEMM_CASE(ACTV)                                                                                       \
    if (Cpre) gemm_bf16_launch<BM, BN, STAGES, OCC, false, false, EPI_ACT_SAVE, ACTV>(                           \
                  A, B, C, Cpre, G, M, N, K, gather, gather_rows, stream, nullptr, nullptr, Clo);                \
    else gemm_bf16_launch<BM, BN, STAGES, OCC, false, false, EPI_ACT, ACTV>(A, B, C, nullptr, G, M, N, K, gather, \
                                                                           gather_rows, stream, nullptr, nullptr, Clo)
    if (act == EC_ACT_RELU) { EC_GEMM_CASE(EC_ACT_RELU); }
    else if (act == EC_ACT_GELU) { EC_GEMM_CASE(EC_ACT_GELU); }
    else { EC_GEMM_CASE(EC_ACT_IDENTITY); }
#undef EC_GEMM_CASE
    return check_launch();
}

// Tile configuration of a grouped product: the candidate with the lowest estimated time, taken as
// (rounds of 256 compute units) x (tile area) / (relative rate of that configuration).
static int gemm_tile_pick(int G, int M, int N, int K) {
    auto cost = [&](int bm, int bn, int occ, double rate) {
        double tiles = (double)G * ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        double rounds = std::ceil(tiles / (256.0 * occ)) * occ;
        return rounds * bm * bn / rate;
    };
    const double c0 = cost(256, 256, 1, 1.0), c1 = cost(256, 128, 1, 0.85), c2 = cost(128, 128, 2, 0.6);
    const double c4 = cost(256, 192, 1, 0.95);  // fills the chip exactly when 256 x 256 tiles leave units idle
    int pick = (c0 <= c1 && c0 <= c2) ? 0 : (c1 <= c2 ? 1 : 2);
    if (c4 < c0 && c4 < c1 && c4 < c2) pick = 4;
    // Short contractions leave the epilogue (activation, stores) as large as the MFMA phase: 128 x 128 tiles, two
    // workgroups per compute unit, overlap one's epilogue with the other's MFMAs.  Measured with the GeLU epilogue:
    // K = 768 (16 x 1024 x 3072): 103 us against 105 (256 x 256) and 111 (256 x 128 pairs); from K = 1024 on
    // (64 x 512 x 4096) the 256 x 256 tile wins, 344 us against 356 and 369.
    if (pick == 0 && K <= 768 && cost(128, 128, 2, 1.0) <= 1.25 * c0) pick = 2;
    return pick;
}

// Clo (optional): receives act(acc) - C, the part of the activated value that the bf16 rounding of C dropped.
static int gemm_bf16_dispatch(const bf16_t* A, const bf16_t* B, bf16_t* C, bf16_t* Cpre, int G, int M, int N,
                              int K, int act, const int32_t* gather, int gather_rows, hipStream_t stream,
                              bf16_t* Clo = nullptr) {
    if (!gemm_bf16_fast_ok(M, N, K, gather != nullptr, gather_rows)) return EC_ERR_UNSUPPORTED;
    switch (gemm_tile_pick(G, M, N, K)) {
        case 1: return launch_gemm_bf16<256, 128, 2, 1>(A, B, C, Cpre, G, M, N, K, act, gather, gather_rows, stream, Clo);
        case 2: return launch_gemm_bf16<128, 128, 1, 2>(A, B, C, Cpre, G, M, N, K, act, gather, gather_rows, stream, Clo);
        case 4: return launch_gemm_bf16<256, 192, 2, 1>(A, B, C, Cpre, G, M, N, K, act, gather, gather_rows, stream, Clo);
        default: return launch_gemm_bf16<256, 256, 2, 1>(A, B, C, Cpre, G, M, N, K, act, gather, gather_rows, stream, Clo);
    }
}

// The second product of Eq. 3 with its left operand carried as high part + remainder (A + Alo): C32 (fp32) = the
// product unrounded, Cb (bf16, optional) = the same rounded.  The tile is chosen for the doubled contraction.
static int gemm_bf16_dispatch_split(const bf16_t* A, const bf16_t* Alo, const bf16_t* B, float* C32, bf16_t* Cb, int G,
                                    int M, int N, int K, hipStream_t stream) {
    if (!gemm_bf16_shape_ok(M, N, K)) return EC_ERR_UNSUPPORTED;
#define EC_SPLIT_CASE(BM, BN, ST, OCC)                                                                              \
    gemm_bf16_launch<BM, BN, ST, OCC, false, false, EPI_F32, EC_ACT_IDENTITY, SPLIT_LEFT>(A, B, C32, nullptr, G, M, N, K, \
                                                                                         nullptr, 0, stream, nullptr, Alo, Cb)
    switch (gemm_tile_pick(G, M, N, 2 * K)) {
        case 1: EC_SPLIT_CASE(256, 128, 2, 1); break;
        case 2: EC_SPLIT_CASE(128, 128, 1, 2); break;
        case 4: EC_SPLIT_CASE(256, 192, 2, 1); break;
        default: EC_SPLIT_CASE(256, 256, 2, 1); break;
    }
#undef EC_SPLIT_CASE
    return check_launch();
}

// ===========================================================================
// fp32 products (gemm_f32.h): C = act(A.B), optionally the pre-activations too.
// ===========================================================================
static int launch_gemm_f32(const float* A, const float* B, float* C, float* Cpre, int G, int M, int N, int K,
                           int act, const int32_t* gather, hipStream_t stream) {
    GemmF32Args<float, float, float> p = {};
    p.A = A; p.B = B; p.C = C; p.Cpre = Cpre; p.gather = gather;
    p.M = M; p.N = N; p.K = K; p.G = G;
    p.sA = (long long)M * K; p.sB = (long long)K * N; p.sC = (long long)M * N;
    if (act == EC_ACT_RELU) return gemm_f32<false, true, F32_ACT, EC_ACT_RELU>(p, stream);
    if (act == EC_ACT_GELU) return gemm_f32<false, true, F32_ACT, EC_ACT_GELU>(p, stream);
    return gemm_f32<false, true, F32_ACT, EC_ACT_IDENTITY>(p, stream);
}

// ---------------------------------------------------------------------------
// Xe = act(Xin.W1).W2 ; H is the [e,k,d_ff] hidden buffer (workspace or caller's).
// ---------------------------------------------------------------------------
// True when the first product can gather its rows straight from X (no X_in buffer needed).
// It is used only while X is small (16 MiB: it then stays in the L2 caches): the tile loader reads every bucket row
// once per column of tiles, and rows scattered over a large X cost more there than one pass of the dispatch kernel
// (measured: 8192 x 768 tokens, gathered product 99 us against 103 + 13 for the dispatch; 16384 x 1024 tokens,
// 383 us against 344 + 25).
bool ffn_can_gather(int dtype, int64_t n, int64_t k, int64_t d, int64_t d_ff) {
    if (dtype == EC_F32) return n * d * 4 <= ((int64_t)16 << 20);
    return dtype == EC_BF16 && k > 0 && n * d * 2 <= ((int64_t)16 << 20) && gemm_bf16_fast_ok(k, d_ff, d, true, n);
}


// True when the products can carry H as high part + remainder (the matrix-core kernel covers both shapes).
bool ffn_can_hilo(int dtype, int64_t k, int64_t d, int64_t d_ff) {
    return dtype == EC_BF16 && k > 0 && gemm_bf16_shape_ok(k, d_ff, d) && gemm_bf16_shape_ok(k, d, d_ff);
}

// Xin == nullptr: gather mode, rows of the buckets are read from X through I (needs ffn_can_gather).
// H_lo / Xe32 (both or neither; need ffn_can_hilo): the first product also leaves H_lo = act(A) - H, the second
// multiplies (H + H_lo) by W2 and writes X_e unrounded to Xe32 [e,k,d] (fp32), and rounded to Xe if Xe is given.
int launch_ffn(const void* Xin, const void* X, const int32_t* I, int64_t n, const void* W1, const void* W2, void* Xe,
               void* A_save, void* H, int64_t e, int64_t k, int64_t d, int64_t d_ff, int act, int dtype,
               hipStream_t stream, void* H_lo, float* Xe32) {
    const int G = (int)e, M = (int)k;
    if (dtype == EC_BF16) {
        int rc;
        if (Xin == nullptr)
            rc = gemm_bf16_dispatch((const bf16_t*)X, (const bf16_t*)W1, (bf16_t*)H, (bf16_t*)A_save, G, M, (int)d_ff,
                                    (int)d, act, I, (int)n, stream, (bf16_t*)H_lo);
        else
            rc = gemm_bf16_dispatch((const bf16_t*)Xin, (const bf16_t*)W1, (bf16_t*)H, (bf16_t*)A_save, G, M, (int)d_ff,
                                    (int)d, act, nullptr, 0, stream, (bf16_t*)H_lo);
        if (rc != EC_OK) return rc;
        if (H_lo != nullptr)
            return gemm_bf16_dispatch_split((const bf16_t*)H, (const bf16_t*)H_lo, (const bf16_t*)W2, Xe32, (bf16_t*)Xe, G,
                                            M, (int)d, (int)d_ff, stream);
        return gemm_bf16_dispatch((const bf16_t*)H, (const bf16_t*)W2, (bf16_t*)Xe, nullptr, G, M, (int)d, (int)d_ff,
                                  EC_ACT_IDENTITY, nullptr, 0, stream);
    }
    if (H_lo != nullptr) return EC_ERR_UNSUPPORTED;
    int rc = launch_gemm_f32((const float*)(Xin ? Xin : X), (const float*)W1, (float*)H, (float*)A_save, G, M, (int)d_ff,
                             (int)d, act, Xin ? nullptr : I, stream);
    if (rc != EC_OK) return rc;
    return launch_gemm_f32((const float*)H, (const float*)W2, (float*)Xe, nullptr, G, M, (int)d, (int)d_ff,
                           EC_ACT_IDENTITY, nullptr, stream);
}

}  // namespace ecmoe
