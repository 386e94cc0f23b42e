// Grouped fp32 GEMM on the matrix cores: every product of the fp32 layer, forward and backward, and the products of
// the bf16 backward pass whose operands are carried in fp32 (operands stored as bf16 are widened on their way to LDS):
//   C[g] = epilogue( opA(A[g]) . opB(B[g]) ),   M x K times K x N, any M, N, K; one launch for all groups g.
//
// v_mfma_f32_32x32x2_f32 multiplies and adds in full fp32 at 256 flop per cycle and compute unit, the same as the
// vector pipes could do at best, but without an LDS read per multiplication: the 64 x 64 vector-FMA tile that ran
// here before read two LDS words for every two FMAs of a thread and reached 20-30 TFLOP/s of the 157 the chip has.
// Measured (8 groups, 512 x 2048 x 512): 157 -> 94 us with act and pre-activations, transposed operands 160 -> 84 us
// (103 TFLOP/s); 8 groups of 64 x 64 x 256: 34 -> 5 us; X^T dZ of 8192 x 768 x 16 in 16 splits 110 -> 12 us.
//
// Operand storage:  A_MC / B_NC false: [rows][K], contraction-contiguous;  true: [K][rows], k is the row index.
// A contraction-contiguous tile sits in LDS as [rows][32 + 4] (fragments are 16-byte reads, 9 r mod 16 is a
// permutation: no bank conflicts), the other kind as [32][rows + 8] (4-byte reads; the two half-waves read rows k
// and k + 4, 32 banks apart).  The contraction is consumed in groups of 8: half-wave h multiplies elements
// 8 g + 4 h + s in step s, the same for both operands, so one 16-byte read feeds four steps.
//
// Tiling: WM x WN x KW = 4 wavefronts; a wavefront owns TM x TN tiles of 32 x 32 and, with KW = 4, a quarter of
// every K stage (the four partial tiles are added in wavefront order through LDS): that form is for products with
// so few tiles that the chip would wait for one long chain of K stages.
#pragma once

#include "ec_common.h"

namespace ecmoe {

enum GemmF32Epilogue {
    F32_ACT = 0,      // C = act(acc); optionally Cpre = acc
    F32_MULGRAD = 1,  // C = acc * act'(aux[m][n])
};

template <typename TA, typename TB, typename TAux>
struct GemmF32Args {
    const TA* A;
    const TB* B;
    float* C;
    float* Cpre;          // F32_ACT: optional [G, M, N]
    const TAux* aux;      // F32_MULGRAD: [G, M, N]
    const int32_t* gather;  // A contraction-contiguous: row m of group g is row gather[g*M + m] of A (-1: zeros)
    int M, N, K, G;
    long long sA, sB, sC;  // elements from one group's matrix to the next
    long long k_total;     // groups cut one long contraction into pieces of K: group g has min(K, k_total - g*K)
    int tiles_m, tiles_n;
};

constexpr int F32_KS = 32;  // contraction elements per wavefront and stage

template <int WM, int WN, int KW, int TM, int TN, bool A_MC, bool B_NC, int VEC, int EPI, int ACT, typename TA, typename TB,
          typename TAux>
__global__ void __launch_bounds__(256)
gemm_f32_kernel(GemmF32Args<TA, TB, TAux> p) {
    static_assert(WM * WN * KW == 4, "four wavefronts");
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = KW * F32_KS;
    // row pitch: contraction-contiguous rows hold BK elements, the other kind holds one tile row per k
    constexpr int A_PITCH = A_MC ? BM + 8 : BK + 4, B_PITCH = B_NC ? BN + 8 : BK + 4;
    constexpr int A_ELEMS = A_MC ? BK * A_PITCH : BM * A_PITCH, B_ELEMS = B_NC ? BK * B_PITCH : BN * B_PITCH;
    constexpr int STAGE = A_ELEMS + B_ELEMS;
    constexpr int A_CH = BM * BK / VEC / 256, B_CH = BN * BK / VEC / 256;  // chunks of VEC elements per thread
    constexpr int RED = KW > 1 ? (KW - 1) * TM * TN * WM * WN * 1024 : 0;  // partial tiles of the other K slices
    __shared__ __attribute__((aligned(16))) float smem[2 * STAGE > RED ? 2 * STAGE : RED];
    typedef float vec_t __attribute__((ext_vector_type(VEC)));
    typedef TA avec_t __attribute__((ext_vector_type(VEC)));
    typedef TB bvec_t __attribute__((ext_vector_type(VEC)));

    // XCD-aware order: every XCD gets a contiguous run of tiles, the axis with fewer tiles fastest
    const int total = p.G * p.tiles_m * p.tiles_n;
    const int per_xcd = (total + 7) / 8;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= total) return;
    const bool n_fast = p.tiles_m > p.tiles_n;
    const int tm = n_fast ? (logical / p.tiles_n) % p.tiles_m : logical % p.tiles_m;
    const int tn = n_fast ? logical % p.tiles_n : (logical / p.tiles_m) % p.tiles_n;
    const int g = logical / (p.tiles_m * p.tiles_n);
    const int m0 = tm * BM, n0 = tn * BN, M = p.M, N = p.N;
    const long long left = p.k_total - (long long)g * p.K;
    const int K = left < p.K ? (int)left : p.K;
    const TA* __restrict__ A = p.A + (p.gather != nullptr ? 0 : g * p.sA);
    const TB* __restrict__ B = p.B + g * p.sB;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kw = wave / (WM * WN), wr = (wave / WN) % WM, wc = wave % WN;
    const int col = lane & 31, half = lane >> 5;

    // Chunks of this thread: pointer at stage 0, LDS element offset, and (as a limit on k) whether it exists at all.
    const TA* a_ptr[A_CH];
    const TB* b_ptr[B_CH];
    int a_lds[A_CH], b_lds[B_CH], a_k[A_CH], b_k[B_CH];
#pragma unroll
    for (int r = 0; r < A_CH; ++r) {
        const int c = tid + 256 * r;
        const int row = A_MC ? (c % (BM / VEC)) * VEC : c / (BK / VEC), k = A_MC ? c / (BM / VEC) : (c % (BK / VEC)) * VEC;
        bool in = m0 + row < M;
        size_t src = (size_t)(m0 + row);
        if (!A_MC && p.gather != nullptr && in) {
            const int s = p.gather[(size_t)g * M + m0 + row];
            in = s >= 0;
            src = (size_t)(in ? s : 0);
        }
        a_k[r] = in ? k : 0x40000000;
        a_ptr[r] = A + (A_MC ? (size_t)k * M + m0 + row : src * p.K + k);
        a_lds[r] = A_MC ? k * A_PITCH + row : row * A_PITCH + k;
    }
#pragma unroll
    for (int r = 0; r < B_CH; ++r) {
        const int c = tid + 256 * r;
        const int row = B_NC ? (c % (BN / VEC)) * VEC : c / (BK / VEC), k = B_NC ? c / (BN / VEC) : (c % (BK / VEC)) * VEC;
        b_k[r] = n0 + row < N ? k : 0x40000000;
        b_ptr[r] = B + (B_NC ? (size_t)k * N + n0 + row : (size_t)(n0 + row) * p.K + k);
        b_lds[r] = A_ELEMS + (B_NC ? k * B_PITCH + row : row * B_PITCH + k);
    }
    const size_t a_step = A_MC ? (size_t)M : 1, b_step = B_NC ? (size_t)N : 1;

    avec_t areg[A_CH];
    bvec_t breg[B_CH];
    auto load = [&](int k0) {
#pragma unroll
        for (int r = 0; r < A_CH; ++r) {
            areg[r] = avec_t(static_cast<TA>(0.0f));
            if (a_k[r] + k0 < K) areg[r] = *reinterpret_cast<const avec_t*>(a_ptr[r] + (size_t)k0 * a_step);
        }
#pragma unroll
        for (int r = 0; r < B_CH; ++r) {
            breg[r] = bvec_t(static_cast<TB>(0.0f));
            if (b_k[r] + k0 < K) breg[r] = *reinterpret_cast<const bvec_t*>(b_ptr[r] + (size_t)k0 * b_step);
        }
    };
    auto store = [&](int buf) {
        float* base = smem + buf * STAGE;
#pragma unroll
        for (int r = 0; r < A_CH; ++r) *reinterpret_cast<vec_t*>(&base[a_lds[r]]) = __builtin_convertvector(areg[r], vec_t);
#pragma unroll
        for (int r = 0; r < B_CH; ++r) *reinterpret_cast<vec_t*>(&base[b_lds[r]]) = __builtin_convertvector(breg[r], vec_t);
    };

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // fragment offsets of k group 0: element 4*half of this wavefront's slice
    const int kf = kw * F32_KS + 4 * half;
    const int a_frag = A_MC ? kf * A_PITCH + wr * TM * 32 + col : (wr * TM * 32 + col) * A_PITCH + kf;
    const int b_frag = A_ELEMS + (B_NC ? kf * B_PITCH + wc * TN * 32 + col : (wc * TN * 32 + col) * B_PITCH + kf);

    const int nk = (K + BK - 1) / BK;
    load(0);
    store(0);
    if (nk > 1) load(BK);
    __syncthreads();
    for (int kc = 0; kc < nk; ++kc) {
        const float* st = smem + (kc & 1) * STAGE;
        if (kc + 1 < nk) {
            store((kc & 1) ^ 1);  // last read before the barrier that ended stage kc - 1
            if (kc + 2 < nk) load((kc + 2) * BK);
        }
#pragma unroll
        for (int q = 0; q < F32_KS / 8; ++q) {
            floatx4 a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (A_MC) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) a[i][s] = st[a_frag + (8 * q + s) * A_PITCH + i * 32];
                } else {
                    a[i] = *reinterpret_cast<const floatx4*>(&st[a_frag + i * 32 * A_PITCH + 8 * q]);
                }
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (B_NC) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) b[j][s] = st[b_frag + (8 * q + s) * B_PITCH + j * 32];
                } else {
                    b[j] = *reinterpret_cast<const floatx4*>(&st[b_frag + j * 32 * B_PITCH + 8 * q]);
                }
            }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

    if (KW > 1) {  // slices 1.. leave their partial tiles in LDS, slice 0 adds them in slice order
        constexpr int PER_SLICE = TM * TN * WM * WN * 1024;
        float* mine = smem + (kw - 1) * PER_SLICE + (wr * WN + wc) * TM * TN * 1024;
        if (kw > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mine[((i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll
        for (int s = 0; s < KW - 1; ++s)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[i][j][r] += smem[s * PER_SLICE + (wr * WN + wc) * TM * TN * 1024 + ((i * TN + j) * 16 + r) * 64 + lane];
    }

    // acc[i][j][r] = C[row i*32 + 8*(r/4) + 4*half + r%4][column j*32 + col]: a store covers 128 contiguous bytes of two rows
    float* __restrict__ C = p.C + g * p.sC;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int gn = n0 + (wc * TN + j) * 32 + col;
            const int gm0 = m0 + (wr * TM + i) * 32 + 4 * half;
            if (gn >= N) continue;
            float aux[EPI == F32_MULGRAD ? 16 : 1];
            if (EPI == F32_MULGRAD) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int gm = gm0 + 8 * (r >> 2) + (r & 3);
                    aux[r] = gm < M ? Cvt<TAux>::to_f32(p.aux[g * p.sC + (size_t)gm * N + gn]) : 0.0f;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int gm = gm0 + 8 * (r >> 2) + (r & 3);
                if (gm >= M) continue;
                const size_t at = (size_t)gm * N + gn;
                const float v = acc[i][j][r];
                if (EPI == F32_MULGRAD) {
                    C[at] = v * act_grad<ACT>(aux[r]);
                } else {
                    if (p.Cpre != nullptr) p.Cpre[g * p.sC + at] = v;
                    C[at] = apply_act<ACT>(v);
                }
            }
        }
}

template <int WM, int WN, int KW, int TM, int TN, bool A_MC, bool B_NC, int EPI, int ACT, typename TA, typename TB,
          typename TAux>
static void gemm_f32_launch_tile(GemmF32Args<TA, TB, TAux> p, bool vec4, hipStream_t stream) {
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    const long long total = (long long)p.G * p.tiles_m * p.tiles_n;
    const dim3 grid((unsigned)((total + 7) / 8 * 8)), block(256);
    auto k4 = gemm_f32_kernel<WM, WN, KW, TM, TN, A_MC, B_NC, 4, EPI, ACT, TA, TB, TAux>;
    auto k1 = gemm_f32_kernel<WM, WN, KW, TM, TN, A_MC, B_NC, 1, EPI, ACT, TA, TB, TAux>;
    hipLaunchKernelGGL(vec4 ? k4 : k1, grid, block, 0, stream, p);
}

// One grouped product.  The largest tile that still gives every compute unit a workgroup: 128 x 128 moves half the
// operand bytes of 64 x 64 per flop, and below 256 tiles of 64 x 64 the four wavefronts of a 32 x 32 tile share K.
template <bool A_MC, bool B_NC, int EPI, int ACT, typename TA, typename TB, typename TAux>
static int gemm_f32(GemmF32Args<TA, TB, TAux> p, hipStream_t stream) {
    if (p.k_total == 0) p.k_total = (long long)p.G * p.K;
    const long long t32 = (long long)p.G * ((p.M + 31) / 32) * ((p.N + 31) / 32);
    if (t32 + 8 >= (long long)1 << 31) return EC_ERR_UNSUPPORTED;
    const bool vec4 = (A_MC ? p.M % 4 == 0 : p.K % 4 == 0) && (B_NC ? p.N % 4 == 0 : p.K % 4 == 0) && p.sA % 4 == 0 &&
                      p.sB % 4 == 0 && aligned16(p.A) && aligned16(p.B);
    auto tiles = [&](int t) { return (long long)p.G * ((p.M + t - 1) / t) * ((p.N + t - 1) / t); };
    if (tiles(128) >= 256) gemm_f32_launch_tile<2, 2, 1, 2, 2, A_MC, B_NC, EPI, ACT>(p, vec4, stream);
    else if (tiles(64) >= 256 || p.K <= F32_KS) gemm_f32_launch_tile<2, 2, 1, 1, 1, A_MC, B_NC, EPI, ACT>(p, vec4, stream);
    else gemm_f32_launch_tile<1, 1, 4, 1, 1, A_MC, B_NC, EPI, ACT>(p, vec4, stream);
    return check_launch();
}

}  // namespace ecmoe
