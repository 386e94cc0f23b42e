// Gating scores S = Softmax(X.Wg) over the expert axis (Sec. 3.2, Eq. 2; Sec. 3.4).
//
//  * gate_kernel          up to 256 experts, any storage type and width.  Computes Z^T = Wg^T.X^T on the matrix cores
//    with experts as the MFMA row axis and tokens as the column axis, 32 tokens per workgroup.
//  * gate_generic_kernel  more than 256 experts; one wavefront per token, plain fp32 FMAs.
// With more than 64 experts and enough tokens to fill the chip the product runs on the grouped-GEMM
// kernel instead (gemm_bf16.h, softmax epilogue).
#include "ec_common.h"
#include "gemm_bf16.h"

namespace ecmoe {

// ---------------------------------------------------------------------------
// A gate is bound by latency, not by bytes or flops: 8192 x 768 tokens are 12.6 MB (3 us) and two MFMAs per 16 columns
// of d.  So the four wavefronts of a workgroup all fetch -- PD phases of KC columns of 32 rows of X and of Wg are in
// flight, through registers, before the first of them is needed -- and share the staged phase in LDS; wavefront w runs
// the MFMA chains of expert tiles w, w + 4.  One wavefront per 32 tokens that fetched its own 64-column stages between
// two barriers each took 11 us on 8192 x 768 x 16 and 20 us on 16384 x 1024 x 64.
//   bf16: v_mfma_f32_32x32x16_bf16; Wg stays row-major in LDS, transposing reads (ds_read_b64_tr_b16) hand each lane
//         2 x 4 consecutive k of its expert.  Half-wave h takes columns 32 h + 8 s .. + 7 of a 64-column stage in step s.
//   fp32: v_mfma_f32_32x32x2_f32; half-wave h takes columns 4 h + s of a group of 8.  Its chain is eight times as long
//         per column, so wavefronts left over by few expert tiles take a slice of every phase instead of idling, and
//         the slices are added in order.
// Logits then go to LDS and all threads share maximum, exponentials and stores; the sum of a token runs over the
// experts with bit 2 clear in ascending order, then over those with bit 2 set, then adds the two.
// The launch also clears `zero_words` 32-bit words at `zero_buf` (counters the later stages use).
// ---------------------------------------------------------------------------
constexpr int GATE_TOK = 32;

template <typename T, int ET, bool EVEC, bool XVEC>  // EVEC / XVEC: rows of Wg / X can be read 16 bytes at a time
__global__ void __launch_bounds__(256)
gate_kernel(const T* __restrict__ X, const T* __restrict__ Wg, float* __restrict__ S, float* __restrict__ St, int n, int d,
            int e, uint32_t* __restrict__ zero_buf, int zero_words) {
    constexpr bool BF = sizeof(T) == 2;
    constexpr int E_PAD = 32 * ET;
    constexpr int VEC = 16 / (int)sizeof(T);
    constexpr int KC = BF ? (ET <= 4 ? 128 : 64) : (ET <= 4 ? 64 : 32);  // columns of d per phase
    constexpr int PD = ET <= 2 ? 3 : 2;                                   // phases in flight
    constexpr int X_PITCH = KC + VEC;
    // bf16: four consecutive rows in four 64-byte bank groups; fp32: rows k and k + 4 32 banks apart
    constexpr int W_PITCH = BF ? (ET == 1 ? 32 : E_PAD + 32) : E_PAD + 8;
    constexpr int XCH = GATE_TOK * KC / VEC, WCH = KC * E_PAD / VEC;  // 16-byte chunks per phase
    constexpr int XC = (XCH + 255) / 256, WC = (WCH + 255) / 256;
    constexpr int SLICES = BF ? 1 : (ET == 1 ? 4 : ET == 2 ? 2 : 1);  // wavefronts that share a phase of one expert tile
    constexpr int TPW = ET > 4 ? 2 : 1;                               // expert tiles per wavefront
    constexpr int Z_PITCH = GATE_TOK + 1;
    constexpr int STAGE_BYTES = (GATE_TOK * X_PITCH + KC * W_PITCH) * (int)sizeof(T);
    constexpr int Z_BYTES = (E_PAD * Z_PITCH + 10 * GATE_TOK) * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[STAGE_BYTES > Z_BYTES ? STAGE_BYTES : Z_BYTES];
    T* Xs = reinterpret_cast<T*>(smem);
    T* Ws = Xs + GATE_TOK * X_PITCH;
    typedef T vec_t __attribute__((ext_vector_type(VEC)));
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

    const int tid = threadIdx.x;
    for (int i = blockIdx.x * 256 + tid; i < zero_words; i += gridDim.x * 256) zero_buf[i] = 0u;

    const int lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5, l16 = lane & 15;
    const int tok0 = blockIdx.x * GATE_TOK;

    const vec_t zero = vec_t(static_cast<T>(0.0f));
    vec_t xq[PD][XC], wq[PD][WC];
    auto load_phase = [&](int k0, vec_t (&xr)[XC], vec_t (&wr)[WC]) {
#pragma unroll
        for (int r = 0; r < XC; ++r) {
            const int c = tid + 256 * r, row = c / (KC / VEC), k = k0 + (c % (KC / VEC)) * VEC;
            const int tok = tok0 + row < n ? tok0 + row : n - 1;  // loads are clamped, stores predicated
            const T* src = X + (size_t)tok * d + k;
            vec_t v = zero;
            if (XCH % 256 == 0 || c < XCH) {
                if (XVEC) {
                    if (k < d) v = *reinterpret_cast<const vec_t*>(src);
                } else {
#pragma unroll
                    for (int q = 0; q < VEC; ++q)
                        if (k + q < d) v[q] = src[q];
                }
            }
            xr[r] = v;
        }
#pragma unroll
        for (int r = 0; r < WC; ++r) {
            const int c = tid + 256 * r, k = k0 + c / (E_PAD / VEC), ex = (c % (E_PAD / VEC)) * VEC;
            const T* src = Wg + (size_t)k * e + ex;
            vec_t v = zero;
            if ((WCH % 256 == 0 || c < WCH) && k < d) {
                if (EVEC) {
                    if (ex < e) v = *reinterpret_cast<const vec_t*>(src);
                } else {
#pragma unroll
                    for (int q = 0; q < VEC; ++q)
                        if (ex + q < e) v[q] = src[q];
                }
            }
            wr[r] = v;
        }
    };

    floatx16 acc[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
    const int te0 = SLICES > 1 ? wave % ET : wave, slice = SLICES > 1 ? wave / ET : 0;

    const int phases = (d + KC - 1) / KC;
#pragma unroll
    for (int u = 0; u < PD; ++u)
        if (u < phases) load_phase(u * KC, xq[u], wq[u]);
    for (int p0 = 0; p0 < phases; p0 += PD) {
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            const int p = p0 + u;
            if (p >= phases) break;  // uniform
            __syncthreads();
#pragma unroll
            for (int r = 0; r < XC; ++r) {
                const int c = tid + 256 * r;
                if (XCH % 256 == 0 || c < XCH)
                    *reinterpret_cast<vec_t*>(&Xs[c / (KC / VEC) * X_PITCH + c % (KC / VEC) * VEC]) = xq[u][r];
            }
#pragma unroll
            for (int r = 0; r < WC; ++r) {
                const int c = tid + 256 * r;
                if (WCH % 256 == 0 || c < WCH)
                    *reinterpret_cast<vec_t*>(&Ws[c / (E_PAD / VEC) * W_PITCH + c % (E_PAD / VEC) * VEC]) = wq[u][r];
            }
            __syncthreads();
            if (p + PD < phases) load_phase((p + PD) * KC, xq[u], wq[u]);
            if constexpr (BF) {
                if (te0 < ET) {
#pragma unroll
                    for (int q = 0; q < KC / 64; ++q) {
                        if (p * KC + q * 64 >= d) break;
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const int k = q * 64 + half * 32 + s * 8;
                            const bf16x8 x = *reinterpret_cast<const bf16x8*>(&Xs[col * X_PITCH + k]);
#pragma unroll
                            for (int t = 0; t < TPW; ++t) {
                                const bf16_t* p0w = &Ws[(k + (l16 >> 2)) * W_PITCH + (te0 + 4 * t) * 32 +
                                                        ((lane >> 4) & 1) * 16 + (l16 & 3) * 4];
                                const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p0w));
                                const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p0w + 4 * W_PITCH));
                                const bf16x8 w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, x, acc[t], 0, 0, 0);
                            }
                        }
                    }
                }
            } else {
                if (te0 < ET) {
                    constexpr int KS = KC / SLICES;
#pragma unroll
                    for (int q = 0; q < KS / 8; ++q) {
                        const int k = slice * KS + q * 8 + half * 4;
                        const floatx4 x = *reinterpret_cast<const floatx4*>(&Xs[col * X_PITCH + k]);
#pragma unroll
                        for (int s = 0; s < 4; ++s)
#pragma unroll
                            for (int t = 0; t < TPW; ++t)
                                acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                                    Ws[(k + s) * W_PITCH + (te0 + 4 * t) * 32 + col], x[s], acc[t], 0, 0, 0);
                    }
                }
            }
        }
    }

    // acc[t][r] = Z[expert = 32*te + 8*(r/4) + 4*half + r%4][token = col]
    float* Z = reinterpret_cast<float*>(smem);         // [expert][token]
    float* red = Z + E_PAD * Z_PITCH;                  // [8][token]
    float* tot = red + 8 * GATE_TOK;                   // [2][token]
#pragma unroll
    for (int sl = 0; sl < SLICES; ++sl) {
        __syncthreads();  // the staged phase, or the previous slice, has been read
        if (te0 < ET && slice == sl) {
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float* z = &Z[((te0 + 4 * t) * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * Z_PITCH + col];
                    *z = sl == 0 ? acc[t][r] : *z + acc[t][r];
                }
        }
    }
    __syncthreads();
    const int tk = tid & 31, grp = tid >> 5;  // a token and one of eight runs through its experts
    float m = -INFINITY;
    for (int ex = grp; ex < e; ex += 8) m = fmaxf(m, Z[ex * Z_PITCH + tk]);
    red[grp * GATE_TOK + tk] = m;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) m = fmaxf(m, red[q * GATE_TOK + tk]);
    for (int ex = grp; ex < e; ex += 8) {
        const float z = Z[ex * Z_PITCH + tk] - m;
        // bf16: exp through the hardware exp2 (relative 6e-8 * |z - max| from rounding the scaled argument)
        Z[ex * Z_PITCH + tk] = BF ? __builtin_amdgcn_exp2f(z * 1.44269504088896340736f) : expf(z);
    }
    __syncthreads();
    if (grp < 2) {
        float sum = 0.0f;
        for (int ex = 4 * grp; ex < e; ex += 8)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (ex + j < e) sum += Z[(ex + j) * Z_PITCH + tk];
        tot[grp * GATE_TOK + tk] = sum;
    }
    __syncthreads();
    const float sum = tot[tk] + tot[GATE_TOK + tk];
    const float inv_sum = 1.0f / sum;
    const bool live = tok0 + tk < n;
    for (int ex = grp; ex < e; ex += 8) {
        const float p = Z[ex * Z_PITCH + tk];
        const float v = BF ? p * inv_sum : p / sum;
        if (St != nullptr && live) St[(size_t)ex * n + tok0 + tk] = v;
        if (S != nullptr) Z[ex * Z_PITCH + tk] = v;
    }
    if (S == nullptr) return;
    __syncthreads();
    const int rows = n - tok0 < GATE_TOK ? n - tok0 : GATE_TOK;
    float* out = S + (size_t)tok0 * e;  // the rows of the block are contiguous in S
    for (int i = tid; i < rows * e; i += 256) out[i] = Z[(i % e) * Z_PITCH + i / e];
}

__global__ void __launch_bounds__(256)
zero_words_kernel(uint32_t* __restrict__ p, long long count) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long long)gridDim.x * 256) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Generic gate: one wavefront per token, lanes split the model dimension,
// experts in chunks of 16, logits staged in LDS, softmax by the same wavefront.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
gate_generic_kernel(const T* __restrict__ X, const T* __restrict__ Wg, float* __restrict__ S,
                    float* __restrict__ St, int n, int d, int e) {
    __shared__ float z[4][EC_MOE_MAX_EXPERTS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int tok = blockIdx.x * 4 + wave; tok < n; tok += gridDim.x * 4) {
        const T* xrow = X + (size_t)tok * d;
        for (int i0 = 0; i0 < e; i0 += 16) {
            float acc[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = 0.0f;
            for (int t = lane; t < d; t += kWave) {
                float x = Cvt<T>::to_f32(xrow[t]);
                const T* wrow = Wg + (size_t)t * e + i0;
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (i0 + j < e) acc[j] = fmaf(x, Cvt<T>::to_f32(wrow[j]), acc[j]);
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                float v = wave_reduce_sum(acc[j]);
                if (lane == 0 && i0 + j < e) z[wave][i0 + j] = v;
            }
        }
        __builtin_amdgcn_wave_barrier();
        __threadfence_block();
        float m = -INFINITY;
        for (int i = lane; i < e; i += kWave) m = fmaxf(m, z[wave][i]);
        m = wave_reduce_max(m);
        float sum = 0.0f;
        for (int i = lane; i < e; i += kWave) sum += expf(z[wave][i] - m);
        sum = wave_reduce_sum(sum);
        for (int i = lane; i < e; i += kWave) {
            float v = expf(z[wave][i] - m) / sum;
            if (S != nullptr) S[(size_t)tok * e + i] = v;
            if (St != nullptr) St[(size_t)i * n + tok] = v;
        }
        __builtin_amdgcn_wave_barrier();
        __threadfence_block();
    }
}

int launch_gate(const void* X, const void* Wg, float* S, float* St, int64_t n, int64_t d, int64_t e,
                int dtype, uint32_t* zero_buf, int64_t zero_words, hipStream_t stream) {
    // Many experts and many tokens: X.Wg is a real matrix product.  It runs on the grouped-GEMM kernel
    // (one group, all experts inside one tile) whose epilogue does the softmax and clears the counters.
    if (dtype == EC_BF16 && (d % 64) == 0 && (e % 8) == 0 && e > 64 && e <= 256 && gemm_bf16_shape_ok(n, e, d)) {
        if (e > 128 && n >= 128 * 256) {
            gemm_bf16_launch<256, 256, 2, 1, false, false, EPI_SOFTMAX, EC_ACT_IDENTITY>(
                (const bf16_t*)X, (const bf16_t*)Wg, St, S, 1, (int)n, (int)e, (int)d,
                reinterpret_cast<const int32_t*>(zero_buf), (int)zero_words, stream);
            return check_launch();
        }
        if (e <= 128 && n >= 128 * 128) {
            gemm_bf16_launch<128, 128, 1, 2, false, false, EPI_SOFTMAX, EC_ACT_IDENTITY>(
                (const bf16_t*)X, (const bf16_t*)Wg, St, S, 1, (int)n, (int)e, (int)d,
                reinterpret_cast<const int32_t*>(zero_buf), (int)zero_words, stream);
            return check_launch();
        }
    }
    if (e <= 256) {
        const int vec = 16 / (int)elem_size(dtype);
        const bool ev = e % vec == 0, xv = d % vec == 0;
        const dim3 grid((unsigned)ceil_div(n, GATE_TOK)), block(256);
#define EC_GATE_LAUNCH(T, ETV, EV, XV)                                                                              \
    hipLaunchKernelGGL((gate_kernel<T, ETV, EV, XV>), grid, block, 0, stream, (const T*)X, (const T*)Wg, S, St, (int)n, \
                       (int)d, (int)e, zero_buf, (int)zero_words)
#define EC_GATE_ET(T, EV, XV)                                  \
    do {                                                       \
        if (e <= 32) EC_GATE_LAUNCH(T, 1, EV, XV);             \
        else if (e <= 64) EC_GATE_LAUNCH(T, 2, EV, XV);        \
        else if (e <= 128) EC_GATE_LAUNCH(T, 4, EV, XV);       \
        else EC_GATE_LAUNCH(T, 8, EV, XV);                     \
    } while (0)
#define EC_GATE_TYPE(T)                                        \
    do {                                                       \
        if (ev && xv) EC_GATE_ET(T, true, true);               \
        else if (xv) EC_GATE_ET(T, false, true);               \
        else EC_GATE_ET(T, false, false);                      \
    } while (0)
        if (dtype == EC_BF16) EC_GATE_TYPE(bf16_t);
        else EC_GATE_TYPE(float);
#undef EC_GATE_TYPE
#undef EC_GATE_ET
#undef EC_GATE_LAUNCH
        return check_launch();
    }
    if (zero_words > 0) {
        long long zb = (zero_words + 255) / 256;
        hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)(zb > 4096 ? 4096 : zb)), dim3(256), 0, stream, zero_buf,
                           (long long)zero_words);
    }
    int64_t blocks = ceil_div(n, 4);
    if (blocks > 65536) blocks = 65536;
    if (dtype == EC_BF16)
        hipLaunchKernelGGL(gate_generic_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, stream,
                           (const bf16_t*)X, (const bf16_t*)Wg, S, St, (int)n, (int)d, (int)e);
    else
        hipLaunchKernelGGL(gate_generic_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream,
                           (const float*)X, (const float*)Wg, S, St, (int)n, (int)d, (int)e);
    return check_launch();
}

}  // namespace ecmoe
