// Dispatch ("shuffle", Sec. 3.2 Eq. 3 first line) and combine ("unshuffle", Eq. 4).
//
// dispatch: X_in[i,j,:] = X[I[i,j],:] -- a row gather with 16-byte lanes (I = -1: a row of zeros).
// combine:  X_out[l,:] = sum_{(i,j): I[i,j]=l} G[i,j] X_e[i,j,:], deterministic.
//   A token-major index is built from I with integer atomics only (see below); one group of
//   lanes per token then adds that token's bucket rows in ascending expert order in fp32.
#include <mutex>

#include "ec_common.h"

namespace ecmoe {

// Scratch of ec_moe_combine_static: the token-major index lives here instead of in a caller's
// workspace.  One copy per GPU, held until the process ends; every call on a GPU shares it.
static __device__ __align__(256) unsigned char scratch[EC_MOE_STATIC_SCRATCH_BYTES];

// ------------------------------------------------------------------ dispatch
// One row per group of `tpr` threads; each thread moves 16 bytes per step.
__global__ void __launch_bounds__(256)
dispatch_kernel(const uint4* __restrict__ X, const int32_t* __restrict__ I, uint4* __restrict__ Xin,
                long long rows, int vec_per_row, int tpr) {
    const int rows_per_block = 256 / tpr;
    const int sub = threadIdx.x / tpr, t = threadIdx.x % tpr;
    for (long long r = (long long)blockIdx.x * rows_per_block + sub; r < rows;
         r += (long long)gridDim.x * rows_per_block) {
        const int tok = I[r];  // -1: an empty buffer row (token-choice routing), filled with zeros
        const uint4* src = X + (size_t)(tok < 0 ? 0 : tok) * vec_per_row;
        uint4* dst = Xin + (size_t)r * vec_per_row;
        for (int v = t; v < vec_per_row; v += tpr) dst[v] = tok < 0 ? make_uint4(0u, 0u, 0u, 0u) : src[v];
    }
}

// Rows whose byte length is not a multiple of 16 (fp32 with d % 4 != 0).
__global__ void __launch_bounds__(256)
dispatch_scalar_kernel(const float* __restrict__ X, const int32_t* __restrict__ I, float* __restrict__ Xin,
                       long long rows, int d) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (long long r = (long long)blockIdx.x * 4 + wave; r < rows; r += (long long)gridDim.x * 4) {
        const int tok = I[r];
        const float* src = X + (size_t)(tok < 0 ? 0 : tok) * d;
        float* dst = Xin + (size_t)r * d;
        for (int v = lane; v < d; v += kWave) dst[v] = tok < 0 ? 0.0f : src[v];
    }
}

static int pick_threads_per_row(int64_t vec_per_row) {
    int tpr = 8;
    while (tpr < 256 && tpr < vec_per_row) tpr <<= 1;
    return tpr;
}

int launch_dispatch(const void* X, const int32_t* I, void* Xin, int64_t n, int64_t d, int64_t e, int64_t k,
                    int dtype, hipStream_t stream) {
    (void)n;
    const long long rows = (long long)e * k;
    const size_t row_bytes = (size_t)d * elem_size(dtype);
    if (row_bytes % 16 == 0) {
        int vec = (int)(row_bytes / 16);
        int tpr = pick_threads_per_row(vec);
        long long blocks = ceil_div(rows, 256 / tpr);
        if (blocks > (1 << 20)) blocks = 1 << 20;
        hipLaunchKernelGGL(dispatch_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint4*)X, I,
                           (uint4*)Xin, rows, vec, tpr);
    } else {
        long long blocks = ceil_div(rows, 4);
        if (blocks > (1 << 20)) blocks = 1 << 20;
        hipLaunchKernelGGL(dispatch_scalar_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const float*)X,
                           I, (float*)Xin, rows, (int)d);
    }
    return check_launch();
}

// ------------------------------------------------------------------- combine
// Token-major index of the routing (CombineIndex), built with integer stores and ORs only, so it never depends on
// timing.  Lists of the other form: offsets = exclusive scan of the bitmap's popcounts,
// inv[offsets[l] + (number of set bits below i)] = i*k + j -- expert-ascending.
__global__ void __launch_bounds__(256)
fill_u32_kernel(uint32_t* __restrict__ p, long long count, uint32_t v) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long long)gridDim.x * 256) p[i] = v;
}

__global__ void __launch_bounds__(256)
index_kernel(const int32_t* __restrict__ I, uint32_t* __restrict__ bitmap, int32_t* __restrict__ pos, long long rows, int k,
             int words, int e) {
    for (long long r = (long long)blockIdx.x * 256 + threadIdx.x; r < rows; r += (long long)gridDim.x * 256) {
        const int i = (int)(r / k), l = I[r];
        if (l < 0) continue;  // empty buffer row
        if (pos != nullptr) pos[(size_t)l * e + i] = (int32_t)r;
        atomicOr(&bitmap[(size_t)l * words + (i >> 5)], 1u << (i & 31));
    }
}

// Exclusive scan of per-token expert counts (popcounts of the bitmap rows) in two launches:
// block_counts_kernel sums the counts of each block's token range; offsets_kernel adds up the
// totals of the blocks before it (at most 1024 of them, one per thread) and scans its own range.
// A block owns `tpb` consecutive tokens (a multiple of 1024), walked 1024 at a time so that
// loads stay coalesced.
__device__ __forceinline__ unsigned int token_count(const uint32_t* __restrict__ bitmap, int l, int n, int words) {
    unsigned int v = 0;
    if (l < n)
        for (int w = 0; w < words; ++w) v += __popc(bitmap[(size_t)l * words + w]);
    return v;
}

__device__ __forceinline__ unsigned int block_sum_1024(unsigned int v, unsigned int* red /*[16]*/) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    __syncthreads();  // red may still be read from a previous use
    if (lane == 0) red[wave] = v;
    __syncthreads();
    unsigned int total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) total += red[w];
    return total;
}

__global__ void __launch_bounds__(1024)
block_counts_kernel(const uint32_t* __restrict__ bitmap, uint32_t* __restrict__ block_tot, int n, int words, int tpb) {
    __shared__ unsigned int red[16];
    const int beg = blockIdx.x * tpb;
    unsigned int v = 0;
    for (int l0 = beg; l0 < beg + tpb && l0 < n; l0 += 1024) v += token_count(bitmap, l0 + threadIdx.x, n, words);
    const unsigned int total = block_sum_1024(v, red);
    if (threadIdx.x == 0) block_tot[blockIdx.x] = total;
}

__global__ void __launch_bounds__(1024)
offsets_kernel(const uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ block_tot,
               int32_t* __restrict__ offsets, int n, int words, int tpb) {
    __shared__ unsigned int red[16];
    __shared__ unsigned int wave_tot[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned int carry = block_sum_1024(tid < (int)blockIdx.x ? block_tot[tid] : 0u, red);  // gridDim.x <= 1024
    const int beg = blockIdx.x * tpb;
    for (int l0 = beg; l0 < beg + tpb && l0 < n; l0 += 1024) {
        const int l = l0 + tid;
        const unsigned int c = token_count(bitmap, l, n, words);
        unsigned int incl = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            unsigned int o = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += o;
        }
        __syncthreads();  // wave_tot of the previous round has been read
        if (lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        unsigned int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            unsigned int t = wave_tot[w];
            before += w < wave ? t : 0u;
            total += t;
        }
        if (l < n) offsets[l] = (int32_t)(carry + before + incl - c);
        carry += total;
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) offsets[n] = (int32_t)carry;
}

__global__ void __launch_bounds__(256)
inverse_index_kernel(const int32_t* __restrict__ I, const uint32_t* __restrict__ bitmap,
                     const int32_t* __restrict__ offsets, int32_t* __restrict__ inv, long long rows, int k,
                     int words) {
    for (long long r = (long long)blockIdx.x * 256 + threadIdx.x; r < rows; r += (long long)gridDim.x * 256) {
        int i = (int)(r / k);
        int l = I[r];
        if (l < 0) continue;  // empty buffer row
        const uint32_t* bm = bitmap + (size_t)l * words;
        int rank = 0;
        for (int w = 0; w < (i >> 5); ++w) rank += __popc(bm[w]);
        rank += __popc(bm[i >> 5] & ((1u << (i & 31)) - 1u));
        inv[offsets[l] + rank] = (int32_t)r;
    }
}

// One token per group of `tpr` lanes of a wavefront, nothing shared between groups.  Bound by memory, and on small
// batches by the chain bitmap -> bucket row -> weight -> row: lane q of the group resolves entry q of the token's list, so
// the chain is walked once per token however many experts chose it, all tokens a wavefront slot can hold are in flight,
// and no barrier ties them together (blocks that resolved a run of tokens into LDS first took 19 us on 8192 x 768, 42 on
// 16384 x 1024 and 199 on 65536 x 4096; now 10, 23 and 160, the last at 6 TB/s).  Then the group streams the rows, U pieces
// of 16 bytes per lane at a time (8 bf16 / 4 fp32), entry by entry in list order, fp32 sums, rounded once.
template <typename T, int VEC, int U, bool LISTS, typename TRow = T>
__global__ void __launch_bounds__(256)
combine_kernel(const TRow* __restrict__ Xe, const float* __restrict__ G, const uint32_t* __restrict__ bitmap,
               const int32_t* __restrict__ pos, const int32_t* __restrict__ offsets, const int32_t* __restrict__ inv,
               T* __restrict__ Xout, int n, int d, int e, int tpr, const float* __restrict__ addend,
               const int32_t* __restrict__ src_rows) {
    typedef T vec_t __attribute__((ext_vector_type(VEC)));
    typedef TRow row_vec_t __attribute__((ext_vector_type(VEC)));  // bucket rows may be fp32 where the output is bf16
    typedef float add_vec_t __attribute__((ext_vector_type(VEC)));
    const int t = threadIdx.x & (tpr - 1);
    const long long l = (long long)blockIdx.x * (256 / tpr) + threadIdx.x / tpr;
    if (l >= n) return;
    const int vec_per_row = d / VEC, words = (e + 31) >> 5;
    // Entry q of the token's list (expert-ascending): source row and weight.  src_rows: bucket row r is row src_rows[r] of
    // Xe (identity experts: X_e[i,j,:] = X[I[i,j],:], the gather of Eq. 3 read in place instead of through a materialised
    // X_in); no weights: plain scatter-add of rows.  Returns the length of the list.
    auto entry = [&](int q, int& src, float& g) -> int {
        int cnt = 0, r = -1;
        if (LISTS) {
            const int beg = offsets[l];
            cnt = offsets[l + 1] - beg;
            if (q < cnt) r = inv[beg + q];
        } else {
            uint32_t mine = 0u;
            int at = 0, ex = 0;
#pragma unroll 4
            for (int w = 0; w < words; ++w) {
                const uint32_t m = bitmap[l * words + w];
                const int c = __popc(m);
                if (q >= cnt && q < cnt + c) {
                    mine = m;
                    at = q - cnt;
                    ex = 32 * w;
                }
                cnt += c;
            }
            if (q < cnt) {
                for (; at > 0; --at) mine &= mine - 1u;
                r = pos[l * e + ex + __ffs(mine) - 1];
            }
        }
        src = r;
        g = 1.0f;
        if (r >= 0) {
            if (src_rows != nullptr) src = src_rows[r];
            if (G != nullptr) g = G[r];
        }
        return cnt;
    };
    int src;
    float g;
    const int cnt = entry(t, src, g);
    for (int v0 = 0; v0 < vec_per_row; v0 += tpr * U) {
        float acc[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = v0 + u * tpr + t;
            add_vec_t a = add_vec_t(0.0f);
            if (addend != nullptr && v < vec_per_row) a = *reinterpret_cast<const add_vec_t*>(addend + l * d + (long long)v * VEC);
#pragma unroll
            for (int q = 0; q < VEC; ++q) acc[u][q] = a[q];
        }
        for (int p0 = 0; p0 < cnt; p0 += tpr) {
            if (cnt > tpr) entry(p0 + t, src, g);  // more experts than lanes: a batch of the list at a time
            const int batch = cnt - p0 < tpr ? cnt - p0 : tpr;
            for (int p = 0; p < batch; ++p) {
                const TRow* row = Xe + (size_t)__shfl(src, p, tpr) * d;
                const float w = __shfl(g, p, tpr);
                row_vec_t x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int v = v0 + u * tpr + t;
                    if (v < vec_per_row) x[u] = *reinterpret_cast<const row_vec_t*>(row + (size_t)v * VEC);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[u][q] = fmaf(w, Cvt<TRow>::to_f32(x[u][q]), acc[u][q]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = v0 + u * tpr + t;
            vec_t o;
#pragma unroll
            for (int q = 0; q < VEC; ++q) o[q] = Cvt<T>::from_f32(acc[u][q]);
            if (v < vec_per_row) *reinterpret_cast<vec_t*>(Xout + l * d + (long long)v * VEC) = o;
        }
    }
}

// Lanes per token: as many as the row fills without leaving more than it must idle in the last step.
static int combine_threads_per_row(int64_t vec_per_row) {
    int tpr = 64;
    while (tpr > 16 && align_up((size_t)vec_per_row, tpr / 2) < align_up((size_t)vec_per_row, tpr)) tpr /= 2;
    return tpr;
}

static unsigned blocks_for(long long items) {
    long long b = (items + 255) / 256;
    return (unsigned)(b > 16384 ? 16384 : (b < 1 ? 1 : b));
}

// Lists from a filled bitmap: offsets (exclusive scan) and the expert-ascending row lists.
static void launch_index_lists(const int32_t* I, int64_t n, int64_t e, int64_t k, const CombineIndex& ix, hipStream_t stream) {
    const long long rows = (long long)e * k;
    const int words = (int)ceil_div(e, 32);
    // token range of a scan block: 1024 tokens, more only when that would need over 1024 blocks
    const int tpb = (int)(ceil_div(ceil_div(n, 1024), 1024) * 1024);
    const unsigned scan_blocks = (unsigned)ceil_div(n, tpb);
    hipLaunchKernelGGL(block_counts_kernel, dim3(scan_blocks), dim3(1024), 0, stream, ix.bitmap, ix.block_tot, (int)n,
                       words, tpb);
    hipLaunchKernelGGL(offsets_kernel, dim3(scan_blocks), dim3(1024), 0, stream, ix.bitmap, ix.block_tot, ix.offsets,
                       (int)n, words, tpb);
    hipLaunchKernelGGL(inverse_index_kernel, dim3(blocks_for(rows)), dim3(256), 0, stream, I, ix.bitmap, ix.offsets,
                       ix.inv, rows, (int)k, words);
}

// Builds the token-major index from I alone (stand-alone combine, backward pass; the forward pass gets it
// from the gate and top-k kernels instead).
int launch_combine_index(const int32_t* I, int64_t n, int64_t e, int64_t k, const CombineIndex& ix,
                         hipStream_t stream, bool bitmap_is_zero) {
    const long long rows = (long long)e * k;
    if (!bitmap_is_zero)
        hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks_for(combine_zero_words(n, e))), dim3(256), 0, stream, ix.bitmap,
                           (long long)combine_zero_words(n, e), 0u);
    hipLaunchKernelGGL(index_kernel, dim3(blocks_for(rows)), dim3(256), 0, stream, I, ix.bitmap, ix.pos, rows, (int)k,
                       (int)ceil_div(e, 32), (int)e);
    if (ix.pos == nullptr) launch_index_lists(I, n, e, k, ix, stream);
    return check_launch();
}

// Applies Eq. 4 given a filled index.
// G == nullptr adds the rows unweighted; `addend` (fp32 [n,d], optional) is the starting value of every row;
// `src_rows` (optional, [e*k]) redirects bucket row r to row src_rows[r] of Xe; `rows_f32`: the bucket rows are
// fp32 although the output is bf16 (the last product of the backward pass is kept unrounded).
int launch_combine(const void* Xe, const float* G, const int32_t* I, void* Xout, int64_t n, int64_t d,
                   int64_t e, int64_t k, int dtype, const CombineIndex& ix, hipStream_t stream,
                   const float* addend, const int32_t* src_rows, bool rows_f32) {
    (void)I; (void)k;
#define EC_COMBINE_LAUNCH(TYPE, VECV, TROW)                                                                              \
    do {                                                                                                                 \
        const int tpr = combine_threads_per_row(d / VECV);                                                               \
        auto dense2 = combine_kernel<TYPE, VECV, 2, false, TROW>;                                                        \
        auto dense4 = combine_kernel<TYPE, VECV, 4, false, TROW>;                                                        \
        auto lists = combine_kernel<TYPE, VECV, 4, true, TROW>;                                                          \
        hipLaunchKernelGGL(ix.pos == nullptr ? lists : d / VECV <= 2 * tpr ? dense2 : dense4, dim3((unsigned)ceil_div(n, 256 / tpr)), dim3(256), 0,      \
                           stream, (const TROW*)Xe, G, ix.bitmap, ix.pos, ix.offsets, ix.inv, (TYPE*)Xout, (int)n, (int)d, \
                           (int)e, tpr, addend, src_rows);                                                               \
    } while (0)
    if (dtype == EC_BF16 && rows_f32) EC_COMBINE_LAUNCH(bf16_t, 8, float);
    else if (dtype == EC_BF16) EC_COMBINE_LAUNCH(bf16_t, 8, bf16_t);
    else if (d % 4 == 0) EC_COMBINE_LAUNCH(float, 4, float);
    else EC_COMBINE_LAUNCH(float, 1, float);
#undef EC_COMBINE_LAUNCH
    return check_launch();
}

// Eq. 4 with the token-major index in the library's own static device array (nothing is allocated).
// The array's device address is looked up once per GPU, with that GPU current; host code only ever
// uses that address, never the array's name.
int combine_static(const void* Xe, const float* G, const int32_t* I, void* Xout, int64_t n, int64_t d, int64_t e,
                   int64_t k, int dtype, hipStream_t stream) {
    // The documented limit, stated in what earlier forms of the index took: sizes stay accepted or refused as they were.
    // Up to 16 experts the dense form takes 4 n (1 + e) bytes and fits whenever the limit admits the call.
    auto part = [](size_t words) { return align_up(words * 4, 256); };
    const size_t cap = e <= 4 ? 4 : e <= 8 ? 8 : 16;
    const size_t need = e <= 16 ? part((size_t)n) + part((size_t)n * cap)
                                : part(1024) + part((size_t)combine_zero_words(n, e)) + part((size_t)n + 1) + part((size_t)e * k);
    if (need > (size_t)EC_MOE_STATIC_SCRATCH_BYTES) return EC_ERR_UNSUPPORTED;
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static unsigned char* scratch_ptr[MAX_DEVICES] = {};
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        set_last_hip_error(err != hipSuccess ? err : hipErrorInvalidDevice);
        return EC_ERR_HIP;
    }
    unsigned char* base;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (scratch_ptr[dev] == nullptr) {
            void* p = nullptr;
            err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (err != hipSuccess || p == nullptr) {
                set_last_hip_error(err != hipSuccess ? err : hipErrorInvalidSymbol);
                return EC_ERR_HIP;
            }
            scratch_ptr[dev] = static_cast<unsigned char*>(p);
        }
        base = scratch_ptr[dev];
    }
    // carve-up: the dense index if it fits, the lists otherwise
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t a = off; off = align_up(off + bytes, 256); return base + a; };
    CombineIndex ix = {};
    ix.bitmap = reinterpret_cast<uint32_t*>(take((size_t)combine_zero_words(n, e) * 4));
    if (off + (size_t)n * e * 4 <= (size_t)EC_MOE_STATIC_SCRATCH_BYTES) {
        ix.pos = reinterpret_cast<int32_t*>(base + off);
    } else {
        ix.block_tot = reinterpret_cast<uint32_t*>(take(1024 * 4));
        ix.offsets = reinterpret_cast<int32_t*>(take((size_t)(n + 1) * 4));
        ix.inv = reinterpret_cast<int32_t*>(take((size_t)e * k * 4));
    }
    int rc = launch_combine_index(I, n, e, k, ix, stream);  // clears the counters / bitmap with a fill kernel first
    if (rc != EC_OK) return rc;
    return launch_combine(Xe, G, I, Xout, n, d, e, k, dtype, ix, stream);
}

}  // namespace ecmoe
