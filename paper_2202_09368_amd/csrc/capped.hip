// Expert choice with a cap on the experts per token (Sec. 3.3): the matrix A[e,n] of the
// entropy-regularised linear programme
//     max <S^T, A> + lambda H(A),  rows sum to k, columns sum to at most b, 0 <= A <= 1,
// by Dykstra's algorithm over the three constraint sets; the buckets are then TopK(A, k).
// The paper prints neither the projections nor a stopping rule.  Here the projections are the KL
// (Bregman) ones, which are scalings -- rows by k / rowsum, columns by min(1, b / colsum), entries
// clipped at 1 -- with Dykstra's correction terms for the two inequality sets (one scale per column,
// one value per entry), and a fixed number of sweeps (rows, columns, box) is run.  Everything is
// kept in the log domain in float64: exp(S / lambda) overflows any float type for lambda = 0.001.
//
// Two forms:
//  * capped_solve_kernel, one launch for all sweeps: the state stays in the registers of at most 256 workgroups, which
//    exchange their partial row sums through memory once per sweep.
//  * two launches per sweep over a state in memory, for problems the first form does not hold (more than 128 experts,
//    more than 256 workgroups of 16 entries per thread), for caps of no practical use, and inside a stream capture:
//      capped_row_kernel   per expert row: r[i] = log k - logsumexp_j logA[i,j]   (read only)
//      capped_col_kernel   per token column: applies r, the column scale and the box step, and keeps
//                          the two correction terms.  Lanes run along the token axis (contiguous).
//    Bound: launches for small problems, then L2 / HBM traffic, 2 reads + 2 writes of 8 e n bytes per sweep plus one
//    more read for the row sums.
// Reductions use a fixed order in both, so results do not depend on timing.
#include <cmath>
#include <mutex>

#include "ec_common.h"

namespace ecmoe {

struct Lse {  // running log-sum-exp: sum = s * exp(m)
    double m, s;
};
__device__ __forceinline__ Lse lse_empty() { return {-INFINITY, 0.0}; }
__device__ __forceinline__ Lse lse_add(Lse a, double x) {
    if (x > a.m) { a.s = a.s * exp(a.m - x) + 1.0; a.m = x; }
    else if (x > -INFINITY) a.s += exp(x - a.m);
    return a;
}
__device__ __forceinline__ Lse lse_merge(Lse a, Lse b) {
    if (b.m > a.m) { Lse t = a; a = b; b = t; }
    if (b.m > -INFINITY) a.s += b.s * exp(b.m - a.m);
    return a;
}
__device__ __forceinline__ double lse_value(Lse a) { return a.m + log(a.s); }

__global__ void __launch_bounds__(256)
capped_init_kernel(const float* __restrict__ St, double inv_lambda, double* __restrict__ logA,
                   double* __restrict__ lq_box, double* __restrict__ lq_col, long long count, int n) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long long)gridDim.x * 256) {
        logA[i] = (double)St[i] * inv_lambda;
        lq_box[i] = 0.0;
        if (i < n) lq_col[i] = 0.0;
    }
}

__global__ void __launch_bounds__(1024)
capped_row_kernel(const double* __restrict__ logA, double* __restrict__ r, int n, double log_k) {
    __shared__ double sm[16], ss[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double* row = logA + (size_t)blockIdx.x * n;
    Lse a = lse_empty();
    for (int j = tid; j < n; j += 1024) a = lse_add(a, row[j]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        Lse o = {__shfl_xor(a.m, off, kWave), __shfl_xor(a.s, off, kWave)};
        a = lse_merge(a, o);  // symmetric in its arguments: both partners end with the same value
    }
    if (lane == 0) { sm[wave] = a.m; ss[wave] = a.s; }
    __syncthreads();
    if (tid == 0) {
        Lse t = {sm[0], ss[0]};
        for (int w = 1; w < 16; ++w) t = lse_merge(t, Lse{sm[w], ss[w]});
        r[blockIdx.x] = log_k - lse_value(t);
    }
}

// Block = 64 tokens x 4 slices of the expert axis (wavefront w takes experts w, w+4, ...).
__global__ void __launch_bounds__(256)
capped_col_kernel(double* __restrict__ logA, double* __restrict__ lq_box, double* __restrict__ lq_col,
                  const double* __restrict__ r, int n, int e, double log_b) {
    __shared__ double sm[4][64], ss[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + lane;
    const bool live = j < n;
    const double qc = live ? lq_col[j] : 0.0;
    Lse a = lse_empty();
    if (live)
        for (int i = wave; i < e; i += 4) a = lse_add(a, logA[(size_t)i * n + j] + r[i] + qc);
    sm[wave][lane] = a.m;
    ss[wave][lane] = a.s;
    __syncthreads();
    Lse t = {sm[0][lane], ss[0][lane]};
#pragma unroll
    for (int w = 1; w < 4; ++w) t = lse_merge(t, Lse{sm[w][lane], ss[w][lane]});
    if (!live) return;
    const double s = fmin(0.0, log_b - lse_value(t));  // log of the column's scale
    for (int i = wave; i < e; i += 4) {
        const size_t at = (size_t)i * n + j;
        const double B = logA[at] + r[i] + qc + s + lq_box[at];
        logA[at] = fmin(B, 0.0);
        lq_box[at] = fmax(B, 0.0);
    }
    if (wave == 0) lq_col[j] = -s;
}

// ---------------------------------------------------------------------------
// All sweeps in one launch.  What bounds a sweep is the exchange, not the arithmetic: every row sum needs every
// workgroup, a store and a load through the memory shared by the XCDs, about 2 us.  So the state never leaves the
// registers, and a sweep makes one exchange and one block barrier:
//  * wavefront w of a workgroup owns experts w, w + 8, .. (EP of them) of the workgroup's 64 TT tokens; lanes run along
//    the tokens, so a row's partial sum is one wavefront reduction and a column's sum one trip through LDS.
//  * a partial row sum is its own message: slots[sweep & 1][expert][workgroup] (pitch: one expert to the next) holds the sum (a positive double) with
//    bit (sweep >> 1) & 1 as its sign, and the reader polls until the sign is the expected one.  A workgroup overwrites
//    a slot two sweeps later, when it has read everybody's next message, i.e. after everybody has read this one.  The
//    readers of expert i are the wavefronts that own it, so nothing else has to be passed on inside a workgroup.
//  * no logarithm and no exponential: log A plus the box set's correction is one number, to which a sweep adds the row's
//    shift and the column's (the box step only moves it between the two terms).  So an entry is y, scaled by k / rowsum
//    and by the column's factor, and A = min(y, 1); y and the column's correction are doubles with an exponent of their
//    own, since exp(S / lambda) and what many sweeps make of it overflow any double.  Rows sum to [min(1, b / e), n]
//    after every sweep (and to at least 1 at the start, where the row's maximum is taken off); a column whose
//    correction is not 1 sums to at least min(1, b) k / n after the rows' step: plain doubles hold both.
// Measured per sweep of 16 experts: 8192 tokens 17.7 us as two launches, 3.6 here (2.0 with 1024 tokens, 1.3 with 64, where
// the exchange stays inside one workgroup; 64 experts x 8192 tokens 5.0, 128 x 2048 5.6).
// Every workgroup waits for every other, so all of them have to be on the chip together: at most 256 (one per compute
// unit), and the launches of a process follow one another on a GPU (SolverTurn).  A wait gives up after ten seconds,
// and A then reads NaN.
// ---------------------------------------------------------------------------
constexpr int CAP_WAVES = 8;
constexpr int CAP_MAX_BLOCKS = 256;
constexpr int CAP_TARGET_BLOCKS = 32;
constexpr unsigned long long CAP_SIGN = 1ull << 63;

// Row maxima of S^T, and every slot marked as not yet written (the first two sweeps write positive numbers).
__global__ void __launch_bounds__(1024)
capped_start_kernel(const float* __restrict__ St, float* __restrict__ row_max, unsigned long long* __restrict__ slots,
                    int nslots, int n) {
    __shared__ float red[16];
    const int tid = threadIdx.x;
    for (int i = blockIdx.x * 1024 + tid; i < nslots; i += gridDim.x * 1024) slots[i] = CAP_SIGN;
    const float* row = St + (size_t)blockIdx.x * n;
    float m = -INFINITY;
    for (int j = tid; j < n; j += 1024) m = fmaxf(m, row[j]);
    m = wave_reduce_max(m);
    if ((tid & 63) == 0) red[tid >> 6] = m;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 16; ++w) m = fmaxf(m, red[w]);
        row_max[blockIdx.x] = m;
    }
}

// Lane exchanges without the LDS crossbar (a trip of a hundred cycles on the path of every sweep).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// Adds the halves (W = 32) or the rows of 16 in pairs (W = 16) of two vectors: the lower half / even rows of the result
// belong to x, the others to y.
template <int W>
__device__ __forceinline__ double fold_pair_f64(double x, double y) {
    const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
    double d[2];
    if (W == 32) {
        const auto lo = __builtin_amdgcn_permlane32_swap((unsigned int)bx, (unsigned int)by, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((unsigned int)(bx >> 32), (unsigned int)(by >> 32), false, false);
        for (int q = 0; q < 2; ++q) d[q] = __longlong_as_double((long long)(((unsigned long long)hi[q] << 32) | lo[q]));
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap((unsigned int)bx, (unsigned int)by, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((unsigned int)(bx >> 32), (unsigned int)(by >> 32), false, false);
        for (int q = 0; q < 2; ++q) d[q] = __longlong_as_double((long long)(((unsigned long long)hi[q] << 32) | lo[q]));
    }
    return d[0] + d[1];
}
// Sums of EP vectors over the wavefront: v[q] of row g of 16 lanes (all of them) ends as the sum of vector
// sums_index<EP>(q, g), q < sums_kept<EP>.
template <int EP>
constexpr int sums_kept() { return EP >= 4 ? EP / 4 : 1; }
template <int EP>
__device__ __forceinline__ int sums_index(int q, int g) {
    return EP >= 4 ? q + (g & 1) * (EP / 4) + (g >> 1) * (EP / 2) : (EP == 2 ? g >> 1 : 0);
}
template <int EP>
__device__ __forceinline__ void wave_sums_f64(double (&v)[EP]) {
    if (EP >= 2) {
#pragma unroll
        for (int q = 0; q < EP / 2; ++q) v[q] = fold_pair_f64<32>(v[q], v[q + EP / 2]);
    } else {
        v[0] = fold_pair_f64<32>(v[0], v[0]);
    }
    if (EP >= 4) {
#pragma unroll
        for (int q = 0; q < EP / 4; ++q) v[q] = fold_pair_f64<16>(v[q], v[q + EP / 4]);
    } else {
        v[0] = fold_pair_f64<16>(v[0], v[0]);
    }
#pragma unroll
    for (int q = 0; q < sums_kept<EP>(); ++q) {
        v[q] += dpp_f64<0xB1>(v[q]);   // quad_perm 1 0 3 2
        v[q] += dpp_f64<0x4E>(v[q]);   // quad_perm 2 3 0 1
        v[q] += dpp_f64<0x141>(v[q]);  // row_half_mirror: the other quad
        v[q] += dpp_f64<0x140>(v[q]);  // row_mirror: the other eight
    }
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int EP, int TT>
__global__ void __launch_bounds__(64 * CAP_WAVES)
capped_solve_kernel(const float* __restrict__ St, const float* __restrict__ row_max, float* __restrict__ A,
                    unsigned long long* slots, int pitch, int n, int e, double inv_lambda, double k, double b, int iters) {
    __shared__ double col[2][CAP_WAVES][64 * TT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int blk = blockIdx.x, nb = gridDim.x;
    const int j0 = blk * 64 * TT + lane;
    // y = ym 2^yx with ym in [0.5, 1), a = min(y, 1); the column's correction is qm 2^qx
    double ym[EP][TT], a[EP][TT], qm[TT];
    int yx[EP][TT], qx[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        qm[t] = 0.5;
        qx[t] = 1;
    }
#pragma unroll
    for (int p = 0; p < EP; ++p) {
        const int i = wave + CAP_WAVES * p;
        const double mx = i < e ? (double)row_max[i] : 0.0;
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            const int j = j0 + 64 * t;
            const bool live = i < e && j < n;
            const double z = live ? ((double)St[(size_t)i * n + j] - mx) * inv_lambda : 0.0;
            const double z1 = z * 1.4426950408889634074, z2 = fmax(rint(z1), -1e9);
            const double f = exp2(z1 - z2);
            ym[p][t] = live && z2 > -1e9 ? __builtin_amdgcn_frexp_mant(f) : 0.0;
            yx[p][t] = live ? (int)z2 + __builtin_amdgcn_frexp_exp(f) : -1000000000;
            a[p][t] = yx[p][t] > 0 ? 1.0 : ldexp(ym[p][t], yx[p][t]);
        }
    }
    bool gave_up = false;
    const unsigned long long start = __builtin_amdgcn_s_memrealtime();  // 100 MHz
    for (int it = 0; it < iters; ++it) {
        unsigned long long* slot = slots + (size_t)(it & 1) * e * pitch;
        const unsigned long long sign = (it >> 1) & 1 ? CAP_SIGN : 0ull;
        // rows: publish this workgroup's part, collect everybody's
        double part[EP];
#pragma unroll
        for (int p = 0; p < EP; ++p) {
            part[p] = a[p][0];
#pragma unroll
            for (int t = 1; t < TT; ++t) part[p] += a[p][t];
        }
        wave_sums_f64<EP>(part);
#pragma unroll
        for (int q = 0; q < sums_kept<EP>(); ++q) {
            const int i = wave + CAP_WAVES * sums_index<EP>(q, lane >> 4);
            if (i < e && (lane & (EP >= 4 ? 15 : EP == 2 ? 31 : 63)) == 0)
                __hip_atomic_store(&slot[(size_t)i * pitch + blk],
                                   ((unsigned long long)__double_as_longlong(part[q]) & ~CAP_SIGN) | sign, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        double row[EP];
#pragma unroll
        for (int p = 0; p < EP; ++p) row[p] = 0.0;
        for (int b0 = 0; b0 < nb; b0 += 64) {
            unsigned long long v[EP];
            const bool mine = b0 + lane < nb;
#pragma unroll
            for (int p = 0; p < EP; ++p) v[p] = mine && wave + CAP_WAVES * p < e ? ~sign : sign;  // ~sign: not read yet
            for (int polls = 1;; ++polls) {  // all that is missing is asked for together: one trip to memory per round
                bool missing = false;
#pragma unroll
                for (int p = 0; p < EP; ++p)
                    if (((v[p] ^ sign) & CAP_SIGN) != 0ull)
                        v[p] = __hip_atomic_load(&slot[(size_t)(wave + CAP_WAVES * p) * pitch + b0 + lane], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int p = 0; p < EP; ++p) missing |= ((v[p] ^ sign) & CAP_SIGN) != 0ull;
                if (__ballot(missing) == 0ull || gave_up) break;
                if ((polls & 255) == 0) gave_up = __builtin_amdgcn_s_memrealtime() - start > 1000000000ull;
            }
#pragma unroll
            for (int p = 0; p < EP; ++p) row[p] += __longlong_as_double((long long)(v[p] & ~CAP_SIGN));
        }
        wave_sums_f64<EP>(row);
        double rho[EP];
#pragma unroll
        for (int q = 0; q < sums_kept<EP>(); ++q) {  // four rows of lanes, four experts at a time
            const double scale = k / row[q];
#pragma unroll
            for (int g = 0; g < 4; g += EP >= 4 ? 1 : EP == 2 ? 2 : 4) {
                const int p = sums_index<EP>(q, g);
                rho[p] = wave + CAP_WAVES * p < e ? readlane_f64(scale, 16 * g) : 0.0;
            }
        }
        // columns
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            double s = 0.0;
#pragma unroll
            for (int p = 0; p < EP; ++p) s = fma(a[p][t], rho[p], s);
            col[it & 1][wave][64 * t + lane] = s;
        }
        __syncthreads();  // the other buffer is rewritten after the next one of these
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < CAP_WAVES; ++w) s += col[it & 1][w][64 * t + lane];
            // the column times its correction is scaled down to b if it is above; what that takes off is the next correction
            const double sm = __builtin_amdgcn_frexp_mant(s);
            const int sx = __builtin_amdgcn_frexp_exp(s);
            const double qs = qm[t] * sm;
            const bool over = ldexp(qs, qx[t] + sx) > b;
            const double fm = over ? b / sm : qm[t];
            const int fx = over ? -sx : qx[t];
            const double nq = over ? qs / b : 0.5;
            qx[t] = over ? qx[t] + sx + __builtin_amdgcn_frexp_exp(nq) : 1;
            qm[t] = __builtin_amdgcn_frexp_mant(nq);
            // box
#pragma unroll
            for (int p = 0; p < EP; ++p) {
                const double v = (ym[p][t] * rho[p]) * fm;
                ym[p][t] = __builtin_amdgcn_frexp_mant(v);
                yx[p][t] += fx + __builtin_amdgcn_frexp_exp(v);
                a[p][t] = yx[p][t] > 0 ? 1.0 : ldexp(ym[p][t], yx[p][t]);
            }
        }
    }
    const bool bad = __ballot(gave_up) != 0ull;
#pragma unroll
    for (int p = 0; p < EP; ++p) {
        const int i = wave + CAP_WAVES * p;
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            const int j = j0 + 64 * t;
            if (i < e && j < n) A[(size_t)i * n + j] = bad ? __uint_as_float(0x7FC00000u) : (float)a[p][t];
        }
    }
}

// One solver launch at a time on a GPU: a later one waits for the event behind the earlier one, whatever its stream.
struct SolverTurn {
    std::mutex mu;
    hipEvent_t done = nullptr;
};
static SolverTurn g_turn[64];

template <typename F>
static int with_solver_turn(hipStream_t stream, F&& launch) {
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err == hipSuccess && (dev < 0 || dev >= 64)) err = hipErrorInvalidDevice;
    if (err == hipSuccess) {
        SolverTurn& turn = g_turn[dev];
        std::lock_guard<std::mutex> lock(turn.mu);
        if (turn.done == nullptr) err = hipEventCreateWithFlags(&turn.done, hipEventDisableTiming);
        else err = hipStreamWaitEvent(stream, turn.done, 0);
        if (err == hipSuccess) {
            launch();
            err = hipGetLastError();
            const hipError_t rec = hipEventRecord(turn.done, stream);
            if (err == hipSuccess) err = rec;
        }
    }
    if (err != hipSuccess) {
        set_last_hip_error(err);
        return EC_ERR_HIP;
    }
    return EC_OK;
}

// Form of the one-launch solver: EP experts per wavefront, TT tokens per lane (at most 16 entries per
// thread, and the column sums of 8 tokens per lane in LDS).
struct SolverForm {
    int ep, tt;
    int64_t blocks;
};
static SolverForm solver_form(int64_t n, int64_t e) {
    SolverForm f = {1, 0, 0};
    if (e > 16 * CAP_WAVES) return f;
    while (f.ep * CAP_WAVES < e) f.ep *= 2;
    // few workgroups make the exchange cheap, many the arithmetic between two: 8192 x 16 takes 4.1 / 3.6 / 3.8 us a sweep
    // with 16 / 32 / 64 of them, 4096 x 16 2.6 / 3.3 / 3.9
    for (int tt = 1; tt <= 8 && tt * f.ep <= 16; tt *= 2) {
        f.tt = tt;
        f.blocks = ceil_div(n, 64 * tt);
        if (f.blocks <= CAP_TARGET_BLOCKS) break;
    }
    return f;
}

__global__ void __launch_bounds__(256)
capped_exp_kernel(const double* __restrict__ logA, float* __restrict__ A, long long count) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long long)gridDim.x * 256)
        A[i] = (float)exp(logA[i]);
}

size_t capped_ws_bytes(int64_t n, int64_t e) {
    return 2 * align_up((size_t)e * n * 8, 256) + align_up((size_t)n * 8, 256) + align_up((size_t)e * 8, 256);
}

static unsigned grid_for(long long items) {
    long long b = (items + 255) / 256;
    return (unsigned)(b > 65536 ? 65536 : (b < 1 ? 1 : b));
}

int launch_capped_assignment(const float* St, int64_t n, int64_t e, int64_t k, double b, double lambda,
                             int64_t iters, float* A, void* ws, hipStream_t stream) {
    char* p = (char*)ws;
    double* logA = (double*)p;    p += align_up((size_t)e * n * 8, 256);
    double* lq_box = (double*)p;  p += align_up((size_t)e * n * 8, 256);
    double* lq_col = (double*)p;  p += align_up((size_t)n * 8, 256);
    double* r = (double*)p;
    const long long count = (long long)e * n;
    const SolverForm f = solver_form(n, e);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
        (void)hipGetLastError();
        capture = hipStreamCaptureStatusActive;
    }
    if (iters > 0 && f.blocks > 0 && f.blocks <= CAP_MAX_BLOCKS && b >= 1e-100 && b <= 1e100 &&
        capture == hipStreamCaptureStatusNone) {
        // The regions of the state in memory hold the row maxima and the slots, at most n words per expert and buffer.
        // 17 x 256 bytes from one expert's slots to the next spread them over the memory channels.
        const int pitch = (int)(n < 544 ? n : 544);
        unsigned long long* slots = (unsigned long long*)logA;
        float* row_max = (float*)r;
        hipLaunchKernelGGL(capped_start_kernel, dim3((unsigned)e), dim3(1024), 0, stream, St, row_max, slots,
                           (int)(2 * e * pitch), (int)n);
        return with_solver_turn(stream, [&]() {
#define EC_SOLVE(EPV, TTV)                                                                                               \
    if (f.ep == EPV && f.tt == TTV)                                                                                      \
        hipLaunchKernelGGL((capped_solve_kernel<EPV, TTV>), dim3((unsigned)f.blocks), dim3(64 * CAP_WAVES), 0, stream, St, \
                           row_max, A, slots, pitch, (int)n, (int)e, 1.0 / lambda, (double)k, b, (int)iters)
            EC_SOLVE(1, 1); EC_SOLVE(1, 2); EC_SOLVE(1, 4); EC_SOLVE(1, 8);
            EC_SOLVE(2, 1); EC_SOLVE(2, 2); EC_SOLVE(2, 4); EC_SOLVE(2, 8);
            EC_SOLVE(4, 1); EC_SOLVE(4, 2); EC_SOLVE(4, 4);
            EC_SOLVE(8, 1); EC_SOLVE(8, 2);
            EC_SOLVE(16, 1);
#undef EC_SOLVE
        });
    }
    hipLaunchKernelGGL(capped_init_kernel, dim3(grid_for(count)), dim3(256), 0, stream, St, 1.0 / lambda, logA, lq_box,
                       lq_col, count, (int)n);
    const double log_k = std::log((double)k), log_b = std::log(b);
    for (int64_t it = 0; it < iters; ++it) {
        hipLaunchKernelGGL(capped_row_kernel, dim3((unsigned)e), dim3(1024), 0, stream, logA, r, (int)n, log_k);
        hipLaunchKernelGGL(capped_col_kernel, dim3((unsigned)ceil_div(n, 64)), dim3(256), 0, stream, logA, lq_box, lq_col,
                           r, (int)n, (int)e, log_b);
    }
    hipLaunchKernelGGL(capped_exp_kernel, dim3(grid_for(count)), dim3(256), 0, stream, logA, A, count);
    return check_launch();
}

}  // namespace ecmoe
