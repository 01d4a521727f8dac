// Arithmetic of the calibration-set construction (paper Sec. 3.3, Noise-Filtered Diverse Sampling): the two reductions
// that read whole activation tensors (per-layer mean / variance of a sample, frame-to-first-frame cosine of a feature
// map) and the small per-pool steps built on their results (noise score, percentile filter, one K-Means iteration).
//
// The reductions are bound by HBM: every element is read once with 16-byte loads, converted to double and summed in
// double (sum, sum of squares / dot product), so that the variance formula E[x^2] - E[x]^2 has no cancellation problem
// and the result does not depend on the size of the tensor.  A row is split over several blocks; each block leaves a
// pair of partial sums in the workspace and a second, tiny kernel adds them in a fixed order (deterministic results).
// 24 frames of 1374 x 1024 bf16: moments 15.3 us, correlation 18.8, of which 6.5 are the two launches of a call that reads next to nothing; 100
// frames, past the caches, 47.2 and 46.7 (6 TB/s).  Lane sums go through DPP moves (reads of other lanes through LDS were 1 us of every call).
// The per-pool steps handle a few hundred samples: one block each, double arithmetic, written for clarity.
#include "qvggt_common.h"

#include <algorithm>
#include <type_traits>

namespace qvggt {

namespace nfds {
constexpr int THREADS = 256;
constexpr int MAX_BLOCKS_PER_ROW = 1024;
constexpr int TARGET_BLOCKS = 2048;          // blocks in flight on the 256 compute units
constexpr int MIN_VEC_PER_BLOCK = 4 * THREADS;  // 16-byte vectors a block handles at least: keeps the partials few for small rows

__host__ inline int blocks_per_row(int rows, long long count, int elt_bytes)
{
    const long long vecs = count * elt_bytes / 16;
    long long want = std::max(1LL, (long long)TARGET_BLOCKS / std::max(rows, 1));
    const long long cap = std::max(1LL, vecs / MIN_VEC_PER_BLOCK);
    want = std::min(std::min(want, cap), (long long)MAX_BLOCKS_PER_ROW);
    return (int)want;
}

// The frame correlation's blocks take four frames of a share where that leaves at least this many blocks, and two otherwise (us a call of 1374 x 1024
// bf16 values a frame, one frame a block / two / four: 4 samples of 20 frames 52.1 / 49.1 / 44.0, 100 frames 53.3 / 46.8 / 46.7, 24 frames 20.7 / 19.3 /
// 18.8, 5 frames (342 blocks of four) 9.8 / 8.3 / 8.7; 20 samples of 10 frames of 200 x 64 (60 blocks) 7.1 / 7.1 / 8.5).
constexpr int CORR_BLOCKS = 400;
constexpr int MAX_PAIRS_PER_THREAD = 8;      // a row's partial sums are added by one thread up to here, by a wave beyond

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// the 8 bf16 or 4 f32 values of one 16-byte vector, as doubles
template <bool F32>
__device__ inline int unpack(const v4u &v, double (&x)[8])
{
    if constexpr (F32) {
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = (double)__uint_as_float(v[q]);
        return 4;
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x[2 * q] = (double)__uint_as_float(v[q] << 16);
            x[2 * q + 1] = (double)__uint_as_float(v[q] & 0xFFFF0000u);
        }
        return 8;
    }
}

// v of the lane that a DPP control names
template <int CTRL>
__device__ inline double from_lane(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false), hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned int)hi << 32) | (unsigned int)lo));
}

// the sum over the wave's 64 lanes, fixed order, in the last lane (the other lanes hold parts): pairs, quads, 8, 16, then rows of 16 onto the next ones
__device__ inline double wave_sum(double v)
{
    v += from_lane<0xB1>(v);         // lane ^ 1
    v += from_lane<0x4E>(v);         // lane ^ 2
    v += from_lane<0x141>(v);        // mirrored in 8
    v += from_lane<0x140>(v);        // mirrored in 16
    v += from_lane<0x142>(v);        // row 0's sum to row 1, 2's to 3 (and 0 to row 0)
    v += from_lane<0x143>(v);        // rows 0 and 1's sum to rows 2 and 3
    return v;
}

// sum[k] over the block's threads, in thread k < N
template <int N>
__device__ inline double block_sums(double (&sum)[N])
{
    __shared__ double lds[THREADS / kWave][N];
    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        sum[k] = wave_sum(sum[k]);
        if (threadIdx.x % kWave == kWave - 1) lds[wave][k] = sum[k];
    }
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < N)
        for (int w = 0; w < THREADS / kWave; ++w) t += lds[w][threadIdx.x];
    return t;
}
}  // namespace nfds

// partial[row * bpr + b] = (sum, sum of squares) over block b's share of row `row`
template <bool F32>
__global__ __launch_bounds__(nfds::THREADS) void nfds_moments_partial_kernel(const void *__restrict__ A, long long count, int bpr,
                                                                             double2 *__restrict__ partial)
{
    const int row = blockIdx.x / bpr, b = blockIdx.x % bpr;
    const long long vecs = count * (F32 ? 4 : 2) / 16;
    const long long v0 = vecs * b / bpr, v1 = vecs * (b + 1) / bpr;
    const nfds::v4u *x = reinterpret_cast<const nfds::v4u *>(A) + row * vecs;
    double sum[2] = {0.0, 0.0};
    for (long long v = v0 + threadIdx.x; v < v1; v += nfds::THREADS) {
        double xv[8];
        const int n = nfds::unpack<F32>(x[v], xv);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < n) { sum[0] += xv[i]; sum[1] += xv[i] * xv[i]; }
    }
    const double s = nfds::block_sums(sum);
    if (threadIdx.x < 2) reinterpret_cast<double *>(partial + (size_t)row * bpr + b)[threadIdx.x] = s;
}

// (<a_0, a_t>, |a_t|^2) over vectors v0 .. v1 of frames t0 .. t0 + G - 1 to out[0], out[bpr], ...
template <bool F32, int G>
__device__ inline void corr_share(const nfds::v4u *__restrict__ ref, long long vecs, int t0, long long v0, long long v1, double2 *out, int bpr)
{
    const nfds::v4u *x[G];
#pragma unroll
    for (int k = 0; k < G; ++k) x[k] = ref + (t0 + k) * vecs;
    double sum[2 * G];
#pragma unroll
    for (int k = 0; k < 2 * G; ++k) sum[k] = 0.0;
    for (long long v = v0 + threadIdx.x; v < v1; v += nfds::THREADS) {
        nfds::v4u raw[G];
#pragma unroll
        for (int k = 0; k < G; ++k) raw[k] = x[k][v];
        double rv[8], xv[8];
        const int n = nfds::unpack<F32>(ref[v], rv);
#pragma unroll
        for (int k = 0; k < G; ++k) {
            nfds::unpack<F32>(raw[k], xv);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < n) { sum[2 * k] += rv[i] * xv[i]; sum[2 * k + 1] += xv[i] * xv[i]; }
        }
    }
    const double s = nfds::block_sums(sum);
    const int k = threadIdx.x;
    if (k < 2 * G) reinterpret_cast<double *>(out + (size_t)(k / 2) * bpr)[k % 2] = s;
}

// partial[row * bpr + b] = (<a_0, a_t>, |a_t|^2) over share b of frame t of a sample, row = sample * f + t.  A block takes its share of G frames, so
// that the first frame is read and converted to double once for all of them.
template <bool F32, int G>
__global__ __launch_bounds__(nfds::THREADS) void nfds_corr_partial_kernel(const void *__restrict__ A, long long count, int bpr, int f, int groups,
                                                                          double2 *__restrict__ partial)
{
    const int b = blockIdx.x % bpr, g = blockIdx.x / bpr;
    const int first = g / groups * f, t0 = g % groups * G;           // the sample's first row, the group's first frame
    const long long vecs = count * (F32 ? 4 : 2) / 16;
    const long long v0 = vecs * b / bpr, v1 = vecs * (b + 1) / bpr;
    const nfds::v4u *ref = reinterpret_cast<const nfds::v4u *>(A) + first * vecs;
    double2 *out = partial + (size_t)(first + t0) * bpr + b;
    const int frames = min(G, f - t0);
    if (frames == G) corr_share<F32, G>(ref, vecs, t0, v0, v1, out, bpr);
    else if (G > 3 && frames == 3) corr_share<F32, 3>(ref, vecs, t0, v0, v1, out, bpr);
    else if (G > 2 && frames == 2) corr_share<F32, 2>(ref, vecs, t0, v0, v1, out, bpr);
    else corr_share<F32, 1>(ref, vecs, t0, v0, v1, out, bpr);
}

// The partial sums of a row (up to MAX_BLOCKS_PER_ROW pairs) are added by LANES lanes: a wave, since one thread walking them pays a memory
// round trip for every few (25 us for the 85 pairs per row of a 24-frame sample, 3.4 us this way), or one thread where there are few pairs
// and many rows (the whole call on 4000 rows of one pair: 9.3 us with a thread each, 10.5 with a wave; 300 rows of two pairs 6.6 / 7.2,
// 100 rows of 20 pairs 12.3 / 11.1; measured when the lanes' sums cost some 0.5 us more).
// mean = S1 / n, var = S2 / n - mean^2 (population variance)
template <int LANES>
__global__ __launch_bounds__(nfds::THREADS) void nfds_moments_final_kernel(const double2 *__restrict__ partial, int rows, int bpr,
                                                                           long long count, float *__restrict__ mean, float *__restrict__ var)
{
    const int row = blockIdx.x * (nfds::THREADS / LANES) + threadIdx.x / LANES, lane = threadIdx.x % LANES;
    if (row >= rows) return;
    double s1 = 0.0, s2 = 0.0;
#pragma unroll 4
    for (int b = lane; b < bpr; b += LANES) {
        const double2 p = partial[(size_t)row * bpr + b];
        s1 += p.x; s2 += p.y;
    }
    if constexpr (LANES > 1) {
        s1 = nfds::wave_sum(s1);
        s2 = nfds::wave_sum(s2);
    }
    if (lane != LANES - 1) return;
    const double m = s1 / (double)count;
    mean[row] = (float)m;
    var[row] = (float)fmax(s2 / (double)count - m * m, 0.0);
}

// c[sample, t - 1] = <a_0, a_t> / (|a_0| |a_t|), LANES lanes per (sample, t >= 1)
template <int LANES>
__global__ __launch_bounds__(nfds::THREADS) void nfds_corr_final_kernel(const double2 *__restrict__ partial, int samples, int f, int bpr,
                                                                        float *__restrict__ c)
{
    const int idx = blockIdx.x * (nfds::THREADS / LANES) + threadIdx.x / LANES, lane = threadIdx.x % LANES;
    if (idx >= samples * (f - 1)) return;
    const int i = idx / (f - 1), t = idx % (f - 1) + 1;
    double dot = 0.0, nt = 0.0, n0 = 0.0;
#pragma unroll 4
    for (int b = lane; b < bpr; b += LANES) {
        const double2 p = partial[(size_t)(i * f + t) * bpr + b];
        dot += p.x; nt += p.y;
        n0 += partial[(size_t)(i * f) * bpr + b].y;
    }
    if constexpr (LANES > 1) {
        dot = nfds::wave_sum(dot);
        nt = nfds::wave_sum(nt);
        n0 = nfds::wave_sum(n0);
    }
    if (lane == LANES - 1) c[idx] = (float)(dot / (sqrt(n0) * sqrt(nt)));
}

// noise score of every sample of the pool from its per-layer moments: one block, layers then samples dealt to threads
__global__ __launch_bounds__(nfds::THREADS) void nfds_scores_kernel(const float *__restrict__ m, const float *__restrict__ s, int D,
                                                                   int L, double eps, float *__restrict__ score)
{
    extern __shared__ double stat[];     // mu, sigma, nu, tau: 4 * L
    for (int j = threadIdx.x; j < L; j += nfds::THREADS) {
        double mu = 0.0, nu = 0.0;
        for (int i = 0; i < D; ++i) { mu += (double)m[(size_t)i * L + j]; nu += (double)s[(size_t)i * L + j]; }
        mu /= D; nu /= D;
        double vm = 0.0, vs = 0.0;
        for (int i = 0; i < D; ++i) {
            const double dm = (double)m[(size_t)i * L + j] - mu, ds = (double)s[(size_t)i * L + j] - nu;
            vm += dm * dm; vs += ds * ds;
        }
        stat[j] = mu; stat[L + j] = sqrt(vm / D + eps);
        stat[2 * L + j] = nu; stat[3 * L + j] = sqrt(vs / D + eps);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < D; i += nfds::THREADS) {
        double acc_m = 0.0, acc_s = 0.0;
        for (int j = 0; j < L; ++j) {
            const double zm = ((double)m[(size_t)i * L + j] - stat[j]) / stat[L + j];
            const double zs = ((double)s[(size_t)i * L + j] - stat[2 * L + j]) / stat[3 * L + j];
            acc_m += zm * zm; acc_s += zs * zs;
        }
        score[i] = (float)sqrt(acc_m + acc_s);
    }
}

// keep[i] = 1 for the n_keep samples of lowest score, equal scores ordered by index
__global__ void nfds_keep_lowest_kernel(const float *__restrict__ score, int D, int n_keep, uint8_t *__restrict__ keep)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= D) return;
    const float si = score[i];
    int rank = 0;
    for (int k = 0; k < D; ++k) {
        const float sk = score[k];
        rank += (sk < si || (sk == si && k < i)) ? 1 : 0;
    }
    keep[i] = rank < n_keep ? 1 : 0;
}

// one Lloyd iteration: labels, then every centre coordinate as the mean of its points (one block)
__global__ __launch_bounds__(nfds::THREADS) void nfds_kmeans_step_kernel(const float *__restrict__ c, int n, int dim, int K,
                                                                        const float *__restrict__ cin, float *__restrict__ cout,
                                                                        int32_t *__restrict__ labels)
{
    for (int i = threadIdx.x; i < n; i += nfds::THREADS) {
        int best = 0;
        double best_d = 0.0;
        for (int k = 0; k < K; ++k) {
            double d = 0.0;
            for (int j = 0; j < dim; ++j) {
                const double e = (double)c[(size_t)i * dim + j] - (double)cin[(size_t)k * dim + j];
                d += e * e;
            }
            if (k == 0 || d < best_d) { best = k; best_d = d; }
        }
        labels[i] = best;
    }
    __threadfence_block();
    __syncthreads();
    for (int e = threadIdx.x; e < K * dim; e += nfds::THREADS) {
        const int k = e / dim, j = e % dim;
        double sum = 0.0;
        int cnt = 0;
        for (int i = 0; i < n; ++i)
            if (labels[i] == k) { sum += (double)c[(size_t)i * dim + j]; ++cnt; }
        cout[e] = cnt > 0 ? (float)(sum / cnt) : cin[e];
    }
}

// ---------------------------------------------------------------------------------------------------------------
size_t nfds_workspace_bytes(int rows, long long count, bool f32)
{
    return (size_t)rows * nfds::blocks_per_row(rows, count, f32 ? 4 : 2) * 2 * sizeof(double);
}

hipError_t run_nfds_moments(const void *A, bool f32, int rows, long long count, float *mean, float *var, double *ws,
                            hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    const int bpr = nfds::blocks_per_row(rows, count, f32 ? 4 : 2);
    double2 *pairs = reinterpret_cast<double2 *>(ws);
    if (f32) nfds_moments_partial_kernel<true><<<rows * bpr, nfds::THREADS, 0, stream>>>(A, count, bpr, pairs);
    else nfds_moments_partial_kernel<false><<<rows * bpr, nfds::THREADS, 0, stream>>>(A, count, bpr, pairs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (bpr <= nfds::MAX_PAIRS_PER_THREAD) nfds_moments_final_kernel<1><<<(rows + 255) / 256, nfds::THREADS, 0, stream>>>(pairs, rows, bpr, count, mean, var);
    else nfds_moments_final_kernel<kWave><<<(rows + 3) / 4, nfds::THREADS, 0, stream>>>(pairs, rows, bpr, count, mean, var);
    return hipGetLastError();
}

hipError_t run_nfds_frame_correlation(const void *A, bool f32, int samples, int f, long long dhat, float *c, double *ws,
                                      hipStream_t stream)
{
    if (samples <= 0) return hipSuccess;
    const int rows = samples * f;
    const int bpr = nfds::blocks_per_row(rows, dhat, f32 ? 4 : 2);
    double2 *pairs = reinterpret_cast<double2 *>(ws);
    const auto start = [&](auto frames) {
        constexpr int G = decltype(frames)::value;
        const int groups = (f + G - 1) / G, blocks = samples * groups * bpr;
        if (G > 2 && blocks < nfds::CORR_BLOCKS) return false;
        if (f32) nfds_corr_partial_kernel<true, G><<<blocks, nfds::THREADS, 0, stream>>>(A, dhat, bpr, f, groups, pairs);
        else nfds_corr_partial_kernel<false, G><<<blocks, nfds::THREADS, 0, stream>>>(A, dhat, bpr, f, groups, pairs);
        return true;
    };
    if (!start(std::integral_constant<int, 4>())) start(std::integral_constant<int, 2>());
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int n = samples * (f - 1);
    if (bpr <= nfds::MAX_PAIRS_PER_THREAD) nfds_corr_final_kernel<1><<<(n + 255) / 256, nfds::THREADS, 0, stream>>>(pairs, samples, f, bpr, c);
    else nfds_corr_final_kernel<kWave><<<(n + 3) / 4, nfds::THREADS, 0, stream>>>(pairs, samples, f, bpr, c);
    return hipGetLastError();
}

hipError_t run_nfds_scores(const float *m, const float *s, int D, int L, double eps, float *score, hipStream_t stream)
{
    nfds_scores_kernel<<<1, nfds::THREADS, 4 * L * sizeof(double), stream>>>(m, s, D, L, eps, score);
    return hipGetLastError();
}

hipError_t run_nfds_keep_lowest(const float *score, int D, int n_keep, uint8_t *keep, hipStream_t stream)
{
    nfds_keep_lowest_kernel<<<(D + 255) / 256, 256, 0, stream>>>(score, D, n_keep, keep);
    return hipGetLastError();
}

hipError_t run_nfds_kmeans_step(const float *c, int n, int dim, int K, const float *cin, float *cout, int32_t *labels,
                                hipStream_t stream)
{
    nfds_kmeans_step_kernel<<<1, nfds::THREADS, 0, stream>>>(c, n, dim, K, cin, cout, labels);
    return hipGetLastError();
}

}  // namespace qvggt
