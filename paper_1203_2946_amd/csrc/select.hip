// Learned configuration selection: matrix features and a small MLP
// (40 -> 64 -> 64 -> 24, ReLU, fp32) with forward, backward and Adam kernels.
//
// The paper picks the strip height and kernel options by brute-force search
// over measured times (Sec. 6.3) and notes how much per-matrix tuning could
// still gain (Sec. 6.8).  Here the measured times of every (height, schedule)
// class train a network that predicts, from cheap features of the CSR
// structure, the log time of each class relative to the fastest; the
// selector takes the class with the lowest prediction.
//
// Features (kSelFeatures = 40), all from row_ptr / col_ind:
//   [0, 20)   fraction of rows by length in half octaves: bin 0 empty; a
//             length with p = floor(log2 len) goes to 1 + 2p, or 2 + 2p when
//             2 len >= 3 * 2^p; bins above 19 fold into 19 (len >= 512)
//   [20, 36)  fraction of entries by |col - row * cols / rows|: bin 0 for 0,
//             bin b >= 1 for distances in [2^(b-1), 2^b), last bin open
//   36..39    log2(rows)/22, log2(nnz+1)/26, log2(mean length+1)/14,
//             log2(max length+1)/14
// Parameters, packed: W1[40][64], b1[64], W2[64][64], b2[64], W3[64][24], b3[24]
// (8344 floats); activations row-major [batch][width].
#include <math.h>

#include <algorithm>

#include "cmrs_device.hpp"
#include "cmrs_ext.hpp"

namespace cmrs {

constexpr int kSelFeatures = 40, kSelHidden = 64, kSelClasses = 24;
constexpr int kRowBins = 20, kDistBins = 16;
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kSelFeatures * kSelHidden;
constexpr int kOffW2 = kOffB1 + kSelHidden;
constexpr int kOffB2 = kOffW2 + kSelHidden * kSelHidden;
constexpr int kOffW3 = kOffB2 + kSelHidden;
constexpr int kOffB3 = kOffW3 + kSelHidden * kSelClasses;
constexpr int kSelParams = kOffB3 + kSelClasses;
static_assert(kSelParams == 8344, "parameter count");

// ------------------------------------------------------------------ features

__device__ inline int row_len_bin(int len) {
    if (len <= 0) return 0;
    const int p = 31 - __clz(len);
    const int b = 1 + 2 * p + ((2LL * len >= (3LL << p)) ? 1 : 0);
    return b < kRowBins - 1 ? b : kRowBins - 1;
}

__device__ inline int dist_bin(uint32_t d) {
    if (d == 0) return 0;
    const int b = 32 - __clz(static_cast<int>(d));  // d in [2^(b-1), 2^b)
    return b < kDistBins - 1 ? b : kDistBins - 1;
}

// Counts of one CSR structure.  ws: int counts [kRowBins + kDistBins], int max
// length, zeroed first.
//
// One wave per 64-row group; the group's entries are walked 4 consecutive ones
// per lane (one 16-byte load), kFeatVec such runs in flight.  The rows' pointers
// and centres sit in LDS: a lane finds its run's first row by binary search and
// steps to the next row from there.  Each lane counts in its own column of its
// wave's histogram, so no two lanes of an instruction meet in an LDS atomic, and
// at most kFeatMaxBlocks workgroups (4 of 8 waves on a CU; 512 and 4096 were
// slower) each add their sums to ws once.  10^6 rows, band of 41 columns, 98 MB
// of columns: 94 us with one entry per lane, six shuffles to find its row and
// one histogram per workgroup, whose few bins a banded matrix's lanes hit one
// after the other; 41 us now (2.4 TB/s), without the atomics 38, so the issue
// of searches and row steps is what remains.  A number of lanes per row instead
// of the search was slower (52 us: more slots past the rows' ends).
constexpr int kFeatWaves = 8;
constexpr int kFeatThreads = kFeatWaves * kWave;
constexpr int kFeatVec = 2;
constexpr int kFeatMaxBlocks = 1024;
typedef int feat_int4 __attribute__((ext_vector_type(4), aligned(4)));

__global__ __launch_bounds__(kFeatThreads) void feature_count_kernel(int rows, int cols,
                                                                     const int* __restrict__ row_ptr,
                                                                     const int* __restrict__ col_ind,
                                                                     int* __restrict__ ws) {
    __shared__ int2 rp[kFeatWaves][kWave + 1];  // row pointer; column the row's entries are measured from
    __shared__ int dist[kFeatWaves][kDistBins][kWave];
    __shared__ int hist[kRowBins + kDistBins];
    __shared__ int maxlen;
    const int tid = static_cast<int>(threadIdx.x);
    const int lane = lane_id();
    const int wave = uniform(tid / kWave);
    if (tid < kRowBins + kDistBins) hist[tid] = 0;
    if (tid == 0) maxlen = 0;
    int2* R = rp[wave];
    int* D = &dist[wave][0][lane];
#pragma unroll
    for (int b = 0; b < kDistBins; ++b) D[b * kWave] = 0;
    __syncthreads();
    const double scale = rows > 0 ? static_cast<double>(cols) / rows : 0.0;
    const long long stride = static_cast<long long>(gridDim.x) * kFeatWaves * kWave;
    for (long long r0l = (static_cast<long long>(blockIdx.x) * kFeatWaves + wave) * kWave; r0l < rows; r0l += stride) {
        const int r0 = static_cast<int>(r0l);
        const int nr = min(kWave, rows - r0);
        wave_lds_sync();  // the last group's searches are done
        // The centre of a row is below cols, so 32 bits hold it and the distances.
        R[lane] = make_int2(lane <= nr ? row_ptr[r0 + lane] : 0x7fffffff,
                            static_cast<int>(static_cast<double>(min(r0 + lane, rows - 1)) * scale));
        if (lane == 0 && nr == kWave) R[kWave].x = row_ptr[r0 + kWave];
        wave_lds_sync();
        const int e0 = uniform(R[0].x), e1 = uniform(R[nr].x);
        if (lane < nr) {
            const int len = R[lane + 1].x - R[lane].x;
            atomicAdd(&hist[row_len_bin(len)], 1);
            atomicMax(&maxlen, len);
        }
        for (int base = e0; base < e1; base += 4 * kWave * kFeatVec) {
            feat_int4 c[kFeatVec];
#pragma unroll
            for (int k = 0; k < kFeatVec; ++k) {
                const int j = base + 4 * (k * kWave + lane);
                if (j < e1 - 3) {
                    c[k] = *reinterpret_cast<const feat_int4*>(col_ind + j);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) c[k][i] = j < e1 - i ? col_ind[j + i] : 0;
                }
            }
#pragma unroll
            for (int k = 0; k < kFeatVec; ++k) {
                const int j = base + 4 * (k * kWave + lane);
                const int first = min(j, e1 - 1);
                int t = 0;  // last row of the group starting at or before entry `first`
#pragma unroll
                for (int step = kWave / 2; step >= 1; step >>= 1)
                    if (R[t + step].x <= first) t += step;
                int center = R[t].y, next = R[t + 1].x;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (j < e1 - i) {
                        while (j + i >= next) {
                            center = R[++t].y;
                            next = R[t + 1].x;
                        }
                        const uint32_t d = c[k][i] > center ? static_cast<uint32_t>(c[k][i]) - center
                                                            : static_cast<uint32_t>(center) - c[k][i];
                        atomicAdd(&D[dist_bin(d) * kWave], 1);
                    }
                }
            }
        }
    }
    __syncthreads();
    // 32 threads sum one bin.
    static_assert(kDistBins * 32 == kFeatThreads, "one thread set per bin");
    const int bin = tid / 32;
    int sum = 0;
#pragma unroll
    for (int w = 0; w < kFeatWaves; ++w) sum += dist[w][bin][tid % 32] + dist[w][bin][32 + tid % 32];
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if (tid % 32 == 0) hist[kRowBins + bin] = sum;
    __syncthreads();
    if (tid < kRowBins + kDistBins && hist[tid]) atomicAdd(&ws[tid], hist[tid]);
    if (tid == 0 && maxlen) atomicMax(&ws[kRowBins + kDistBins], maxlen);
}

__global__ void feature_finish_kernel(int rows, int nnz, const int* __restrict__ ws, float* __restrict__ feat) {
    const int t = static_cast<int>(threadIdx.x);
    if (t < kRowBins) feat[t] = rows > 0 ? static_cast<float>(ws[t]) / rows : 0.0f;
    if (t >= kRowBins && t < kRowBins + kDistBins) feat[t] = nnz > 0 ? static_cast<float>(ws[t]) / nnz : 0.0f;
    if (t == 0) {
        const float mean = rows > 0 ? static_cast<float>(nnz) / rows : 0.0f;
        feat[36] = log2f(static_cast<float>(rows > 0 ? rows : 1)) / 22.0f;
        feat[37] = log2f(static_cast<float>(nnz) + 1.0f) / 26.0f;
        feat[38] = log2f(mean + 1.0f) / 14.0f;
        feat[39] = log2f(static_cast<float>(ws[kRowBins + kDistBins]) + 1.0f) / 14.0f;
    }
}

// ------------------------------------------------------------------ MLP

// The network of one workgroup's rows.  The parameters sit in LDS (W2 and W3
// with a row stride one above their width: the backward pass reads them with
// the lanes along the rows, which at a stride of 64 would all meet in one
// bank); a wave computes kMlpRows / kMlpWaves rows, lane j output j, so only
// the load of the parameters needs the workgroup.  One launch for the whole
// pass: as one launch per layer with the weights read from L2 for each product,
// a forward pass of one row took 54 us, nearly all of it load latency in chains
// of 40 to 64 products, and now 6 us; forward, loss gradient and input gradients
// of 1500 rows took 62 us in six launches and now 9 us in one.  Every sum runs
// in index order, as before.
constexpr int kMlpWaves = 4;
constexpr int kMlpThreads = kMlpWaves * kWave;
constexpr int kMlpRowsPerWave = 2;
constexpr int kMlpRows = kMlpWaves * kMlpRowsPerWave;
constexpr int kLdW2 = kSelHidden + 1, kLdW3 = kSelClasses + 1;

struct MlpLds {
    float w1[kSelFeatures * kSelHidden], b1[kSelHidden];
    float w2[kSelHidden * kLdW2], b2[kSelHidden];
    float w3[kSelHidden * kLdW3], b3[kSelClasses];
    float act[kMlpWaves][kMlpRowsPerWave][kSelHidden];  // a wave's layer input
};

typedef float mlp_float4 __attribute__((ext_vector_type(4), aligned(4)));

// `n` floats (a multiple of 4) in rows of `width` (a multiple of 4) to rows of
// `ld` in LDS.
__device__ inline void mlp_stage(const float* __restrict__ src, float* dst, int n, int width, int ld) {
    for (int i = 4 * static_cast<int>(threadIdx.x); i < n; i += 4 * kMlpThreads) {
        const mlp_float4 v = *reinterpret_cast<const mlp_float4*>(src + i);
        float* d = dst + i / width * ld + i % width;
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = v[k];
    }
}

__device__ inline void mlp_stage_all(const float* __restrict__ params, MlpLds& L) {
    mlp_stage(params + kOffW1, L.w1, kSelFeatures * kSelHidden, kSelHidden, kSelHidden);
    mlp_stage(params + kOffB1, L.b1, kSelHidden, kSelHidden, kSelHidden);
    mlp_stage(params + kOffW2, L.w2, kSelHidden * kSelHidden, kSelHidden, kLdW2);
    mlp_stage(params + kOffB2, L.b2, kSelHidden, kSelHidden, kSelHidden);
    mlp_stage(params + kOffW3, L.w3, kSelHidden * kSelClasses, kSelClasses, kLdW3);
    mlp_stage(params + kOffB3, L.b3, kSelClasses, kSelClasses, kSelClasses);
}

// s[r] = start + sum over i < N of act[r][i] * w[i * stride], i ascending.
template <int N>
__device__ inline void mlp_dot(const float (*act)[kSelHidden], const float* w, int stride, float (&s)[kMlpRowsPerWave]) {
#pragma unroll 4
    for (int i = 0; i < N; i += 4) {
        float wv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) wv[k] = w[(i + k) * stride];
#pragma unroll
        for (int r = 0; r < kMlpRowsPerWave; ++r) {
            const float4 a = *reinterpret_cast<const float4*>(&act[r][i]);
            s[r] = fmaf(a.x, wv[0], s[r]);
            s[r] = fmaf(a.y, wv[1], s[r]);
            s[r] = fmaf(a.z, wv[2], s[r]);
            s[r] = fmaf(a.w, wv[3], s[r]);
        }
    }
}

// A wave's rows of one hidden layer, to `out` and to the wave's next input.
template <int NIN>
__device__ inline void mlp_hidden(MlpLds& L, const float* w, int ldw, const float* bias, int wave, int lane, int row0,
                                  int batch, float* __restrict__ out) {
    float s[kMlpRowsPerWave];
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) s[r] = bias[lane];
    mlp_dot<NIN>(L.act[wave], w + lane, ldw, s);
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) {
        const float v = s[r] < 0.0f ? 0.0f : s[r];
        L.act[wave][r][lane] = v;
        if (row0 + r < batch) out[static_cast<size_t>(row0 + r) * kSelHidden + lane] = v;
    }
    wave_lds_sync();
}

// A wave's rows of the input gradient through a layer and the ReLU of its
// input: din[i] = (act[i] > 0) * sum_j dout[j] W[i][j], j ascending, with dout
// in the wave's LDS rows; to `din` and to those rows.
template <int NOUT>
__device__ inline void mlp_input_grad(MlpLds& L, const float* w, int ldw, int wave, int lane, int row0, int batch,
                                      const float (&act)[kMlpRowsPerWave], float* __restrict__ din) {
    float s[kMlpRowsPerWave];
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) s[r] = 0.0f;
    mlp_dot<NOUT>(L.act[wave], w + lane * ldw, 1, s);
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) {
        const float v = act[r] > 0.0f ? s[r] : 0.0f;
        L.act[wave][r][lane] = v;
        if (row0 + r < batch) din[static_cast<size_t>(row0 + r) * kSelHidden + lane] = v;
    }
    wave_lds_sync();
}

// Forward pass (H1, H2, Y); with GRAD also dY = scale (Y - T) and the input
// gradients dH2 and dH1, whose layers' weights and activations are at hand.
template <bool GRAD>
__global__ __launch_bounds__(kMlpThreads) void mlp_rows_kernel(int batch, const float* __restrict__ X,
                                                               const float* __restrict__ params,
                                                               float* __restrict__ H1, float* __restrict__ H2,
                                                               float* __restrict__ Y, const float* __restrict__ T,
                                                               float scale, float* __restrict__ dY,
                                                               float* __restrict__ dH2, float* __restrict__ dH1) {
    __shared__ __align__(16) MlpLds L;
    const int lane = lane_id();
    const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int row0 = static_cast<int>(blockIdx.x) * kMlpRows + wave * kMlpRowsPerWave;
    mlp_stage_all(params, L);
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r)
        L.act[wave][r][lane] = row0 + r < batch && lane < kSelFeatures
                                   ? X[static_cast<size_t>(row0 + r) * kSelFeatures + lane]
                                   : 0.0f;
    __syncthreads();
    if (row0 >= batch) return;
    float h1[kMlpRowsPerWave], h2[kMlpRowsPerWave];
    mlp_hidden<kSelFeatures>(L, L.w1, kSelHidden, L.b1, wave, lane, row0, batch, H1);
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) h1[r] = L.act[wave][r][lane];
    mlp_hidden<kSelHidden>(L, L.w2, kLdW2, L.b2, wave, lane, row0, batch, H2);
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) h2[r] = L.act[wave][r][lane];
    const int j = min(lane, kSelClasses - 1);
    float y[kMlpRowsPerWave];
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) y[r] = L.b3[j];
    mlp_dot<kSelHidden>(L.act[wave], L.w3 + j, kLdW3, y);
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) {
        const size_t at = static_cast<size_t>(row0 + r) * kSelClasses + lane;
        if (lane < kSelClasses && row0 + r < batch) {
            Y[at] = y[r];
            if constexpr (GRAD) {
                const float d = scale * (y[r] - T[at]);
                dY[at] = d;
                L.act[wave][r][lane] = d;
            }
        }
    }
    if constexpr (GRAD) {
        wave_lds_sync();
        mlp_input_grad<kSelClasses>(L, L.w3, kLdW3, wave, lane, row0, batch, h2, dH2);
        mlp_input_grad<kSelHidden>(L, L.w2, kLdW2, wave, lane, row0, batch, h1, dH1);
    }
}

// The two input gradients from a given dY and the forward activations.
__global__ __launch_bounds__(kMlpThreads) void mlp_input_grads_kernel(int batch, const float* __restrict__ params,
                                                                      const float* __restrict__ H1,
                                                                      const float* __restrict__ H2,
                                                                      const float* __restrict__ dY,
                                                                      float* __restrict__ dH2,
                                                                      float* __restrict__ dH1) {
    __shared__ __align__(16) MlpLds L;
    const int lane = lane_id();
    const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int row0 = static_cast<int>(blockIdx.x) * kMlpRows + wave * kMlpRowsPerWave;
    mlp_stage(params + kOffW2, L.w2, kSelHidden * kSelHidden, kSelHidden, kLdW2);
    mlp_stage(params + kOffW3, L.w3, kSelHidden * kSelClasses, kSelClasses, kLdW3);
    float h1[kMlpRowsPerWave], h2[kMlpRowsPerWave];
#pragma unroll
    for (int r = 0; r < kMlpRowsPerWave; ++r) {
        const bool in = row0 + r < batch;
        const size_t row = static_cast<size_t>(row0 + r);
        h1[r] = in ? H1[row * kSelHidden + lane] : 0.0f;
        h2[r] = in ? H2[row * kSelHidden + lane] : 0.0f;
        L.act[wave][r][lane] = in && lane < kSelClasses ? dY[row * kSelClasses + lane] : 0.0f;
    }
    __syncthreads();
    if (row0 >= batch) return;
    mlp_input_grad<kSelClasses>(L, L.w3, kLdW3, wave, lane, row0, batch, h2, dH2);
    mlp_input_grad<kSelHidden>(L, L.w2, kLdW2, wave, lane, row0, batch, h1, dH1);
}

// dL/dY for L = mean over batch and classes of (Y - T)^2.
__global__ __launch_bounds__(256) void mse_grad_kernel(int n, const float* __restrict__ Y, const float* __restrict__ T,
                                                       float* __restrict__ dY, float scale) {
    const int t = static_cast<int>(blockIdx.x * blockDim.x + threadIdx.x);
    if (t < n) dY[t] = scale * (Y[t] - T[t]);
}

// Weight and bias gradients of all three layers: dW = in^T dOut, db = the column
// sums of dOut.  One workgroup per 16 x 16 tile of a weight matrix (12 + 16 +
// 8 tiles); its 16 waves split the batch, each with fp32 matrix instructions
// over 4 rows at a time and kGradU steps of loads in flight, and the waves'
// tiles are added in wave order, so the result depends on the batch size
// only.  One thread per weight summing the whole batch was a serial chain of
// 1500 loads and products: 357 to 410 us a layer at batch 1500, and now
// 7 us for the three.  (The sums are also shorter: the error against 64 bits fell.)
constexpr int kGradWaves = 16;
constexpr int kGradThreads = kGradWaves * kWave;
constexpr int kGradU = 8;
constexpr int kTile = 16;
constexpr int tiles_of(int n) { return (n + kTile - 1) / kTile; }
constexpr int kTiles1 = tiles_of(kSelFeatures) * tiles_of(kSelHidden);
constexpr int kTiles2 = tiles_of(kSelHidden) * tiles_of(kSelHidden);
constexpr int kTiles3 = tiles_of(kSelHidden) * tiles_of(kSelClasses);
typedef float grad_float4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kGradThreads) void mlp_weight_grads_kernel(
    int batch, const float* __restrict__ X, const float* __restrict__ H1, const float* __restrict__ H2,
    const float* __restrict__ dY, const float* __restrict__ dH2, const float* __restrict__ dH1,
    float* __restrict__ grads) {
    __shared__ float part[kGradWaves][kTile * kTile];
    __shared__ float bpart[kGradWaves][kWave];
    int tile = static_cast<int>(blockIdx.x);
    const float *in, *dout;
    int nin, nout, offw, offb;
    if (tile < kTiles1) {
        in = X, dout = dH1, nin = kSelFeatures, nout = kSelHidden, offw = kOffW1, offb = kOffB1;
    } else if (tile < kTiles1 + kTiles2) {
        tile -= kTiles1;
        in = H1, dout = dH2, nin = kSelHidden, nout = kSelHidden, offw = kOffW2, offb = kOffB2;
    } else {
        tile -= kTiles1 + kTiles2;
        in = H2, dout = dY, nin = kSelHidden, nout = kSelClasses, offw = kOffW3, offb = kOffB3;
    }
    const int jt = (nout + kTile - 1) / kTile;
    const int i0 = tile / jt * kTile, j0 = tile % jt * kTile;
    const int tid = static_cast<int>(threadIdx.x);
    const int lane = lane_id();
    const int wave = uniform(tid / kWave);
    // Operands of the 16 x 16 x 4 instruction: lane l holds row l / 16 of the
    // step's four, column i0 + l % 16 of `in` and j0 + l % 16 of dOut.
    const int kr = lane / kTile, i = i0 + lane % kTile, j = j0 + lane % kTile;
    const bool ai = i < nin, bj = j < nout;
    const int ic = min(i, nin - 1), jc = min(j, nout - 1);
    const int steps = (batch + 3) / 4;
    const int s0 = static_cast<int>(static_cast<long long>(steps) * wave / kGradWaves);
    const int s1 = static_cast<int>(static_cast<long long>(steps) * (wave + 1) / kGradWaves);
    grad_float4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    float bsum = 0.0f;
    for (int s = s0; s < s1; s += kGradU) {
        float a[kGradU], b[kGradU];
#pragma unroll
        for (int u = 0; u < kGradU; ++u) {
            const int row = min(4 * (s + u) + kr, batch - 1);
            a[u] = in[static_cast<size_t>(row) * nin + ic];
            b[u] = dout[static_cast<size_t>(row) * nout + jc];
        }
#pragma unroll
        for (int u = 0; u < kGradU; ++u) {
            const bool live = s + u < s1 && 4 * (s + u) + kr < batch;
            const float av = live && ai ? a[u] : 0.0f, bv = live && bj ? b[u] : 0.0f;
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc, 0, 0, 0);
            bsum += bv;
        }
    }
    // Lane l holds column l % 16 of rows 4 (l / 16) .. + 3 of the wave's tile.
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][(4 * kr + v) * kTile + lane % kTile] = acc[v];
    bpart[wave][lane] = bsum;
    __syncthreads();
    if (tid < kTile * kTile) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kGradWaves; ++w) t += part[w][tid];
        const int ti = i0 + tid / kTile, tj = j0 + tid % kTile;
        if (ti < nin && tj < nout) grads[offw + ti * nout + tj] = t;
    } else if (i0 == 0 && tid < kTile * kTile + kTile) {
        const int c = tid - kTile * kTile;
        float t = 0.0f;
        for (int w = 0; w < kGradWaves; ++w)
#pragma unroll
            for (int k = 0; k < 4; ++k) t += bpart[w][k * kTile + c];
        if (j0 + c < nout) grads[offb + j0 + c] = t;
    }
}

// Adam (Kingma & Ba), bias-corrected, fp32.
__global__ __launch_bounds__(256) void adam_kernel(int n, float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                                   float b2, float eps, float c1, float c2) {
    const int t = static_cast<int>(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= n) return;
    const float gt = g[t];
    const float mt = b1 * m[t] + (1.0f - b1) * gt;
    const float vt = b2 * v[t] + (1.0f - b2) * gt * gt;
    m[t] = mt;
    v[t] = vt;
    p[t] -= lr * (mt / c1) / (sqrtf(vt / c2) + eps);
}

__global__ void feature_zero_kernel(int* __restrict__ ws, int n) {
    if (static_cast<int>(threadIdx.x) < n) ws[threadIdx.x] = 0;
}

namespace {
inline int blocks_for(long long n) { return static_cast<int>((n + 255) / 256); }
}  // namespace

hipError_t launch_features(int rows, int cols, int nnz, const int* row_ptr, const int* col_ind, float* feat,
                           int* ws, hipStream_t stream) {
    hipLaunchKernelGGL(feature_zero_kernel, dim3(1), dim3(64), 0, stream, ws, kRowBins + kDistBins + 1);
    const int groups = rows / kWave + (rows % kWave != 0);
    const int g = std::max(1, std::min((groups + kFeatWaves - 1) / kFeatWaves, kFeatMaxBlocks));
    hipLaunchKernelGGL(feature_count_kernel, dim3(g), dim3(kFeatThreads), 0, stream, rows, cols, row_ptr, col_ind, ws);
    hipLaunchKernelGGL(feature_finish_kernel, dim3(1), dim3(64), 0, stream, rows, nnz, ws, feat);
    return hipGetLastError();
}

namespace {
int mlp_blocks(int batch) { return batch / kMlpRows + (batch % kMlpRows != 0); }

hipError_t launch_weight_grads(int batch, const float* X, const float* H1, const float* H2, const float* dY,
                               const float* dH2, const float* dH1, float* grads, hipStream_t stream) {
    hipLaunchKernelGGL(mlp_weight_grads_kernel, dim3(kTiles1 + kTiles2 + kTiles3), dim3(kGradThreads), 0, stream,
                       batch, X, H1, H2, dY, dH2, dH1, grads);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_mlp_forward(int batch, const float* X, const float* params, float* H1, float* H2, float* Y,
                              hipStream_t stream) {
    hipLaunchKernelGGL((mlp_rows_kernel<false>), dim3(mlp_blocks(batch)), dim3(kMlpThreads), 0, stream, batch, X,
                       params, H1, H2, Y, static_cast<const float*>(nullptr), 0.0f, static_cast<float*>(nullptr),
                       static_cast<float*>(nullptr), static_cast<float*>(nullptr));
    return hipGetLastError();
}

hipError_t launch_mlp_backward(int batch, const float* X, const float* params, const float* H1, const float* H2,
                               const float* dY, float* dH2, float* dH1, float* grads, hipStream_t stream) {
    hipLaunchKernelGGL(mlp_input_grads_kernel, dim3(mlp_blocks(batch)), dim3(kMlpThreads), 0, stream, batch, params,
                       H1, H2, dY, dH2, dH1);
    return launch_weight_grads(batch, X, H1, H2, dY, dH2, dH1, grads, stream);
}

hipError_t launch_mlp_grads(int batch, const float* X, const float* T, const float* params, float scale, float* H1,
                            float* H2, float* Y, float* dY, float* dH2, float* dH1, float* grads,
                            hipStream_t stream) {
    hipLaunchKernelGGL((mlp_rows_kernel<true>), dim3(mlp_blocks(batch)), dim3(kMlpThreads), 0, stream, batch, X,
                       params, H1, H2, Y, T, scale, dY, dH2, dH1);
    return launch_weight_grads(batch, X, H1, H2, dY, dH2, dH1, grads, stream);
}

hipError_t launch_mse_grad(int n, const float* Y, const float* T, float* dY, float scale, hipStream_t stream) {
    hipLaunchKernelGGL(mse_grad_kernel, dim3(blocks_for(n)), dim3(256), 0, stream, n, Y, T, dY, scale);
    return hipGetLastError();
}

hipError_t launch_adam(int n, float* p, const float* g, float* m, float* v, float lr, float b1, float b2, float eps,
                       int step, hipStream_t stream) {
    const float c1 = 1.0f - powf(b1, static_cast<float>(step));
    const float c2 = 1.0f - powf(b2, static_cast<float>(step));
    hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n)), dim3(256), 0, stream, n, p, g, m, v, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace cmrs
