// Learning from label proportions with a linear classifier (the LLP and
// Label-DP use cases): the classifier labels every row of a bag, a grouped
// soft COUNT per (bag, class) of its softmax is the relaxed query answer,
// and the backward returns the classifier's weight and bias gradients.
//
// Forward: bags are consecutive runs of `bag` rows (a power of two).  For
// bag <= 64 a wave takes 64 consecutive rows, one per lane, and adds each
// bag's probabilities with a butterfly over the bag's aligned group of
// lanes; for larger bags a wave takes whole bags, lanes striding over the
// rows, then a butterfly over the wave.  Each bag's sum is formed inside one
// wave in a fixed order (float64), so results do not depend on scheduling.
// Backward: every thread recomputes its rows' probabilities, keeps the
// gradient terms in registers, the workgroup reduces them in float64 into
// one partial row, and a one-workgroup kernel adds the rows in a fixed order.
#include "common.hpp"

namespace tdp {

namespace {

constexpr int kLlpMaxF = 16;
constexpr int kLlpMaxC = 4;
constexpr int kLlpThreads = 256;
constexpr int kLlpMaxGrid = 1024;
constexpr int kLlpFinThreads = 1024;  // threads of the one-workgroup finishing kernels

struct LlpArgs {
    const float* X;
    int64_t n;
    int F;
    const float* W;  // [C][F]
    const float* b;  // [C]
    int64_t bag;
    int bag_shift;   // log2(bag): a 64-bit division per row cost more than the rest of it
};

// The classifier in registers (features past F are zero).
template <int C, int FM>
struct LlpParams {
    float w[C][FM], b[C];
    __device__ __forceinline__ explicit LlpParams(const LlpArgs& a) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            b[c] = a.b[c];
#pragma unroll
            for (int f = 0; f < FM; ++f) w[c][f] = f < a.F ? a.W[c * a.F + f] : 0.0f;
        }
    }
};

// Class probabilities of one row: softmax of W x + b, float32.
template <int C, int FM>
__device__ __forceinline__ void llp_probs(const LlpParams<C, FM>& m, const float x[FM], float p[C]) {
    float z[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        float a = m.b[c];
#pragma unroll
        for (int f = 0; f < FM; ++f) a = fmaf(m.w[c][f], x[f], a);  // zeros past F
        z[c] = a;
    }
    float top = z[0];
#pragma unroll
    for (int c = 1; c < C; ++c) top = fmaxf(top, z[c]);
    float sum = 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        z[c] = __expf(z[c] - top);
        sum += z[c];
    }
    const float inv = 1.0f / sum;
#pragma unroll
    for (int c = 0; c < C; ++c) p[c] = z[c] * inv;
}

template <int FM>
__device__ __forceinline__ void llp_load_row(const LlpArgs& a, int64_t row, float x[FM]) {
#pragma unroll
    for (int f = 0; f < FM; ++f) x[f] = 0.0f;
    if (row >= a.n) return;
    const float* src = a.X + row * a.F;
    if ((a.F & 3) == 0) {
#pragma unroll
        for (int f = 0; f < FM; f += 4) {
            if (f < a.F) {
                const float4 q = *(const float4*)(src + f);
                x[f] = q.x; x[f + 1] = q.y; x[f + 2] = q.z; x[f + 3] = q.w;
            }
        }
    } else {
#pragma unroll
        for (int f = 0; f < FM; ++f)
            if (f < a.F) x[f] = src[f];
    }
}

// Squared error of one cell's count against T, its gradient written to dS
// (float64 arithmetic, as the oracle's mean squared error).
__device__ __forceinline__ double llp_cell_loss(int64_t cell, double acc, float* S, const float* T, float* dS,
                                                double inv_cells) {
    const float sv = (float)acc;
    S[cell] = sv;
    if (!T) return 0.0;
    const double d = (double)sv - (double)T[cell];
    dS[cell] = (float)(2.0 * d * inv_cells);
    return d * d;
}

// One butterfly step that also halves the values: the lanes with the bit
// `off` keep the pair sum of b, the others that of a.
__device__ __forceinline__ double llp_fold(double a, double b, int off, int lane) {
    const bool hi = lane & off;
    return (hi ? b : a) + __shfl_xor(hi ? a : b, off, kWave);
}

// FM: the features the kernel is built for, 8 or 16.  Two rows per lane are in
// flight.
template <int C, int FM>
__global__ __launch_bounds__(kLlpThreads) void llp_fwd_kernel(LlpArgs a, float* S, const float* T, float* dS,
                                                              double* loss_part) {
    __shared__ double s_l[kLlpThreads / kWave];
    const LlpParams<C, FM> m(a);
    double lsum = 0.0;  // this lane's squared errors (lanes that write bags)
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * kLlpThreads + threadIdx.x) / kWave;
    const int64_t n_waves = (int64_t)gridDim.x * kLlpThreads / kWave;
    const int64_t n_bags = (a.n + a.bag - 1) >> a.bag_shift;
    const double inv_cells = 1.0 / (double)(n_bags * C);
    if (a.bag <= kWave) {
        const int64_t units = (a.n + kWave - 1) / kWave;
        for (int64_t u = wave; u < units; u += 2 * n_waves) {
            float x[2][FM], p[C];
            double acc[2][C];
#pragma unroll
            for (int k = 0; k < 2; ++k) llp_load_row<FM>(a, (u + k * n_waves) * kWave + lane, x[k]);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                llp_probs<C, FM>(m, x[k], p);
#pragma unroll
                for (int c = 0; c < C; ++c) acc[k][c] = (u + k * n_waves) * kWave + lane < a.n ? (double)p[c] : 0.0;
            }
            // each bag's aligned group of lanes: the two units, then (even C)
            // the classes, are folded into one another first, so that a
            // step moves half the values of the one before
            int off = (int)a.bag / 2, k = 0;
            double v[C];
            if (off == 0) {  // bags of one row: nothing to add
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int64_t row = (u + q * n_waves) * kWave + lane;
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (row < a.n) lsum += llp_cell_loss(row * C + c, acc[q][c], S, T, dS, inv_cells);
                }
                continue;
            }
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] = llp_fold(acc[0][c], acc[1][c], off, lane);
            k = lane & off ? 1 : 0;
            off >>= 1;
            int c0 = 0;
            constexpr int H = C % 2 == 0 ? C / 2 : C;  // values after the classes are folded
            const bool folded = C % 2 == 0 && off > 0;
            if (folded) {
#pragma unroll
                for (int c = 0; c < H; ++c) v[c] = llp_fold(v[c], v[(c + H) % C], off, lane);
                c0 = lane & off ? H : 0;
                off >>= 1;
            }
            const int own = 2 * off - (off > 0);  // the lanes below this position repeat one sum
            for (; off > 0; off >>= 1) {
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (c < H || !folded) v[c] += __shfl_xor(v[c], off, kWave);
            }
            // the first row of the lane's bag: a bag without one has no cells
            const int64_t row = ((u + k * n_waves) * kWave + lane) & ~(a.bag - 1);
            if ((lane & own) == 0 && row < a.n)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (c < H || !folded)
                        lsum += llp_cell_loss((row >> a.bag_shift) * C + c0 + c, v[c], S, T, dS, inv_cells);
        }
    } else {
        for (int64_t j = wave; j < n_bags; j += n_waves) {
            const int64_t r0 = j * a.bag, r1 = r0 + a.bag < a.n ? r0 + a.bag : a.n;
            double acc[C];
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = 0.0;
            for (int64_t row = r0 + lane; row < r1; row += 2 * kWave) {
                float x[2][FM], p[C];
#pragma unroll
                for (int k = 0; k < 2; ++k) llp_load_row<FM>(a, row + k * kWave < r1 ? row + k * kWave : a.n, x[k]);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    llp_probs<C, FM>(m, x[k], p);
#pragma unroll
                    for (int c = 0; c < C; ++c) acc[c] += row + k * kWave < r1 ? (double)p[c] : 0.0;
                }
            }
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
#pragma unroll
                for (int c = 0; c < C; ++c) acc[c] += __shfl_xor(acc[c], off, kWave);
            }
            if (lane == 0)
#pragma unroll
                for (int c = 0; c < C; ++c) lsum += llp_cell_loss(j * C + c, acc[c], S, T, dS, inv_cells);
        }
    }
    if (T) {  // the workgroup's squared errors, in a fixed order
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off, kWave);
        if (lane == 0) s_l[threadIdx.x / kWave] = lsum;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < kLlpThreads / kWave; ++w) t += s_l[w];
            loss_part[blockIdx.x] = t;
        }
    }
}

// One workgroup: the loss, the partials added in workgroup order.
__global__ __launch_bounds__(kLlpFinThreads) void llp_loss_finish_kernel(const double* part, int n_parts,
                                                                         double inv_cells, float* d_loss) {
    constexpr int kW = kLlpFinThreads / kWave;
    __shared__ double s_w[kW];
    double t = 0.0;
    for (int b = threadIdx.x; b < n_parts; b += kLlpFinThreads) t += part[b];  // each thread's strided share, in order
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, kWave);
    if (lane_id() == 0) s_w[threadIdx.x / kWave] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int w = 0; w < kW; ++w) tot += s_w[w];
        *d_loss = (float)(tot * inv_cells);
    }
}

// Per-thread gradient terms over a grid-stride of rows, reduced to one
// float64 partial row per workgroup: [C][kLlpMaxF] weights then [C] biases.
template <int C, int FM>
__global__ __launch_bounds__(kLlpThreads) void llp_bwd_kernel(LlpArgs a, const float* __restrict__ dS, double* part) {
    __shared__ double s_red[kLlpThreads / kWave][C * (FM + 1)];
    const LlpParams<C, FM> m(a);
    float gw[C][FM], gb[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        gb[c] = 0.0f;
#pragma unroll
        for (int f = 0; f < FM; ++f) gw[c][f] = 0.0f;
    }
    const int64_t stride = (int64_t)gridDim.x * kLlpThreads;
    for (int64_t r0 = (int64_t)blockIdx.x * kLlpThreads + threadIdx.x; r0 < a.n; r0 += 2 * stride) {
        float x[2][FM], dp[2][C];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int64_t row = r0 + k * stride;
            llp_load_row<FM>(a, row, x[k]);
            const float* d = dS + ((row < a.n ? row : r0) >> a.bag_shift) * C;
#pragma unroll
            for (int c = 0; c < C; ++c) dp[k][c] = d[c];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (r0 + k * stride >= a.n) continue;
            float p[C], s = 0.0f;
            llp_probs<C, FM>(m, x[k], p);
#pragma unroll
            for (int c = 0; c < C; ++c) s = fmaf(p[c], dp[k][c], s);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float dz = p[c] * (dp[k][c] - s);
                gb[c] += dz;
#pragma unroll
                for (int f = 0; f < FM; ++f) gw[c][f] = fmaf(dz, x[k][f], gw[c][f]);
            }
        }
    }
    // workgroup sums in float64, written as this workgroup's partial row
    const int lane = lane_id(), wv = threadIdx.x / kWave;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int f = 0; f <= FM; ++f) {
            const double t = wave_sum((double)(f < FM ? gw[c][f < FM ? f : 0] : gb[c]));
            if (lane == 0) s_red[wv][c * (FM + 1) + f] = t;
        }
    __syncthreads();
    double* row = part + (int64_t)blockIdx.x * C * (kLlpMaxF + 1);
    for (int k = threadIdx.x; k < C * (kLlpMaxF + 1); k += kLlpThreads) {
        const int c = k / (kLlpMaxF + 1), f = k % (kLlpMaxF + 1), at = f < FM ? f : FM;
        double tot = 0.0;
        if (f < FM || f == kLlpMaxF)
            for (int w = 0; w < kLlpThreads / kWave; ++w) tot += s_red[w][c * (FM + 1) + at];
        row[k] = tot;
    }
}

// One workgroup: the partial rows added in a fixed order, to float32.
// Thread (slice s, column k) adds rows s, s + slices, ... (16 loads in
// flight), then the slices are added in order: one thread per column walking
// every row one dependent load at a time took 245 us for 1024 rows.

__global__ __launch_bounds__(kLlpFinThreads) void llp_bwd_finish_kernel(const double* part, int n_parts, int C, int F,
                                                                        float* dW, float* db) {
    __shared__ double s_acc[kLlpFinThreads];
    const int cols = C * (kLlpMaxF + 1);  // <= 68
    const int slices = kLlpFinThreads / cols;
    const int k = threadIdx.x % cols, sl = threadIdx.x / cols;
    double t = 0.0;
    if (sl < slices) {
        for (int b0 = sl; b0 < n_parts; b0 += 16 * slices) {
            double v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int b = b0 + q * slices;
                v[q] = b < n_parts ? part[(int64_t)b * cols + k] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < 16; ++q) t += v[q];
        }
    }
    s_acc[threadIdx.x] = t;
    __syncthreads();
    if (threadIdx.x < cols) {
        double tot = 0.0;
        for (int q = 0; q < slices; ++q) tot += s_acc[q * cols + threadIdx.x];
        const int c = threadIdx.x / (kLlpMaxF + 1), f = threadIdx.x % (kLlpMaxF + 1);
        if (f < F) dW[c * F + f] = (float)tot;
        else if (f == kLlpMaxF) db[c] = (float)tot;
    }
}

// Argmax of the logits, accumulated in float64 as b, then one fused
// multiply-add per feature in feature order; ties to the smallest class.
__global__ void llp_predict_kernel(LlpArgs a, int C, int8_t* out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < a.n; row += stride) {
        int best = 0;
        double bz = 0.0;
        for (int c = 0; c < C; ++c) {
            double z = (double)a.b[c];
            for (int f = 0; f < a.F; ++f) z = fma((double)a.W[c * a.F + f], (double)a.X[row * a.F + f], z);
            if (c == 0 || z > bz) {
                best = c;
                bz = z;
            }
        }
        out[row] = (int8_t)best;
    }
}

__global__ void count_fill_kernel(float* out, int64_t cells, const float* noise) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < cells; j += stride)
        out[j] = noise ? noise[j] : 0.0f;
}

__global__ void count_place_kernel(const int64_t* k0, const int64_t* k1, const int64_t* count,
                                   const int64_t* d_n_groups, int64_t lo0, int64_t card0, int64_t lo1, int64_t card1,
                                   const float* noise, float* out, int32_t* status) {
    const int64_t m = *d_n_groups;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const int64_t u0 = k0[i] - lo0, u1 = k1 ? k1[i] - lo1 : 0;
        if (u0 < 0 || u0 >= card0 || u1 < 0 || u1 >= card1) {
            raise_flag(status, TDP_FLAG_KEY_DOMAIN);
            continue;
        }
        const int64_t j = u0 * card1 + u1;
        out[j] = (float)count[i] + (noise ? noise[j] : 0.0f);
    }
}

int llp_check(const LlpArgs& a, int C, const char* fn) {
    if (a.n < 0 || (a.n > 0 && (!a.X || !a.W || !a.b))) return fail(TDP_EINVAL, "%s: null pointer or n < 0", fn);
    if (a.F < 1 || a.F > kLlpMaxF) return fail(TDP_EINVAL, "%s: F=%d outside 1..%d", fn, a.F, kLlpMaxF);
    if (C < 2 || C > kLlpMaxC) return fail(TDP_EINVAL, "%s: C=%d outside 2..%d", fn, C, kLlpMaxC);
    if (a.bag < 1 || a.bag > (1 << 20) || (a.bag & (a.bag - 1)))
        return fail(TDP_EINVAL, "%s: bag=%lld is not a power of two in 1..2^20", fn, (long long)a.bag);
    if ((uintptr_t)a.X & 15) return fail(TDP_EINVAL, "%s: X must be 16-byte aligned", fn);
    return TDP_OK;
}

int log2_of(int64_t v) {
    int s = 0;
    while (s < 62 && ((int64_t)1 << s) < v) ++s;
    return s;
}

template <int C>
void llp_fwd(const LlpArgs& a, int grid, float* S, const float* T, float* dS, double* lp, hipStream_t s) {
    if (a.F <= 8) llp_fwd_kernel<C, 8><<<grid, kLlpThreads, 0, s>>>(a, S, T, dS, lp);
    else llp_fwd_kernel<C, kLlpMaxF><<<grid, kLlpThreads, 0, s>>>(a, S, T, dS, lp);
}

template <int C>
void llp_bwd(const LlpArgs& a, int grid, const float* dS, double* part, hipStream_t s) {
    if (a.F <= 8) llp_bwd_kernel<C, 8><<<grid, kLlpThreads, 0, s>>>(a, dS, part);
    else llp_bwd_kernel<C, kLlpMaxF><<<grid, kLlpThreads, 0, s>>>(a, dS, part);
}

int llp_grid(int64_t n) {
    return (int)std::min<int64_t>(std::max<int64_t>(ceil_div(n, (int64_t)kLlpThreads * 16), 1), kLlpMaxGrid);
}

}  // namespace

}  // namespace tdp

using namespace tdp;

namespace {
constexpr int kLlpFwdMaxGrid = 4096;
}

extern "C" size_t tdp_llp_workspace_size(int32_t C) {
    WsAlloc wa(nullptr);
    wa.take<double>((size_t)kLlpMaxGrid * std::max(C, 1) * (kLlpMaxF + 1));
    wa.take<double>(kLlpFwdMaxGrid);
    return wa.bytes();
}

extern "C" int tdp_llp_bag_count(const float* X, int64_t n, int32_t F, const float* W, const float* b, int32_t C,
                                 int64_t bag, float* S, const float* T, float* d_loss, float* dS, void* ws,
                                 size_t ws_bytes, hipStream_t stream) {
    LlpArgs a{X, n, F, W, b, bag, log2_of(bag)};
    int rc = llp_check(a, C, "tdp_llp_bag_count");
    if (rc) return rc;
    if (n > 0 && !S) return fail(TDP_EINVAL, "tdp_llp_bag_count: null S");
    if (T && (!d_loss || !dS)) return fail(TDP_EINVAL, "tdp_llp_bag_count: T given without d_loss and dS");
    if (T && (!ws || ws_bytes < tdp_llp_workspace_size(C)))
        return fail_need(TDP_EWORKSPACE, (int64_t)tdp_llp_workspace_size(C), "tdp_llp_bag_count: workspace %zu < %zu",
                         ws_bytes, tdp_llp_workspace_size(C));
    if (n == 0) return TDP_OK;
    WsAlloc wa(ws);
    wa.take<double>((size_t)kLlpMaxGrid * std::max(C, 1) * (kLlpMaxF + 1));
    double* lp = T ? wa.take<double>(kLlpFwdMaxGrid) : nullptr;
    const int grid = (int)std::min<int64_t>(std::max<int64_t>(ceil_div(n, (int64_t)kLlpThreads * 8), 1), kLlpFwdMaxGrid);
    switch (C) {
        case 2: llp_fwd<2>(a, grid, S, T, dS, lp, stream); break;
        case 3: llp_fwd<3>(a, grid, S, T, dS, lp, stream); break;
        default: llp_fwd<4>(a, grid, S, T, dS, lp, stream); break;
    }
    if (T) {
        const int64_t n_bags = (n + bag - 1) / bag;
        llp_loss_finish_kernel<<<1, kLlpFinThreads, 0, stream>>>(lp, grid, 1.0 / (double)(n_bags * C), d_loss);
    }
    return launch_status("tdp_llp_bag_count");
}

extern "C" int tdp_llp_bag_count_bwd(const float* X, int64_t n, int32_t F, const float* W, const float* b, int32_t C,
                                     int64_t bag, const float* dS, float* dW, float* db, void* ws, size_t ws_bytes,
                                     hipStream_t stream) {
    LlpArgs a{X, n, F, W, b, bag, log2_of(bag)};
    int rc = llp_check(a, C, "tdp_llp_bag_count_bwd");
    if (rc) return rc;
    if (!dW || !db || (n > 0 && !dS)) return fail(TDP_EINVAL, "tdp_llp_bag_count_bwd: null dS, dW or db");
    if (!ws || ws_bytes < tdp_llp_workspace_size(C))
        return fail_need(TDP_EWORKSPACE, (int64_t)tdp_llp_workspace_size(C), "tdp_llp_bag_count_bwd: workspace %zu < %zu",
                         ws_bytes, tdp_llp_workspace_size(C));
    double* part = (double*)ws;
    const int grid = llp_grid(n);
    switch (C) {
        case 2: llp_bwd<2>(a, grid, dS, part, stream); break;
        case 3: llp_bwd<3>(a, grid, dS, part, stream); break;
        default: llp_bwd<4>(a, grid, dS, part, stream); break;
    }
    llp_bwd_finish_kernel<<<1, kLlpFinThreads, 0, stream>>>(part, grid, C, F, dW, db);
    return launch_status("tdp_llp_bag_count_bwd");
}

extern "C" int tdp_llp_predict(const float* X, int64_t n, int32_t F, const float* W, const float* b, int32_t C,
                               int8_t* out, hipStream_t stream) {
    LlpArgs a{X, n, F, W, b, 1, 0};
    int rc = llp_check(a, C, "tdp_llp_predict");
    if (rc) return rc;
    if (n > 0 && !out) return fail(TDP_EINVAL, "tdp_llp_predict: null out");
    if (n == 0) return TDP_OK;
    llp_predict_kernel<<<(int)std::min<int64_t>(ceil_div(n, 256), 4096), 256, 0, stream>>>(a, C, out);
    return launch_status("tdp_llp_predict");
}

extern "C" int tdp_count_table(const int64_t* key0, const int64_t* key1, const int64_t* count,
                               const int64_t* d_n_groups, int64_t lo0, int64_t card0, int64_t lo1, int64_t card1,
                               const float* noise, float* out, int32_t* d_status, hipStream_t stream) {
    if (!key0 || !count || !d_n_groups || !out) return fail(TDP_EINVAL, "tdp_count_table: null pointer");
    if (card0 < 1 || card1 < 1 || card0 > (1ll << 31) / card1)
        return fail(TDP_EINVAL, "tdp_count_table: table of %lld x %lld cells", (long long)card0, (long long)card1);
    if (!key1 && card1 != 1) return fail(TDP_EINVAL, "tdp_count_table: key1 == NULL requires card1 == 1");
    const int64_t cells = card0 * card1;
    count_fill_kernel<<<(int)std::min<int64_t>(ceil_div(cells, 256), 4096), 256, 0, stream>>>(out, cells, noise);
    count_place_kernel<<<(int)std::min<int64_t>(ceil_div(cells, 256), 4096), 256, 0, stream>>>(
        key0, key1, count, d_n_groups, lo0, card0, lo1, card1, noise, out, d_status);
    return launch_status("tdp_count_table");
}

namespace {
__global__ void segment_ids_kernel(int64_t n, int64_t width, int32_t* out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = (int32_t)(i / width);
}
}  // namespace

extern "C" int tdp_segment_ids(int64_t n, int64_t width, int32_t* out, hipStream_t stream) {
    if (n < 0 || width < 1 || (n > 0 && !out)) return fail(TDP_EINVAL, "tdp_segment_ids: n=%lld width=%lld", (long long)n, (long long)width);
    if ((n - 1) / width > INT32_MAX) return fail(TDP_EINVAL, "tdp_segment_ids: more than 2^31 segments");
    if (n == 0) return TDP_OK;
    segment_ids_kernel<<<(int)std::min<int64_t>(ceil_div(n, 256), 4096), 256, 0, stream>>>(n, width, out);
    return launch_status("tdp_segment_ids");
}
