// Non-GEMM kernels of the PPO learner for gfx950: Philox4x32-10 action noise,
// the policy/critic output heads fused with sampling (rollout) or with the
// PPO loss and its output gradients (update), GAE with the float64 advantage
// statistics, gradient assembly with the float64 global norm, and Adam.
#include "common.hpp"

#include <algorithm>
#include <mutex>
#include "philox.hpp"

namespace ppo {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2Pi = 1.8378770664093453f;
constexpr int kMaxAct = 16;

// ------------------------------------------------------------------ Philox
__global__ void philox_blocks_kernel(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2,
                                     uint32_t c3, long long n, uint32_t *out) {
    for (long long i = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<long long>(gridDim.x) * blockDim.x) {
        uint32_t c[4] = {c0 + static_cast<uint32_t>(i), c1, c2, c3};
        philox4x32_10(c, k0, k1);
        *reinterpret_cast<u32x4 *>(out + 4 * i) = u32x4{c[0], c[1], c[2], c[3]};
    }
}

// --------------------------------------------------------------- reductions
__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ inline double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// ------------------------------------------------------------ obs gather
template <typename T>
__global__ void gather_obs_kernel(const float *obs, const int32_t *idx, int src_rows, int rows, int D, int ld,
                                  T *out) {
    const long long total = static_cast<long long>(rows) * ld;
    for (long long e = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; e < total;
         e += static_cast<long long>(gridDim.x) * blockDim.x) {
        const int r = static_cast<int>(e / ld);
        const int k = static_cast<int>(e - static_cast<long long>(r) * ld);
        // indices outside [0, src_rows) are clamped so a bad permutation cannot fault
        const long long src_row = idx ? min(max(idx[r], 0), src_rows - 1) : r;
        const float v = k < D ? obs[src_row * D + k] : 0.0f;
        out[e] = Elem<T>::from_f(v);
    }
}

// ------------------------------------------------- output-layer helpers
constexpr int kHeadThreads = 256;
constexpr int kLossRows = 32;     // mini-batch samples per block (loss)
constexpr int kSampleRows = 16;   // environments per block (rollout)
constexpr int kWPad = 4;          // floats of row padding for staged output-layer weights

// 8 consecutive activations of one row as float32.
template <typename T>
__device__ inline void load8(const T *src, float (&x)[8]) {
    if constexpr (sizeof(T) == 2) {
        const u32x4 r = *reinterpret_cast<const u32x4 *>(src);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            x[2 * w] = __uint_as_float(r[w] << 16);
            x[2 * w + 1] = __uint_as_float(r[w] & 0xFFFF0000u);
        }
    } else {
        const float4 p = reinterpret_cast<const float4 *>(src)[0];
        const float4 q = reinterpret_cast<const float4 *>(src)[1];
        x[0] = p.x; x[1] = p.y; x[2] = p.z; x[3] = p.w;
        x[4] = q.x; x[5] = q.y; x[6] = q.z; x[7] = q.w;
    }
}

// Output-layer weights of both networks: rows j < A are the actor's, row A
// the critic's, each padded to Hl + kWPad floats.  Staged in LDS when they
// fit (dynamic shared memory), else read from global memory.
struct HeadWeights {
    const float *w;
    int pitch;
};

__device__ inline HeadWeights stage_head_weights(float *s_w, bool in_lds, const float *Wa, const float *Wc, int A,
                                                 int Hl) {
    if (!in_lds) return HeadWeights{nullptr, 0};
    const int pitch = Hl + kWPad;
    const int n = (A + 1) * Hl;
    // eight loads in flight per thread before any store
    constexpr int U = 8;
    for (int q0 = threadIdx.x; q0 < n; q0 += U * blockDim.x) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * blockDim.x;
            const int j = q / Hl, k = q - (q / Hl) * Hl;
            v[u] = q < n ? (j < A ? Wa[static_cast<long long>(j) * Hl + k] : Wc[k]) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * blockDim.x;
            const int j = q / Hl, k = q - (q / Hl) * Hl;
            if (q < n) s_w[j * pitch + k] = v[u];
        }
    }
    __syncthreads();
    return HeadWeights{s_w, pitch};
}

__device__ inline const float *head_row(const HeadWeights &hw, const float *Wa, const float *Wc, int A, int Hl,
                                        int j) {
    if (hw.w) return hw.w + j * hw.pitch;
    return j < A ? Wa + static_cast<long long>(j) * Hl : Wc;
}

// out[i][j] = b_j + h_i . W_j for the A actor outputs (j < A) and the critic
// value (j == A); one dot product per thread.  Hl is a multiple of 16.
// The block's rows of both last hidden layers, staged in LDS (pitch Hl + 8
// elements) with coalesced 16-byte loads, four in flight per thread.
template <typename T>
__device__ inline void stage_hidden_rows(T *ha_l, T *hc_l, const T *ha, const T *hc, int r0, int rows, int Hl,
                                         bool actor, bool critic) {
    constexpr int VEC = 16 / sizeof(T);
    const int pitch = Hl + 8;
    const int per_row = Hl / VEC;
    const int n = 2 * rows * per_row;
    constexpr int U = 4;
    for (int q0 = threadIdx.x; q0 < n; q0 += U * blockDim.x) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * blockDim.x;
            const int net = q / (rows * per_row);
            const int rem = q - net * rows * per_row;
            const int i = rem / per_row, c = (rem - i * per_row) * VEC;
            const bool want = q < n && (net == 0 ? actor : critic);
            if (want)
                v[u] = *reinterpret_cast<const u32x4 *>((net == 0 ? ha : hc) + static_cast<long long>(r0 + i) * Hl + c);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * blockDim.x;
            const int net = q / (rows * per_row);
            const int rem = q - net * rows * per_row;
            const int i = rem / per_row, c = (rem - i * per_row) * VEC;
            const bool want = q < n && (net == 0 ? actor : critic);
            if (want) *reinterpret_cast<u32x4 *>((net == 0 ? ha_l : hc_l) + i * pitch + c) = v[u];
        }
    }
    __syncthreads();
}

// Bytes of dynamic LDS for `rows` staged rows of both last hidden layers,
// 0 when they do not fit next to the output-layer weights.
template <typename T>
size_t head_rows_lds(int rows, int Hl, size_t weight_bytes) {
    const size_t bytes = 2 * static_cast<size_t>(rows) * (Hl + 8) * sizeof(T);
    return weight_bytes + bytes <= 48 * 1024 ? bytes : 0;
}

template <typename T, int ROWS>
__device__ inline void output_layers(const T *ha, const T *hc, const T *ha_l, const T *hc_l,
                                     const HeadWeights &hw, const float *Wa,
                                     const float *ba, const float *Wc, const float *bc, int r0, int rows, int A,
                                     int Hl, bool actor, float (*out)[kMaxAct + 1]) {
    const int n_out = A + 1;
    for (int q = threadIdx.x; q < ROWS * n_out; q += kHeadThreads) {
        const int i = q / n_out, j = q - (q / n_out) * n_out;
        if (i >= rows || (j < A && !actor)) continue;
        const T *h = ha_l ? (j < A ? ha_l : hc_l) + i * (Hl + 8)
                          : (j < A ? ha : hc) + static_cast<long long>(r0 + i) * Hl;
        const float *w = head_row(hw, Wa, Wc, A, Hl, j);
        float acc = j < A ? ba[j] : bc[0];
        // 64 activations (eight 8-wide loads) in flight per step; Hl is a multiple of 16
        for (int k0 = 0; k0 < Hl; k0 += 64) {
            float x[8][8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + 8 * u < Hl) load8<T>(h + k0 + 8 * u, x[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + 8 * u < Hl)
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc += x[u][e] * w[k0 + 8 * u + e];
        }
        out[i][j] = acc;
    }
}

// ----------------------------------------------------------- head + sample
// Rollout: mu = h_a Wa^T + ba and V = h_c Wc^T + bc for 16 environments per
// block, then one lane per environment draws the diagonal-Gaussian action
// a = mu + sigma * eps with Philox noise and its log-density
// sum_j(-eps_j^2 / 2 - log sigma_j) - (A/2) log(2 pi).
template <typename T>
__global__ __launch_bounds__(kHeadThreads) void head_sample_kernel(const HeadSampleArgs a, int w_in_lds,
                                                                    int rows_lds_offset) {
    extern __shared__ float s_w[];
    __shared__ float s_out[kSampleRows][kMaxAct + 1];
    const int r0 = blockIdx.x * kSampleRows;
    const int rows = min(kSampleRows, a.N - r0);
    const int A = a.A;
    const HeadWeights hw = stage_head_weights(s_w, w_in_lds, a.Wa, a.Wc, A, a.Hl);
    const T *ha = static_cast<const T *>(a.ha);
    const T *hc = static_cast<const T *>(a.hc);
    T *ha_l = nullptr, *hc_l = nullptr;
    if (rows_lds_offset >= 0) {
        ha_l = reinterpret_cast<T *>(reinterpret_cast<char *>(s_w) + rows_lds_offset);
        hc_l = ha_l + kSampleRows * (a.Hl + 8);
        stage_hidden_rows<T>(ha_l, hc_l, ha, hc, r0, rows, a.Hl, !a.value_only, true);
    }
    output_layers<T, kSampleRows>(ha, hc, ha_l, hc_l, hw, a.Wa, a.ba, a.Wc, a.bc, r0, rows, A, a.Hl,
                                  !a.value_only, s_out);
    __syncthreads();
    const int i = threadIdx.x;
    if (i >= rows) return;
    const int n = r0 + i;
    if (a.values) a.values[n] = s_out[i][A];
    if (a.value_only) return;
    const int groups = (A + 3) / 4;
    CompSum lp;   // log-density in float32 with compensated summation
    for (int g = 0; g < groups; ++g) {
        uint32_t c[4] = {static_cast<uint32_t>(n) * groups + g, a.t, a.iteration, 1u};
        philox4x32_10(c, a.key0, a.key1);
        float eps[4];
        box_muller(c[0], c[1], eps[0], eps[1]);
        box_muller(c[2], c[3], eps[2], eps[3]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = 4 * g + q;
            if (j >= A) break;
            const float m = s_out[i][j];
            const float ls = a.logstd[j];
            lp.add_gauss(eps[q], ls);
            if (a.actions) a.actions[static_cast<long long>(n) * A + j] = m + expf(ls) * eps[q];
            if (a.mu) a.mu[static_cast<long long>(n) * A + j] = m;
        }
    }
    if (a.logp) a.logp[n] = lp.value();
}

// ------------------------------------------------------------- head + loss
// Update: for 32 mini-batch samples per block, the output layers, the
// log-probability of the stored action, the ratio, clipped surrogate and
// value loss with their gradients wrt mu and V (one lane per sample), then
// the gradient through the output layers and the last ELU into the last
// hidden pre-activations (8-wide row segments, coalesced).  Per-block sums of
// the loss terms and of the log-std gradient go to `partials` (wave-0
// shuffle reduction, fixed order).
template <typename T>
__global__ __launch_bounds__(kHeadThreads) void head_loss_kernel(const HeadLossArgs a, int w_in_lds,
                                                                  int rows_lds_offset) {
    extern __shared__ float s_w[];
    __shared__ float s_out[kLossRows][kMaxAct + 1];
    const int r0 = blockIdx.x * kLossRows;
    const int rows = min(kLossRows, a.M - r0);
    const int A = a.A, Hl = a.Hl;
    const int W = A + 8;
    const T *ha = static_cast<const T *>(a.ha);
    const T *hc = static_cast<const T *>(a.hc);
    const HeadWeights hw = stage_head_weights(s_w, w_in_lds, a.Wa, a.Wc, A, Hl);
    // the block's activation rows, read once from HBM and reused by the
    // output layers and the backward below
    T *ha_l = nullptr, *hc_l = nullptr;
    if (rows_lds_offset >= 0) {
        ha_l = reinterpret_cast<T *>(reinterpret_cast<char *>(s_w) + rows_lds_offset);
        hc_l = ha_l + kLossRows * (Hl + 8);
        stage_hidden_rows<T>(ha_l, hc_l, ha, hc, r0, rows, Hl, true, true);
    }
    output_layers<T, kLossRows>(ha, hc, ha_l, hc_l, hw, a.Wa, a.ba, a.Wc, a.bc, r0, rows, A, Hl, true, s_out);
    __syncthreads();

    const int tid = threadIdx.x;
    if (tid < 64) {
        float pl = 0.0f, vl = 0.0f, clipped = 0.0f, kl = 0.0f, kl_mu = 0.0f;
        float dls[kMaxAct];
#pragma unroll
        for (int j = 0; j < kMaxAct; ++j) dls[j] = 0.0f;
        if (tid < rows) {
            const int i = tid;
            const long long row = a.idx ? min(max(a.idx[r0 + i], 0), a.B - 1) : r0 + i;
            // Log-ratio log pi(a|s) - lp_old: the A log-density terms and -lp_old
            // summed with compensation in float32 (terms of order 1 that nearly
            // cancel against lp_old).
            float z[kMaxAct];
            CompSum lr;
#pragma unroll
            for (int j = 0; j < kMaxAct; ++j) {
                z[j] = 0.0f;
                if (j < A) {
                    const float ls = a.logstd[j];
                    const float inv_sigma = expf(-ls);
                    z[j] = (a.actions[row * A + j] - s_out[i][j]) * inv_sigma;
                    lr.add_gauss(z[j], ls);
                    if (a.mu_old) {
                        // mean-shift part of KL(pi_old || pi_new): (mu_old - mu)^2 / (2 sigma^2)
                        const float dm = (a.mu_old[row * A + j] - s_out[i][j]) * inv_sigma;
                        kl_mu += 0.5f * dm * dm;
                    }
                }
            }
            const float adv = a.adv[row];
            lr.add(-a.logp_old[row]);
            const float ratio = expf(lr.value());
            const float lo = 1.0f - a.clip, hi = 1.0f + a.clip;
            pl = -fminf(ratio * adv, fminf(fmaxf(ratio, lo), hi) * adv);
            const bool active = adv >= 0.0f ? (ratio <= hi) : (ratio >= lo);
            if (a.active_out) a.active_out[r0 + i] = active ? 1 : 0;
            if (a.ratio_out) a.ratio_out[r0 + i] = ratio;
            clipped = fabsf(ratio - 1.0f) > a.clip ? 1.0f : 0.0f;
            kl = (ratio - 1.0f) - logf(ratio);
            const float g_lp = active ? -a.inv_m * adv * ratio : 0.0f;

            const float V = s_out[i][A];
            const float ret = a.returns[row];
            const float diff = V - ret;
            float pass = 1.0f;
            vl = diff * diff;
            if (a.clip_value) {
                const float v_old = a.values_old[row];
                const float vc = v_old + fminf(fmaxf(V - v_old, -a.clip), a.clip);
                const float sqc = (vc - ret) * (vc - ret);
                pass = vl >= sqc ? 1.0f : 0.0f;
                vl = fmaxf(vl, sqc);
            }
            const float g_v = 2.0f * a.value_coef * a.inv_m * diff * pass;

            T *dha = static_cast<T *>(a.dz_head_a) + static_cast<long long>(r0 + i) * kHeadPad;
            T *dhc = static_cast<T *>(a.dz_head_c) + static_cast<long long>(r0 + i) * kHeadPad;
#pragma unroll
            for (int j = 0; j < kMaxAct; ++j) {
                float gm = 0.0f;
                if (j < A) {
                    gm = g_lp * z[j] * expf(-a.logstd[j]);
                    dls[j] = g_lp * __builtin_fmaf(z[j], z[j], -1.0f);
                    s_out[i][j] = gm;
                }
                dha[j] = Elem<T>::from_f(gm);
                dhc[j] = Elem<T>::from_f(j == 0 ? g_v : 0.0f);
            }
            s_out[i][A] = g_v;
        }
        // wave 0 holds every sample of the block: shuffle-reduce in a fixed order
        const float w_pl = wave_sum(pl), w_vl = wave_sum(vl), w_cl = wave_sum(clipped), w_kl = wave_sum(kl);
        const float w_klmu = wave_sum(kl_mu);
        float w_dls[kMaxAct];
#pragma unroll
        for (int j = 0; j < kMaxAct; ++j) w_dls[j] = wave_sum(dls[j]);
        if (tid == 0) {
            float *out = a.partials + static_cast<long long>(blockIdx.x) * W;
            out[0] = w_pl;
            out[1] = w_vl;
            out[2] = w_cl;
            out[3] = w_kl;
#pragma unroll
            for (int j = 0; j < kMaxAct; ++j)
                if (j < A) out[4 + j] = w_dls[j];
            float ent = 0.0f, kl_ls = 0.0f;
            if (blockIdx.x == 0) {
                // entropy of the state-independent policy at this step's parameters
                ent = 0.5f * A * (1.0f + kLog2Pi);
                for (int j = 0; j < A; ++j) ent += a.logstd[j];
                // sample-independent part of the KL:
                //   sum_j log(sigma / sigma_old) + sigma_old^2 / (2 sigma^2) - 1/2
                if (a.mu_old)
                    for (int j = 0; j < A; ++j) {
                        const float d = a.logstd_old[j] - a.logstd[j];
                        kl_ls += -d + 0.5f * expf(2.0f * d) - 0.5f;
                    }
            }
            out[4 + A] = ent;
            out[5 + A] = w_klmu;
            out[6 + A] = kl_ls;
        }
    }
    __syncthreads();

    // gradient into the last hidden pre-activations, both networks
    const int chunks = Hl / 8;
    const int n_q = 2 * kLossRows * chunks;
    // four 8-wide activation loads in flight per thread before the arithmetic
    constexpr int U = 4;
    for (int q0 = tid; q0 < n_q; q0 += U * kHeadThreads) {
        float xs[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * kHeadThreads;
            const int net = q / (kLossRows * chunks);
            const int rem = q - net * kLossRows * chunks;
            const int i = rem / chunks;
            const int k = (rem - i * chunks) * 8;
            if (q < n_q && i < rows) {
                if (ha_l)
                    load8<T>((net == 0 ? ha_l : hc_l) + i * (Hl + 8) + k, xs[u]);
                else
                    load8<T>((net == 0 ? ha : hc) + static_cast<long long>(r0 + i) * Hl + k, xs[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
        const int q = q0 + u * kHeadThreads;
        const int net = q / (kLossRows * chunks);
        const int rem = q - net * kLossRows * chunks;
        const int i = rem / chunks;
        const int k = (rem - i * chunks) * 8;
        if (q >= n_q || i >= rows) continue;
        const long long off = static_cast<long long>(r0 + i) * Hl + k;
        const float *x = xs[u];
        float g[8];
        if (net == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = 0.0f;
            for (int j = 0; j < A; ++j) {
                const float gm = s_out[i][j];
                const float *w = head_row(hw, a.Wa, a.Wc, A, Hl, j) + k;
#pragma unroll
                for (int e = 0; e < 8; ++e) g[e] += gm * w[e];
            }
        } else {
            const float gv = s_out[i][A];
            const float *w = head_row(hw, a.Wa, a.Wc, A, Hl, A) + k;
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = gv * w[e];
        }
        T o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = Elem<T>::from_f(g[e] * (x[e] > 0.0f ? 1.0f : x[e] + 1.0f));
        T *dst = static_cast<T *>(net == 0 ? a.dza : a.dzc) + off;
        if constexpr (sizeof(T) == 2) {
            *reinterpret_cast<u32x4 *>(dst) = *reinterpret_cast<const u32x4 *>(o);
        } else {
            reinterpret_cast<u32x4 *>(dst)[0] = reinterpret_cast<const u32x4 *>(o)[0];
            reinterpret_cast<u32x4 *>(dst)[1] = reinterpret_cast<const u32x4 *>(o)[1];
        }
        }
    }
}

// ------------------------------------------------------------------- GAE
// One lane walks VEC environments t = T-1 .. 0 (coalesced across lanes):
//   r' = r + gamma V timeout;  delta = r' + gamma (1 - d) V_next - V;
//   A = delta + gamma lambda (1 - d) A_next;  R = A + V.
// A lane's inputs load CHUNK steps at a time; their advantages' float64 mean
// and sum of squared deviations follow in two passes over the registers (no
// division per step), then the lanes' and waves' (count, mean, M2) combine by
// sums in a fixed order into one partial per block.
//
// Few environments: a latency chain.  Blocks of one wave spread 4096
// environments over 64 CUs instead of 16, and up to 32 steps load at once (a
// rollout of 24 waits for memory once).  Many: bandwidth.  Four environments
// per lane take 16-byte loads and 4-byte loads of the flags.  One environment
// per lane in blocks of four waves, 16 steps at a time, with a Welford update
// (a float64 division) per step and a tree of merges: 4096 x 24 in 8.9 us and
// the normalisation in 4.7 us, now 5.4 and 3.4; 2^20 x 24 with normalisation
// 146 us a call, now 125 (gae_shape has what lies between).
constexpr int kFinalizeThreads = 256;

template <int VEC, int CHUNK, int THREADS>
__global__ __launch_bounds__(THREADS) void gae_kernel(const GaeArgs a) {
    const unsigned n = (blockIdx.x * THREADS + threadIdx.x) * VEC;
    double cnt = 0.0, mean = 0.0, m2 = 0.0;
    if (n < static_cast<unsigned>(a.N)) {
        auto load_f = [](const float *p, float (&x)[VEC]) {
            if constexpr (VEC == 4) {
                const float4 q = *reinterpret_cast<const float4 *>(p);
                x[0] = q.x; x[1] = q.y; x[2] = q.z; x[3] = q.w;
            } else {
                x[0] = p[0];
            }
        };
        auto store_f = [](float *p, const float (&x)[VEC]) {
            if constexpr (VEC == 4)
                *reinterpret_cast<float4 *>(p) = make_float4(x[0], x[1], x[2], x[3]);
            else
                p[0] = x[0];
        };
        auto load_b = [](const uint8_t *p) -> uint32_t {
            if constexpr (VEC == 4) return *reinterpret_cast<const uint32_t *>(p);
            else return p[0];
        };
        float next_v[VEC], next_a[VEC];
        load_f(a.last_values + n, next_v);
#pragma unroll
        for (int c = 0; c < VEC; ++c) next_a[c] = 0.0f;
        const float gl = a.gamma * a.lam;
        for (int t0 = a.T - 1; t0 >= 0; t0 -= CHUNK) {
            float vv[CHUNK][VEC], rr[CHUNK][VEC];
            uint32_t dd[CHUNK], tt[CHUNK];
#pragma unroll
            for (int i = 0; i < CHUNK; ++i) {
                // past the first step its row again (no branches between loads)
                const long long s = static_cast<long long>(max(t0 - i, 0)) * a.N + n;
                load_f(a.values + s, vv[i]);
                load_f(a.rewards + s, rr[i]);
                dd[i] = load_b(a.dones + s);
            }
            if (a.timeouts) {
#pragma unroll
                for (int i = 0; i < CHUNK; ++i)
                    tt[i] = load_b(a.timeouts + static_cast<long long>(max(t0 - i, 0)) * a.N + n);
            } else {
#pragma unroll
                for (int i = 0; i < CHUNK; ++i) tt[i] = 0u;
            }
            double sum = 0.0;
#pragma unroll
            for (int i = 0; i < CHUNK; ++i) {
                const int t = t0 - i;
                if (t >= 0) {
                    const long long s = static_cast<long long>(t) * a.N + n;
                    float ret[VEC];
#pragma unroll
                    for (int c = 0; c < VEC; ++c) {
                        const float v = vv[i][c];
                        float r = rr[i][c];
                        if ((tt[i] >> (8 * c)) & 0xFFu) r += a.gamma * v;
                        const float nd = (dd[i] >> (8 * c)) & 0xFFu ? 0.0f : 1.0f;
                        const float delta = r + a.gamma * nd * next_v[c] - v;
                        const float adv = delta + gl * nd * next_a[c];
                        ret[c] = adv + v;
                        rr[i][c] = adv;
                        next_v[c] = v;
                        next_a[c] = adv;
                        sum += static_cast<double>(adv);
                    }
                    store_f(a.adv + s, rr[i]);
                    store_f(a.returns + s, ret);
                }
            }
            // this chunk's (count, mean, M2), merged with the earlier ones
            const double nc = static_cast<double>(min(CHUNK, t0 + 1) * VEC);
            const double mc = sum / nc;
            double qc = 0.0;
#pragma unroll
            for (int i = 0; i < CHUNK; ++i)
                if (t0 - i >= 0)
#pragma unroll
                    for (int c = 0; c < VEC; ++c) {
                        const double d = static_cast<double>(rr[i][c]) - mc;
                        qc += d * d;
                    }
            const double d = mc - mean, w = nc / (cnt + nc);
            m2 += qc + d * d * cnt * w;
            mean += d * w;
            cnt += nc;
        }
    }
    // the block's mean, then its squared deviations around it
    __shared__ double s_red[2][THREADS / 64];
    auto block_sum = [&](double v, double *red) {
        v = wave_sum_d(v);
        if constexpr (THREADS == 64) return v;
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < THREADS / 64; ++i) t += red[i];
        return t;
    };
    const long long here = min(static_cast<long long>(a.N) - static_cast<long long>(blockIdx.x) * THREADS * VEC,
                               static_cast<long long>(THREADS) * VEC);
    const double total = static_cast<double>(here) * a.T;
    const double bmean = block_sum(cnt * mean, s_red[0]) / total;
    const double bm2 = block_sum(m2 + cnt * (mean - bmean) * (mean - bmean), s_red[1]);
    if (threadIdx.x == 0) {
        a.partials[3 * blockIdx.x + 0] = total;
        a.partials[3 * blockIdx.x + 1] = bmean;
        a.partials[3 * blockIdx.x + 2] = bm2;
    }
}

// Every block combines all partials the same way, so each holds the identical
// result: the mean of all, then the squared deviations around it, each summed
// per thread, over the wave and over the waves in order.  Block 0 publishes
// (mean, unbiased std), and all blocks optionally normalise; a thread's first
// advantages load ahead of the partials.
__global__ __launch_bounds__(kFinalizeThreads) void adv_finalize_kernel(const double *partials, int nparts,
                                                                        float *adv, long long count,
                                                                        double *stats_out, int normalize) {
    __shared__ double s_red[2][kFinalizeThreads / 64];
    const int tid = threadIdx.x;
    const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
    const long long first = blockIdx.x * static_cast<long long>(blockDim.x) + tid;
    const long long n4 = count / 4;
    float4 *adv4 = reinterpret_cast<float4 *>(adv);
    const bool pre = normalize && first < n4;
    const float4 v_first = pre ? adv4[first] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    auto block_sum = [&](double v, double *red) {
        v = wave_sum_d(v);
        if ((tid & 63) == 0) red[tid >> 6] = v;
        __syncthreads();
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < kFinalizeThreads / 64; ++i) t += red[i];
        return t;
    };
    const double n = static_cast<double>(count);
    double s = 0.0;
    for (int p = tid; p < nparts; p += kFinalizeThreads) s += partials[3 * p] * partials[3 * p + 1];
    const double mean = block_sum(s, s_red[0]) / n;
    double q = 0.0;
    for (int p = tid; p < nparts; p += kFinalizeThreads) {
        const double d = partials[3 * p + 1] - mean;
        q += partials[3 * p + 2] + partials[3 * p] * d * d;
    }
    const double m2 = block_sum(q, s_red[1]);
    const double std = n > 1.0 ? sqrt(m2 / (n - 1.0)) : 0.0;
    if (blockIdx.x == 0 && tid == 0) {
        stats_out[0] = mean;
        stats_out[1] = std;
    }
    if (!normalize) return;
    const double inv = 1.0 / (std + 1e-8);
    auto norm = [&](float x) { return static_cast<float>((static_cast<double>(x) - mean) * inv); };
    // 16-byte accesses (adv is 16-byte aligned), then the tail of count % 4
    auto put = [&](long long e, float4 v) {
        adv4[e] = make_float4(norm(v.x), norm(v.y), norm(v.z), norm(v.w));
    };
    if (pre) put(first, v_first);
    for (long long e = first + stride; e < n4; e += stride) put(e, adv4[e]);
    for (long long e = 4 * n4 + first; e < count; e += stride) adv[e] = norm(adv[e]);
}

// -------------------------------------------------------- gradient reduce
// Sums the split partials of every segment into the flat gradient; the last
// block sums the loss partials column-wise (8 row stripes, then the stripes in
// order) into the log-std gradient and the loss sums.  Every block writes the
// float64 sum of squares of what it wrote.
//
// A latency chain at these sizes (17 MB of partials at [512, 256, 128]), not
// bandwidth: every block belongs to one segment, whose descriptor it reads
// with scalar loads, and a thread has the loads of four elements by up to 16
// partials in flight.  One element and 8 partials at a time, the segment
// searched by every lane: 9.4 us at [512, 256, 128] and 21.8 us at
// [1024, 512, 256] with 235 inputs; now 7.4 and 9.6 us.
constexpr int kReduceThreads = 256;

// Four elements (or one) of segment S summed over its partials, 16 loads in
// flight at a time, added in split order.
template <typename V>
__device__ inline V sum_partials(const float *src, long long stride, int splits) {
    V sum{};
    for (int s0 = 0; s0 < splits; s0 += 16) {
        V v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (s0 + u < splits) v[u] = *reinterpret_cast<const V *>(src + (s0 + u) * stride);
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (s0 + u < splits) sum += v[u];
    }
    return sum;
}

__global__ __launch_bounds__(kReduceThreads) void grad_reduce_kernel(const ReduceArgs a) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    __shared__ double red[kReduceThreads / 64];
    double ss = 0.0;
    const int blk = blockIdx.x;
    if (blk + 1 < static_cast<int>(gridDim.x)) {
        int si = 0;
#pragma unroll
        for (int q = 1; q < kMaxSegments; ++q)
            if (q < a.count && blk >= a.block[q]) si = q;
        si = __builtin_amdgcn_readfirstlane(si);
        const ReduceSegment &S = a.seg[si];
        const int i0 = (blk - a.block[si]) * a.per_block, i1 = min(S.count, i0 + a.per_block);
        float *dst = a.grad + S.dst_offset;
        if (S.vec) {
            for (int i = i0 + 4 * static_cast<int>(threadIdx.x); i < i1; i += 4 * kReduceThreads) {
                const f32x4 sum = sum_partials<f32x4>(S.src + i, S.split_stride, S.splits);
                *reinterpret_cast<f32x4 *>(dst + i) = sum;
#pragma unroll
                for (int e = 0; e < 4; ++e) ss += static_cast<double>(sum[e]) * sum[e];
            }
        } else {
            for (int i = i0 + static_cast<int>(threadIdx.x); i < i1; i += kReduceThreads) {
                const float sum = sum_partials<float>(S.src + i, S.split_stride, S.splits);
                dst[i] = sum;
                ss += static_cast<double>(sum) * sum;
            }
        }
    } else {
        // columns: 4 loss sums, A log-std gradients, entropy, mean-shift KL, log-std KL
        __shared__ float stripe[8][kMaxAct + 8];
        __shared__ float total[kMaxAct + 8];
        const int cols = 7 + a.A;
        const int c = threadIdx.x & 31, st = threadIdx.x >> 5;
        if (c < cols) {
            // sixteen independent running sums keep sixteen loads in flight (the
            // partials come from every XCD, so each round trip is long); they
            // are combined in a fixed pairwise order, so the result does not
            // depend on timing
            constexpr int U = 16;
            float acc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = 0.0f;
            int b = st;
            for (; b + 8 * (U - 1) < a.n_loss; b += 8 * U)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    acc[u] += a.loss_partials[static_cast<long long>(b + 8 * u) * a.loss_width + c];
            for (; b < a.n_loss; b += 8) acc[0] += a.loss_partials[static_cast<long long>(b) * a.loss_width + c];
#pragma unroll
            for (int w = 1; w < U; w *= 2)
#pragma unroll
                for (int u = 0; u < U; u += 2 * w) acc[u] += acc[u + w];
            stripe[st][c] = acc[0];
        }
        __syncthreads();
        if (threadIdx.x < cols) {
            float v = 0.0f;
            for (int q = 0; q < 8; ++q) v += stripe[q][threadIdx.x];
            total[threadIdx.x] = v;
            if (threadIdx.x < 4) {
                a.loss_sums[threadIdx.x] = v;
            } else if (threadIdx.x < 4 + a.A && a.grad) {
                const float g = v - a.entropy_coef;
                a.grad[a.logstd_offset + threadIdx.x - 4] = g;
                ss = static_cast<double>(g) * g;
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            a.loss_sums[4] = total[4 + a.A];
            const float kl = total[5 + a.A] * a.inv_m + total[6 + a.A];
            a.loss_sums[5] = kl;
            if (a.lr && a.desired_kl > 0.0f) {
                // Algorithm 1: shrink the rate when the step moved the policy too
                // far, grow it when it moved too little, within [lr_min, lr_max]
                float lr = *a.lr;
                if (kl > 2.0f * a.desired_kl)
                    lr = fmaxf(a.lr_min, lr / a.lr_factor);
                else if (kl < 0.5f * a.desired_kl)
                    lr = fminf(a.lr_max, lr * a.lr_factor);
                *a.lr = lr;
            }
            if (a.step) *a.step += a.step_add;
        }
    }
    ss = wave_sum_d(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kReduceThreads / 64; ++w) t += red[w];
        a.sumsq_partials[blockIdx.x] = t;
    }
}

// ------------------------------------------------------------------ Adam
// Clip coefficient from the reduction's sums of squares, then Adam on the flat
// vector, with the bf16 shadow and the fragment copies of the hidden weights.
//
// A latency chain too: every block adds up the norm's partials (in the same
// order), and its elements can only be written after that.  So a thread's
// first kAdamUnroll elements load together with the partials, the two bias
// corrections (float64 powers) are computed by two other waves than the one
// that finishes the norm, and a block lies within one matrix, whose descriptor
// is scalar.  One element per lane and step: the bf16 copies coalesce only when
// neighbouring lanes own neighbouring elements.  With one element loaded ahead,
// the powers behind the norm and every matrix tested per element: 9.7 us at
// [512, 256, 128] and 23.5 us at [1024, 512, 256] with 235 inputs; now 9.2 and
// 20.4 us (6.6 us without the fragment copies).
constexpr int kAdamThreads = 256;
constexpr int kAdamUnroll = 4;

__global__ __launch_bounds__(kAdamThreads) void adam_kernel(const AdamArgs a) {
    __shared__ double s_sumsq;
    __shared__ double red[kAdamThreads / 64];
    __shared__ float s_bc[2];
    const int tid = threadIdx.x, blk = blockIdx.x;
    int ri = 0;
#pragma unroll
    for (int q = 1; q < kMaxAdamRegions; ++q)
        if (q < a.n_regions && blk >= a.block[q]) ri = q;
    ri = __builtin_amdgcn_readfirstlane(ri);
    const int e0 = a.region[ri] + (blk - a.block[ri]) * a.per_block;
    const int e1 = min(a.region[ri + 1], e0 + a.per_block);
    // this thread's first elements go out before the norm is known
    float g_pre[kAdamUnroll], m_pre[kAdamUnroll], v_pre[kAdamUnroll], th_pre[kAdamUnroll];
#pragma unroll
    for (int u = 0; u < kAdamUnroll; ++u) {
        const int e = e0 + tid + kAdamThreads * u;
        const bool in = a.apply && e < e1;
        g_pre[u] = in ? a.grad[e] : 0.0f;
        m_pre[u] = in ? a.m[e] : 0.0f;
        v_pre[u] = in ? a.v[e] : 0.0f;
        th_pre[u] = in ? a.theta[e] : 0.0f;
    }
    const float lr = a.lr ? *a.lr : 0.0f;
    // global norm: every block sums the same partials in the same order
    // (four loads in flight, added in index order)
    double ss = 0.0;
    int p = tid;
    for (; p + 3 * kAdamThreads < a.n_sumsq; p += 4 * kAdamThreads) {
        const double s0 = a.sumsq_partials[p], s1 = a.sumsq_partials[p + kAdamThreads];
        const double s2 = a.sumsq_partials[p + 2 * kAdamThreads], s3 = a.sumsq_partials[p + 3 * kAdamThreads];
        ss += s0;
        ss += s1;
        ss += s2;
        ss += s3;
    }
    for (; p < a.n_sumsq; p += kAdamThreads) ss += a.sumsq_partials[p];
    if (a.apply && (tid == 64 || tid == 128)) {
        // bias corrections of this step, once per block
        const int step = *a.step + a.step_offset + 1;
        s_bc[tid == 64 ? 0 : 1] =
            static_cast<float>(1.0 - pow(static_cast<double>(tid == 64 ? a.beta1 : a.beta2), step));
    }
    ss = wave_sum_d(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < kAdamThreads / 64; ++w) t += red[w];
        s_sumsq = t;
    }
    __syncthreads();
    const double norm = sqrt(s_sumsq);
    const bool finite = isfinite(norm);
    const float coef = static_cast<float>(fmin(1.0, static_cast<double>(a.max_grad_norm) / (norm + 1e-6)));

    if (blk == 0 && tid == 0) {
        const float pl = a.loss_sums[0] * a.inv_m, vl = a.loss_sums[1] * a.inv_m;
        const float ent = a.loss_sums[4];
        a.stats[0] = pl + a.value_coef * vl - a.entropy_coef * ent;
        a.stats[1] = pl;
        a.stats[2] = vl;
        a.stats[3] = ent;
        a.stats[4] = a.loss_sums[2] * a.inv_m;
        a.stats[5] = a.loss_sums[3] * a.inv_m;
        a.stats[6] = static_cast<float>(norm);
        a.stats[7] = finite ? 0.0f : 1.0f;
        a.stats[8] = a.loss_sums[5];
        a.stats[9] = lr;
    }
    if (!a.apply || !finite) return;

    const float bc1 = s_bc[0], bc2 = s_bc[1];
    const int fi = a.region_frag[ri];
    const AdamFrag &F = a.frag[fi < 0 ? 0 : fi];
    auto update = [&](int e, float g_raw, float m_old, float v_old, float th_old) {
        const float g = g_raw * coef;
        const float m = a.beta1 * m_old + (1.0f - a.beta1) * g;
        const float v = a.beta2 * v_old + (1.0f - a.beta2) * g * g;
        a.m[e] = m;
        a.v[e] = v;
        const float th = th_old - lr * (m / bc1) / (sqrtf(v / bc2) + a.eps);
        a.theta[e] = th;
        const uint16_t bits = f32_to_bf16(th);
        if (a.shadow) a.shadow[e] = bits;
        if (fi < 0) return;
        // the same bf16 value into the fragment copies of its weight matrix:
        // element (r, c) of W [rows][cols] sits in fragment (r / 32, c / 16),
        // lane r % 32 + 32 ((c % 16) / 8), element c % 8; in the transposed
        // copy the roles of r and c swap.  rows * cols < 2^31 (width and
        // observation limits): 32-bit division
        const unsigned li = static_cast<unsigned>(e - a.region[ri]), cols = static_cast<unsigned>(F.cols);
        const int r = static_cast<int>(li / cols), c = static_cast<int>(li - static_cast<unsigned>(r) * cols);
        const int li_in = (r & 31) + 32 * ((c & 15) >> 3);
        if (F.split) {
            // split layout: the feature block's S bf16 fragments, then its S
            // residual fragments
            const long long f0 = static_cast<long long>(2 * (r >> 5)) * F.S + (c >> 4);
            F.dst[(f0 * 64 + li_in) * 8 + (c & 7)] = bits;
            F.dst[((f0 + F.S) * 64 + li_in) * 8 + (c & 7)] = f32_to_bf16(th - bf16_to_f32(bits));
        } else {
            const long long fs = static_cast<long long>(r >> 5) * F.S + (c >> 4);
            F.dst[(fs * 64 + li_in) * 8 + (c & 7)] = bits;
        }
        if (F.dst_t)
            F.dst_t[((static_cast<long long>(c >> 5) * F.S_t + (r >> 4)) * 64 + (c & 31) + 32 * ((r & 15) >> 3)) * 8 +
                    (r & 7)] = bits;
    };
#pragma unroll
    for (int u = 0; u < kAdamUnroll; ++u) {
        const int e = e0 + tid + kAdamThreads * u;
        if (e < e1) update(e, g_pre[u], m_pre[u], v_pre[u], th_pre[u]);
    }
    for (int e = e0 + tid + kAdamThreads * kAdamUnroll; e < e1; e += kAdamThreads)
        update(e, a.grad[e], a.m[e], a.v[e], a.theta[e]);
}

// ------------------------------------------------------- weight staging
// One 64 x 64 tile of one job per block: coalesced reads of source rows into
// LDS, coalesced writes of destination rows (transposed or padded).
constexpr int kStageTile = 64;

template <typename T>
__global__ __launch_bounds__(256) void stage_weights_kernel(const StageArgs a) {
    __shared__ T tile[kStageTile][kStageTile + 1];
    int ji = 0;
    while (ji + 1 < a.count && static_cast<int>(blockIdx.x) >= a.job[ji + 1].tile_begin) ++ji;
    const StageJob &j = a.job[ji];
    const int local = blockIdx.x - j.tile_begin;
    // tiles cover the source (transpose) or the padded destination (copy)
    const int cols_t = j.transpose ? j.cols : j.dst_ld;
    const int tiles_c = (cols_t + kStageTile - 1) / kStageTile;
    const int r0 = (local / tiles_c) * kStageTile;
    const int c0 = (local % tiles_c) * kStageTile;
    const T *src = static_cast<const T *>(j.src);
    T *dst = static_cast<T *>(j.dst);
    for (int e = threadIdx.x; e < kStageTile * kStageTile; e += blockDim.x) {
        const int r = e / kStageTile, c = e % kStageTile;
        const int gr = r0 + r, gc = c0 + c;
        T v = T(0);
        if (gr < j.rows && gc < j.cols) {
            if constexpr (sizeof(T) == 2) {
                if (j.lo_src) {
                    // bf16 residual of the float32 weight (exact subtraction)
                    const float x = j.lo_src[static_cast<long long>(gr) * j.src_ld + gc];
                    v = f32_to_bf16(x - bf16_to_f32(f32_to_bf16(x)));
                } else {
                    v = src[static_cast<long long>(gr) * j.src_ld + gc];
                }
            } else {
                v = src[static_cast<long long>(gr) * j.src_ld + gc];
            }
        }
        tile[r][c] = v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kStageTile * kStageTile; e += blockDim.x) {
        const int r = e / kStageTile, c = e % kStageTile;
        if (j.transpose) {
            // destination row c0 + r holds source column c0 + r
            const int dr = c0 + r, dc = r0 + c;
            if (dr < j.cols && dc < j.rows) dst[static_cast<long long>(dr) * j.dst_ld + dc] = tile[c][r];
        } else {
            const int dr = r0 + r, dc = c0 + c;
            if (dr < j.rows && dc < j.dst_ld) dst[static_cast<long long>(dr) * j.dst_ld + dc] = tile[r][c];
        }
    }
}

__global__ void step_advance_kernel(int32_t *step, int k) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *step += k;
}

__global__ void pack_bf16_kernel(const float *theta, uint16_t *shadow, long long n) {
    for (long long e = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; e < n;
         e += static_cast<long long>(gridDim.x) * blockDim.x)
        shadow[e] = f32_to_bf16(theta[e]);
}

int grid_for(long long n, int threads, int cap) {
    long long b = (n + threads - 1) / threads;
    if (b < 1) b = 1;
    return static_cast<int>(b < cap ? b : cap);
}

}  // namespace

hipError_t launch_philox_blocks(hipStream_t s, uint64_t seed, uint32_t c0, uint32_t c1, uint32_t c2,
                                uint32_t c3, long long n, uint32_t *out) {
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    hipLaunchKernelGGL(philox_blocks_kernel, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, k0, k1, c0, c1, c2, c3,
                       n, out);
    return hipGetLastError();
}

hipError_t launch_gather_obs(Precision prec, hipStream_t s, const float *obs, const int32_t *idx, int src_rows,
                             int rows, int D, int ld, void *out) {
    const long long total = static_cast<long long>(rows) * ld;
    const dim3 grid(grid_for(total, 256, 8192)), block(256);
    if (prec == kBF16)
        hipLaunchKernelGGL(gather_obs_kernel<uint16_t>, grid, block, 0, s, obs, idx, src_rows, rows, D, ld,
                           static_cast<uint16_t *>(out));
    else
        hipLaunchKernelGGL(gather_obs_kernel<float>, grid, block, 0, s, obs, idx, src_rows, rows, D, ld,
                           static_cast<float *>(out));
    return hipGetLastError();
}

// Dynamic LDS for the staged output-layer weights, 0 when they do not fit.
size_t head_weight_lds(int A, int Hl) {
    const size_t bytes = static_cast<size_t>(A + 1) * (Hl + kWPad) * sizeof(float);
    return bytes <= 48 * 1024 ? bytes : 0;
}

hipError_t launch_head_sample(Precision prec, const HeadSampleArgs &a, hipStream_t s) {
    const dim3 grid((a.N + kSampleRows - 1) / kSampleRows), block(kHeadThreads);
    const size_t wsh = head_weight_lds(a.A, a.Hl);
    if (prec == kBF16) {
        const size_t rsh = head_rows_lds<uint16_t>(kSampleRows, a.Hl, wsh);
        hipLaunchKernelGGL(head_sample_kernel<uint16_t>, grid, block, wsh + rsh, s, a, wsh > 0 ? 1 : 0,
                           rsh > 0 ? static_cast<int>(wsh) : -1);
    } else {
        const size_t rsh = head_rows_lds<float>(kSampleRows, a.Hl, wsh);
        hipLaunchKernelGGL(head_sample_kernel<float>, grid, block, wsh + rsh, s, a, wsh > 0 ? 1 : 0,
                           rsh > 0 ? static_cast<int>(wsh) : -1);
    }
    return hipGetLastError();
}

void add_stage_job(StageArgs &a, const StageJob &j) {
    StageJob q = j;
    const int cols_t = q.transpose ? q.cols : q.dst_ld;
    q.tile_begin = a.total_tiles;
    a.job[a.count++] = q;
    a.total_tiles += ((q.rows + kStageTile - 1) / kStageTile) * ((cols_t + kStageTile - 1) / kStageTile);
}

hipError_t launch_stage_weights(Precision prec, const StageArgs &a, hipStream_t s) {
    if (a.count == 0 || a.total_tiles == 0) return hipSuccess;
    const dim3 grid(a.total_tiles), block(256);
    if (prec == kBF16)
        hipLaunchKernelGGL(stage_weights_kernel<uint16_t>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(stage_weights_kernel<float>, grid, block, 0, s, a);
    return hipGetLastError();
}

int head_loss_blocks(int M) { return (M + kLossRows - 1) / kLossRows; }
int head_loss_partial_width(int A) { return A + 8; }

hipError_t launch_head_loss(Precision prec, const HeadLossArgs &a, hipStream_t s) {
    const dim3 grid(head_loss_blocks(a.M)), block(kHeadThreads);
    const size_t wsh = head_weight_lds(a.A, a.Hl);
    if (prec == kBF16) {
        const size_t rsh = head_rows_lds<uint16_t>(kLossRows, a.Hl, wsh);
        hipLaunchKernelGGL(head_loss_kernel<uint16_t>, grid, block, wsh + rsh, s, a, wsh > 0 ? 1 : 0,
                           rsh > 0 ? static_cast<int>(wsh) : -1);
    } else {
        const size_t rsh = head_rows_lds<float>(kLossRows, a.Hl, wsh);
        hipLaunchKernelGGL(head_loss_kernel<float>, grid, block, wsh + rsh, s, a, wsh > 0 ? 1 : 0,
                           rsh > 0 ? static_cast<int>(wsh) : -1);
    }
    return hipGetLastError();
}

// The scan's kernel for N environments of T steps.  Times of the scan and its
// statistics, in us.
//
// Few environments: one per lane and blocks of one wave, in the smallest chunk
// that holds the horizon, since steps past it load its first row again.  Chunks
// of 8, 16 and 24 against one of 32 for all, 4096 environments: 8 steps 5.6
// against 7.0, 16 steps 6.4 against 7.4, 24 steps 7.3 against 7.9; 256 and 65536
// environments gain as much.  Longer horizons go 32 steps at a time.
// More: one per lane, blocks of four waves, 16 steps at a time.  A horizon of 25
// to 256 steps is better off so from 49152 environments on (65536 x 128: 28.8
// against 35.3 in blocks of one wave; 49152 x 64: 17.8 and 18.5; 32768 x 128: 24.9
// and 23.8), a shorter one from 65536 on (65536 x 24: 10.4 and 10.9).
// Many: four per lane where the rows stay 16-byte aligned (N a multiple of 4) and
// the lanes still fill the chip, from 163840 environments on (200000 x 128: 91
// against 102; 131072 x 128: 79 against 62), from 131072 on up to 96 steps, whose
// 16 MB rows stay in the memory-side cache.  From 2^18 on four steps at a time,
// past 64 steps in blocks of one wave: 2^20 x 24 92 against 96 with eight steps,
// 2^18 x 256 207 against 222, 2^20 x 96 353 against 426.
struct GaeShape { int vec, chunk, threads; };
constexpr int kGaeSmallN = 1 << 16;
GaeShape gae_shape(int N, int T) {
    if (N <= 3 << 14 || (N <= kGaeSmallN && (T <= 24 || T > 256)))
        return {1, T <= 8 ? 8 : T <= 16 ? 16 : T <= 24 ? 24 : 32, 64};
    if (N % 4 == 0 && (N >= 5 << 15 || (N >= 1 << 17 && T <= 96))) {
        if (N < 1 << 18) return {4, 8, 256};
        return {4, 4, T <= 64 ? 256 : 64};
    }
    return {1, 16, 256};
}

int gae_blocks(int N, int T) {
    const GaeShape sh = gae_shape(N, T);
    const int per = sh.vec * sh.threads;
    return static_cast<int>((static_cast<long long>(N) + per - 1) / per);
}

int gae_max_blocks(int N) {
    return N <= kGaeSmallN ? (N + 63) / 64 : std::max(kGaeSmallN / 64, static_cast<int>((N + 255LL) / 256));
}

// Scratch of the allocation-free GAE entry point: the partials (three doubles
// per gae_kernel block, at most one per 256 environments past 2^16 and 1024 up
// to there) of up to kGaeNoAllocMaxN environments, one copy per device for the
// life of the process.
static __device__ __align__(256) double scratch[3 * (kGaeNoAllocMaxN / 256)];

hipError_t gae_scratch(double **out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *ptr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        // the host-side name of the array is not a device address: ask the
        // runtime for this device's copy once, with the device current
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        ptr[dev] = static_cast<double *>(p);
    }
    *out = ptr[dev];
    return hipSuccess;
}

hipError_t launch_gae(const GaeArgs &a, hipStream_t s) {
    static const struct {
        GaeShape shape;
        void (*fn)(const GaeArgs);
    } kernels[] = {{{1, 8, 64}, &gae_kernel<1, 8, 64>},     {{1, 16, 64}, &gae_kernel<1, 16, 64>},
                   {{1, 24, 64}, &gae_kernel<1, 24, 64>},   {{1, 32, 64}, &gae_kernel<1, 32, 64>},
                   {{1, 16, 256}, &gae_kernel<1, 16, 256>}, {{4, 8, 256}, &gae_kernel<4, 8, 256>},
                   {{4, 4, 256}, &gae_kernel<4, 4, 256>},   {{4, 4, 64}, &gae_kernel<4, 4, 64>}};
    const GaeShape sh = gae_shape(a.N, a.T);
    for (const auto &k : kernels)
        if (k.shape.vec == sh.vec && k.shape.chunk == sh.chunk && k.shape.threads == sh.threads) {
            hipLaunchKernelGGL(k.fn, dim3(gae_blocks(a.N, a.T)), dim3(sh.threads), 0, s, a);
            return hipGetLastError();
        }
    return hipErrorInvalidValue;
}

hipError_t launch_adv_finalize(const double *partials, int nparts, float *adv, long long count, double *stats_out,
                               int normalize, hipStream_t s) {
    const int blocks = normalize ? grid_for(count / 4, kFinalizeThreads, 1024) : 1;
    hipLaunchKernelGGL(adv_finalize_kernel, dim3(blocks), dim3(kFinalizeThreads), 0, s, partials, nparts, adv, count,
                       stats_out,
                       normalize);
    return hipGetLastError();
}

// At most about 960 blocks of whole passes over the threads (their sums of
// squares have 1024 places), one pass each where that is enough.
void plan_reduce(ReduceArgs &a) {
    long long total = 0;
    for (int q = 0; q < a.count; ++q) total += a.seg[q].count;
    constexpr long long pass = 4 * kReduceThreads;
    a.per_block = static_cast<int>(pass * std::max<long long>(1, (total + pass * 960 - 1) / (pass * 960)));
    a.block[0] = 0;
    for (int q = 0; q < a.count; ++q)
        a.block[q + 1] = a.block[q] + (a.seg[q].count + a.per_block - 1) / a.per_block;
}

hipError_t launch_grad_reduce(const ReduceArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(grad_reduce_kernel, dim3(reduce_blocks(a)), dim3(kReduceThreads), 0, s, a);
    return hipGetLastError();
}

void plan_adam(AdamArgs &a) {
    int n = 0;
    long long at = 0;
    auto add = [&](long long end, int frag) {
        if (end > at) {
            a.region[n] = static_cast<int>(at);
            a.region_frag[n++] = frag;
            at = end;
        }
    };
    for (int f = 0; f < a.n_frag; ++f) {   // in flat order
        add(a.frag[f].begin, -1);
        add(a.frag[f].begin + static_cast<long long>(a.frag[f].rows) * a.frag[f].cols, f);
    }
    add(a.P, -1);
    a.n_regions = n;
    a.region[n] = static_cast<int>(a.P);
    // one pass of kAdamUnroll elements per thread up to 2048 blocks (as many as
    // fit on the device at once), several from there on
    constexpr long long pass = kAdamUnroll * kAdamThreads;
    a.per_block = static_cast<int>(pass * std::max<long long>(1, (a.P + pass * 2048 - 1) / (pass * 2048)));
    a.block[0] = 0;
    for (int q = 0; q < n; ++q)
        a.block[q + 1] = a.block[q] + (a.region[q + 1] - a.region[q] + a.per_block - 1) / a.per_block;
}

hipError_t launch_adam(const AdamArgs &a, hipStream_t s) {
    // without a step only the statistics, by one block
    hipLaunchKernelGGL(adam_kernel, dim3(a.apply ? a.block[a.n_regions] : 1), dim3(kAdamThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_step_advance(int32_t *step, int k, hipStream_t s) {
    hipLaunchKernelGGL(step_advance_kernel, dim3(1), dim3(64), 0, s, step, k);
    return hipGetLastError();
}

hipError_t launch_pack_bf16(const float *theta, uint16_t *shadow, long long n, hipStream_t s) {
    hipLaunchKernelGGL(pack_bf16_kernel, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, theta, shadow, n);
    return hipGetLastError();
}

}  // namespace ppo
