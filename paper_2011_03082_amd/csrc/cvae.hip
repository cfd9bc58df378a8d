// cvae.hip -- conditional VAEs of Sec. 3.2 / Sec. 4.2 on gfx950: parameter
// init, training features, FP64 column moments, fused forward + backward on
// bfloat16 MFMA with FP32 master weights and AdamW, packing of the decoder
// for inference, and decoder-only sampling.
#include <math.h>

#include <mutex>

#include "host.hpp"
#include "packed.hpp"

namespace msst {

constexpr float kLvMin = -12.0f, kLvMax = 8.0f;
constexpr float kLog2Pi = 1.83787706640934548f;
constexpr int kTrainWaves = 4;  // waves per training block
constexpr int kMaxNL = 4;       // linear maps per network: 2 .. 4 (one to three hidden layers)
constexpr int kMaxDevices = 64; // devices whose noalloc scratch address is kept

struct Shape {
    int model, p_in, p_out, latent, width, n_linear;
};

__device__ __forceinline__ float clamp_lv(float x) { return __builtin_fminf(kLvMax, __builtin_fmaxf(kLvMin, x)); }
__device__ __forceinline__ float clamp_mask(float x) { return (x > kLvMin && x < kLvMax) ? 1.0f : 0.0f; }

// Normals n[4 j .. 4 j + 3] of Philox block c0 + j: Box-Muller on the word
// pairs (0, 1) and (2, 3).
__device__ __forceinline__ void normals4(const Rng& r, uint32_t c0, float* n) {
    const uint4 w = r.block(c0);
    box_muller(u01(w.x), u01(w.y), n[0], n[1]);
    box_muller(u01(w.z), u01(w.w), n[2], n[3]);
}

// ---------------------------------------------------------------------------
// init

struct LayerDims {
    int n_in, n_out;
};

// Feature blocks per layer dimension: every layer is stored and computed as
// a (16 T) x (16 T) grid of 16 x 16 MFMA tiles, T = 1 when all of the
// network's widths (hidden units, both networks' inputs and outputs) fit one
// tile and T = 2 up to 32 (Table 1's widest settings: 20 hidden units, or
// 2 x 9 encoder outputs).
__host__ __device__ inline int shape_blocks(const Shape& s) {
    int m = s.width;
    m = m > s.p_out + s.p_in ? m : s.p_out + s.p_in;
    m = m > s.latent + s.p_in ? m : s.latent + s.p_in;
    m = m > 2 * s.p_out ? m : 2 * s.p_out;
    m = m > 2 * s.latent ? m : 2 * s.latent;
    return m <= kTile ? 1 : 2;
}
// Floats of one layer: (16 T)^2 row-major weights, then 16 T biases.
__host__ __device__ inline int layer_floats(const Shape& s) {
    const int S = kTile * shape_blocks(s);
    return S * S + S;
}
constexpr int kMaxBlocks = 2;
constexpr int kMaxLayerFloats = (kTile * kMaxBlocks) * (kTile * kMaxBlocks) + kTile * kMaxBlocks;
__host__ __device__ inline LayerDims layer_dims(const Shape& s, int layer) {
    const int nl = s.n_linear;
    const bool dec = layer >= nl;
    const int j = dec ? layer - nl : layer;
    const int in0 = dec ? s.latent + s.p_in : s.p_out + s.p_in;
    const int outl = dec ? 2 * s.p_out : 2 * s.latent;
    return LayerDims{j == 0 ? in0 : s.width, j == nl - 1 ? outl : s.width};
}

__global__ void cvae_init_kernel(Shape s, uint64_t seed, float* master, int n_params) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_params) return;
    const int lf = layer_floats(s), S = kTile * shape_blocks(s);
    const int layer = p / lf, flat = p % lf;
    const LayerDims d = layer_dims(s, layer);
    int row, col;
    if (flat < S * S) {
        row = flat / S;
        col = flat % S;
    } else {
        row = flat - S * S;
        col = 0;
    }
    float v = 0.0f;
    if (row < d.n_out && col < d.n_in) {
        const Rng r = make_rng(seed, MS_TAG_CVAE_INIT, (uint64_t)s.model);
        const uint4 w = r.block((uint32_t)p >> 2);
        const uint32_t word = (p & 3) == 0 ? w.x : (p & 3) == 1 ? w.y : (p & 3) == 2 ? w.z : w.w;
        v = (2.0f * u01(word) - 1.0f) / sqrtf((float)d.n_in);
    }
    master[p] = v;
}

// ---------------------------------------------------------------------------
// features (Sec. 4.2 model inputs; LengthGen target dequantised)

// (float)((c - mean) / std) in FP64 through the reciprocal and one correction
// (three operations; FP64 division takes a dozen), the division itself where
// the reciprocal or the quotient is not finite.
__device__ __forceinline__ float standardised(float c, double mean, double std, double inv) {
    const double d = (double)c - mean, q = d * inv;
    const double r = __builtin_fma(__builtin_fma(-q, std, d), inv, q);
    return (float)(__builtin_isfinite(r) ? r : d / std);
}

constexpr int kFeatThreads = 256;

// Bound by HBM (EventGen: 60 bytes gathered and 52 written per row): a
// block's rows go through LDS so that they are written in whole lines.  2^22
// records, 2.6e6 EventGen rows 112 -> 66 us.
template <int MODEL>
__global__ __launch_bounds__(kFeatThreads) void cvae_features_kernel(int64_t n_out, const int64_t* rows, int64_t n,
                                                                     const float* params3, const uint32_t* n_scatter,
                                                                     const float* exit_param, const float* event_pos,
                                                                     const float* event_dir, uint64_t seed,
                                                                     uint64_t id_offset, const double* stats,
                                                                     float* cond, float* target) {
    constexpr int PC = MODEL == MS_MODEL_LENGTH ? 2 : MODEL == MS_MODEL_PATH ? 3 : 7;
    constexpr int PY = MODEL == MS_MODEL_LENGTH ? 1 : MODEL == MS_MODEL_PATH ? 3 : 6;
    __shared__ float cs[kFeatThreads * PC], ys[kFeatThreads * PY];
    __shared__ double inv_std[PC + PY];
    const int t = threadIdx.x;
    if (stats && t < PC + PY) inv_std[t] = 1.0 / stats[t < PC ? 16 + t : 48 + t - PC];
    __syncthreads();
    for (int64_t o0 = blockIdx.x * (int64_t)kFeatThreads; o0 < n_out; o0 += (int64_t)gridDim.x * kFeatThreads) {
        const int64_t o = o0 + t;
        if (o < n_out) {
            const int64_t i = rows ? rows[o] : o;
            const float lst = logf(params3[i]), g = params3[n + i];
            const float N = (float)n_scatter[i];
            float c[PC], y[PY];
            c[0] = lst;
            c[1] = g;
            if (MODEL == MS_MODEL_LENGTH) {
                const Rng r = make_rng(seed, MS_TAG_DEQUANT, id_offset + (uint64_t)i);
                const float u = u01(r.block(0).x);
                y[0] = logf(N + u - 0.5f);
            } else if (MODEL == MS_MODEL_PATH) {
                c[PC - 1] = logf(N);
#pragma unroll
                for (int k = 0; k < 3; ++k) y[k % PY] = exit_param[k * n + i];
            } else {
                c[2 % PC] = params3[2 * n + i];
#pragma unroll
                for (int k = 0; k < 3; ++k) c[(3 + k) % PC] = exit_param[k * n + i];
                c[PC - 1] = logf(N);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    y[k % PY] = event_pos[k * n + i];
                    y[(3 + k) % PY] = event_dir[k * n + i];
                }
            }
#pragma unroll
            for (int k = 0; k < PC; ++k)
                cs[t * PC + k] = stats ? standardised(c[k], stats[k], stats[16 + k], inv_std[k]) : c[k];
#pragma unroll
            for (int k = 0; k < PY; ++k)
                ys[t * PY + k] = stats ? standardised(y[k], stats[32 + k], stats[48 + k], inv_std[PC + k]) : y[k];
        }
        __syncthreads();
        const int m = n_out - o0 < kFeatThreads ? (int)(n_out - o0) : kFeatThreads;
        for (int q = t; q < m * PC; q += kFeatThreads) cond[o0 * PC + q] = cs[q];
        for (int q = t; q < m * PY; q += kFeatThreads) target[o0 * PY + q] = ys[q];
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// deterministic row selection (stream compaction in index order)

constexpr int kSelPerBlock = 2048;  // 256 threads x 8 consecutive rows

// Which of rows base .. base + 7 are selected, one bit each; VEC: both arrays
// are 16-byte aligned and read 16 bytes at a time.
template <bool VEC>
__device__ __forceinline__ uint32_t rows_selected(int64_t base, int64_t n, const uint32_t* ns, const uint32_t* ek,
                                                  uint32_t min_n, uint32_t min_k) {
    uint32_t f = 0;
    if (VEC && base + 8 <= n) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint4 a = *reinterpret_cast<const uint4*>(ns + base + 4 * h);
            uint4 e = make_uint4(min_k, min_k, min_k, min_k);
            if (ek) e = *reinterpret_cast<const uint4*>(ek + base + 4 * h);
            f |= (uint32_t)(a.x >= min_n && e.x >= min_k) << (4 * h);
            f |= (uint32_t)(a.y >= min_n && e.y >= min_k) << (4 * h + 1);
            f |= (uint32_t)(a.z >= min_n && e.z >= min_k) << (4 * h + 2);
            f |= (uint32_t)(a.w >= min_n && e.w >= min_k) << (4 * h + 3);
        }
        return f;
    }
    for (int j = 0; j < 8; ++j)
        if (base + j < n && ns[base + j] >= min_n && (ek == nullptr || ek[base + j] >= min_k)) f |= 1u << j;
    return f;
}

// Inclusive prefix sum over a wave.
__device__ __forceinline__ int wave_scan(int v) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(v, off);
        if (lane_id() >= off) v += o;
    }
    return v;
}

template <bool VEC>
__global__ __launch_bounds__(256) void select_count_kernel(int64_t n, const uint32_t* ns, const uint32_t* ek,
                                                           uint32_t min_n, uint32_t min_k, int64_t* block_count) {
    __shared__ int wave_sum[4];
    const int64_t base = blockIdx.x * (int64_t)kSelPerBlock + threadIdx.x * 8;
    int c = __popc(rows_selected<VEC>(base, n, ns, ek, min_n, min_k));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if (lane_id() == 0) wave_sum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) block_count[blockIdx.x] = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
}

// Exclusive prefix of the blocks' counts and their total, by one block: each
// thread adds up four consecutive counts, a scan over the threads, and the
// total carried to the next 4096.  (One thread over 2048 counts: 216 us.)
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void select_scan_kernel(int64_t nb, int64_t* block_count, int64_t* total) {
    __shared__ int wave_sum[kScanThreads / 64];
    int64_t carry = 0;
    for (int64_t at = 0; at < nb; at += 4 * kScanThreads) {
        const int64_t i = at + 4 * (int64_t)threadIdx.x;
        int c[4], s = 0;  // a block counts at most 2048 rows: 4096 of them fit 32 bits
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = i + j < nb ? (int)block_count[i + j] : 0;
            s += c[j];
        }
        const int incl = wave_scan(s);
        if (lane_id() == 63) wave_sum[threadIdx.x >> 6] = incl;
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kScanThreads / 64; ++w) {
            before += w < (int)(threadIdx.x >> 6) ? wave_sum[w] : 0;
            all += wave_sum[w];
        }
        int64_t p = carry + before + incl - s;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i + j < nb) block_count[i + j] = p;
            p += c[j];
        }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// The block's rows go through LDS so that they are written in whole lines.
template <bool VEC>
__global__ __launch_bounds__(256) void select_write_kernel(int64_t n, const uint32_t* ns, const uint32_t* ek,
                                                           uint32_t min_n, uint32_t min_k, const int64_t* block_offset,
                                                           int64_t* rows) {
    __shared__ int wave_sum[4];
    __shared__ uint16_t kept[kSelPerBlock];
    const int64_t first = blockIdx.x * (int64_t)kSelPerBlock;
    const uint32_t f = rows_selected<VEC>(first + threadIdx.x * 8, n, ns, ek, min_n, min_k);
    // exclusive prefix of the counts over the block: within the wave, then across waves
    const int incl = wave_scan(__popc(f));
    const int wave = threadIdx.x >> 6;
    if (lane_id() == 63) wave_sum[wave] = incl;
    __syncthreads();
    int pos = incl - __popc(f), all = 0;
    for (int w = 0; w < 4; ++w) {
        if (w < wave) pos += wave_sum[w];
        all += wave_sum[w];
    }
    for (int j = 0; j < 8; ++j)
        if ((f >> j) & 1u) kept[pos++] = (uint16_t)(threadIdx.x * 8 + j);
    __syncthreads();
    int64_t* dst = rows + block_offset[blockIdx.x];
    for (int q = threadIdx.x; q < all; q += 256) dst[q] = first + kept[q];
}

// ---------------------------------------------------------------------------
// FP64 column moments: deterministic two-pass (mean, then centred squares).

constexpr int kMomBlocks = 1024, kMomMinBlocks = 256, kMomThreads = 256;

// Sums of the columns over this block's share of the matrix, read as one flat
// array of V floats per thread (V = 4: 16-byte aligned).  The number of blocks
// is a multiple of dim, so a thread meets the same columns in every round.
// HBM-bound: 2.6e6 x 7 floats 50 -> 15 us (rows per thread and 256 blocks left
// one wave per SIMD).
template <int V>
__global__ __launch_bounds__(kMomThreads) void moments_partial_kernel(const float* x, int64_t total, int dim,
                                                                      const double* mean, double* partial) {
    __shared__ double red[kMomThreads * V];
    __shared__ double sums[16][17];
    const int t = threadIdx.x;
    const int64_t at = (blockIdx.x * (int64_t)kMomThreads + t) * V, stride = (int64_t)gridDim.x * kMomThreads * V;
    double mu[V], acc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = mean ? mean[(at + j) % dim] : 0.0;
        acc[j] = 0.0;
    }
    auto add = [&](const float* p) __attribute__((always_inline)) {
        float v[V];
        if constexpr (V == 4) {
            const float4 f = *reinterpret_cast<const float4*>(p);
            v[0] = f.x;
            v[1] = f.y;
            v[2] = f.z;
            v[3] = f.w;
        } else {
            v[0] = *p;
        }
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const double d = (double)v[j] - mu[j];
            acc[j] += mean ? d * d : d;
        }
    };
#pragma unroll 4
    for (int64_t p = at; p + V <= total; p += stride) add(x + p);
#pragma unroll
    for (int j = 0; j < V; ++j) red[t * V + j] = acc[j];
    __syncthreads();
    if (V > 1 && blockIdx.x == 0 && t == 0) {
        // the matrix's last elements, fewer than V: entry e % dim of block 0
        // is one of column e % dim
        for (int64_t e = total - total % V; e < total; ++e) {
            const int c = (int)(e % dim);
            const double d = (double)x[e] - (mean ? mean[c] : 0.0);
            red[c] += mean ? d * d : d;
        }
    }
    __syncthreads();
    // column k = t % 16: entries k', k' + dim, ... of red, 16 threads each
    const int k = t & 15, r = t >> 4;
    double s = 0.0;
    if (k < dim) {
        const int off = (int)((blockIdx.x * (int64_t)kMomThreads * V) % dim);
        const int e0 = k >= off ? k - off : k - off + dim;
        for (int e = e0 + dim * r; e < kMomThreads * V; e += dim * 16) s += red[e];
    }
    sums[k][r] = s;
    __syncthreads();
    if (t < 16) {
        s = 0.0;
        for (int q = 0; q < 16; ++q) s += sums[t][q];
        partial[blockIdx.x * 16 + t] = s;
    }
}

__global__ __launch_bounds__(256) void moments_final_kernel(const double* partial, int nblocks, int64_t n, int dim,
                                                            double* out, int second_pass) {
    __shared__ double sums[16][17];
    const int k = threadIdx.x & 15, r = threadIdx.x >> 4;
    double s = 0.0;
#pragma unroll 8
    for (int b = r; b < nblocks; b += 16) s += partial[b * 16 + k];
    sums[k][r] = s;
    __syncthreads();
    if ((int)threadIdx.x >= dim) return;
    s = 0.0;
    for (int q = 0; q < 16; ++q) s += sums[threadIdx.x][q];
    if (!second_pass) out[threadIdx.x] = s / (double)n;
    else out[16 + threadIdx.x] = sqrt(s / (double)n);
}

// ---------------------------------------------------------------------------
// Training: fused forward + backward of encoder and decoder on 16-sample
// tiles, one tile at a time per wave; per-block gradient partials.

struct TrainArgs {
    Shape s;
    const float* master;
    const float* cond;
    const float* target;
    int64_t n_rows;
    int batch;
    int sample_rows;
    uint64_t seed;
    int64_t step;
    uint64_t id_offset;
    float kl_weight;      // weight of the KL term in the gradient
    float* partial;       // [blocks][n_params]
    double* loss_partial; // [blocks][2]
};

// Per-wave LDS: what passes between lanes, 16 T feature rows (T stacked 16 x 16
// tiles) of 16 samples each.  Layer inputs and their gradients are held as the
// bfloat16 values that the products take.
template <int NL, int T>
struct WaveLds {
    __bf16 act[2 * NL][kTile * T][kTile];   // inputs of the 2 NL layers
    __bf16 dpre[2 * NL][kTile * T][kTile];  // gradients of their linear outputs
    float enc[kTile * T][kTile];            // encoder output: mean, log variance
    float dec[kTile * T][kTile];            // decoder output
    float y[kTile][kTile];                  // target
    float eps[kTile][kTile], dz[kTile][kTile];
    float kl[kTile][kTile], nll[kTile][kTile];  // a sample's loss, term by term
};

// Weight fragments of block (o, k) of a layer with row stride 16 T: the A
// operand of the forward product (output rows 16 o .., input columns
// 16 k ..), its transpose (for dX = W^T dPre) and the biases of output block o.
template <int T>
__device__ __forceinline__ bf16x4 w_frag(const float* layer, int o, int k) {
    constexpr int S = kTile * T;
    const f32x4 v = *reinterpret_cast<const f32x4*>(layer + (kTile * o + frag_row()) * S + kTile * k + frag_k0());
    return to_bf16x4(v);
}
template <int T>
__device__ __forceinline__ bf16x4 wt_frag(const float* layer, int o, int k) {
    constexpr int S = kTile * T;
    const float* p = layer + (kTile * o + frag_k0()) * S + kTile * k + frag_row();
    return to_bf16x4(p[0], p[S], p[2 * S], p[3 * S]);
}
template <int T>
__device__ __forceinline__ f32x4 bias_d(const float* layer, int o) {
    constexpr int S = kTile * T;
    return *reinterpret_cast<const f32x4*>(layer + S * S + kTile * o + frag_k0());
}

// A tile of 16 features by 16 samples in LDS as bfloat16: stored from the D
// layout (this lane's four rows of its column), and read transposed (row
// frag_row(), four consecutive samples: an operand of dPre X^T).
__device__ __forceinline__ void tile_put(__bf16 (*t)[kTile], bf16x4 v) {
    const int c = frag_row(), k0 = frag_k0();
#pragma unroll
    for (int q = 0; q < 4; ++q) t[k0 + q][c] = v[q];
}
__device__ __forceinline__ bf16x4 tile_get_t(const __bf16 (*t)[kTile]) {
    return *reinterpret_cast<const bf16x4*>(&t[frag_row()][frag_k0()]);
}

// Forward of one net (NL layers starting at FIRST) from its input x, the B
// operand of this lane (which act[FIRST] holds for the backward pass); the
// last layer's output blocks go to `out`.  The D layout of a layer's output is
// the next one's B operand, so the chain stays in registers.  Hidden units at
// or beyond `width` do not exist: their activations are forced to 0, so their
// (zero-initialised) weights and biases receive zero gradients.
template <int FIRST, int NL, int T>
__device__ __forceinline__ void net_forward(const bf16x4 (*wf)[T][T], const f32x4 (*bs)[T], WaveLds<NL, T>& L,
                                            f32x4 (*pre)[T], int width, bf16x4* x, f32x4* out) {
    const int k0 = frag_k0();
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int layer = FIRST + j;
#pragma unroll
        for (int o = 0; o < T; ++o) {
            f32x4 acc = bs[layer][o];
#pragma unroll
            for (int k = 0; k < T; ++k) acc = mfma_bf16(wf[layer][o][k], x[k], acc);
            pre[layer][o] = acc;
            out[o] = acc;
        }
        if (j < NL - 1) {
#pragma unroll
            for (int o = 0; o < T; ++o) {
                f32x4 a;
#pragma unroll
                for (int q = 0; q < 4; ++q) a[q] = kTile * o + k0 + q < width ? softplus(pre[layer][o][q]) : 0.0f;
                x[o] = to_bf16x4(a);
                tile_put(L.act[layer + 1] + kTile * o, x[o]);
            }
        }
    }
}

// Backward of one net given d loss / d (last linear output) in D layout, which
// is also the B operand of dX = W^T dPre: the chain stays in registers.  Adds
// db, leaves the rounded dPre of every layer in LDS for the weight gradients,
// and writes d loss / d (input of the first layer) in D layout to dx.
template <int FIRST, int NL, int T>
__device__ __forceinline__ void net_backward(const bf16x4 (*wt)[T][T], WaveLds<NL, T>& L, const f32x4 (*pre)[T],
                                             f32x4* dpre, f32x4 (*db)[T], f32x4* dx) {
#pragma unroll
    for (int j = NL - 1; j >= 0; --j) {
        const int layer = FIRST + j;
        bf16x4 d[T];
#pragma unroll
        for (int o = 0; o < T; ++o) {
            db[layer][o] += dpre[o];
            d[o] = to_bf16x4(dpre[o]);
            tile_put(L.dpre[layer] + kTile * o, d[o]);
        }
#pragma unroll
        for (int k = 0; k < T; ++k) {
            f32x4 acc = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int o = 0; o < T; ++o) acc = mfma_bf16(wt[layer][o][k], d[o], acc);
            dx[k] = acc;
        }
        if (j > 0) {
#pragma unroll
            for (int k = 0; k < T; ++k) {
#pragma unroll
                for (int q = 0; q < 4; ++q) dpre[k][q] = dx[k][q] * sigmoid(pre[layer - 1][k][q]);
            }
        }
    }
}

// Sum over the 16 lanes of a row (the same in every lane): each step adds the
// value of a lane whose partial sum covers the other half.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_sum(float v) {
    v = dpp_add<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v = dpp_add<0x141>(v);  // row_half_mirror
    return dpp_add<0x140>(v);  // row_mirror
}

// A step of 4096 samples is one tile per wave, one wave per SIMD: bound by the
// latency of one tile's chain of dependent steps, so all 64 lanes take part in
// each (a lane holds 4 T of the 16 T rows of its sample), the layers chain in
// registers, rows are gathered ahead of the weights, and the weight gradients'
// transposed products wait for the end of the tile.
template <int NL, int T>
__global__ __launch_bounds__(256) void cvae_train_kernel(const TrainArgs a) {
    constexpr int S = kTile * T;   // row stride of a layer's weights
    constexpr int LF = S * S + S;  // floats per layer
    constexpr int kParams = 2 * NL * LF;
    typedef WaveLds<NL, T> Lds;
    __shared__ __align__(16) Lds lds_all[kTrainWaves];
    const int wave = uniform_u32(threadIdx.x >> 6);
    Lds& L = lds_all[wave];
    const Shape s = a.s;
    const int P = s.p_out, Lt = s.latent, C = s.p_in;
    const int lane = lane_id(), c = frag_row(), k0 = frag_k0();
    const float inv_b = 1.0f / (float)a.batch;

    // this lane's rows k0 .. k0 + 3 of each block of (target, cond), sample
    // column c of a tile
    auto gather = [&](int tile, f32x4* x) __attribute__((always_inline)) {
        const int b = tile * kTile + c;
        int64_t row = b;
        if (a.sample_rows) {
            const Rng rb = make_rng(a.seed, MS_TAG_CVAE_BATCH, (uint64_t)b);
            row = (int64_t)(((uint64_t)rb.block((uint32_t)a.step).x * (uint64_t)a.n_rows) >> 32);
        }
#pragma unroll
        for (int k = 0; k < T; ++k) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = kTile * k + k0 + q;
                float v = 0.0f;
                if (r < P) v = a.target[row * P + r];
                else if (r < P + C) v = a.cond[row * C + (r - P)];
                x[k][q] = v;
            }
        }
    };
    const int n_tiles = a.batch / kTile;
    const int wave_global = blockIdx.x * kTrainWaves + wave;
    const int n_waves = gridDim.x * kTrainWaves;
    f32x4 x_next[T];
    if (wave_global < n_tiles) gather(wave_global, x_next);

    // all layers' weight fragments (both orientations) and biases of this
    // lane, loaded once
    bf16x4 wf[2 * NL][T][T], wt[2 * NL][T][T];
    f32x4 bs[2 * NL][T];
#pragma unroll
    for (int i = 0; i < 2 * NL; ++i) {
        const float* layer = a.master + i * LF;
#pragma unroll
        for (int o = 0; o < T; ++o) {
            bs[i][o] = bias_d<T>(layer, o);
#pragma unroll
            for (int k = 0; k < T; ++k) {
                wf[i][o][k] = w_frag<T>(layer, o, k);
                wt[i][o][k] = wt_frag<T>(layer, o, k);
            }
        }
    }
    f32x4 dw[2 * NL][T][T], db[2 * NL][T], pre[2 * NL][T];
#pragma unroll
    for (int i = 0; i < 2 * NL; ++i) {
#pragma unroll
        for (int o = 0; o < T; ++o) {
            db[i][o] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < T; ++k) dw[i][o][k] = f32x4{0, 0, 0, 0};
        }
    }
    double kl_acc = 0.0, nll_acc = 0.0;

    for (int tile = wave_global; tile < n_tiles; tile += n_waves) {
        // noise of latents k0 .. k0 + 3 (Philox block k0 / 4)
        float eps[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (k0 < Lt)
            normals4(make_rng(a.seed, MS_TAG_CVAE_REPARAM, a.id_offset + (uint64_t)(tile * kTile + c)),
                     (uint32_t)(4 * a.step + (k0 >> 2)), eps);
        bf16x4 x[T];
#pragma unroll
        for (int k = 0; k < T; ++k) {
            x[k] = to_bf16x4(x_next[k]);
            tile_put(L.act[0] + kTile * k, x[k]);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (kTile * k + k0 + q < P) L.y[(kTile * k + k0 + q) & 15][c] = x_next[k][q];
        }
        if (tile + n_waves < n_tiles) gather(tile + n_waves, x_next);
        // encoder
        f32x4 out[T];
        net_forward<0, NL, T>(wf, bs, L, pre, s.width, x, out);
#pragma unroll
        for (int o = 0; o < T; ++o) tile_store_d(&L.enc[kTile * o][0], out[o]);
        wave_sync();
        // z after the reparametrisation, then the condition
#pragma unroll
        for (int k = 0; k < T; ++k) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = kTile * k + k0 + q;
                __bf16 v = (__bf16)0.0f;
                if (r < Lt) {
                    const float mu = L.enc[r][c], lv = clamp_lv(L.enc[Lt + r][c]);
                    v = (__bf16)__builtin_fmaf(fast_exp(0.5f * lv), eps[q], mu);
                    L.kl[r & 15][c] = __builtin_fmaf(mu, mu, fast_exp(lv)) - lv - 1.0f;
                    L.eps[r & 15][c] = eps[q];
                } else if (r < Lt + C) {
                    v = L.act[0][P + r - Lt][c];
                }
                x[k][q] = v;
            }
            tile_put(L.act[NL] + kTile * k, x[k]);
        }
        // decoder
        net_forward<NL, NL, T>(wf, bs, L, pre, s.width, x, out);
#pragma unroll
        for (int o = 0; o < T; ++o) tile_store_d(&L.dec[kTile * o][0], out[o]);
        wave_sync();
        f32x4 dcur[T], dzc[T];
#pragma unroll
        for (int o = 0; o < T; ++o) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = kTile * o + k0 + q, k = r < P ? r : r - P;
                float v = 0.0f;
                if (r < 2 * P) {
                    const float mu = L.dec[k][c], lvr = L.dec[P + k][c], lv = clamp_lv(lvr);
                    const float e = L.y[k & 15][c] - mu, iv = fast_exp(-lv);
                    if (r < P) {
                        L.nll[k & 15][c] = __builtin_fmaf(e * e, iv, kLog2Pi + lv);
                        v = -e * iv * inv_b;
                    } else {
                        v = 0.5f * __builtin_fmaf(-(e * e), iv, 1.0f) * clamp_mask(lvr) * inv_b;
                    }
                }
                dcur[o][q] = v;
            }
        }
        net_backward<NL, NL, T>(wt, L, pre, dcur, db, dzc);
        tile_store_d(&L.dz[0][0], dzc[0]);
        wave_sync();
#pragma unroll
        for (int o = 0; o < T; ++o) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = kTile * o + k0 + q, i = r < Lt ? r : r - Lt;
                float v = 0.0f;
                if (r < Lt) {
                    v = __builtin_fmaf(a.kl_weight * L.enc[r][c], inv_b, L.dz[r & 15][c]);
                } else if (r < 2 * Lt) {
                    const float lvr = L.enc[r][c], lv = clamp_lv(lvr), sd = fast_exp(0.5f * lv);
                    const float kl = a.kl_weight * 0.5f * (fast_exp(lv) - 1.0f) * inv_b;
                    v = __builtin_fmaf(0.5f * L.dz[i & 15][c] * L.eps[i & 15][c], sd, kl) * clamp_mask(lvr);
                }
                dcur[o][q] = v;
            }
        }
        net_backward<0, NL, T>(wt, L, pre, dcur, db, dzc);
        wave_sync();
        // dW += dPre X^T, both operands read transposed
#pragma unroll
        for (int i = 0; i < 2 * NL; ++i) {
            bf16x4 xt[T];
#pragma unroll
            for (int k = 0; k < T; ++k) xt[k] = tile_get_t(L.act[i] + kTile * k);
#pragma unroll
            for (int o = 0; o < T; ++o) {
                const bf16x4 dt = tile_get_t(L.dpre[i] + kTile * o);
#pragma unroll
                for (int k = 0; k < T; ++k) dw[i][o][k] = mfma_bf16(dt, xt[k], dw[i][o][k]);
            }
        }
        if (lane < 16) {
            float kl = 0.0f, nll = 0.0f;
            for (int i = 0; i < Lt; ++i) kl = __builtin_fmaf(0.5f, L.kl[i][c], kl);
            for (int k = 0; k < P; ++k) nll = __builtin_fmaf(0.5f, L.nll[k][c], nll);
            kl_acc += (double)kl;
            nll_acc += (double)nll;
        }
        wave_sync();
    }

    // bias gradients: sum over the 16 sample columns of each lane group
#pragma unroll
    for (int i = 0; i < 2 * NL; ++i) {
#pragma unroll
        for (int o = 0; o < T; ++o) {
#pragma unroll
            for (int q = 0; q < 4; ++q) db[i][o][q] = row_sum(db[i][o][q]);
        }
    }
    // Block sum through LDS (reusing the tile space), ((w0 + w1) + w2) + w3 of
    // the waves' gradients: as many waves at a time as there is room for (four,
    // or three of the two-tile networks).
    constexpr int kFit = (int)(sizeof(lds_all) / (sizeof(float) * kParams));
    constexpr int kRegions = kFit < kTrainWaves ? kFit : kTrainWaves;
    static_assert(kRegions >= 3, "the block sum takes at most two rounds");
    float* red = reinterpret_cast<float*>(lds_all);  // [kRegions][kParams]
    auto put = [&](int region) __attribute__((always_inline)) {
        float* dst = red + region * kParams;
#pragma unroll
        for (int i = 0; i < 2 * NL; ++i) {
#pragma unroll
            for (int o = 0; o < T; ++o) {
#pragma unroll
                for (int k = 0; k < T; ++k) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        dst[i * LF + (kTile * o + k0 + q) * S + kTile * k + c] = dw[i][o][k][q];
                }
                if (c == 0) *reinterpret_cast<f32x4*>(dst + i * LF + S * S + kTile * o + k0) = db[i][o];
            }
        }
    };
    float* partial = a.partial + (int64_t)blockIdx.x * kParams;
    __syncthreads();
    if (wave < kRegions) put(wave);
    __syncthreads();
    if (kRegions < kTrainWaves) {
        for (int p = threadIdx.x; p < kParams; p += 256) red[p] = (red[p] + red[kParams + p]) + red[2 * kParams + p];
        __syncthreads();
        if (wave == kTrainWaves - 1) put(1);
        __syncthreads();
        for (int p = threadIdx.x; p < kParams; p += 256) partial[p] = red[p] + red[kParams + p];
    } else {
        for (int p = threadIdx.x; p < kParams; p += 256)
            partial[p] = ((red[p] + red[kParams + p]) + red[2 * kParams + p]) + red[3 * kParams + p];
    }
    // loss partials: lanes 0..15 of each wave hold sums
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
        kl_acc += __shfl_xor(kl_acc, off);
        nll_acc += __shfl_xor(nll_acc, off);
    }
    __shared__ double loss_w[kTrainWaves][2];
    if (lane == 0) {
        loss_w[wave][0] = kl_acc;
        loss_w[wave][1] = nll_acc;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double v = 0.0;
        for (int w = 0; w < kTrainWaves; ++w) v += loss_w[w][threadIdx.x];
        a.loss_partial[blockIdx.x * 2 + threadIdx.x] = v;
    }
}

struct AdamArgs {
    int n_params, n_blocks, batch;
    const float* partial;
    const double* loss_partial;
    float* master;
    float* m;
    float* v;
    float* grad_out;
    double* loss_out;
    int do_update;
    float lr, beta1, beta2, one_m_beta1, one_m_beta2, eps, wd, bc1, bc2;
};

// Gradient = sum of the per-block partials, then the AdamW update.  The sum
// over blocks is latency-bound (one dependent load per block), so each block
// of this kernel takes 32 parameters x 8 groups of partial blocks: group q adds
// blocks q, q + 8, ... with its loads in flight together, and the 8 group sums
// are added in fixed order.  The loss partials are reduced by wave 0 of block 0
// with a fixed butterfly.
constexpr int kAdamParams = 32, kAdamGroups = 8;

__global__ __launch_bounds__(256) void cvae_adam_kernel(const AdamArgs a) {
    __shared__ float red[kAdamGroups][kAdamParams];
    const int pl = threadIdx.x % kAdamParams, grp = threadIdx.x / kAdamParams;
    const int p = blockIdx.x * kAdamParams + pl;
    float part = 0.0f;
    if (p < a.n_params) {
#pragma unroll 8
        for (int b = grp; b < a.n_blocks; b += kAdamGroups) part += a.partial[(int64_t)b * a.n_params + p];
    }
    red[grp][pl] = part;
    __syncthreads();
    if (grp == 0 && p < a.n_params) {
        float g = 0.0f;
#pragma unroll
        for (int q = 0; q < kAdamGroups; ++q) g += red[q][pl];
        if (a.grad_out) a.grad_out[p] = g;
        if (a.do_update) {
            const float m = a.beta1 * a.m[p] + a.one_m_beta1 * g;
            const float v = a.beta2 * a.v[p] + a.one_m_beta2 * g * g;
            a.m[p] = m;
            a.v[p] = v;
            const float mh = m / a.bc1, vh = v / a.bc2;
            const float th = a.master[p];
            a.master[p] = th - a.lr * (mh / (sqrtf(vh) + a.eps) + a.wd * th);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < 64 && a.loss_out) {
        double k = 0.0, n = 0.0;
        for (int b = threadIdx.x; b < a.n_blocks; b += 64) {
            k += a.loss_partial[b * 2 + 0];
            n += a.loss_partial[b * 2 + 1];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            k += __shfl_xor(k, off);
            n += __shfl_xor(n, off);
        }
        if (threadIdx.x == 0) {
            a.loss_out[0] = (k + n) / a.batch;
            a.loss_out[1] = k / a.batch;
            a.loss_out[2] = n / a.batch;
        }
    }
}

// ---------------------------------------------------------------------------
// pack

__device__ __forceinline__ uint32_t fp8_e4m3_bits(float x) {
    // OCP E4M3: bias 7, 3 mantissa bits, max 448, round to nearest even,
    // saturating.
    const uint32_t sign = x < 0.0f ? 0x80u : 0u;
    float a = __builtin_fabsf(x);
    if (!(a == a)) return 0x7fu | sign;
    if (a >= 448.0f) return 0x7eu | sign;
    if (a < 0x1p-10f) return sign;  // rounds to zero (half of the smallest subnormal 2^-9)
    int e;
    frexpf(a, &e);
    int eu = e - 1;
    if (eu < -6) eu = -6;
    const float q = ldexpf(1.0f, eu - 3);
    float m = rintf(a / q);  // ties to even
    float v = m * q;
    if (v > 448.0f) v = 448.0f;
    // encode v
    if (v < 0x1p-6f) return sign | (uint32_t)(v / 0x1p-9f);
    int ev;
    frexpf(v, &ev);
    const int eb = ev - 1 + 7;
    const uint32_t mant = (uint32_t)((v / ldexpf(1.0f, ev - 1) - 1.0f) * 8.0f + 0.5f);
    return sign | ((uint32_t)eb << 3) | (mant & 7u);
}

// FP8 activation scales from calibration rows (one block of 256 threads):
// decoder layer j's inputs a_j, computed in FP32 from the master weights for
// every row i < n -- the standardised condition cond[i] after the latent z,
// z the first `latent` normals of the sampler's stream for seed 0 and id i
// -- give s_j, the smallest power of two with max_i |a_j| / s_j <= 448 (the
// largest E4M3 value; 1 where the maximum is 0).  Writes in_scale = 1 / s_j;
// cvae_pack_kernel then folds s_j into out_scale.
__global__ __launch_bounds__(256) void cvae_calib_kernel(Shape s, const float* master, const double* stats,
                                                         const float* cond, int64_t n, PackedModel* pm) {
    const int nl = s.n_linear, L = s.latent, C = s.p_in;
    const int S = kTile * shape_blocks(s), lf = layer_floats(s);
    float mx[kMaxLayers] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
        float a[2 * kTile], nrm[2 * kTile];
        const Rng r = make_rng(0, MS_TAG_CVAE_SAMPLE, (uint64_t)i);
        for (int j = 0; 4 * j < L; ++j) normals4(r, (uint32_t)j, nrm + 4 * j);
        for (int k = 0; k < 2 * kTile; ++k) a[k] = 0.0f;
        for (int k = 0; k < L; ++k) a[k] = nrm[k];
        for (int k = 0; k < C; ++k) a[L + k] = (float)((cond[i * C + k] - stats[k]) / stats[16 + k]);
        for (int j = 0; j < nl; ++j) {
            const LayerDims d = layer_dims(s, nl + j);
            for (int k = 0; k < d.n_in; ++k) mx[j] = fmaxf(mx[j], fabsf(a[k]));
            if (j == nl - 1) break;
            const float* layer = master + (nl + j) * lf;
            float o[2 * kTile];
            for (int row = 0; row < d.n_out; ++row) {
                float acc = layer[S * S + row];
                for (int k = 0; k < d.n_in; ++k) acc = fmaf(layer[row * S + k], a[k], acc);
                o[row] = softplus(acc);
            }
            for (int k = 0; k < 2 * kTile; ++k) a[k] = k < d.n_out ? o[k] : 0.0f;
        }
    }
    __shared__ float red[kMaxLayers][256];
    for (int j = 0; j < kMaxLayers; ++j) red[j][threadIdx.x] = mx[j];
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off)
            for (int j = 0; j < kMaxLayers; ++j) red[j][threadIdx.x] = fmaxf(red[j][threadIdx.x], red[j][threadIdx.x + off]);
        __syncthreads();
    }
    if (threadIdx.x < kMaxLayers) {
        const float m = red[threadIdx.x][0];
        float inv = 1.0f;
        if (m > 0.0f) {
            int e;
            const float f = frexpf(m / 448.0f, &e);  // m / 448 = f 2^e, f in [0.5, 1)
            inv = ldexpf(1.0f, -(f == 0.5f ? e - 1 : e));
        }
        pm->in_scale[threadIdx.x] = inv;
    }
}

// With `calibrated`, in_scale was written by cvae_calib_kernel earlier on the
// same stream; otherwise activations enter E4M3 unscaled.
__global__ void cvae_pack_kernel(Shape s, const float* master, const double* stats, int precision, bool calibrated,
                                 PackedModel* pm) {
    const int lane = threadIdx.x;  // 64 threads
    const int nl = s.n_linear;
    const int T = shape_blocks(s), S = kTile * T, lf = layer_floats(s);
    if (lane == 0) {
        pm->magic = (int32_t)kPackedMagic;
        pm->model = s.model;
        pm->p_in = s.p_in;
        pm->p_out = s.p_out;
        pm->latent = s.latent;
        pm->width = s.width;
        pm->n_linear = nl;
        pm->precision = precision;
        pm->blocks = T;
        pm->pad_[0] = pm->pad_[1] = pm->pad_[2] = 0;
    }
    if (lane < 16) {
        pm->mean_c[lane] = stats ? (float)stats[lane] : 0.0f;
        pm->inv_std_c[lane] = stats ? (float)(1.0 / stats[16 + lane]) : 1.0f;
        pm->mean_y[lane] = stats ? (float)stats[32 + lane] : 0.0f;
        pm->std_y[lane] = stats ? (float)stats[48 + lane] : 1.0f;
    }
    __shared__ float smax[64];
    for (int j = 0; j < kMaxLayers; ++j) {
        const bool real = j < nl;
        const float* layer = master + (nl + (real ? j : 0)) * lf;
        float scale = 1.0f;
        if (precision == MS_PREC_FP8) {
            float mx = 0.0f;
            for (int q = lane; q < S * S; q += 64) mx = fmaxf(mx, real ? fabsf(layer[q]) : 0.0f);
            smax[lane] = mx;
            __syncthreads();
            for (int off = 32; off > 0; off >>= 1) {
                if (lane < off) smax[lane] = fmaxf(smax[lane], smax[lane + off]);
                __syncthreads();
            }
            scale = smax[0] > 0.0f ? smax[0] / 448.0f : 1.0f;
            __syncthreads();
        }
        if (lane == 0) {
            const float in_sc = precision == MS_PREC_FP8 && calibrated ? pm->in_scale[j] : 1.0f;
            pm->in_scale[j] = in_sc;
            pm->out_scale[j] = scale / in_sc;  // s_w s_a, exact: s_a is a power of two
        }
        if (lane < 2 * kTile) {
            const float b = real && lane < S ? layer[S * S + lane] : 0.0f;
            if (lane < kTile) pm->bias[j][lane] = b;
            else pm->bias_hi[j][lane - kTile] = b;
        }
        const int r = lane & 15, kg = lane >> 4;
        for (int ti = 0; ti < 4; ++ti) {
            uint32_t w0 = 0, w1 = 0;
            if (real && precision == MS_PREC_FP8 && ti < T) {
                // K = 32 operand in the permuted order of the FP8 decoders:
                // bytes 0..3 = columns 4 kg .. 4 kg + 3 of input block 0,
                // bytes 4..7 = the same columns of input block 1 (0 when
                // the layer has one block)
                const float* row = layer + (kTile * ti + r) * S + 4 * kg;
                uint32_t lo[4], hi[4];
                for (int q = 0; q < 4; ++q) {
                    lo[q] = fp8_e4m3_bits(row[q] / scale);
                    hi[q] = T == 2 ? fp8_e4m3_bits(row[kTile + q] / scale) : 0u;
                }
                w0 = lo[0] | (lo[1] << 8) | (lo[2] << 16) | (lo[3] << 24);
                w1 = hi[0] | (hi[1] << 8) | (hi[2] << 16) | (hi[3] << 24);
            } else if (real && precision != MS_PREC_FP8 && ti < T * T) {
                const int o = ti >> 1, k = ti & 1;
                const float* row = layer + (kTile * o + r) * S + kTile * k + 4 * kg;
                w0 = (uint32_t)bf16_bits(row[0]) | ((uint32_t)bf16_bits(row[1]) << 16);
                w1 = (uint32_t)bf16_bits(row[2]) | ((uint32_t)bf16_bits(row[3]) << 16);
            }
            uint32_t* dst = ti == 0 ? pm->frag[j][lane] : pm->frag_hi[j][ti - 1][lane];
            dst[0] = w0;
            dst[1] = w1;
        }
    }
}

// ---------------------------------------------------------------------------
// decoder-only sampling: a wave takes 64 / T rows at a time, T lanes each to
// draw and standardise, then 16-row MFMA tiles

constexpr int kSampleWaves = 4;

// A wave's rows in LDS, feature-major: 16 T decoder inputs, which the outputs
// overwrite, then 8 T normals of the posterior noise.  Four more columns than
// rows put a tile's four feature groups on banks of their own, and a lane's
// own row is without conflicts (row-major, 64 lanes' rows lay on four banks).
template <int T>
struct SampleLds {
    static constexpr int kRows = 64 / T;
    static constexpr int kEps = kTile * T;
    float x[kEps + kTile / 2 * T][kRows + 4];  // inputs, then normals from kEps on
};

// T: tiles per layer dimension of the packed model (pm->blocks).  Bound by
// instruction issue: of about 600 a row set the softplus is half, the normals a
// third.  Hence no constants of the model held across rows (scalar loads where
// they are used leave registers for a fifth wave), matrix instructions on
// vector registers (the attribute of the kernel: without it every tile moves
// 24 values to and from accumulators), and values converted in pairs.  2^24
// EventGen samples 557 -> 338 us in BF16, 579 -> 403 in FP8 (moving their 52
// bytes a row takes 173), of Table 1's widest 1769 -> 863; 1000 samples 8.7 ->
// 6.2 us.
template <int T>
__device__ __forceinline__ void sample_rows(const PackedModel* pm, const float* cond, int64_t n, uint64_t seed,
                                            uint64_t id_offset, float* out, SampleLds<T>& L) {
    constexpr int R = SampleLds<T>::kRows, kEps = SampleLds<T>::kEps, kCond = kTile / T, kOut = kTile / 2;
    const ConstModel c = (ConstModel)pm;
    const int P = c->p_out, Lt = c->latent, C = c->p_in;
    // this lane's row of a chunk; of a row's T lanes it takes every T-th
    // condition, block of normals and output from `part` on
    const int row = T == 1 ? lane_id() : lane_id() % R, part = T == 1 ? 0 : lane_id() / R;
    const int col = frag_row(), k0 = frag_k0();
    const bool three = c->n_linear == kDecLayers, fp8 = c->precision == MS_PREC_FP8;
    const DecoderRegs w = load_decoder(pm);
    const int64_t n_chunks = (n + R - 1) / R;
    const int64_t wave_global = blockIdx.x * (int64_t)kSampleWaves + uniform_u32(threadIdx.x >> 6);
    const int64_t n_waves = (int64_t)gridDim.x * kSampleWaves;
    for (int64_t chunk = wave_global; chunk < n_chunks; chunk += n_waves) {
        const int64_t i = chunk * R + row;
        const bool valid = i < n;
        float cv[kCond] = {};
        if (valid) {
#pragma unroll
            for (int q = 0; q < kCond; ++q) {
                const int k = q * T + part;
                if (k < C) cv[q] = cond[i * C + k];
            }
        }
        const Rng r = make_rng(seed, MS_TAG_CVAE_SAMPLE, id_offset + (uint64_t)i);
        for (int j = part; 4 * j < Lt + P; j += T) {
            float nv[4];
            const uint4 u = r.block((uint32_t)j);
            box_muller(u01(u.x), u01(u.y), nv[0], nv[1]);
            if (4 * j + 2 < Lt + P) box_muller(u01(u.z), u01(u.w), nv[2], nv[3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = 4 * j + q;
                if (e < Lt + P) L.x[e < Lt ? e : e + (kEps - Lt)][row] = nv[q];
            }
        }
#pragma unroll
        for (int q = 0; q < kCond; ++q) {
            const int k = q * T + part;
            if (k < C) L.x[Lt + k][row] = (cv[q] - c->mean_c[k]) * c->inv_std_c[k];
        }
        for (int q = Lt + C + part; q < kEps; q += T) L.x[q][row] = 0.0f;
        wave_sync();
        // each lane overwrites exactly the values that it read
        auto load = [&](int path, int f0) {
            return f32x4{L.x[f0 + k0][path], L.x[f0 + k0 + 1][path], L.x[f0 + k0 + 2][path], L.x[f0 + k0 + 3][path]};
        };
        auto store = [&](int path, int f0, f32x4 v) {
#pragma unroll
            for (int q = 0; q < 4; ++q) L.x[f0 + k0 + q][path] = v[q];
        };
        if constexpr (T == 1) {
            if (!three) {
                for (int t = 0; t < R; t += kTile) store(t + col, 0, decoder_tile_layers(pm, load(t + col, 0)));
            } else if (fp8) {
#pragma unroll
                for (int t = 0; t < R; t += kTile) store(t + col, 0, decoder_tile_fp8(w, load(t + col, 0)));
            } else {
#pragma unroll
                for (int t = 0; t < R; t += kTile) store(t + col, 0, decoder_tile(w, load(t + col, 0)));
            }
        } else {
            f32x4 v[R / kTile][2];
#pragma unroll
            for (int t = 0; t < R / kTile; ++t)
                v[t][0] = load(kTile * t + col, 0), v[t][1] = load(kTile * t + col, kTile);
            decoder_tiles_wide<R / kTile>(pm, v);
#pragma unroll
            for (int t = 0; t < R / kTile; ++t)
                store(kTile * t + col, 0, v[t][0]), store(kTile * t + col, kTile, v[t][1]);
        }
        wave_sync();
        if (valid) {
#pragma unroll
            for (int q = 0; q < kOut; ++q) {
                const int k = q * T + part;
                if (k >= P) break;
                const float y = __builtin_fmaf(fast_exp(0.5f * clamp_lv(L.x[P + k][row])), L.x[kEps + k][row], L.x[k][row]);
                out[i * P + k] = __builtin_fmaf(y, c->std_y[k], c->mean_y[k]);
            }
        }
        wave_sync();
    }
}

// One kernel for both widths: the packed model's block count is on the device.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void cvae_sample_kernel(
    const PackedModel* pm, const float* cond, int64_t n, uint64_t seed, uint64_t id_offset, float* out) {
    union Lds {
        SampleLds<1> one;
        SampleLds<2> two;
    };
    __shared__ Lds lds_all[kSampleWaves];
    Lds& L = lds_all[threadIdx.x >> 6];
    if (pm->blocks == 2) sample_rows<2>(pm, cond, n, seed, id_offset, out, L.two);
    else sample_rows<1>(pm, cond, n, seed, id_offset, out, L.one);
}

// ---------------------------------------------------------------------------

static ms_status check_shape(const ms_cvae_shape* sh, Shape* out) {
    MS_REQUIRE(sh != nullptr, "CVAE shape is NULL");
    MS_REQUIRE(sh->model >= 0 && sh->model <= 2, "CVAE model must be 0, 1 or 2");
    MS_REQUIRE(sh->p_in >= 1 && sh->p_out >= 1 && sh->latent >= 1 && sh->width >= 1, "CVAE sizes must be positive");
    if (sh->width > 32 || sh->p_out + sh->p_in > 32 || sh->latent + sh->p_in > 32 || 2 * sh->p_out > 32 ||
        2 * sh->latent > 32 || sh->p_in > 16 || sh->n_linear < 2 || sh->n_linear > kMaxNL)
        return set_error(MS_ERR_UNSUPPORTED,
                         "CVAE shape unsupported: needs width <= 32, 2 <= n_linear <= 4, p_in <= 16, "
                         "p_out + p_in <= 32, latent + p_in <= 32, 2 p_out <= 32, 2 latent <= 32");
    *out = Shape{sh->model, sh->p_in, sh->p_out, sh->latent, sh->width, sh->n_linear};
    return MS_OK;
}

constexpr int kMaxTrainBatch = 1 << 20;
constexpr int kMaxTrainWaveCount = 1024;

constexpr int train_blocks(int batch) {
    return ((batch / kTile < kMaxTrainWaveCount ? batch / kTile : kMaxTrainWaveCount) + kTrainWaves - 1) /
           kTrainWaves;
}

// Scratch of one training step: per-block gradient partials [blocks][params]
// (FP32), then per-block loss partials [blocks][2] (FP64).  Every block
// writes all of its partials on every step, so nothing needs clearing.
constexpr size_t train_partial_bytes(int nb, int n_params) {
    return ((size_t)nb * n_params * sizeof(float) + 255) / 256 * 256;
}
constexpr size_t train_scratch_bytes(int nb, int n_params) {
    return train_partial_bytes(nb, n_params) + (size_t)nb * 2 * sizeof(double);
}

// Device-resident scratch of cvae_train_step_noalloc, sized for the largest
// batch and network the training kernels accept (about 8.7 MB); each device
// holds its own copy for the life of the process.  Host code must not pass
// this name to a kernel: it is a host-side stand-in, not a device address.
// Its per-device address comes from hipGetSymbolAddress (noalloc_scratch).
constexpr size_t kTrainScratchBytes = train_scratch_bytes(train_blocks(kMaxTrainBatch), 2 * kMaxNL * kMaxLayerFloats);
static __device__ __align__(256) unsigned char scratch[kTrainScratchBytes];

}  // namespace msst

extern "C" {

ms_status cvae_param_count(const ms_cvae_shape* shape, size_t* n_floats) {
    msst::Shape s;
    ms_status st = msst::check_shape(shape, &s);
    if (st != MS_OK) return st;
    MS_REQUIRE(n_floats != nullptr, "cvae_param_count: n_floats is NULL");
    *n_floats = (size_t)(2 * s.n_linear * msst::layer_floats(s));
    return MS_OK;
}

ms_status cvae_init(const ms_cvae_shape* shape, uint64_t seed, float* master_dev, void* stream) {
    using namespace msst;
    Shape s;
    ms_status st = check_shape(shape, &s);
    if (st != MS_OK) return st;
    MS_REQUIRE(master_dev != nullptr, "cvae_init: master_dev is NULL");
    int cus;
    if ((st = device_cu_count(&cus)) != MS_OK) return st;
    const int n = 2 * s.n_linear * layer_floats(s);
    hipLaunchKernelGGL(cvae_init_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, s, seed,
                       master_dev, n);
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

ms_status cvae_features(int32_t model, int64_t n, const int64_t* rows_dev, int64_t n_records,
                        const float* params3_dev, const uint32_t* n_scatter_dev, const float* exit_param_dev,
                        const float* event_pos_dev, const float* event_dir_dev, uint64_t seed, uint64_t id_offset,
                        const double* stats_dev, float* cond_dev, float* target_dev, void* stream) {
    using namespace msst;
    MS_REQUIRE(model >= 0 && model <= 2, "cvae_features: model must be 0, 1 or 2");
    MS_REQUIRE(n > 0 && n_records > 0, "cvae_features: n and n_records must be positive");
    MS_REQUIRE(rows_dev != nullptr || n <= n_records, "cvae_features: n > n_records without a row list");
    MS_REQUIRE(params3_dev && n_scatter_dev && cond_dev && target_dev, "cvae_features: NULL array");
    MS_REQUIRE(model == 0 || exit_param_dev, "cvae_features: exit_param is required for PathGen and EventGen");
    MS_REQUIRE(model != 2 || (event_pos_dev && event_dir_dev), "cvae_features: event arrays required for EventGen");
    int cus;
    ms_status st = device_cu_count(&cus);
    if (st != MS_OK) return st;
    int64_t blocks = (n + kFeatThreads - 1) / kFeatThreads;
    if (blocks > cus * 8) blocks = cus * 8;
    const auto kernel = model == MS_MODEL_LENGTH ? cvae_features_kernel<MS_MODEL_LENGTH>
                        : model == MS_MODEL_PATH ? cvae_features_kernel<MS_MODEL_PATH>
                                                 : cvae_features_kernel<MS_MODEL_EVENT>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kFeatThreads), 0, (hipStream_t)stream, n, rows_dev,
                       n_records, params3_dev, n_scatter_dev, exit_param_dev, event_pos_dev, event_dir_dev, seed,
                       id_offset, stats_dev, cond_dev, target_dev);
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

ms_status ms_select_rows_workspace_size(int64_t n, size_t* bytes) {
    MS_REQUIRE(bytes != nullptr && n > 0, "ms_select_rows_workspace_size: need n > 0 and bytes");
    *bytes = (size_t)((n + msst::kSelPerBlock - 1) / msst::kSelPerBlock) * sizeof(int64_t) + 256;
    return MS_OK;
}

ms_status ms_select_rows(int64_t n, const uint32_t* n_scatter_dev, const uint32_t* event_index_dev,
                         uint32_t min_scatter, uint32_t min_event, int64_t* rows_dev, int64_t* count_dev,
                         void* workspace_dev, size_t workspace_bytes, void* stream) {
    using namespace msst;
    MS_REQUIRE(n > 0 && n < ((int64_t)1 << 40), "ms_select_rows: n must be in [1, 2^40)");
    MS_REQUIRE(n_scatter_dev && rows_dev && count_dev && workspace_dev, "ms_select_rows: NULL array");
    size_t need = 0;
    ms_select_rows_workspace_size(n, &need);
    if (workspace_bytes < need) return set_error(MS_ERR_WORKSPACE_TOO_SMALL, "ms_select_rows: workspace needs %zu bytes", need);
    int cus;
    ms_status st = device_cu_count(&cus);
    if (st != MS_OK) return st;
    const int64_t nb = (n + kSelPerBlock - 1) / kSelPerBlock;
    int64_t* bc = reinterpret_cast<int64_t*>(workspace_dev);
    hipStream_t s = (hipStream_t)stream;
    const bool vec = (((uintptr_t)n_scatter_dev | (uintptr_t)event_index_dev) & 15u) == 0;
    hipLaunchKernelGGL(vec ? select_count_kernel<true> : select_count_kernel<false>, dim3((unsigned)nb), dim3(256), 0, s,
                       n, n_scatter_dev, event_index_dev, min_scatter, min_event, bc);
    hipLaunchKernelGGL(select_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, nb, bc, count_dev);
    hipLaunchKernelGGL(vec ? select_write_kernel<true> : select_write_kernel<false>, dim3((unsigned)nb), dim3(256), 0, s,
                       n, n_scatter_dev, event_index_dev, min_scatter, min_event, (const int64_t*)bc, rows_dev);
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

ms_status ms_column_moments_workspace_size(int64_t n, int32_t dim, size_t* bytes) {
    MS_REQUIRE(bytes != nullptr, "ms_column_moments_workspace_size: bytes is NULL");
    *bytes = (size_t)msst::kMomBlocks * 16 * sizeof(double);
    return MS_OK;
}

ms_status ms_column_moments(const float* x_dev, int64_t n, int32_t dim, double* out_dev, void* workspace_dev,
                            size_t workspace_bytes, void* stream) {
    using namespace msst;
    MS_REQUIRE(x_dev && out_dev, "ms_column_moments: NULL array");
    MS_REQUIRE(n > 0 && dim >= 1 && dim <= 16, "ms_column_moments: need n > 0 and 1 <= dim <= 16");
    MS_REQUIRE(workspace_dev != nullptr, "ms_column_moments: workspace is NULL");
    if (workspace_bytes < (size_t)kMomMinBlocks * 16 * sizeof(double))
        return set_error(MS_ERR_WORKSPACE_TOO_SMALL, "ms_column_moments: workspace too small");
    int cus;
    ms_status st = device_cu_count(&cus);
    if (st != MS_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    double* partial = reinterpret_cast<double*>(workspace_dev);
    const int64_t total = n * dim;
    const bool vec = ((uintptr_t)x_dev & 15u) == 0;
    const auto sums = vec ? moments_partial_kernel<4> : moments_partial_kernel<1>;
    // a multiple of dim, no more than the matrix fills or the workspace holds
    int64_t fill = (total + kMomThreads * 4 - 1) / (kMomThreads * 4);
    const int64_t room = (int64_t)(workspace_bytes / (16 * sizeof(double)));
    if (fill > kMomBlocks) fill = kMomBlocks;
    if (fill > room) fill = room;
    const int nb = (int)(fill / dim > 0 ? fill / dim : 1) * dim;
    for (int pass = 0; pass < 2; ++pass) {
        hipLaunchKernelGGL(sums, dim3(nb), dim3(kMomThreads), 0, s, x_dev, total, dim,
                           pass ? (const double*)out_dev : nullptr, partial);
        hipLaunchKernelGGL(moments_final_kernel, dim3(1), dim3(256), 0, s, (const double*)partial, nb, n, dim, out_dev, pass);
    }
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

ms_status cvae_workspace_size(const ms_cvae_shape* shape, int32_t batch, size_t* bytes) {
    using namespace msst;
    Shape s;
    ms_status st = check_shape(shape, &s);
    if (st != MS_OK) return st;
    MS_REQUIRE(bytes != nullptr, "cvae_workspace_size: bytes is NULL");
    MS_REQUIRE(batch > 0 && batch % 16 == 0 && batch <= kMaxTrainBatch, "cvae_workspace_size: batch must be a positive multiple of 16, <= 2^20");
    *bytes = train_scratch_bytes(train_blocks(batch), 2 * s.n_linear * layer_floats(s));
    return MS_OK;
}

}  // extern "C"

namespace msst {

// Address of this device's noalloc scratch, looked up once per device
// (hipGetSymbolAddress with the device current) and kept for the process.
static ms_status noalloc_scratch(void** out) {
    static std::mutex mu;
    static void* ptr[kMaxDevices] = {};
    int dev = -1;
    MS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return set_error(MS_ERR_UNSUPPORTED, "device %d is beyond the %d supported", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(mu);
    if (ptr[dev] == nullptr) {
        void* p = nullptr;
        MS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (p == nullptr) return set_error(MS_ERR_DEVICE, "hipGetSymbolAddress returned NULL for the training scratch");
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return MS_OK;
}

// Validation and launches of one training step on a scratch buffer of at
// least train_scratch_bytes(train_blocks(batch), params) bytes: the caller's
// workspace (ws_dev, ws_bytes), or with `noalloc` this device's scratch
// array, looked up after the arguments have been validated.
static ms_status train_step_launch(const char* who, bool noalloc, const ms_cvae_shape* shape, float* master_dev, float* adam_m_dev,
                                   float* adam_v_dev, const ms_adam* adam, const float* cond_dev,
                                   const float* target_dev, int64_t n_rows, int32_t batch, int32_t sample_rows,
                                   uint64_t seed, int64_t step, uint64_t id_offset, double kl_weight, void* ws_dev,
                                   size_t ws_bytes, double* loss_dev, float* grad_dev, void* stream) {
    Shape s;
    ms_status st = check_shape(shape, &s);
    if (st != MS_OK) return st;
    MS_REQUIRE(master_dev && cond_dev && target_dev, "%s: NULL array", who);
    MS_REQUIRE(batch > 0 && batch % 16 == 0 && batch <= kMaxTrainBatch, "%s: batch must be a positive multiple of 16, <= 2^20", who);
    MS_REQUIRE(n_rows > 0 && n_rows < ((int64_t)1 << 32), "%s: n_rows must be in [1, 2^32)", who);
    MS_REQUIRE(sample_rows || n_rows >= batch, "%s: n_rows < batch without row sampling", who);
    MS_REQUIRE(step >= 0 && step < ((int64_t)1 << 30), "%s: step must be in [0, 2^30)", who);
    MS_REQUIRE(kl_weight >= 0.0 && kl_weight <= 1e6, "%s: kl_weight must be in [0, 1e6]", who);
    if (adam) {
        MS_REQUIRE(adam_m_dev && adam_v_dev, "%s: AdamW moments are NULL", who);
        MS_REQUIRE(adam->step >= 1, "%s: AdamW step must be >= 1", who);
        MS_REQUIRE(adam->lr > 0 && adam->beta1 >= 0 && adam->beta1 < 1 && adam->beta2 >= 0 && adam->beta2 < 1 &&
                       adam->eps > 0 && adam->weight_decay >= 0,
                   "%s: invalid AdamW hyper-parameters", who);
    }
    const int nb = train_blocks(batch);
    const int n_params = 2 * s.n_linear * layer_floats(s);
    const size_t need = train_scratch_bytes(nb, n_params);
    if (!noalloc) {
        MS_REQUIRE(ws_dev != nullptr, "%s: workspace is NULL", who);
        if (ws_bytes < need) return set_error(MS_ERR_WORKSPACE_TOO_SMALL, "%s: workspace needs %zu bytes", who, need);
    }
    int cus;
    if ((st = device_cu_count(&cus)) != MS_OK) return st;
    if (noalloc) {
        if (need > kTrainScratchBytes)
            return set_error(MS_ERR_WORKSPACE_TOO_SMALL, "%s: needs %zu bytes of scratch, the static maximum is %zu",
                             who, need, kTrainScratchBytes);
        if ((st = noalloc_scratch(&ws_dev)) != MS_OK) return st;
    }

    TrainArgs ta{};
    ta.s = s;
    ta.master = master_dev;
    ta.cond = cond_dev;
    ta.target = target_dev;
    ta.n_rows = n_rows;
    ta.batch = batch;
    ta.sample_rows = sample_rows;
    ta.seed = seed;
    ta.step = step;
    ta.id_offset = id_offset;
    ta.kl_weight = (float)kl_weight;
    ta.partial = reinterpret_cast<float*>(ws_dev);
    ta.loss_partial = reinterpret_cast<double*>(reinterpret_cast<char*>(ws_dev) + train_partial_bytes(nb, n_params));
    hipStream_t hs = (hipStream_t)stream;
    const dim3 grid(nb), block(64 * kTrainWaves);
    if (shape_blocks(s) == 1) {
        switch (s.n_linear) {
            case 2: hipLaunchKernelGGL((cvae_train_kernel<2, 1>), grid, block, 0, hs, ta); break;
            case 3: hipLaunchKernelGGL((cvae_train_kernel<3, 1>), grid, block, 0, hs, ta); break;
            default: hipLaunchKernelGGL((cvae_train_kernel<4, 1>), grid, block, 0, hs, ta); break;
        }
    } else {
        switch (s.n_linear) {
            case 2: hipLaunchKernelGGL((cvae_train_kernel<2, 2>), grid, block, 0, hs, ta); break;
            case 3: hipLaunchKernelGGL((cvae_train_kernel<3, 2>), grid, block, 0, hs, ta); break;
            default: hipLaunchKernelGGL((cvae_train_kernel<4, 2>), grid, block, 0, hs, ta); break;
        }
    }
    MS_LAUNCHED();
    AdamArgs aa{};
    aa.n_params = n_params;
    aa.n_blocks = nb;
    aa.batch = batch;
    aa.partial = ta.partial;
    aa.loss_partial = ta.loss_partial;
    aa.master = master_dev;
    aa.m = adam_m_dev;
    aa.v = adam_v_dev;
    aa.grad_out = grad_dev;
    aa.loss_out = loss_dev;
    aa.do_update = adam != nullptr;
    if (adam) {
        aa.lr = (float)adam->lr;
        aa.beta1 = (float)adam->beta1;
        aa.beta2 = (float)adam->beta2;
        aa.one_m_beta1 = (float)(1.0 - adam->beta1);  // 1 - beta in FP32 would lose ~1e-5 relative
        aa.one_m_beta2 = (float)(1.0 - adam->beta2);
        aa.eps = (float)adam->eps;
        aa.wd = (float)adam->weight_decay;
        aa.bc1 = (float)(1.0 - pow(adam->beta1, (double)adam->step));
        aa.bc2 = (float)(1.0 - pow(adam->beta2, (double)adam->step));
    }
    hipLaunchKernelGGL(cvae_adam_kernel, dim3((n_params + kAdamParams - 1) / kAdamParams), dim3(256), 0, hs, aa);
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

}  // namespace msst

extern "C" {

ms_status cvae_train_step(const ms_cvae_shape* shape, float* master_dev, float* adam_m_dev, float* adam_v_dev,
                          const ms_adam* adam, const float* cond_dev, const float* target_dev, int64_t n_rows,
                          int32_t batch, int32_t sample_rows, uint64_t seed, int64_t step, uint64_t id_offset,
                          double kl_weight, void* workspace_dev, size_t workspace_bytes, double* loss_dev,
                          float* grad_dev, void* stream) {
    return msst::train_step_launch("cvae_train_step", false, shape, master_dev, adam_m_dev, adam_v_dev, adam, cond_dev,
                                   target_dev, n_rows, batch, sample_rows, seed, step, id_offset, kl_weight,
                                   workspace_dev, workspace_bytes, loss_dev, grad_dev, stream);
}

ms_status cvae_train_step_noalloc(const ms_cvae_shape* shape, float* master_dev, float* adam_m_dev,
                                  float* adam_v_dev, const ms_adam* adam, const float* cond_dev,
                                  const float* target_dev, int64_t n_rows, int32_t batch, int32_t sample_rows,
                                  uint64_t seed, int64_t step, uint64_t id_offset, double kl_weight,
                                  double* loss_dev, float* grad_dev, void* stream) {
    return msst::train_step_launch("cvae_train_step_noalloc", true, shape, master_dev, adam_m_dev, adam_v_dev, adam,
                                   cond_dev, target_dev, n_rows, batch, sample_rows, seed, step, id_offset, kl_weight,
                                   nullptr, 0, loss_dev, grad_dev, stream);
}

size_t cvae_packed_bytes(void) { return sizeof(msst::PackedModel); }

ms_status cvae_pack(const ms_cvae_shape* shape, const float* master_dev, const double* stats_dev, int32_t precision,
                    const float* calib_cond_dev, int64_t n_calib, void* packed_dev, size_t packed_bytes,
                    void* stream) {
    using namespace msst;
    Shape s;
    ms_status st = check_shape(shape, &s);
    if (st != MS_OK) return st;
    MS_REQUIRE(master_dev && packed_dev, "cvae_pack: NULL array");
    MS_REQUIRE(precision == MS_PREC_BF16 || precision == MS_PREC_FP8, "cvae_pack: precision must be BF16 or FP8");
    MS_REQUIRE(n_calib >= 0 && n_calib <= (1 << 20), "cvae_pack: n_calib must be in [0, 2^20]");
    MS_REQUIRE(n_calib == 0 || (calib_cond_dev && stats_dev), "cvae_pack: calibration rows need calib_cond and stats");
    MS_REQUIRE(((uintptr_t)packed_dev & 15u) == 0, "cvae_pack: packed buffer must be 16-byte aligned");
    if (packed_bytes < sizeof(PackedModel))
        return set_error(MS_ERR_WORKSPACE_TOO_SMALL, "cvae_pack: packed buffer needs %zu bytes", sizeof(PackedModel));
    int cus;
    if ((st = device_cu_count(&cus)) != MS_OK) return st;
    const bool calib = precision == MS_PREC_FP8 && n_calib > 0;
    if (calib)
        hipLaunchKernelGGL(cvae_calib_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, s, master_dev, stats_dev,
                           calib_cond_dev, n_calib, reinterpret_cast<PackedModel*>(packed_dev));
    hipLaunchKernelGGL(cvae_pack_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, s, master_dev, stats_dev, precision,
                       calib, reinterpret_cast<PackedModel*>(packed_dev));
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

ms_status cvae_sample(const void* packed_dev, const float* cond_dev, int64_t n, uint64_t seed, uint64_t id_offset,
                      float* out_dev, void* stream) {
    using namespace msst;
    MS_REQUIRE(packed_dev && cond_dev && out_dev, "cvae_sample: NULL array");
    MS_REQUIRE(n > 0 && n < ((int64_t)1 << 40), "cvae_sample: n must be in [1, 2^40)");
    MS_REQUIRE(((uintptr_t)packed_dev & 15u) == 0, "cvae_sample: packed buffer must be 16-byte aligned");
    int cus;
    ms_status st = device_cu_count(&cus);
    if (st != MS_OK) return st;
    int64_t blocks = (n + 64 * kSampleWaves - 1) / (64 * kSampleWaves);
    // five blocks fit a CU; shares of a sixth of that even out the end (2^24
    // samples 349 us with 8 blocks per CU, 336 to 338 with 20, 32 and 64)
    if (blocks > cus * 32) blocks = cus * 32;
    const PackedModel* pm = reinterpret_cast<const PackedModel*>(packed_dev);
    hipLaunchKernelGGL(cvae_sample_kernel, dim3((unsigned)blocks), dim3(64 * kSampleWaves), 0, (hipStream_t)stream, pm,
                       cond_dev, n, seed, id_offset, out_dev);
    MS_LAUNCHED();
    clear_error();
    return MS_OK;
}

}  // extern "C"
