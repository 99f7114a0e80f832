// The paper's readout and decode on gfx950 (Sec. Encoder, last paragraph;
// Sec. Losses for the seven quantiles and their median; the seed-anchored
// output of Sec. Method).
//
// Per track, with z = [f; b] the last layer's forward state at the last hit
// and reverse state at the first hit (2d floats, from fit_tracks_states):
// y = g (.) z / rms(z); h = SiLU(W1 y + b1) with NH hidden units (the paper's
// head has 128); q = W2 h + b2 (35 values, seven quantiles at ascending levels
// for each of d0, z0, phi, theta, q/p); the point estimate of each parameter
// is its median quantile, the middle output q[7p + 3]; it is added to the
// fp64 seed (phi wrapped to [-pi, pi)), q/p through the seed's scale
// |q/p_seed| + 0.02/GeV.
//
// A wave takes 32 tracks at a time, both layers as matrix-core products with the
// tracks on the 32 columns: hid^T = W1' z^T with W1' = W1 diag(g) (the gain
// folded in on the host), then the per-track 1/rms scales the columns;
// q^T = W2 h^T takes the layer-1 accumulators as its B operand as they lie.
// The reduction order over k is free, so the host packs both weight matrices
// in the order in which the lanes hold their operands, and in layer 2 a lane
// (half s, column t) supplies the hidden units it holds.
//
// Two number types: fp32 products (32x32x2) for the fp32 model; for the
// 16-bit models bf16 weights (W1 and W2 as given, exact for bf16-valued
// weights; the gain is applied to the fp32 activations instead of being
// folded in, which would round the products to 8 bits) against fp32
// activations split into a high and a low bf16 part (32x32x16, two products
// per k-step), which keeps the activations to about 16 significant bits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "common.h"
#include "trackfit.h"

namespace {

constexpr int kNq = 7;          // quantiles per parameter
constexpr int kNout = 35;       // outputs of the head
constexpr float kRoEps = 1e-6f; // RMSNorm epsilon
constexpr double kQopEps = 0.02;  // 1/GeV, scale floor of the q/p decode
constexpr double kPi = 3.14159265358979323846;
constexpr int kWaves = 4;
constexpr int kWaves16 = 8;     // waves of a workgroup of the 16-bit head: two per SIMD
constexpr int kQBytes = 32 * kNout * 4;  // a wave's 32 rows of 35 outputs in LDS
constexpr int kMaxHidden = 256; // hidden units of the head, at most (a multiple of 32)

__device__ __forceinline__ f32x16 mma(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 mma16(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// v = hi + lo + O(2^-16 |v|), both parts bf16 (round to nearest even)
__device__ __forceinline__ void split16(const f32x8 v, bf16x8 &hi, bf16x8 &lo) {
    hi = __builtin_convertvector(v, bf16x8);
    lo = __builtin_convertvector(v - __builtin_convertvector(hi, f32x8), bf16x8);
}

// Layer 1 bias and SiLU on the accumulators (lane (s, c) holds unit
// 32 m + 8 (q/4) + 4 s + q%4 of track c), in place.
template <int MT>
__device__ __forceinline__ void bias_silu(f32x16 (&acc)[MT], float inv, const float *__restrict__ b1, int s) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float v = fmaf(inv, acc[m][q], b1[32 * m + 8 * (q >> 2) + 4 * s + (q & 3)]);
            acc[m][q] = silu_f32(v);
        }
}

// The decode's inputs for the wave's 32 tracks: element lane + 64 e of their
// contiguous 160 seeds.
constexpr int kSeedRegs = 3;
__device__ __forceinline__ void load_seeds(double (&sd)[kSeedRegs], const double *__restrict__ seeds, int t0, int n,
                                           int lane) {
    const int rows = n - t0 < 32 ? n - t0 : 32;
#pragma unroll
    for (int e = 0; e < kSeedRegs; ++e) {
        const int i = lane + 64 * e;
        sd[e] = i < 5 * rows ? seeds[(size_t)t0 * 5 + i] : 0.0;
    }
}

// Outputs to LDS, then the point estimates, decode and the optional quantile rows.  o[rb]
// holds rows 32 rb + 8 (q/4) + 4 s + q%4 of track c (rows past 34 unused).  The wave's
// rows are contiguous in memory and lie in LDS as they do there, so seeds, outputs
// and quantiles move as whole lines.
__device__ __forceinline__ void finish(const f32x16 (&o)[2], const float *b2, float *qs, int lane, int t0, int n,
                                       const double (&sd)[kSeedRegs], float *__restrict__ quant,
                                       double *__restrict__ out) {
    const int s = lane >> 5, c = lane & 31;
    wave_lds_sync();  // the previous tile's reads of the rows are done
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int row = 32 * rb + 8 * (q >> 2) + 4 * s + (q & 3);
            if (row < kNout) qs[c * kNout + row] = o[rb][q] + b2[row];
        }
    wave_lds_sync();

    // point estimates (each parameter's median quantile, its middle output) and decode
    const int rows = n - t0 < 32 ? n - t0 : 32;
#pragma unroll
    for (int e = 0; e < kSeedRegs; ++e) {
        const int i = lane + 64 * e;
        if (i < 5 * rows) {
            const int tr = i / 5, p = i - 5 * tr;
            const double med = (double)qs[tr * kNout + kNq * p + kNq / 2];
            double v = sd[e] + (p == 4 ? med * (fabs(sd[e]) + kQopEps) : med);
            if (p == 2) v -= 2.0 * kPi * floor((v + kPi) / (2.0 * kPi));
            out[(size_t)t0 * 5 + i] = v;
        }
    }
    if (quant) {
        float *qb = quant + (size_t)t0 * kNout;
        const int nf = rows * kNout;
        int i0 = 0;
        if ((reinterpret_cast<uintptr_t>(qb) & 15) == 0) {  // (32 rows are a multiple of 16 bytes)
            for (int i = 4 * lane; i + 4 <= nf; i += 256)
                *reinterpret_cast<f32x4 *>(qb + i) = *reinterpret_cast<const f32x4 *>(qs + i);
            i0 = nf & ~3;
        }
        for (int i = i0 + lane; i < nf; i += 64) qb[i] = qs[i];
    }
}

// fp32 head: A1 [d/4][MT][64] float4 (4 consecutive k-steps), A2 [MT][4][2][64] float4.
// MT: 32-unit blocks of the hidden layer; D: half the state width (a multiple of 8).
template <int MT>
__global__ __launch_bounds__(64 * kWaves) void tf_readout_kernel(const float *__restrict__ states, int n, int D,
                                                                 const double *__restrict__ seeds,
                                                                 const float4 *__restrict__ A1,
                                                                 const float *__restrict__ b1,
                                                                 const float4 *__restrict__ A2,
                                                                 const float *__restrict__ b2,
                                                                 float *__restrict__ quant, double *__restrict__ out) {
    __shared__ __attribute__((aligned(16))) float qs[kWaves][kQBytes / 4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int t0 = (blockIdx.x * kWaves + wv) * 32;
    if (t0 >= n) return;  // the whole wave
    const int s = lane >> 5, c = lane & 31;
    const int t = t0 + c;
    double sd[kSeedRegs];
    load_seeds(sd, seeds, t0, n, lane);
    // columns past the batch repeat track t0 (in bounds); their results are dropped
    const float4 *zp = reinterpret_cast<const float4 *>(states + (size_t)(t < n ? t : t0) * (2 * D) + s * D);

    // layer 1: acc[m] = rows 32 m .. of W1' z^T, k-step ks of this lane half
    // reading z[t][s d + ks]
    f32x16 acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[m][q] = 0.f;
    float ss = 0.f;
#pragma unroll 2
    for (int g = 0; g < D / 4; ++g) {
        const float4 z = zp[g];
        float4 a[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) a[m] = A1[(g * MT + m) * 64 + lane];
        ss = fmaf(z.x, z.x, fmaf(z.y, z.y, fmaf(z.z, z.z, fmaf(z.w, z.w, ss))));
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            acc[m] = mma(a[m].x, z.x, acc[m]);
            acc[m] = mma(a[m].y, z.y, acc[m]);
            acc[m] = mma(a[m].z, z.z, acc[m]);
            acc[m] = mma(a[m].w, z.w, acc[m]);
        }
    }
    ss += __shfl_xor(ss, 32);  // both halves of the track's row
    bias_silu<MT>(acc, 1.0f / sqrtf(ss * (1.0f / (2 * D)) + kRoEps), b1, s);

    // layer 2: o[rb] = rows 32 rb .. of W2 h^T, k-step (m, q) taking the lane's unit of acc[m][q]
    f32x16 o[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int q = 0; q < 16; ++q) o[rb][q] = 0.f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int qg = 0; qg < 4; ++qg)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                const float4 a = A2[((m * 4 + qg) * 2 + rb) * 64 + lane];
                o[rb] = mma(a.x, acc[m][4 * qg + 0], o[rb]);
                o[rb] = mma(a.y, acc[m][4 * qg + 1], o[rb]);
                o[rb] = mma(a.z, acc[m][4 * qg + 2], o[rb]);
                o[rb] = mma(a.w, acc[m][4 * qg + 3], o[rb]);
            }
    finish(o, b2, qs[wv], lane, t0, n, sd, quant, out);
}

// 16-bit head.  Its weights, one block [A1 | A2 | gain | b1 | b2]: A1 [d/8][MT][64]
// bf16x8 (lane (s, i): W1 row 32 m + i, k = 16 ks + 8 s + e), A2 [MT][2][2][64] bf16x8
// (k-step (m, qh): the lane's units of acc[m][8 qh .. 8 qh + 7]), gain [2d], b1 [32 MT],
// b2 [64] fp32.
struct Head16 {
    int a2, gain, b1, b2, bytes;  // byte offsets and total (a multiple of kCopyBytes)
};
__host__ __device__ inline Head16 head16(int d, int hidden) {
    Head16 h;
    h.a2 = hidden * 2 * d * 2;
    h.gain = h.a2 + hidden / 32 * 2 * 2 * 64 * 16;
    h.b1 = h.gain + 2 * d * 4;
    h.b2 = h.b1 + hidden * 4;
    h.bytes = round_up(h.b2 + 64 * 4, kCopyBytes);
    return h;
}
// Whether the weights and the waves' output rows fit in LDS together (the paper's
// head: 115 + 35 KB).
inline bool head16_in_lds(int d, int hidden) {
    return head16(d, hidden).bytes + kWaves16 * kQBytes <= kLdsBytesMax;
}

// What bounds it is memory: a track is 1.5 KB of states in, 0.26 KB of seeds, outputs
// and quantiles out.  One workgroup per compute unit takes the weights into LDS
// once (with one wave per 32 tracks and the weights read from L2 by each, 0.9 GB
// of them per 262 144 tracks passed through L2 beside 0.46 GB of states and outputs)
// and its waves go on from tile to tile; each holds 64 k-values of its tracks in
// registers while the next 64 (the next tile's first ones at a tile's end) are on
// their way, 8 KB per wave in flight, which is what hides the latency at two
// waves per SIMD.
// Tile t is wave t / grid of workgroup t % grid in the first turn, so that few tiles
// lie on different compute units.
// 262 144 tracks of the paper's head: 168 -> 112 us (2.7 -> 4.1 TB/s; a large
// copy reaches 4.7).
// LDSW: the weights in LDS; otherwise each wave reads them for its one tile and is a
// workgroup of its own, so that few tiles lie on different compute units (eight waves
// that read up to 390 KB of weights through one unit's cache are slower than eight units)
// and a launch's last tiles do not wait for room for eight waves.  Workgroups of eight,
// one: hidden = 256 on d = 256, 500 tracks 43.5, 23.4 us, 20 011 51.2, 36.0, 66 001 100,
// 79; hidden = 192 on d = 192 32.2, 16.8, 35.9, 23.1, 69.9, 54.4 (of two: in between).
template <int MT, bool LDSW>
__global__ __launch_bounds__(LDSW ? 64 * kWaves16 : 64, 2) void tf_readout16_kernel(const float *__restrict__ states, int n, int D,
                                                                     const double *__restrict__ seeds,
                                                                     const char *__restrict__ weights,
                                                                     float *__restrict__ quant,
                                                                     double *__restrict__ out) {
    __shared__ __attribute__((aligned(16))) char smem[LDSW ? kLdsBytesMax : kQBytes];
    const int lane = threadIdx.x & 63, wv = uniform(threadIdx.x >> 6);
    const int s = lane >> 5, c = lane & 31;
    const Head16 L = head16(D, 32 * MT);
    float *qs = reinterpret_cast<float *>(smem + wv * kQBytes);
    const char *w = weights;
    if constexpr (LDSW) {
        const unsigned lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem + kWaves16 * kQBytes;
        for (int p = wv * kCopyBytes; p < L.bytes; p += kWaves16 * kCopyBytes)
            lds_dma16(weights + p + 16 * lane, lds + p);
        w = smem + kWaves16 * kQBytes;
    }
    const bf16x8 *A1 = reinterpret_cast<const bf16x8 *>(w) + lane;
    const bf16x8 *A2 = reinterpret_cast<const bf16x8 *>(w + L.a2) + lane;
    const float4 *gp = reinterpret_cast<const float4 *>(w + L.gain) + 2 * s;
    const float *b1 = reinterpret_cast<const float *>(w + L.b1), *b2 = reinterpret_cast<const float *>(w + L.b2);

    // (!LDSW: one tile per wave, since nothing would be kept for the next)
    const int tiles = (n + 31) / 32, step = (int)gridDim.x * kWaves16;
    int tile = LDSW ? wv * (int)gridDim.x + (int)blockIdx.x : (int)blockIdx.x;
    // this lane's row of a tile, from its half of the first k-step on (columns past the
    // batch repeat the tile's first track, in bounds; their results are dropped)
    auto row = [&](int tl) {
        const int t = tl * 32 + c;
        return reinterpret_cast<const float4 *>(states + (size_t)(t < n ? t : tl * 32) * (2 * D) + 8 * s);
    };
    constexpr int GK = MT <= 6 ? 4 : 2;  // k-steps of a group (2 d is a multiple of 64; registers)
    const int ng = D / (8 * GK);
    float4 z[2 * GK];
    auto load = [&](float4 (&v)[2 * GK], const float4 *p) {
#pragma unroll
        for (int j = 0; j < 2 * GK; ++j) v[j] = p[4 * (j >> 1) + (j & 1)];
    };
    const float4 *zp = row(tile < tiles ? tile : 0);
    if (tile < tiles) load(z, zp);
    if constexpr (LDSW) {
        wait_vmcnt<0>();
        lds_barrier();  // the weights are in place
    }
    for (; tile < tiles; tile += step) {
        const int t0 = tile * 32;
        double sd[kSeedRegs];
        load_seeds(sd, seeds, t0, n, lane);
        const bool more = LDSW && tile + step < tiles;
        const float4 *znext = row(more ? tile + step : tile);
        f32x16 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[m][q] = 0.f;
        float ss = 0.f;
        for (int g = 0; g < ng; ++g) {
            float4 zn[2 * GK];
            load(zn, g + 1 < ng ? zp + (g + 1) * 4 * GK : znext);
#pragma unroll
            for (int j = 0; j < GK; ++j) {
                const int ks = g * GK + j;
                const float4 z0 = z[2 * j], z1 = z[2 * j + 1];
                const float4 g0 = gp[4 * ks], g1 = gp[4 * ks + 1];
                ss = fmaf(z0.x, z0.x, fmaf(z0.y, z0.y, fmaf(z0.z, z0.z, fmaf(z0.w, z0.w, ss))));
                ss = fmaf(z1.x, z1.x, fmaf(z1.y, z1.y, fmaf(z1.z, z1.z, fmaf(z1.w, z1.w, ss))));
                bf16x8 hi, lo;  // g (.) z, split
                split16((f32x8){g0.x * z0.x, g0.y * z0.y, g0.z * z0.z, g0.w * z0.w, g1.x * z1.x, g1.y * z1.y,
                                g1.z * z1.z, g1.w * z1.w},
                        hi, lo);
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const bf16x8 a = A1[(ks * MT + m) * 64];
                    acc[m] = mma16(a, hi, acc[m]);
                    acc[m] = mma16(a, lo, acc[m]);
                }
            }
#pragma unroll
            for (int j = 0; j < 2 * GK; ++j) z[j] = zn[j];
        }
        zp = znext;
        ss += __shfl_xor(ss, 32);
        bias_silu<MT>(acc, 1.0f / sqrtf(ss * (1.0f / (2 * D)) + kRoEps), b1, s);

        f32x16 o[2];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int q = 0; q < 16; ++q) o[rb][q] = 0.f;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int qh = 0; qh < 2; ++qh) {
                bf16x8 hi, lo;
                split16((f32x8){acc[m][8 * qh + 0], acc[m][8 * qh + 1], acc[m][8 * qh + 2], acc[m][8 * qh + 3],
                                acc[m][8 * qh + 4], acc[m][8 * qh + 5], acc[m][8 * qh + 6], acc[m][8 * qh + 7]},
                        hi, lo);
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) {
                    const bf16x8 a = A2[((m * 2 + qh) * 2 + rb) * 64];
                    o[rb] = mma16(a, hi, o[rb]);
                    o[rb] = mma16(a, lo, o[rb]);
                }
            }
        finish(o, b2, qs, lane, t0, n, sd, quant, out);
        if constexpr (!LDSW) break;
    }
}

}  // namespace

struct tf_readout {
    int d = 0;
    int hidden = 0;
    bool half = false;       // 16-bit head (tf_readout16_kernel)
    int cu_count = 0;
    char *dmem = nullptr;
    const void *A1 = nullptr;
    const float *b1 = nullptr;
    const void *A2 = nullptr;
    const float *b2 = nullptr;
};

namespace {

// float -> bf16 bits, round to nearest even (NaN stays a quiet NaN)
uint16_t bf16_bits(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <int MT>
void launch_mt(const tf_readout *h, hipStream_t stream, const float *states, int n, const double *seeds, float *quant,
               double *out) {
    if (h->half) {
        const int tiles = (n + 31) / 32;
        if (head16_in_lds(h->d, h->hidden))  // one workgroup per compute unit, no more than tiles
            hipLaunchKernelGGL((tf_readout16_kernel<MT, true>), dim3((unsigned)std::min(tiles, h->cu_count)),
                               dim3(64 * kWaves16), 0, stream, states, n, h->d, seeds, h->dmem, quant, out);
        else
            hipLaunchKernelGGL((tf_readout16_kernel<MT, false>), dim3((unsigned)tiles), dim3(64), 0, stream, states, n,
                               h->d, seeds, h->dmem, quant, out);
    } else {
        const int per_block = 32 * kWaves;
        const dim3 grid((unsigned)((n + per_block - 1) / per_block)), block(64 * kWaves);
        hipLaunchKernelGGL(tf_readout_kernel<MT>, grid, block, 0, stream, states, n, h->d, seeds,
                           static_cast<const float4 *>(h->A1), h->b1, static_cast<const float4 *>(h->A2), h->b2,
                           quant, out);
    }
}

bool valid_dims(int d, int hidden) {
    return d >= 32 && d <= 256 && d % 32 == 0 && hidden >= 32 && hidden <= kMaxHidden && hidden % 32 == 0;
}

}  // namespace

extern "C" size_t tf_readout_blob_size(int32_t d, int32_t hidden) {
    if (d <= 0 || hidden <= 0) return 0;
    const size_t dd = (size_t)d, nh = (size_t)hidden;
    return 2 * dd + nh * 2 * dd + nh + kNout * nh + kNout;
}

extern "C" tf_status tf_readout_create(int32_t d, int32_t hidden, int32_t dtype, const float *host_blob,
                                       size_t n_floats, tf_readout **out) {
    if (!out) return TF_EINVAL;
    *out = nullptr;
    if (!host_blob || d <= 0 || hidden <= 0 || n_floats != tf_readout_blob_size(d, hidden)) return TF_EINVAL;
    if (dtype != TF_FP32 && dtype != TF_BF16 && dtype != TF_BF16_F16ACT) return TF_EINVAL;
    if (!valid_dims(d, hidden)) return TF_EUNSUPPORTED;
    const bool half = dtype != TF_FP32;
    const size_t dd = (size_t)d, nh = (size_t)hidden;
    const int MT = hidden / 32;
    const float *g = host_blob, *W1 = g + 2 * dd, *b1 = W1 + nh * 2 * dd, *W2 = b1 + nh, *b2 = W2 + kNout * nh;
    // W1 as lane (s, i) holds it: row 32 m + i, column k, with the gain folded in for the
    // fp32 head (the 16-bit head applies it to the activations); W2 as lane (s, i)
    // holds it: row 32 rb + i, the hidden unit that the lane's accumulator slot carries
    auto w1 = [&](int m, int lane, size_t k) {
        const size_t u = 32 * m + (lane & 31);
        return half ? W1[u * 2 * dd + k] : W1[u * 2 * dd + k] * g[k];
    };
    auto w2 = [&](int rb, int lane, int m, int q) {
        const int row = 32 * rb + (lane & 31);
        const size_t u = 32 * m + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
        return row < kNout ? W2[(size_t)row * nh + u] : 0.f;
    };
    const size_t esz = half ? 2 : 4;
    const size_t nA1 = nh * 2 * dd, nA2 = (size_t)MT * 2 * 16 * 64;  // elements (A2: 2 row blocks x 16 slots)
    // the 16-bit head's block as its kernel takes it, the fp32 head's parts one by one
    const Head16 L = head16(d, hidden);
    const size_t oA2 = half ? (size_t)L.a2 : nA1 * esz + nh * 4, oB1 = half ? (size_t)L.b1 : nA1 * esz;
    const size_t oB2 = half ? (size_t)L.b2 : oA2 + nA2 * esz;
    const size_t total = half ? (size_t)L.bytes : oB2 + 64 * 4;
    std::vector<char> hbuf;
    try {
        hbuf.assign(total, 0);
    } catch (const std::bad_alloc &) {
        return TF_ENOMEM;
    }
    char *hp = hbuf.data();
    if (half) {
        // A1 [d/8][MT][64][8]: lane half s of k-step ks covers k = 16 ks + 8 s .. + 7
        uint16_t *A1 = reinterpret_cast<uint16_t *>(hp);
        for (int ks = 0; ks < d / 8; ++ks)
            for (int m = 0; m < MT; ++m)
                for (int lane = 0; lane < 64; ++lane)
                    for (int e = 0; e < 8; ++e)
                        A1[(((size_t)ks * MT + m) * 64 + lane) * 8 + e] = bf16_bits(w1(m, lane, (size_t)16 * ks + 8 * (lane >> 5) + e));
        // A2 [MT][2][2][64][8]: k-step (m, qh) takes accumulator slots 8 qh .. 8 qh + 7
        uint16_t *A2 = reinterpret_cast<uint16_t *>(hp + oA2);
        for (int m = 0; m < MT; ++m)
            for (int qh = 0; qh < 2; ++qh)
                for (int rb = 0; rb < 2; ++rb)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int e = 0; e < 8; ++e)
                            A2[((((size_t)m * 2 + qh) * 2 + rb) * 64 + lane) * 8 + e] =
                                bf16_bits(w2(rb, lane, m, 8 * qh + e));
    } else {
        // A1 [d/4][MT][64][4]: the k-steps 4 grp .. 4 grp + 3, k = s d + 4 grp .. + 3 in lane half s
        float *A1 = reinterpret_cast<float *>(hp);
        for (int grp = 0; grp < d / 4; ++grp)
            for (int m = 0; m < MT; ++m)
                for (int lane = 0; lane < 64; ++lane)
                    for (int e = 0; e < 4; ++e)
                        A1[(((size_t)grp * MT + m) * 64 + lane) * 4 + e] =
                            w1(m, lane, (lane >> 5) * dd + 4 * grp + e);
        // A2 [MT][4][2][64][4]: k-steps (m, 4 qg .. 4 qg + 3)
        float *A2 = reinterpret_cast<float *>(hp + oA2);
        for (int m = 0; m < MT; ++m)
            for (int qg = 0; qg < 4; ++qg)
                for (int rb = 0; rb < 2; ++rb)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int e = 0; e < 4; ++e)
                            A2[((((size_t)m * 4 + qg) * 2 + rb) * 64 + lane) * 4 + e] = w2(rb, lane, m, 4 * qg + e);
    }
    std::memcpy(hp + oB1, b1, nh * 4);
    std::memcpy(hp + oB2, b2, kNout * 4);
    if (half) std::memcpy(hp + L.gain, g, 2 * dd * 4);
    tf_readout *ro = new (std::nothrow) tf_readout;
    if (!ro) return TF_ENOMEM;
    if (hipMalloc((void **)&ro->dmem, total) != hipSuccess) {
        delete ro;
        return TF_ENOMEM;
    }
    int dev = 0;
    if (hipMemcpy(ro->dmem, hp, total, hipMemcpyHostToDevice) != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ro->cu_count, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        ro->cu_count < 1) {
        (void)hipFree(ro->dmem);
        delete ro;
        return TF_EHIP;
    }
    ro->d = d;
    ro->hidden = hidden;
    ro->half = half;
    ro->A1 = ro->dmem;  // (the parts: the fp32 head's)
    ro->b1 = reinterpret_cast<const float *>(ro->dmem + oB1);
    ro->A2 = ro->dmem + oA2;
    ro->b2 = reinterpret_cast<const float *>(ro->dmem + oB2);
    *out = ro;
    return TF_OK;
}

extern "C" void tf_readout_destroy(tf_readout *h) {
    if (!h) return;
    (void)hipDeviceSynchronize();
    (void)hipFree(h->dmem);
    delete h;
}

extern "C" tf_status tf_decode_tracks(const float *states, int32_t n_tracks, const double *seeds,
                                      const tf_readout *h, float *quantiles, double *out, hipStream_t stream) {
    if (!h || n_tracks < 0) return TF_EINVAL;
    if (n_tracks == 0) return TF_OK;
    if (!states || !seeds || !out) return TF_EINVAL;
    if (!valid_dims(h->d, h->hidden)) return TF_EINVAL;
    const int nt = (int)n_tracks;
    switch (h->hidden / 32) {
        case 1: launch_mt<1>(h, stream, states, nt, seeds, quantiles, out); break;
        case 2: launch_mt<2>(h, stream, states, nt, seeds, quantiles, out); break;
        case 3: launch_mt<3>(h, stream, states, nt, seeds, quantiles, out); break;
        case 4: launch_mt<4>(h, stream, states, nt, seeds, quantiles, out); break;
        case 5: launch_mt<5>(h, stream, states, nt, seeds, quantiles, out); break;
        case 6: launch_mt<6>(h, stream, states, nt, seeds, quantiles, out); break;
        case 7: launch_mt<7>(h, stream, states, nt, seeds, quantiles, out); break;
        case 8: launch_mt<8>(h, stream, states, nt, seeds, quantiles, out); break;
        default: return TF_EINVAL;
    }
    return hipGetLastError() == hipSuccess ? TF_OK : TF_EHIP;
}
