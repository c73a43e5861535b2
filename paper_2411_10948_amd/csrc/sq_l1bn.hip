// Fully-quantized L1 batch normalization (L1BNQ), Sec. 4 (Fig. l1bnq) and
// App. C: forward and backward over 8-bit input codes [M, C] (M = N*H*W rows,
// channels contiguous).
//
// Every statistic is an integer sum over a channel's column, so the kernels
// are column reductions plus one elementwise pass:
//   forward   S_c = sum q                 -> m_c (mean code)
//             A_c = sum |q - m_c|, P_c = sum sgn(q - m_c)
//                                         -> k_c (8-bit sigma code), gamma^q,
//                                            beta^q, kappa_c
//             y = fl(fl(kappa_c (q - m_c)) + beta^q_c)
//   backward  (ShiftQuant codes qg of dy, by the quantizer kernels)
//             G1_c = sum qg, G2_c = sum qg (q - m_c)
//                                         -> dgamma, dbeta, a_c, b_c, e_c
//             dx = fl(fl(fl(a_c qg) + fl(b_c sgn(q - m_c))) + e_c)
// Per-channel constants are evaluated in binary64 and rounded once to
// binary32; the library is built without FMA contraction, so the operation
// order written here is the order executed.
//
// Work split: a thread owns 16 channels of a row (one 16-byte code load);
// 256 / (C / 16) rows are in flight per block and each block takes a
// contiguous range of rows, so every load is a coalesced row segment.  A
// block reduces its rows in LDS and writes one partial per channel; a second
// kernel (16 channels per block) adds the partials.  Block partials are int32:
// with M <= 2^24 and at most 512 row blocks a block holds at most 32768 rows,
// and |qg (q - m)| <= 127 * 254.

#include <algorithm>

#include "sq_internal.h"

namespace sq {

namespace {

constexpr int kBnThreads = 256;
constexpr int kBnChunk = 16;                 // channels per thread (one 16-byte load)
constexpr int kBnWaves = 16;                 // waves of a channel-reduction block

struct BnGeom {
    int64_t chunks;   // ceil(C / 16)
    int cis;          // chunks per block column (<= 256)
    int lanes;        // rows in flight per block
    int64_t slabs;    // block columns (gridDim.y)
    int64_t nb;       // row blocks (gridDim.x)
    int64_t rpb;      // rows per block
};

BnGeom bn_geom(int64_t M, int64_t C, int64_t max_blocks, int64_t min_rows) {
    BnGeom g{};
    g.chunks = (C + kBnChunk - 1) / kBnChunk;
    g.cis = (int)std::min<int64_t>(g.chunks, kBnThreads);
    g.lanes = kBnThreads / g.cis;
    g.slabs = (g.chunks + g.cis - 1) / g.cis;
    g.nb = std::max<int64_t>(1, std::min<int64_t>(max_blocks, (M + min_rows - 1) / min_rows));
    g.rpb = (M + g.nb - 1) / g.nb;
    g.nb = (M + g.rpb - 1) / g.rpb;   // no empty block
    return g;
}

constexpr int64_t kSumBlocks = 512, kSumMinRows = 64;
constexpr int64_t kApplyBlocks = 1024, kApplyMinRows = 64;

BnGeom sum_geom(int64_t M, int64_t C) { return bn_geom(M, C, kSumBlocks, kSumMinRows); }

__device__ __forceinline__ void unpack16(const int4 v, int (&out)[16]) {
    const uint32_t w[4] = {(uint32_t)v.x, (uint32_t)v.y, (uint32_t)v.z, (uint32_t)v.w};
#pragma unroll
    for (int i = 0; i < 16; ++i) out[i] = (int)(int8_t)(w[i >> 2] >> (8 * (i & 3)));
}

__device__ __forceinline__ int sgn(int d) { return (d > 0) - (d < 0); }

// round_half_even(num / den), den > 0
__device__ __forceinline__ int64_t div_round_even(int64_t num, int64_t den) {
    int64_t q = num / den, r = num % den;
    if (r < 0) {
        q -= 1;
        r += den;
    }
    if (2 * r > den || (2 * r == den && (q & 1))) q += 1;
    return q;
}

// Block-level sums of NS per-thread accumulator arrays over the lanes that
// share a chunk; writes part[k nb C + blockIdx.x C + c] for the block's channels.
// Accumulator i of thread t sits at word i (kBnThreads + 1) + t, which keeps both
// the stores and the channel-order reads free of bank conflicts.
constexpr int kRedLd = kBnThreads + 1, kRedWords = kBnChunk * kRedLd;

template <int NS>
__device__ __forceinline__ void block_colsum(int32_t (*red)[kRedWords], const int32_t (&acc)[NS][16], const BnGeom& g,
                                             int64_t C, int32_t* __restrict__ part) {
    const int tid = threadIdx.x, width = g.cis * kBnChunk;
#pragma unroll
    for (int n = 0; n < NS; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) red[n][i * kRedLd + tid] = acc[n][i];
    __syncthreads();
    // up to 128 channels: J threads per channel add a strided subset of its
    // lanes each, and the subsets' sums go through LDS once more
    const int64_t cbase = (int64_t)blockIdx.y * width;
    const int J = std::max(1, kBnThreads / width);
    int32_t sub[NS];
    for (int k = tid % (width * J <= kBnThreads ? width : kBnThreads), j = tid / width; k < width; k += kBnThreads) {
        const int first = (k % kBnChunk) * kRedLd + k / kBnChunk;
#pragma unroll
        for (int n = 0; n < NS; ++n) sub[n] = 0;
        if (J == 1 || j < J)
            for (int l = J == 1 ? 0 : j; l < g.lanes; l += J)
#pragma unroll
                for (int n = 0; n < NS; ++n) sub[n] += red[n][first + l * g.cis];
        if (J == 1 && cbase + k < C)
#pragma unroll
            for (int n = 0; n < NS; ++n) part[((int64_t)n * g.nb + blockIdx.x) * C + cbase + k] = sub[n];
    }
    if (J == 1) return;
    __syncthreads();
    if (tid < width * J)
#pragma unroll
        for (int n = 0; n < NS; ++n) red[n][tid] = sub[n];   // tid = j width + k
    __syncthreads();
    if (tid < width && cbase + tid < C) {
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            int32_t t = 0;
            for (int i = 0; i < J; ++i) t += red[n][i * width + tid];
            part[((int64_t)n * g.nb + blockIdx.x) * C + cbase + tid] = t;
        }
    }
}

// OP 0: S = sum q.  OP 1: A = sum |q - m|, P = sum sgn(q - m).
// OP 2: G1 = sum qg, G2 = sum qg (q - m)  (a = qg codes, x = input codes), for
// layers k_quantize_bn does not take.
// part: [2][nb][C] int32.
template <int OP>
__global__ __launch_bounds__(kBnThreads) void k_bn_colsum(const int8_t* __restrict__ a, int64_t lda,
                                                          const int8_t* __restrict__ x, int64_t ldx,
                                                          const sq_l1bn_channel* __restrict__ ch, int64_t M,
                                                          int64_t C, BnGeom g, int32_t* __restrict__ part) {
    constexpr int NS = OP == 0 ? 1 : 2;
    __shared__ int32_t red[NS][kRedWords];
    const int tid = threadIdx.x, cl = tid % g.cis, lane = tid / g.cis;
    const int64_t chunk = (int64_t)blockIdx.y * g.cis + cl, c0 = chunk * kBnChunk;
    const bool active = lane < g.lanes && chunk < g.chunks;
    const int64_t r0 = (int64_t)blockIdx.x * g.rpb, r1 = std::min<int64_t>(M, r0 + g.rpb);
    int32_t acc[NS][16];
    int mu[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
#pragma unroll
        for (int n = 0; n < NS; ++n) acc[n][i] = 0;
        // clamped index, select after the load (no branch per channel)
        mu[i] = OP >= 1 ? ch[std::min<int64_t>(c0 + i, C - 1)].mu : 0;
    }
    if (active) {
        constexpr int U = OP == 2 ? 4 : 8;   // rows in flight per thread
        auto add_row = [&](const int4 va, const int4 vx) {
            int qa[16], qx[16];
            unpack16(va, qa);
            if (OP == 2) unpack16(vx, qx);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (OP == 0) {
                    acc[0][i] += qa[i];
                } else if (OP == 1) {
                    const int d = qa[i] - mu[i];
                    acc[0][i] += d < 0 ? -d : d;
                    acc[NS - 1][i] += min(max(d, -1), 1);
                } else {
                    acc[0][i] += qa[i];
                    acc[NS - 1][i] += qa[i] * (qx[i] - mu[i]);
                }
            }
        };
        // row indices clamped, so that a batch's loads issue back to back
        for (int64_t m = r0 + lane; m < r1; m += U * (int64_t)g.lanes) {
            int4 va[U], vx[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t mm = std::min<int64_t>(m + u * (int64_t)g.lanes, r1 - 1);
                va[u] = *reinterpret_cast<const int4*>(a + mm * lda + c0);
                if (OP == 2) vx[u] = *reinterpret_cast<const int4*>(x + mm * ldx + c0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (m + u * (int64_t)g.lanes < r1) add_row(va[u], OP == 2 ? vx[u] : va[u]);
        }
    }
    block_colsum<NS>(red, acc, g, C, part);
}

// Per-channel totals of the block partials: a block of 16 waves takes
// kChanPer = 16 consecutive channels, 64 partial rows at a time (a wave reads
// 4 rows of 64 bytes, 8 loads in flight per thread); lanes of a channel add up
// by shuffles, waves in LDS.  Bound by latency; with 64 channels per block (one
// block for the 64-channel layer, 512 partial rows) 8.8 us, so 3.8 to 5.4.
//   OP 0: mean code.  OP 1: deviation and sign sums.
//   OP 2: backward constants (a, b, e), dgamma, dbeta.
constexpr int kChanPer = 16;
template <int OP>
__global__ __launch_bounds__(64 * kBnWaves) void k_bn_chan(const int32_t* __restrict__ part, int64_t nb, int64_t M,
                                                           int64_t C, sq_l1bn_channel* __restrict__ ch,
                                                           const sq_l1bn_layer* __restrict__ layer,
                                                           const uint8_t* __restrict__ group,
                                                           const sq_scale* __restrict__ gscale,
                                                           float* __restrict__ coef, float* __restrict__ dgamma,
                                                           float* __restrict__ dbeta) {
    __shared__ int64_t sh0[kBnWaves][kChanPer], sh1[kBnWaves][kChanPer];
    const int k = threadIdx.x % kChanPer, row = threadIdx.x / kChanPer, w = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * kChanPer + k;
    const int64_t cc = std::min<int64_t>(c, C - 1);
    constexpr int U = 8, kRows = 64 * kBnWaves / kChanPer;
    int64_t t0 = 0, t1 = 0;
    for (int64_t b0 = row; b0 < nb; b0 += (int64_t)kRows * U) {
        int32_t v0[U], v1[U];
        // clamped row, select after the load: the loads issue back to back
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t b = std::min<int64_t>(b0 + (int64_t)kRows * u, nb - 1);
            v0[u] = part[b * C + cc];
            v1[u] = OP >= 1 ? part[(nb + b) * C + cc] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = b0 + (int64_t)kRows * u < nb;
            t0 += in ? v0[u] : 0;
            t1 += in ? v1[u] : 0;
        }
    }
#pragma unroll
    for (int o = kChanPer; o < 64; o <<= 1) {
        t0 += __shfl_xor(t0, o, 64);
        if (OP >= 1) t1 += __shfl_xor(t1, o, 64);
    }
    if ((threadIdx.x & 63) < kChanPer) {
        sh0[w][k] = t0;
        sh1[w][k] = t1;
    }
    __syncthreads();
    if (threadIdx.x >= kChanPer || c >= C) return;
    t0 = t1 = 0;
#pragma unroll
    for (int i = 0; i < kBnWaves; ++i) {
        t0 += sh0[i][k];
        t1 += sh1[i][k];
    }
    if (OP == 0) {
        sq_l1bn_channel v{};
        v.mu = (int32_t)div_round_even(t0, M);
        ch[c] = v;
    } else if (OP == 1) {
        ch[c].dev_sum = t0;
        ch[c].sign_sum = (int32_t)t1;
    } else {
        const sq_l1bn_channel cv = ch[c];
        const sq_l1bn_layer L = *layer;
        const double delta = (double)__fmul_rn(gscale->step, pow2f(-(int)group[c]));
        const double db = delta * (double)t0;
        dbeta[c] = (float)db;
        float ca = 0.0f, cb = 0.0f, ce = 0.0f;
        if (L.dev_max == 0) {
            dgamma[c] = 0.0f;
        } else {
            const double rho = (127.0 * (double)M) / ((double)L.dev_max * (double)cv.sigma);
            const double lambda = ((double)cv.gamma * rho) / (double)L.x_step;
            const double dg = (delta * (double)t1) * rho;
            const double D = dg / (double)M;
            const double gbar = db / (double)M;
            const double sbar = (double)cv.sign_sum / (double)M;
            dgamma[c] = (float)dg;
            ca = (float)(lambda * delta);
            cb = (float)(-(lambda * D));
            ce = (float)(lambda * (D * sbar - gbar));
        }
        reinterpret_cast<float4*>(coef)[c] = make_float4(ca, cb, ce, 0.0f);
    }
}

constexpr int kParThreads = 1024;

__device__ __forceinline__ uint32_t abs_bits(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

// 8-bit per-tensor scale of a parameter vector (the quantizer of W and X).
__device__ __forceinline__ sq_scale param_scale(uint32_t amax) {
    sq_scale s{};
    const float a = __uint_as_float(amax);
    s.r_max = a;
    s.flags = amax >= 0x7F800000u ? SQ_FLAG_NONFINITE : (a < pow2f(-96) ? SQ_FLAG_ZERO : 0u);
    if (!s.flags) {
        s.inv = 127.0f / a;
        s.step = a / 127.0f;
    }
    return s;
}

__device__ __forceinline__ float param_value(float v, const sq_scale& s) {
    if (s.flags) return 0.0f;
    // the code is an integer: a negative value that rounds to 0 gives +0
    const int code = (int)fminf(fmaxf(rintf(__fmul_rn(v, s.inv)), -127.0f), 127.0f);
    return __fmul_rn(s.step, (float)code);
}

// Sigma code, gamma^q, beta^q and kappa of a channel with deviation sum dev.
struct BnParam {
    int32_t sigma;
    float gamma, beta, kappa;
};
__device__ __forceinline__ BnParam channel_param(int64_t dev, int64_t amax, float gamma, float beta, const sq_scale& gs,
                                                 const sq_scale& bs, int64_t M) {
    BnParam p{0, param_value(gamma, gs), param_value(beta, bs), 0.0f};
    if (amax != 0) {
        const int64_t k = std::max<int64_t>(1, div_round_even(127 * dev, amax));
        p.sigma = (int32_t)k;
        p.kappa = (float)(((double)p.gamma * (127.0 * (double)M)) / ((double)amax * (double)k));
    }
    return p;
}

__device__ __forceinline__ void write_layer(sq_l1bn_layer* layer, int64_t M, int64_t amax, float x_step,
                                            const sq_scale& gs, const sq_scale& bs) {
    sq_l1bn_layer L{};
    L.rows = M;
    L.dev_max = amax;
    L.x_step = x_step;
    L.flags = amax == 0 ? SQ_FLAG_ZERO : 0u;
    L.gamma_scale = gs;
    L.beta_scale = bs;
    *layer = L;
}

// One block: A_max, the parameter scales, then every channel's constants (more
// than kFuseC channels; else the forward's elementwise pass takes them).
__global__ __launch_bounds__(kParThreads) void k_bn_params(sq_l1bn_channel* __restrict__ ch, int64_t M, int64_t C,
                                                           const float* __restrict__ gamma,
                                                           const float* __restrict__ beta,
                                                           const sq_scale* __restrict__ xs,
                                                           sq_l1bn_layer* __restrict__ layer) {
    __shared__ int64_t sh_a[kParThreads / 64];
    __shared__ uint32_t sh_g[kParThreads / 64], sh_b[kParThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int64_t amax = 0;
    uint32_t gmax = 0u, bmax = 0u;
    for (int64_t c = tid; c < C; c += kParThreads) {
        amax = std::max<int64_t>(amax, ch[c].dev_sum);
        gmax = std::max(gmax, abs_bits(gamma[c]));
        bmax = std::max(bmax, abs_bits(beta[c]));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        amax = std::max<int64_t>(amax, __shfl_xor(amax, o, 64));
        gmax = std::max(gmax, (uint32_t)__shfl_xor((int)gmax, o, 64));
        bmax = std::max(bmax, (uint32_t)__shfl_xor((int)bmax, o, 64));
    }
    if (lane == 0) {
        sh_a[w] = amax;
        sh_g[w] = gmax;
        sh_b[w] = bmax;
    }
    __syncthreads();
    amax = 0;
    gmax = bmax = 0u;
    for (int i = 0; i < kParThreads / 64; ++i) {
        amax = std::max<int64_t>(amax, sh_a[i]);
        gmax = std::max(gmax, sh_g[i]);
        bmax = std::max(bmax, sh_b[i]);
    }
    const sq_scale gs = param_scale(gmax), bs = param_scale(bmax);
    for (int64_t c = tid; c < C; c += kParThreads) {
        sq_l1bn_channel v = ch[c];
        const BnParam p = channel_param(v.dev_sum, amax, gamma[c], beta[c], gs, bs, M);
        v.sigma = p.sigma;
        v.gamma = p.gamma;
        v.beta = p.beta;
        v.kappa = p.kappa;
        ch[c] = v;
    }
    if (tid == 0) write_layer(layer, M, amax, xs->step, gs, bs);
}

// Elementwise pass.  Forward (BWD = false): y = fl(fl(kappa (q - m)) + beta),
// a = input codes.  Backward: dx = fl(fl(fl(a qg) + fl(b sgn(q - m))) + e),
// a = gradient codes, x = input codes; with `ranges`, each block also writes
// the channel maxima of |dx| over its rows (bit patterns) to ranges[block, c].
// A thread owns one channel quad of a row (a 4-byte code load, one float4
// store), so a wave's loads and stores cover contiguous row segments.
struct QuadGeom {
    int64_t quads;    // ceil(C / 4)
    int qis;          // quads per block column (<= 256)
    int lanes;        // rows in flight per block
    int64_t slabs, nb, rpb;
};

QuadGeom quad_geom(int64_t M, int64_t C) {
    QuadGeom g{};
    g.quads = (C + 3) / 4;
    g.qis = (int)std::min<int64_t>(g.quads, kBnThreads);
    g.lanes = kBnThreads / g.qis;
    g.slabs = (g.quads + g.qis - 1) / g.qis;
    g.nb = std::max<int64_t>(1, std::min<int64_t>(kApplyBlocks, (M + kApplyMinRows - 1) / kApplyMinRows));
    g.rpb = (M + g.nb - 1) / g.nb;
    g.nb = (M + g.rpb - 1) / g.rpb;
    return g;
}

__device__ __forceinline__ void unpack4(uint32_t w, int (&out)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = (int)(int8_t)(w >> (8 * i));
}

// PAR (forward, at most kFuseC channels, so one block column): every block
// also takes A_max and the parameter scales and the constants of all channels
// (a few channels per thread, into LDS), and block 0 writes them to ch and
// layer.  As a launch of one block of its own that took 3.9 us and a gap;
// here 0 to 1.2 us (200704 x 64: the step 131.9 -> 128.5 us; 12544 x 256: 67.9 ->
// 65.6; the forward alone at 12544 x 512 33.9 -> 31.0, 16384 x 768 44.4 -> 41.6,
// 800 x 1024 38.3 -> 35.4, 12544 x 1024 46.2 -> 43.0, where a thread takes 4
// channels; more would not fit one block column).
constexpr int kFuseC = 1024;
template <bool BWD, bool PAR = false>
__global__ __launch_bounds__(kBnThreads) void k_bn_apply(const int8_t* __restrict__ a, int64_t lda,
                                                         const int8_t* __restrict__ x, int64_t ldx,
                                                         sq_l1bn_channel* ch, const float* __restrict__ coef,
                                                         int64_t M, int64_t C, QuadGeom g, float* __restrict__ out,
                                                         int64_t ld_out, bool vec_out, uint32_t* __restrict__ ranges,
                                                         const float* __restrict__ gamma,
                                                         const float* __restrict__ beta,
                                                         const sq_scale* __restrict__ xs, sq_l1bn_layer* layer) {
    __shared__ uint32_t red[BWD ? kBnThreads * 4 : 1];
    __shared__ float par[PAR ? 2 : 1][PAR ? kFuseC : 1];   // kappa, beta^q
    const int tid = threadIdx.x, cl = tid % g.qis, lane = tid / g.qis;
    if constexpr (PAR) {
        __shared__ int64_t sh_a[kBnThreads / 64];
        __shared__ uint32_t sh_g[kBnThreads / 64], sh_b[kBnThreads / 64];
        constexpr int N = kFuseC / kBnThreads;
        int64_t dev[N], amax = 0;
        float gv[N], bv[N];
        uint32_t gmax = 0u, bmax = 0u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * kBnThreads;
            const bool in = c < C;
            dev[i] = in ? ch[c].dev_sum : 0;
            gv[i] = in ? gamma[c] : 0.0f;
            bv[i] = in ? beta[c] : 0.0f;
            amax = std::max(amax, dev[i]);
            gmax = std::max(gmax, abs_bits(gv[i]));
            bmax = std::max(bmax, abs_bits(bv[i]));
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            amax = std::max<int64_t>(amax, __shfl_xor(amax, o, 64));
            gmax = std::max(gmax, (uint32_t)__shfl_xor((int)gmax, o, 64));
            bmax = std::max(bmax, (uint32_t)__shfl_xor((int)bmax, o, 64));
        }
        if ((tid & 63) == 0) {
            sh_a[tid >> 6] = amax;
            sh_g[tid >> 6] = gmax;
            sh_b[tid >> 6] = bmax;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kBnThreads / 64; ++i) {
            amax = std::max(amax, sh_a[i]);
            gmax = std::max(gmax, sh_g[i]);
            bmax = std::max(bmax, sh_b[i]);
        }
        const sq_scale gs = param_scale(gmax), bs = param_scale(bmax);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * kBnThreads;
            if (c >= C) continue;
            const BnParam p = channel_param(dev[i], amax, gv[i], bv[i], gs, bs, M);
            par[0][c] = p.kappa;
            par[PAR ? 1 : 0][c] = p.beta;
            if (blockIdx.x == 0) {   // the other blocks read mu and dev_sum only
                ch[c].sigma = p.sigma;
                ch[c].gamma = p.gamma;
                ch[c].beta = p.beta;
                ch[c].kappa = p.kappa;
            }
        }
        if (blockIdx.x == 0 && tid == 0) write_layer(layer, M, amax, xs->step, gs, bs);
        __syncthreads();
    }
    const int64_t quad = (int64_t)blockIdx.y * g.qis + cl, c0 = quad * 4;
    const bool active = lane < g.lanes && quad < g.quads;
    const int64_t r0 = (int64_t)blockIdx.x * g.rpb, r1 = std::min<int64_t>(M, r0 + g.rpb);
    const bool full = c0 + 4 <= C && vec_out;
    int mu[4];
    float k0[4], k1[4], k2[4];
    uint32_t rmax[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // clamped index, select after the load (no branch per channel)
        const int64_t cc = std::min<int64_t>(c0 + i, C - 1);
        const bool ok = c0 + i < C;
        mu[i] = ch[cc].mu;
        if (BWD) {
            const float4 k = reinterpret_cast<const float4*>(coef)[cc];
            k0[i] = ok ? k.x : 0.0f;
            k1[i] = ok ? k.y : 0.0f;
            k2[i] = ok ? k.z : 0.0f;
        } else {
            k0[i] = !ok ? 0.0f : PAR ? par[0][cc] : ch[cc].kappa;
            k1[i] = !ok ? 0.0f : PAR ? par[PAR ? 1 : 0][cc] : ch[cc].beta;
            k2[i] = 0.0f;
        }
        rmax[i] = 0u;
    }
    auto row_out = [&](int64_t m, uint32_t wa, uint32_t wx) {
        int qa[4], qx[4];
        unpack4(wa, qa);
        if (BWD) unpack4(wx, qx);
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (BWD) {
                const float s = (float)sgn(qx[i] - mu[i]);
                v[i] = __fadd_rn(__fadd_rn(__fmul_rn(k0[i], (float)qa[i]), __fmul_rn(k1[i], s)), k2[i]);
                if (c0 + i < C) rmax[i] = std::max(rmax[i], abs_bits(v[i]));
            } else {
                v[i] = __fadd_rn(__fmul_rn(k0[i], (float)(qa[i] - mu[i])), k1[i]);
            }
        }
        float* row = out + m * ld_out + c0;
        if (full) {
            *reinterpret_cast<float4*>(row) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (c0 + i < C) row[i] = v[i];
        }
    };
    if (active) {
        constexpr int U = 8;   // rows in flight per thread
        int64_t m = r0 + lane;
        for (; m + (U - 1) * (int64_t)g.lanes < r1; m += U * (int64_t)g.lanes) {
            uint32_t wa[U], wx[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t mm = m + u * (int64_t)g.lanes;
                wa[u] = *reinterpret_cast<const uint32_t*>(a + mm * lda + c0);
                wx[u] = BWD ? *reinterpret_cast<const uint32_t*>(x + mm * ldx + c0) : 0u;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) row_out(m + u * (int64_t)g.lanes, wa[u], wx[u]);
        }
        for (; m < r1; m += g.lanes)
            row_out(m, *reinterpret_cast<const uint32_t*>(a + m * lda + c0),
                    BWD ? *reinterpret_cast<const uint32_t*>(x + m * ldx + c0) : 0u);
    }
    if (BWD && ranges) {
        const int width = g.qis * 4;
        __syncthreads();
        if (active) {
#pragma unroll
            for (int i = 0; i < 4; ++i) red[lane * width + cl * 4 + i] = rmax[i];
        }
        __syncthreads();
        const int64_t cbase = (int64_t)blockIdx.y * width;
        for (int k = tid; k < width; k += kBnThreads) {
            const int64_t c = cbase + k;
            if (c >= C) continue;
            uint32_t mx = 0u;
            for (int l = 0; l < g.lanes; ++l) mx = std::max(mx, red[l * width + k]);
            ranges[(int64_t)blockIdx.x * C + c] = mx;
        }
    }
}

}  // namespace

int64_t l1bn_range_slabs(int64_t M, int64_t C) { return M > 0 && C > 0 ? quad_geom(M, C).nb : 0; }

int64_t l1bn_part_words(int64_t M, int64_t C) { return 2 * sum_geom(M, C).nb * C; }

hipError_t launch_l1bn_forward(const int8_t* xq, int64_t M, int64_t C, int64_t ld_x, const sq_scale* xs,
                               const float* gamma, const float* beta, float* y, int64_t ld_y, sq_l1bn_channel* ch,
                               sq_l1bn_layer* layer, int32_t* part, hipStream_t s) {
    if (C <= 0) return hipSuccess;
    const BnGeom gs = sum_geom(M, C);
    const QuadGeom ga = quad_geom(M, C);
    const dim3 sum_grid((unsigned)gs.nb, (unsigned)gs.slabs), chan_grid((unsigned)((C + kChanPer - 1) / kChanPer));
    hipLaunchKernelGGL(k_bn_colsum<0>, sum_grid, dim3(kBnThreads), 0, s, xq, ld_x, nullptr, 0, ch, M, C, gs, part);
    hipLaunchKernelGGL(k_bn_chan<0>, chan_grid, dim3(64 * kBnWaves), 0, s, part, gs.nb, M, C, ch, nullptr, nullptr,
                       nullptr, nullptr, nullptr, nullptr);
    hipLaunchKernelGGL(k_bn_colsum<1>, sum_grid, dim3(kBnThreads), 0, s, xq, ld_x, nullptr, 0, ch, M, C, gs, part);
    hipLaunchKernelGGL(k_bn_chan<1>, chan_grid, dim3(64 * kBnWaves), 0, s, part, gs.nb, M, C, ch, nullptr, nullptr,
                       nullptr, nullptr, nullptr, nullptr);
    const bool vec = (ld_y % 4 == 0) && (reinterpret_cast<uintptr_t>(y) % 16 == 0);
    const dim3 apply_grid((unsigned)ga.nb, (unsigned)ga.slabs);
    if (C <= kFuseC) {
        hipLaunchKernelGGL((k_bn_apply<false, true>), apply_grid, dim3(kBnThreads), 0, s, xq, ld_x, nullptr, 0, ch, nullptr,
                           M, C, ga, y, ld_y, vec, nullptr, gamma, beta, xs, layer);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_bn_params, dim3(1), dim3(kParThreads), 0, s, ch, M, C, gamma, beta, xs, layer);
    hipLaunchKernelGGL((k_bn_apply<false, false>), apply_grid, dim3(kBnThreads), 0, s, xq, ld_x, nullptr, 0, ch, nullptr,
                       M, C, ga, y, ld_y, vec, nullptr, nullptr, nullptr, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_l1bn_backward(const int8_t* qg, int64_t ldg, const int8_t* xq, int64_t ld_x, int64_t M, int64_t C,
                                const sq_l1bn_channel* ch, const sq_l1bn_layer* layer, const uint8_t* group,
                                const sq_scale* gscale, float* dx, int64_t ld_dx, float* dgamma, float* dbeta,
                                uint32_t* ranges, int32_t* part, int64_t part_blocks, float* coef, hipStream_t s) {
    if (C <= 0) return hipSuccess;
    const QuadGeom ga = quad_geom(M, C);
    if (part_blocks <= 0) {
        const BnGeom gs = sum_geom(M, C);
        part_blocks = gs.nb;
        hipLaunchKernelGGL(k_bn_colsum<2>, dim3((unsigned)gs.nb, (unsigned)gs.slabs), dim3(kBnThreads), 0, s, qg, ldg, xq,
                           ld_x, ch, M, C, gs, part);
    }
    hipLaunchKernelGGL(k_bn_chan<2>, dim3((unsigned)((C + kChanPer - 1) / kChanPer)), dim3(64 * kBnWaves), 0, s, part,
                       part_blocks, M, C, const_cast<sq_l1bn_channel*>(ch), layer, group, gscale, coef, dgamma, dbeta);
    const bool vec = (ld_dx % 4 == 0) && (reinterpret_cast<uintptr_t>(dx) % 16 == 0);
    hipLaunchKernelGGL(k_bn_apply<true>, dim3((unsigned)ga.nb, (unsigned)ga.slabs), dim3(kBnThreads), 0, s, qg, ldg,
                       xq, ld_x, const_cast<sq_l1bn_channel*>(ch), coef, M, C, ga, dx, ld_dx, vec, ranges, nullptr,
                       nullptr, nullptr, nullptr);
    return hipGetLastError();
}

}  // namespace sq
