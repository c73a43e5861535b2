// ShiftQuant quantizer kernels for gfx950.
//
// Stream-ordered passes (the tensor range r_max is global, so the gradient is
// read twice):
//   k_colmax         per-channel abs-max r_c (Sec. 3.1) as unsigned bit
//                    patterns: coalesced float4 row loads, one maximum per
//                    channel per row slab (plain stores, no atomics) and one
//                    per block
//   finalize         r_max, group ids (power-of-two thresholds, Sec. 3.1),
//                    scales, flags, and the fold layout for dgrad:
//                    k_final_groups over 64-channel groups and, with several
//                    fold windows, k_final_place; k_colmax_reduce before them
//                    for channel ranges that come from the producer of dY
//   quantize         scale, round (ties-to-even or Philox stochastic rounding,
//                    App. B Eq. "sq"), clamp; writes the shift-folded dgrad
//                    operand row-major and the codes transposed: k_quantize8
//                    (8 channels a thread), k_quantize_grid (transposed codes
//                    on the padded pixel grid; k_quantize8 for some widths),
//                    k_quantize (any shape and alignment); per tensor these
//                    also take the scale from the abs-max pass's block maxima
//
// All fp32 arithmetic is IEEE with round-to-nearest-even and no contraction
// (the library is built with -ffp-contract=off and the products below use the
// _rn intrinsics), so the codes are a bit-exact function of the inputs.
#include <algorithm>
#include <type_traits>

#include "sq_internal.h"

namespace sq {

namespace {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): counter-based uniform bits for
// stochastic rounding.  Written independently of any other implementation.
// ---------------------------------------------------------------------------
struct U4 { uint32_t x, y, z, w; };

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;   // one 32x32->64 product each
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
        c = U4{(uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0};
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

__device__ __forceinline__ U4 philox_block(uint64_t blk, const QuantCfg& cfg) {
    return philox4x32_10(U4{(uint32_t)blk, (uint32_t)(blk >> 32), (uint32_t)cfg.offset,
                            (uint32_t)(cfg.offset >> 32)},
                         (uint32_t)cfg.seed, (uint32_t)(cfg.seed >> 32));
}

__device__ __forceinline__ uint32_t pick(const U4& w, int i) {
    return i == 0 ? w.x : (i == 1 ? w.y : (i == 2 ? w.z : w.w));
}

// The 16-bit uniform of the element with logical index idx = m * C + c: one
// Philox block per 8 consecutive indices, half idx % 2 (low first) of word
// (idx / 2) % 4.
__device__ __forceinline__ uint32_t sr_uniform16(uint64_t idx, const QuantCfg& cfg) {
    return (pick(philox_block(idx >> 3, cfg), (int)((idx >> 1) & 3u)) >> (16u * (uint32_t)(idx & 1u))) & 0xFFFFu;
}

// One code: v = fl(x * s); round; clamp to [-Q, Q].  u16 is the 16-bit
// uniform used only by stochastic rounding.
template <bool SR>
__device__ __forceinline__ int quant_one(float x, float s, float Qf, uint32_t u16) {
    const float v = __fmul_rn(x, s);
    float qf;
    if (SR) {
        const float l = floorf(v);
        const float f = __fsub_rn(v, l);
        qf = ((float)u16 < __fmul_rn(f, 65536.0f)) ? __fadd_rn(l, 1.0f) : l;
    } else {
        qf = rintf(v);
    }
    qf = fminf(fmaxf(qf, -Qf), Qf);
    return (int)qf;
}

// The same code as a float (an exact integer in [-Q, Q]).
template <bool SR>
__device__ __forceinline__ float quant_onef(float x, float s, float Qf, uint32_t u16) {
    const float v = __fmul_rn(x, s);
    float qf;
    if (SR) {
        const float l = floorf(v);
        const float f = __fsub_rn(v, l);
        qf = ((float)u16 < __fmul_rn(f, 65536.0f)) ? __fadd_rn(l, 1.0f) : l;
    } else {
        qf = rintf(v);
    }
    return fminf(fmaxf(qf, -Qf), Qf);
}

__device__ __forceinline__ uint32_t absbits(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

// ---------------------------------------------------------------------------
// Per-channel abs-max, first level.  The rows are cut into slabs; block
// (chunk, slab) reduces its slab for the chunk's channels and stores the
// slab maxima to partial[slab * C + c] (plain stores: same-address atomics
// from many blocks serialise, so the slabs are combined in a second step).
// Thread (rl, tc) covers VEC channels starting at (chunk * tpr + tc) * VEC and
// rows rl, rl + kColThreads / tpr, ... of the slab, 8 loads in flight.
// NT: nontemporal loads, for gradients larger than the last-level cache (see
// launch_colmax).
// ---------------------------------------------------------------------------
constexpr uint64_t kLastLevelCacheBytes = 256ull << 20;   // MI355X last-level (memory-side) cache
constexpr int kColThreads = 512;
typedef float v4f __attribute__((ext_vector_type(4)));

template <int VEC, bool NT>
__global__ __launch_bounds__(kColThreads) void k_colmax(const float* __restrict__ x, int64_t M, int64_t C,
                                                        int64_t ld, int tpr, int64_t rows_per_slab,
                                                        uint32_t* __restrict__ partial,
                                                        uint32_t* __restrict__ block_max) {
    __shared__ uint32_t red[kColThreads * VEC];
    const int tid = threadIdx.x;
    const int nrl = kColThreads / tpr;
    const int rl = tid / tpr, tc = tid % tpr;
    const int64_t c0 = ((int64_t)blockIdx.x * tpr + tc) * VEC;
    const int64_t m_begin = (int64_t)blockIdx.y * rows_per_slab;
    const int64_t m_end = min(M, m_begin + rows_per_slab);
    uint32_t best[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) best[j] = 0u;

    if (c0 < C) {
        int64_t m = m_begin + rl;
        if constexpr (VEC == 4) {
            if (c0 + 4 <= C) {
                // batches of 8 rows, the next batch in flight while one is
                // reduced.  Rows past the slab re-read its last row (the
                // maximum is unchanged): no branch between the loads, so the
                // wait before a batch's reduction leaves the next batch in flight.
                const int64_t step = nrl;
                auto load8 = [&](int64_t mm, float4 (&v)[8]) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int64_t row = min(mm + u * step, m_end - 1);
                        if (NT) {
                            const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(x + row * ld + c0));
                            v[u] = make_float4(t.x, t.y, t.z, t.w);
                        } else {
                            v[u] = *reinterpret_cast<const float4*>(x + row * ld + c0);
                        }
                    }
                };
                auto reduce8 = [&](const float4 (&v)[8]) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        best[0] = max(best[0], absbits(v[u].x));
                        best[1] = max(best[1], absbits(v[u].y));
                        best[2] = max(best[2], absbits(v[u].z));
                        best[3] = max(best[3], absbits(v[u].w));
                    }
                };
                if (m < m_end) {
                    float4 va[8], vb[8];
                    load8(m, va);
                    for (; m < m_end; m += 16 * step) {
                        load8(m + 8 * step, vb);
                        reduce8(va);
                        load8(m + 16 * step, va);
                        reduce8(vb);
                    }
                }
                m = m_end;
            }
        }
        for (; m < m_end; m += nrl) {   // scalar path (and the ragged last vector)
#pragma unroll
            for (int j = 0; j < VEC; ++j)
                if (c0 + j < C) best[j] = max(best[j], absbits(x[m * ld + c0 + j]));
        }
    }
#pragma unroll
    for (int j = 0; j < VEC; ++j) red[tid * VEC + j] = best[j];
    __syncthreads();
    if (rl == 0 && c0 < C) {
        for (int r = 1; r < nrl; ++r)
#pragma unroll
            for (int j = 0; j < VEC; ++j) best[j] = max(best[j], red[(r * tpr + tc) * VEC + j]);
        uint32_t* dst = partial + (int64_t)blockIdx.y * C + c0;
#pragma unroll
        for (int j = 0; j < VEC; ++j)
            if (c0 + j < C) dst[j] = best[j];
    }
    // the block's maximum over its channels (the rl == 0 threads, tid < tpr,
    // all in wave 0), so that r_max needs no pass over the channel ranges
    if (block_max && tid < 64) {
        uint32_t mb = 0u;
        if (rl == 0 && c0 < C)
#pragma unroll
            for (int j = 0; j < VEC; ++j)
                if (c0 + j < C) mb = max(mb, best[j]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mb = max(mb, (uint32_t)__shfl_xor((int)mb, o, 64));
        if (tid == 0) block_max[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = mb;
    }
}

// max over the S slab maxima of channel c (8 loads in flight per thread)
__device__ __forceinline__ uint32_t reduce_slabs(const uint32_t* __restrict__ partial, int64_t S, int64_t C,
                                                 int64_t c) {
    uint32_t a[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    int64_t s = 0;
    for (; s + 8 <= S; s += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = max(a[u], partial[(s + u) * C + c]);
    }
    for (; s < S; ++s) a[0] = max(a[0], partial[s * C + c]);
#pragma unroll
    for (int u = 1; u < 8; ++u) a[0] = max(a[0], a[u]);
    return a[0];
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}

// ---------------------------------------------------------------------------
// Second level of the abs-max.  A block of NW waves takes kFinCh = 64
// consecutive channels and reads its slab maxima (slabs s0 <= s < s1) with 8
// loads in flight per thread: four rows of 64 channels per wave and 16-byte
// load where the rows are aligned, else one row per wave (a 256-byte segment,
// a channel per lane).  The waves combine in LDS; the result is valid in wave
// 0, lane c holding channel c.  NW = 0, for many channels in at most 8 slabs:
// every wave of the block takes 64 channels of its own and all of their slabs.
// ---------------------------------------------------------------------------
constexpr int kFinCh = 64, kFinWaves = 16, kWideWaves = 4;
constexpr int64_t kFinRows = 8 * 4 * kFinWaves;   // slabs that a block reads in one batch of 16-byte loads
template <int NW>
constexpr int kFinThreadsOf = 64 * (NW ? NW : kWideWaves);

// the 64-channel group of this thread's wave
template <int NW>
__device__ __forceinline__ int64_t fin_group() {
    return NW ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * kWideWaves + (threadIdx.x >> 6);
}

__device__ __forceinline__ uint4 max4(const uint4& a, const uint4& b) {
    return make_uint4(max(a.x, b.x), max(a.y, b.y), max(a.z, b.z), max(a.w, b.w));
}

template <int NW>
__device__ __forceinline__ uint32_t slab_max64(const uint32_t* partial, int64_t s0, int64_t s1, int64_t C,
                                               uint32_t (*lanes)[kFinCh]) {
    const int ch = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t c = fin_group<NW>() * kFinCh + ch;
    constexpr int U = 8;
    // the rows past the last slab are clamped to it, so the loads issue back
    // to back (a maximum does not mind a repeated row)
    if (NW && (C & 3) == 0 && (reinterpret_cast<uintptr_t>(partial) & 15) == 0) {
        constexpr int step = 4 * (NW ? NW : 1);
        const int q = threadIdx.x & 15;
        const int64_t cq = fin_group<NW>() * kFinCh + 4 * q;
        uint4 r = make_uint4(0u, 0u, 0u, 0u);
        if (cq < C) {
            for (int64_t sl = s0 + (threadIdx.x >> 4); sl < s1; sl += U * step) {
                uint4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[u] = *reinterpret_cast<const uint4*>(partial + min(sl + u * step, s1 - 1) * C + cq);
#pragma unroll
                for (int u = 0; u < U; ++u) r = max4(r, v[u]);
            }
        }
#pragma unroll
        for (int o = 16; o < 64; o <<= 1)
            r = max4(r, make_uint4((uint32_t)__shfl_xor((int)r.x, o, 64), (uint32_t)__shfl_xor((int)r.y, o, 64),
                                   (uint32_t)__shfl_xor((int)r.z, o, 64), (uint32_t)__shfl_xor((int)r.w, o, 64)));
        if (ch < 16) *reinterpret_cast<uint4*>(&lanes[w][4 * q]) = r;
    } else {
        constexpr int step = NW ? NW : 1;
        uint32_t r = 0u;
        if (c < C) {
            uint32_t v[U] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
            int64_t sl = s0 + (NW ? w : 0);
            for (; sl + (U - 1) * step < s1; sl += U * step) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = max(v[u], partial[(sl + u * step) * C + c]);
            }
            if (sl < s1) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = max(v[u], partial[min(sl + u * step, s1 - 1) * C + c]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) r = max(r, v[u]);
        }
        if constexpr (NW == 0) return r;
        lanes[w][ch] = r;
    }
    __syncthreads();
    uint32_t r = 0u;
    if (w == 0) {
#pragma unroll
        for (int i = 0; i < NW; ++i) r = max(r, lanes[i][ch]);
    }
    return r;
}

// Channel ranges over the slabs [y per, (y + 1) per), y = blockIdx.y, in
// rbits[y][c], and the maximum of each 64 channels in bmax[y][group], for slab
// maxima that come from the producer of dY (no block maxima with them).
template <int NW>
__global__ __launch_bounds__(kFinThreadsOf<NW>) void k_colmax_reduce(const uint32_t* __restrict__ partial, int64_t S,
                                                               int64_t per, int64_t C, uint32_t* __restrict__ rbits,
                                                               uint32_t* __restrict__ bmax, int64_t nb) {
    __shared__ __attribute__((aligned(16))) uint32_t lanes[NW ? NW : 1][kFinCh];
    const int64_t y = blockIdx.y, grp = fin_group<NW>();
    uint32_t r = slab_max64<NW>(partial, y * per, min(S, (y + 1) * per), C, lanes);
    if (NW ? threadIdx.x >= 64 : grp >= nb) return;
    const int64_t c = grp * kFinCh + (threadIdx.x & 63);
    if (c < C) rbits[y * C + c] = r;
    r = wave_max(r);
    if ((threadIdx.x & 63) == 0) bmax[y * nb + grp] = r;
}

// Group of a channel: the smallest j < N_G - 1 with r_c * 2^(j+1) > r_max,
// else N_G - 1.  Products with powers of two are exact (an overflow to +Inf
// still compares correctly), so this equals the threshold test
// r_c > r_max * 2^-(j+1) of Sec. 3.1.
__device__ __forceinline__ int group_of(float r_c, float r_max, int num_groups) {
    for (int j = 0; j < num_groups - 1; ++j)
        if (__fmul_rn(r_c, pow2f(j + 1)) > r_max) return j;
    return num_groups - 1;
}

__device__ __forceinline__ sq_scale make_scale(uint32_t mb, float Qf) {
    const float r_max = __uint_as_float(mb);
    uint32_t flags = 0u;
    if (mb >= 0x7F800000u) flags = SQ_FLAG_NONFINITE;
    else if (r_max < pow2f(-96)) flags = SQ_FLAG_ZERO;
    sq_scale s;
    s.r_max = r_max;
    s.inv = flags ? 0.0f : __fdiv_rn(Qf, r_max);
    s.step = flags ? 0.0f : __fdiv_rn(r_max, Qf);
    s.flags = flags;
    return s;
}

// ---------------------------------------------------------------------------
// Finalize of the gradient quantizer, over blocks of kFinCh channels:
//   k_final_groups  r_max (the maximum of the abs-max pass's block maxima, or
//     of the block's own channels when there is one block), the scale and
//     flags, and the group of each of the block's channels; with one fold
//     window the descriptors and the header too, else the block's count of
//     channels per shift;
//   k_final_place   (several windows) every wave plans the windows from the
//     summed counts (the same plan everywhere), takes its region offsets from
//     the counts of the 64-channel groups before it, and ranks its appended
//     channels with wave ballots; block 0 writes the header and the padding.
// Both are bound by latency: a launch of this size takes 2.5 to 4 us whatever
// it does, so the work is spread until its own chain is shorter than that.
// One block reading every slab maximum and planning on one thread took 17 to
// 22 us (several windows, 768 channels x 169 slabs); these two take 4.7 + 4.8 us
// in a kernel trace of 16384 x 768 activations.
// ---------------------------------------------------------------------------
template <int NW>
__global__ __launch_bounds__(kFinThreadsOf<NW>) void k_final_groups(const uint32_t* partial, int64_t S,
                                                              const uint32_t* block_max, int64_t nbm,
                                                              int64_t C, QuantCfg cfg, uint8_t* __restrict__ group,
                                                              sq_scale* __restrict__ scale,
                                                              int32_t* __restrict__ layout, int64_t ext_max,
                                                              int32_t* hist, int hist_ld) {
    constexpr int nt = kFinThreadsOf<NW>;
    __shared__ __attribute__((aligned(16))) uint32_t lanes[NW ? NW : 1][kFinCh];
    __shared__ uint32_t wmax[nt / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t grp = fin_group<NW>();
    uint32_t mb = 0u;
    if (gridDim.x > 1) {
        if (nbm <= nt) {
            if (tid < nbm) mb = block_max[tid];
        } else {
            for (int64_t i = tid; i < nbm; i += 8 * nt) {   // clamped index: the loads issue back to back
#pragma unroll
                for (int u = 0; u < 8; ++u) mb = max(mb, block_max[min(i + u * nt, nbm - 1)]);
            }
        }
        mb = wave_max(mb);
        if (lane == 0) wmax[tid >> 6] = mb;
    }
    const uint32_t rb = slab_max64<NW>(partial, 0, S, C, lanes);   // ends in a barrier, which covers wmax too
    if (NW == 0) __syncthreads();
    if (NW ? tid >= 64 : grp * kFinCh >= C) return;
    if (gridDim.x > 1) mb = wave_max(lane < nt / 64 ? wmax[lane] : 0u);
    else mb = wave_max(rb);
    const sq_scale sc = make_scale(mb, (float)cfg.Q);
    if (grp == 0 && lane == 0) *scale = sc;
    const int Sh = cfg.num_groups - 1;   // largest shift
    const int64_t c = grp * kFinCh + lane;
    int sh = -1;
    if (c < C) {
        const int g = sc.flags ? Sh : group_of(__uint_as_float(rb), sc.r_max, cfg.num_groups);
        group[c] = (uint8_t)g;
        sh = Sh - g;
    }
    if (ext_max == 0) {
        // every shift fits int8 (N_G - 1 <= T): one window at base 0, the
        // code of channel c stored as code << sh_c in its own column
        if (c < C) layout[kLayoutHeader + c] = sh;
        if (grp == 0 && lane < kLayoutHeader) {
            int v = 0;
            if (lane == kLayNR) v = 1;
            else if (lane == kLayBase) v = (int)fold_ext_base(C);
            else if (lane > kLayStart && lane < kLayStart + kMaxRegions) v = 0x7FFFFFFF;
            layout[lane] = v;
        }
        return;
    }
    int n = 0;
#pragma unroll
    for (int q = 0; q < kMaxRegions; ++q) {
        const int m = __popcll(__ballot(sh == q));
        if (lane == q) n = m;
    }
    if (lane < kMaxRegions) hist[grp * hist_ld + lane] = n;
}

// Shift windows of the fold (the layout is documented in sq_internal.h), held
// across the lanes of a wave; every lane must call it.  Window of shift value
// s: key 0 for the main window [B*, B* + T], key j > 0 for [B* + j (T + 1),
// ...] above it, key -j for the j-th window below it (its base clipped at 0).
// Regions are the non-empty windows (and always the main one) in descending
// key order, which is descending base.  Lane k holds the window of key
// k - kKey0; lane s < kMaxRegions the window lane `win` of shift s.
constexpr int kKey0 = kMaxRegions - 1, kKeys = 2 * kMaxRegions - 1;
struct WavePlan {
    int win;                 // lane s: lane of the window of shift s
    int cnt, width, base;    // channels, padded columns and lowest shift of this lane's window
    int ext_start, flat;     // first appended column (other than the main window), first flat K column
    int before;              // appended channels of this window in earlier 64-channel groups
    uint32_t present;        // windows that are regions, a bit per lane (uniform)
    int bstar;
};

__device__ __forceinline__ int lane_val(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

// n, nb: channels at shift `lane` in all groups and in the groups before the caller's
__device__ __forceinline__ WavePlan wave_fold_plan(int n, int nb, int S, int T, int64_t C) {
    const int lane = threadIdx.x & 63;
    WavePlan P;
    n = lane <= S ? n : 0;
    // the window [B, B + T] holding the most channels (lowest B on ties)
    int c = 0;
#pragma unroll
    for (int j = 0; j < kMaxRegions; ++j) {
        const int v = __shfl(n, lane + j, 64);
        c += j <= T && lane + j <= S ? v : 0;
    }
    int best = lane <= max(S - T, 0) ? c * kMaxRegions + (kMaxRegions - 1 - lane) : -1;
#pragma unroll
    for (int o = 1; o < kMaxRegions; o <<= 1) best = max(best, __shfl_xor(best, o, 64));
    P.bstar = kMaxRegions - 1 - (lane_val(best, 0) & (kMaxRegions - 1));
    const int d = lane - P.bstar;
    P.win = kKey0 + (d >= 0 ? (int)((uint32_t)d / (uint32_t)(T + 1)) : -1 - (int)((uint32_t)(-1 - d) / (uint32_t)(T + 1)));
    P.cnt = P.before = 0;
#pragma unroll
    for (int s = 0; s < kMaxRegions; ++s) {
        const bool in = s <= S && lane_val(P.win, s) == lane;
        P.cnt += in ? lane_val(n, s) : 0;
        P.before += in ? lane_val(nb, s) : 0;
    }
    const int key = lane - kKey0;
    const bool here = lane < kKeys && (P.cnt > 0 || key == 0);
    P.present = (uint32_t)__ballot(here);
    P.base = max(0, P.bstar + key * (T + 1));
    P.width = here ? (int)round_up(key == 0 ? C : P.cnt, kFoldPad) : 0;
    P.ext_start = P.flat = 0;
#pragma unroll
    for (int k = 0; k < kKeys; ++k) {
        const int w = lane_val(P.width, k);
        P.flat += k > lane ? w : 0;
        P.ext_start += k > lane && k != kKey0 ? w : 0;
    }
    return P;
}

constexpr int kPlaceThreads = 256;   // four 64-channel groups, one per wave

__global__ __launch_bounds__(kPlaceThreads) void k_final_place(const uint8_t* __restrict__ group,
                                                               const int32_t* __restrict__ hist, int hist_ld,
                                                               int64_t nb, int64_t C, QuantCfg cfg,
                                                               int32_t* __restrict__ layout, int64_t ext_max) {
    __shared__ int tot[kPlaceThreads / 64][kMaxRegions], bef[kPlaceThreads / 64][kMaxRegions];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int Sh = cfg.num_groups - 1;
    const int64_t first = (int64_t)blockIdx.x * (kPlaceThreads / 64);   // this block's first 64-channel group
    const int64_t c = first * kFinCh + tid;
    const int g = c < C ? (int)group[c] : Sh;
    // channels per shift: all groups, and the groups before this block's
    // (thread t sums shift t % 8 over the groups t / 8 mod 32), then those of
    // the earlier waves
    int vt = 0, vb = 0;
    constexpr int64_t kStep = kPlaceThreads / kMaxRegions;
    if (nb <= kStep) {
        const int64_t b = tid / kMaxRegions;
        if (b < nb) {
            vt = hist[b * hist_ld + tid % kMaxRegions];
            vb = b < first ? vt : 0;
        }
    } else {
        for (int64_t b0 = tid / kMaxRegions; b0 < nb; b0 += 8 * kStep) {   // 8 loads in flight
            int h[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) h[u] = hist[min(b0 + u * kStep, nb - 1) * hist_ld + tid % kMaxRegions];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t b = b0 + u * kStep;
                vt += b < nb ? h[u] : 0;
                vb += b < min(first, nb) ? h[u] : 0;
            }
        }
    }
    int vw = 0;
    for (int w = 0; w < wave; ++w)
        if (lane < kMaxRegions && first + w < nb) vw += hist[(first + w) * hist_ld + lane];
#pragma unroll
    for (int o = kMaxRegions; o < 64; o <<= 1) {
        vt += __shfl_xor(vt, o, 64);
        vb += __shfl_xor(vb, o, 64);
    }
    if (lane < kMaxRegions) {
        tot[wave][lane] = vt;
        bef[wave][lane] = vb;
    }
    __syncthreads();
    vt = 0;
    if (lane < kMaxRegions) {
#pragma unroll
        for (int w = 0; w < kPlaceThreads / 64; ++w) {
            vt += tot[w][lane];
            vw += bef[w][lane];
        }
    }
    const WavePlan P = wave_fold_plan(vt, vw, Sh, cfg.T, C);
    int32_t* ext = layout + kLayoutHeader;
    int32_t* desc = ext + ext_max;
    const int sh = Sh - g;
    const int k = __shfl(P.win, sh, 64);   // this channel's window
    const bool is_ext = c < C && k != kKey0;
    int rank = 0;
    for (uint32_t m = P.present & ~(1u << kKey0); m; m &= m - 1) {
        const int q = __builtin_ctz(m);
        const uint64_t same = __ballot(is_ext && k == q);
        if (k == q) rank = __popcll(same & ((1ull << lane) - 1ull));
    }
    const int base = __shfl(P.base, k, 64), start = __shfl(P.ext_start + P.before, k, 64);
    if (c < C) {
        int pos = -1;
        if (is_ext) {
            pos = start + rank;
            ext[pos] = (int32_t)c;
        }
        desc[c] = ((pos + 1) << 4) | (sh - base);
    }
    if (blockIdx.x != 0 || wave != 0) return;
    // region padding (fewer than 64 columns each)
    for (uint32_t m = P.present & ~(1u << kKey0); m; m &= m - 1) {
        const int q = __builtin_ctz(m);
        const int i = lane_val(P.cnt, q) + lane;
        if (i < lane_val(P.width, q)) ext[lane_val(P.ext_start, q) + i] = -1;
    }
    // header: words 0 .. 7, then region r's start and shift by its window's lane
    const int nr = __popc(P.present);
    int D = 0, H = 0;
#pragma unroll
    for (int q = 0; q < kKeys; ++q) {
        const int w = lane_val(P.width, q);
        D += q != kKey0 ? w : 0;
        H += q > kKey0 ? w : 0;
    }
    const int F = lane_val(P.base, __builtin_ctz(P.present));
    if (lane < kLayoutHeader) {
        const bool in_start = lane >= kLayStart && lane < kLayStart + kMaxRegions;
        int v = 0;
        if (lane == kLayNR) v = nr;
        else if (lane == kLayD) v = D;
        else if (lane == kLayBase) v = (int)fold_ext_base(C);
        else if (lane == kLayF) v = F;
        else if (lane == kLayH) v = H;
        else if (in_start) v = 0x7FFFFFFF;
        // region starts and shifts below nr are written by the window lanes
        const bool mine = (in_start && lane - kLayStart < nr) || (lane > kLayShift && lane - kLayShift < nr);
        if (!mine) layout[lane] = v;
    }
    const uint32_t above = lane < kKeys ? P.present >> (lane + 1) : 0u;   // regions before this lane's
    const int prev = __shfl(P.base, above ? lane + 1 + __builtin_ctz(above) : lane, 64);
    if (lane < kKeys && (P.present >> lane & 1u)) {
        const int r = __popc(above);
        layout[kLayStart + r] = P.flat;
        if (r > 0) layout[kLayShift + r] = prev - P.base;
    }
}

// Scale of a per-tensor quantization, taken by every block of the quantize
// pass from the abs-max pass's block maxima (at most about 520 words up to
// 131,072 channels, or 32,768 where the rows are not 16-byte aligned, then one per
// 256 or 64 channels); block 0 writes it out.  A launch of
// its own for this took 2.1 to 3.9 us and a gap.  In two parts, so that the
// block maxima are loaded first and combined while the tile's rows are in
// flight.  sh: 4 words of LDS.
__device__ __forceinline__ uint32_t tensor_max_load(const TensorMax& tm) {
    const int64_t last = tm.n - 1;
    uint32_t mb = max(tm.block_max[min((int64_t)threadIdx.x, last)], tm.block_max[min((int64_t)threadIdx.x + 256, last)]);
    for (int64_t i = threadIdx.x + 512; i < tm.n; i += 256) mb = max(mb, tm.block_max[i]);
    return mb;
}

__device__ __forceinline__ sq_scale tensor_scale(const TensorMax& tm, uint32_t mb, float Qf, uint32_t* sh) {
    mb = wave_max(mb);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mb;
    __syncthreads();
    const sq_scale sc = make_scale(max(max(sh[0], sh[1]), max(sh[2], sh[3])), Qf);
    if (blockIdx.x == 0 && threadIdx.x == 0) *tm.scale = sc;
    return sc;
}

// The maximum of n block maxima into the first of them (one block), where they
// are too many for every block of the quantize pass to read.
__global__ __launch_bounds__(1024) void k_block_max(uint32_t* bm, int64_t n) {
    __shared__ uint32_t sh[16];
    uint32_t mb = 0u;
    for (int64_t i = threadIdx.x; i < n; i += 1024) mb = max(mb, bm[i]);
    mb = wave_max(mb);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mb;
    __syncthreads();   // every wave has read its words
    if (threadIdx.x < 64) {
        mb = wave_max(sh[threadIdx.x & 15]);
        if (threadIdx.x == 0) bm[0] = mb;
    }
}

// An empty tensor, which has no quantize pass.
__global__ void k_empty_scale(int Q, sq_scale* __restrict__ scale) { *scale = make_scale(0u, (float)Q); }

// ---------------------------------------------------------------------------
// Quantize.  A block quantizes tiles of TR rows x TC channels (64 or 128 each,
// smaller where the tensor would give too few tiles to fill the chip),
// striding over the tiles; neighbouring
// channel tiles of a row tile go to consecutive blocks.  Thread (rq, cq)
// handles, in each pass over the tile, the 4 consecutive rows 4 rq .. 4 rq + 3
// of the channel quad 4 cq .. 4 cq + 3: one 16-byte load per row, the row's 4
// shift-folded codes as one 4-byte store into q_fold (a wave writes whole
// row segments), and each channel's 4 codes as one word into an LDS tile
// [channel][row], from which the block writes q_t as 16-byte chunks, so a
// 128-row tile completes whole 128-byte lines of q_t.  Low register use keeps many
// waves per SIMD in flight to hide the memory latency.
// ---------------------------------------------------------------------------
constexpr int kBlock = 256;

template <int TC, int kTR, int VEC, bool SR>
__global__ __launch_bounds__(kBlock) void k_quantize(const float* __restrict__ x, int64_t M, int64_t C,
                                                     int64_t ld, const uint8_t* __restrict__ group,
                                                     const sq_scale* __restrict__ scale, QuantCfg cfg,
                                                     int8_t* __restrict__ q_fold, int64_t ld_fold,
                                                     int8_t* __restrict__ q_t, int64_t ld_t,
                                                     const int32_t* __restrict__ desc, int64_t ext_base,
                                                     PadGrid pg, int tiled, TensorMax tm) {
    constexpr int QD = TC / 4;            // channel quads per tile
    constexpr int RQ = kBlock / QD;       // row quads per pass
    constexpr int RP = 4 * RQ;            // rows per pass
    constexpr int PASSES = kTR / RP;
    constexpr int TW = kTR / 4 + 1;       // LDS words per channel row (padded)
    __shared__ uint32_t tq[TC * TW];
    const int tid = threadIdx.x, cq = tid % QD, rq = tid / QD;
    const int64_t ctiles = (C + TC - 1) / TC, rtiles = (M + kTR - 1) / kTR;

    const float Qf = (float)cfg.Q;
    __shared__ uint32_t sh_max[4];
    const sq_scale sc = tm.block_max ? tensor_scale(tm, tensor_max_load(tm), Qf, sh_max) : *scale;
    const bool zero = sc.flags != 0u;
    // C a multiple of 8: the channel quads 2k and 2k + 1 of a row share one
    // Philox block; the two lanes (adjacent) each run it for two of their four
    // rows and swap the halves the other needs
    const bool sr_pair = SR && ((C & 7) == 0);
    const int par = cq & 1;

    for (int64_t tile = blockIdx.x; tile < ctiles * rtiles; tile += gridDim.x) {
        const int64_t ct = tile % ctiles, rt = tile / ctiles;
        const int64_t c0 = ct * TC + 4 * cq, m_tile = rt * kTR;
        const bool full_vec = VEC == 4 && c0 + 4 <= C;
        float s[4];
        int t[4], pos[4];   // fold: code << t in main column c (pos < 0) or appended column pos
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t c = c0 + j;
            const int g = (group && c < C) ? (int)group[c] : 0;
            s[j] = __fmul_rn(sc.inv, pow2f(g));
            const int d = (desc && c < C) ? desc[c] : 0;
            t[j] = d & 15;
            pos[j] = (d >> 4) - 1;
        }
        // passes unrolled, except under stochastic rounding (its Philox words
        // make an unrolled body too large for the compiler)
        constexpr int kUnrollPasses = SR ? 1 : PASSES;
#pragma unroll kUnrollPasses
        for (int p = 0; p < PASSES; ++p) {
            const int r0 = p * RP + 4 * rq;   // first of this thread's rows within the tile
            float v[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t m = m_tile + r0 + i;
                v[i][0] = v[i][1] = v[i][2] = v[i][3] = 0.f;
                if (m < M && c0 < C) {
                    if (full_vec) {
                        const float4 f = *reinterpret_cast<const float4*>(x + m * ld + c0);
                        v[i][0] = f.x; v[i][1] = f.y; v[i][2] = f.z; v[i][3] = f.w;
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (c0 + j < C) v[i][j] = x[m * ld + c0 + j];
                    }
                }
            }
            uint32_t colw[4] = {0u, 0u, 0u, 0u};   // channel j: rows r0 .. r0 + 3, little-endian
            // this lane's two Philox words (its quad's 4 halves) for each of its 4 rows
            uint32_t sw[4][2];
            if (SR && sr_pair) {
                const int64_t cpair = c0 & ~(int64_t)7;
                uint32_t mine[2][4];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int64_t m = m_tile + r0 + 2 * par + h;
                    const U4 w = philox_block((uint64_t)(m * C + cpair) >> 3, cfg);
                    mine[h][0] = w.x; mine[h][1] = w.y; mine[h][2] = w.z; mine[h][3] = w.w;
                }
                // own rows 2 par + h: words 2 par, 2 par + 1; the partner's rows
                // come through a lane swap of the words 2 par, 2 par + 1 it computed
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const uint32_t give = mine[h][2 * (1 - par) + k];
                        const uint32_t got = (uint32_t)__shfl_xor((int)give, 1, 64);
                        sw[2 * par + h][k] = mine[h][2 * par + k];
                        sw[2 * (1 - par) + h][k] = got;
                    }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t m = m_tile + r0 + i;
                uint32_t u[4] = {0u, 0u, 0u, 0u};
                if (SR && m < M && c0 < C) {
                    if (sr_pair) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) u[j] = (sw[i][j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (c0 + j < C) u[j] = sr_uniform16((uint64_t)(m * C + c0 + j), cfg);
                    }
                }
                int code[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    code[j] = (zero || m >= M || c0 + j >= C) ? 0 : quant_one<SR>(v[i][j], s[j], Qf, u[j]);
                    colw[j] |= (uint32_t)(uint8_t)code[j] << (8 * i);
                }
                if (q_fold && m < M && c0 < C && !tiled) {
                    int8_t* row = q_fold + m * ld_fold;
                    uint32_t word = 0u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t f = (uint32_t)(uint8_t)(code[j] * (1 << t[j]));
                        if (pos[j] < 0) word |= f << (8 * j);
                        else if (c0 + j < C) row[ext_base + pos[j]] = (int8_t)f;
                    }
                    if (c0 + 4 <= C) {
                        *reinterpret_cast<uint32_t*>(row + c0) = word;
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (c0 + j < C) row[c0 + j] = (int8_t)(word >> (8 * j));
                    }
                } else if (q_fold && m < M && c0 < ext_base && tiled) {
                    // tile-major: the quad's 4 bytes are contiguous; codes of
                    // channels >= C (K padding of the main columns) are 0
                    uint32_t word = 0u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t f = (uint32_t)(uint8_t)(code[j] * (1 << t[j]));
                        if (pos[j] < 0) word |= f << (8 * j);
                        else if (c0 + j < C) q_fold[tiled_off(m, ext_base + pos[j], ld_fold)] = (int8_t)f;
                    }
                    *reinterpret_cast<uint32_t*>(q_fold + tiled_off(m, c0, ld_fold)) = word;
                }
            }
            if (q_t) {
#pragma unroll
                for (int j = 0; j < 4; ++j) tq[(4 * cq + j) * TW + r0 / 4] = colw[j];
            }
        }
        if (q_t) {
            __syncthreads();
            // channel row ch of the tile: kTR bytes = kTR / 16 chunks of 16
            // bytes; this thread writes chunk `part` of the channel rows ch0,
            // ch0 + kBlock / CPR, ..., so its pixels (and their place on a
            // padded grid) are the same for every row it writes
            constexpr int CPR = kTR / 16;
            static_assert((TC * CPR) % kBlock == 0 && kBlock % CPR == 0, "whole passes over the tile");
            const int part = tid % CPR, ch0 = tid / CPR;
            const int64_t m = m_tile + 16 * part;
            // padded pixel grid: pixel m = (n, oh, ow) at n HpWp + oh Wp + ow;
            // 16 pixels in one image row as one 16-byte store, else two 8-byte
            // halves (which never cross an image row when Wo % 8 == 0)
            const bool grid_fast = pg.Wo && pg.Wo % 8 == 0 && (pg.off & 7) == 0 && m + 16 <= M;
            int64_t d0 = 0, d1 = 0;
            bool whole = false;
            if (grid_fast) {
                const uint32_t m0 = (uint32_t)m;
                const uint32_t n = m0 / pg.HoWo, rem = m0 - n * pg.HoWo, oh = rem / pg.Wo;
                const uint32_t ow = rem - oh * pg.Wo;
                d0 = (int64_t)n * pg.HpWp + (int64_t)oh * pg.Wp + ow + pg.off;
                whole = ow + 16 <= pg.Wo && (d0 & 15) == 0;
                const uint32_t mh = m0 + 8;
                const uint32_t n1 = mh / pg.HoWo, rem1 = mh - n1 * pg.HoWo, oh1 = rem1 / pg.Wo;
                d1 = (int64_t)n1 * pg.HpWp + (int64_t)oh1 * pg.Wp + (rem1 - oh1 * pg.Wo) + pg.off;
            }
            // kept rolled: unrolled, the 64-channel tiles measured 1.5 us slower
#pragma unroll 1
            for (int it = 0; it < TC * CPR / kBlock; ++it) {
                const int ch = ch0 + it * (kBlock / CPR);
                const int64_t c = ct * TC + ch;
                if (tiled) {
                    // tile-major: 16 codes of a channel row are contiguous;
                    // rows past M hold 0 (K padding up to a multiple of 64)
                    if (c < C && m < round_up(M, 64)) {
                        const uint32_t* src = &tq[ch * TW + 4 * part];
                        *reinterpret_cast<uint4*>(q_t + tiled_off(c, m, ld_t)) =
                            make_uint4(src[0], src[1], src[2], src[3]);
                    }
                    continue;
                }
                if (c >= C || m >= M) continue;
                const uint32_t* src = &tq[ch * TW + 4 * part];
                int8_t* row = q_t + c * ld_t;
                if (grid_fast) {
                    if (whole) {
                        *reinterpret_cast<uint4*>(row + d0) = make_uint4(src[0], src[1], src[2], src[3]);
                    } else {
                        *reinterpret_cast<uint2*>(row + d0) = make_uint2(src[0], src[1]);
                        *reinterpret_cast<uint2*>(row + d1) = make_uint2(src[2], src[3]);
                    }
                } else if (pg.Wo) {
                    for (int i = 0; i < 16 && m + i < M; ++i) {
                        const uint32_t mi = (uint32_t)(m + i);
                        const uint32_t n = mi / pg.HoWo, rem = mi - n * pg.HoWo, oh = rem / pg.Wo;
                        const uint32_t ow = rem - oh * pg.Wo;
                        row[(int64_t)n * pg.HpWp + (int64_t)oh * pg.Wp + ow + pg.off] =
                            (int8_t)(src[i / 4] >> (8 * (i % 4)));
                    }
                } else if (m + 16 <= M) {
                    *reinterpret_cast<uint4*>(row + m) = make_uint4(src[0], src[1], src[2], src[3]);
                } else {
                    for (int i = 0; i < (int)(M - m); ++i) row[m + i] = (int8_t)(src[i / 4] >> (8 * (i % 4)));
                }
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// Quantize, 8-channel form, for 16-byte aligned inputs with C a multiple of 8.
// A thread quantizes 8 consecutive channels of 4 consecutive rows; the 8
// elements of a row form one Philox block (indices m C + c0 .. + 7 with c0 a
// multiple of 8), so each thread draws its own uniforms and no lane exchange
// is needed.  The codes of a tile are transposed through LDS (4 rows per
// word) for q_t; each row's 8 shift-folded codes leave as one 8-byte store.
// The row loads depend on nothing (indices clamped, no branch), so they are in
// flight while the scale, groups and descriptors arrive.  Lanes past the last
// channel load the last 8, as a neighbour does: the row's first channels instead
// would be lines of another tile (247152 x 96, 4 bits: 51.8 -> 49.8 us).
// ---------------------------------------------------------------------------
// Channels c0 .. c0 + 7: scale, fold factor 2^t of the main column (0 for an
// appended channel, whose main column holds 0), fold descriptors.
struct Chan8 {
    float s[8], tf[8];
    int32_t dw[8];
    bool any_ext;
};

__device__ __forceinline__ Chan8 load_chan8(const uint8_t* __restrict__ group, const int32_t* __restrict__ desc,
                                            int64_t c0, bool cin, int meta_vec, float inv) {
    Chan8 ch;
    uint32_t gw[2] = {0u, 0u};
#pragma unroll
    for (int j = 0; j < 8; ++j) ch.dw[j] = 0;
    if (cin) {
        if (meta_vec) {
            if (group) {
                const uint2 g2 = *reinterpret_cast<const uint2*>(group + c0);
                gw[0] = g2.x; gw[1] = g2.y;
            }
            if (desc) {
                const int4 d0 = *reinterpret_cast<const int4*>(desc + c0);
                const int4 d1 = *reinterpret_cast<const int4*>(desc + c0 + 4);
                ch.dw[0] = d0.x; ch.dw[1] = d0.y; ch.dw[2] = d0.z; ch.dw[3] = d0.w;
                ch.dw[4] = d1.x; ch.dw[5] = d1.y; ch.dw[6] = d1.z; ch.dw[7] = d1.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (group) gw[j >> 2] |= (uint32_t)group[c0 + j] << (8 * (j & 3));
                if (desc) ch.dw[j] = desc[c0 + j];
            }
        }
    }
    ch.any_ext = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        ch.s[j] = __fmul_rn(inv, pow2f((int)((gw[j >> 2] >> (8 * (j & 3))) & 0xFFu)));
        const int pos = (ch.dw[j] >> 4) - 1;
        ch.tf[j] = pos < 0 ? pow2f(ch.dw[j] & 15) : 0.0f;
        ch.any_ext |= pos >= 0;
    }
    return ch;
}

// Codes of 4 rows x 8 channels (0 where !ok): colw[j], channel j's codes of
// the 4 rows; fold[i], row i's folded codes of the main columns.  The bytes
// are built as code + 128 (unsigned), then flipped back to two's complement
// with one xor per word.  idx: the logical index of row 0's first element.
// row(i, a, b): the values of row i; emit(i, f): its folded codes, while bits
// 8 i of colw[j] hold code + 128.
template <bool SR, class Row, class Emit>
__device__ __forceinline__ void quant8(Row row, Emit emit, const bool (&ok)[4], int64_t idx, int64_t C, const Chan8& ch,
                                       const QuantCfg& cfg, uint32_t (&colw)[8]) {
    const float Qf = (float)cfg.Q;
#pragma unroll
    for (int j = 0; j < 8; ++j) colw[j] = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float4 a, b;
        row(i, a, b);
        const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        U4 w{0u, 0u, 0u, 0u};
        if (SR && ok[i]) w = philox_block((uint64_t)(idx + i * C) >> 3, cfg);
        uint32_t lo = 0u, hi = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t u = SR ? (pick(w, j >> 1) >> (16 * (j & 1))) & 0xFFFFu : 0u;
            const float q = ok[i] ? quant_onef<SR>(v[j], ch.s[j], Qf, u) : 0.0f;
            colw[j] = __builtin_amdgcn_cvt_pk_u8_f32(__fadd_rn(q, 128.0f), i, colw[j]);
            const float qf = __fadd_rn(__fmul_rn(q, ch.tf[j]), 128.0f);
            if (j < 4) lo = __builtin_amdgcn_cvt_pk_u8_f32(qf, j, lo);
            else hi = __builtin_amdgcn_cvt_pk_u8_f32(qf, j - 4, hi);
        }
        emit(i, make_uint2(lo ^ 0x80808080u, hi ^ 0x80808080u));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) colw[j] ^= 0x80808080u;
}

// The same with the rows loaded ahead and the folded codes kept.
template <bool SR>
__device__ __forceinline__ void quant8(const float4 (&a)[4], const float4 (&b)[4], const bool (&ok)[4], int64_t idx,
                                       int64_t C, const Chan8& ch, const QuantCfg& cfg, uint32_t (&colw)[8],
                                       uint2 (&fold)[4]) {
    quant8<SR>([&](int i, float4& ra, float4& rb) { ra = a[i]; rb = b[i]; }, [&](int i, uint2 f) { fold[i] = f; }, ok, idx,
               C, ch, cfg, colw);
}

// Row i's codes of the appended channels, at their columns ext_base + pos.
template <class At>
__device__ __forceinline__ void store_ext8(const Chan8& ch, const uint32_t (&colw)[8], int i, At at) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int pos = (ch.dw[j] >> 4) - 1;
        if (pos >= 0) *at(pos) = (int8_t)((int)(int8_t)(colw[j] >> (8 * i)) * (1 << (ch.dw[j] & 15)));
    }
}

// Row-major or tile-major (TL) codes: tiles of 128 rows x 64 channels.  GRID:
// q_t on the padded pixel grid (Wo and off multiples of 8; see launch_quantize).
// AHEAD: a thread loads its 4 rows first and stores their folded codes last;
// else it takes row after row, which needs 20 registers less and lets the other
// waves' memory accesses run under this one's arithmetic (launch_quantize).
template <bool SR, bool TL, bool GRID, bool AHEAD>
__global__ __launch_bounds__(kBlock) void k_quantize8(const float* __restrict__ x, int64_t M, int64_t C, int64_t ld,
                                                      const uint8_t* __restrict__ group,
                                                      const sq_scale* __restrict__ scale, QuantCfg cfg,
                                                      int8_t* __restrict__ q_fold, int64_t ld_fold,
                                                      int8_t* __restrict__ q_t, int64_t ld_t,
                                                      const int32_t* __restrict__ desc, int64_t ext_base,
                                                      int meta_vec, TensorMax tm, PadGrid pg) {
    constexpr int TR = 128, TC = 64, TW = TR / 4 + 1;   // LDS words per channel row (padded)
    __shared__ uint32_t tq[TC * TW];
    __shared__ uint32_t sh_max[4];
    sq_scale sc;
    const uint32_t tmax = tm.block_max ? tensor_max_load(tm) : 0u;
    const int tid = threadIdx.x, g8 = tid & 7, rq = tid >> 3;
    const int64_t ctiles = (C + TC - 1) / TC, rtiles = (M + TR - 1) / TR;
    // q_t rows written: the codes, and with the tile-major layout their zero
    // padding up to a multiple of 64
    const int64_t m_t = TL ? round_up(M, 64) : M;
    auto at_fold = [&](int64_t m, int64_t k) { return TL ? tiled_off(m, k, ld_fold) : m * ld_fold + k; };

    for (int64_t tile = blockIdx.x; tile < ctiles * rtiles; tile += gridDim.x) {
        const int64_t ct = tile % ctiles, rt = tile / ctiles;
        const int64_t c0 = ct * TC + 8 * g8, m0 = rt * TR + 4 * rq;
        const bool cin = c0 < C;   // C % 8 == 0: all 8 channels or none
        auto load = [&](int i, float4& a, float4& b) {
            const float* src = x + min(m0 + i, M - 1) * ld + (cin ? c0 : C - 8);
            a = *reinterpret_cast<const float4*>(src);
            b = *reinterpret_cast<const float4*>(src + 4);
        };
        float4 a[4], b[4];
        if constexpr (AHEAD) {
#pragma unroll
            for (int i = 0; i < 4; ++i) load(i, a[i], b[i]);
        }
        if (tile == blockIdx.x) sc = tm.block_max ? tensor_scale(tm, tmax, (float)cfg.Q, sh_max) : *scale;
        const Chan8 ch = load_chan8(group, desc, c0, cin, meta_vec, sc.inv);
        bool ok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ok[i] = cin && sc.flags == 0u && m0 + i < M;
        uint32_t colw[8];
        if constexpr (AHEAD) {
            uint2 fold[4];
            quant8<SR>(a, b, ok, m0 * C + c0, C, ch, cfg, colw, fold);
            if (q_fold) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t m = m0 + i;
                    if (m >= M) continue;
                    if (cin) {
                        if (ch.any_ext)
                            store_ext8(ch, colw, i, [&](int pos) { return q_fold + at_fold(m, ext_base + pos); });
                        *reinterpret_cast<uint2*>(q_fold + at_fold(m, c0)) = fold[i];
                    } else if (TL && c0 < ext_base) {
                        // K padding of the main columns
                        *reinterpret_cast<uint2*>(q_fold + at_fold(m, c0)) = make_uint2(0u, 0u);
                    }
                }
            }
        } else {
            auto row = [&](int i, float4& ra, float4& rb) {
                ra = rb = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (ok[i]) load(i, ra, rb);
            };
            auto emit = [&](int i, uint2 f) {
                const int64_t m = m0 + i;
                if (!q_fold || m >= M) return;
                if (cin) {
                    if (ch.any_ext) {
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int pos = (ch.dw[j] >> 4) - 1, code = (int)((colw[j] >> (8 * i)) & 0xFFu) - 128;
                            if (pos >= 0) q_fold[at_fold(m, ext_base + pos)] = (int8_t)(code * (1 << (ch.dw[j] & 15)));
                        }
                    }
                    *reinterpret_cast<uint2*>(q_fold + at_fold(m, c0)) = f;
                } else if (TL && c0 < ext_base) {
                    *reinterpret_cast<uint2*>(q_fold + at_fold(m, c0)) = make_uint2(0u, 0u);
                }
            };
            quant8<SR>(row, emit, ok, m0 * C + c0, C, ch, cfg, colw);
        }
        if (q_t) {
#pragma unroll
            for (int j = 0; j < 8; ++j) tq[(8 * g8 + j) * TW + rq] = colw[j];
            __syncthreads();
            // channel row c of the tile, rows 32 part .. + 31 (two 16-byte chunks)
            const int cr = tid >> 2, part = tid & 3;
            const int64_t c = ct * TC + cr, mm = rt * TR + 32 * part;
            if (c < C && mm < m_t) {
                const uint32_t* src = &tq[cr * TW + 8 * part];
                const uint4 lo = make_uint4(src[0], src[1], src[2], src[3]);
                const uint4 hi = make_uint4(src[4], src[5], src[6], src[7]);
                if (TL) {
                    *reinterpret_cast<uint4*>(q_t + tiled_off(c, mm, ld_t)) = lo;
                    *reinterpret_cast<uint4*>(q_t + tiled_off(c, mm + 16, ld_t)) = hi;
                } else if (GRID) {
                    // 4 groups of 8 pixels, none across an image row: 8-byte stores
                    const uint32_t p0 = (uint32_t)mm;
                    uint32_t n = p0 / pg.HoWo, rem = p0 - n * pg.HoWo, oh = rem / pg.Wo, ow = rem - oh * pg.Wo;
                    int8_t* row = q_t + c * ld_t + pg.off;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        if (mm + 8 * g < M)
                            *reinterpret_cast<uint2*>(row + (int64_t)n * pg.HpWp + (int64_t)oh * pg.Wp + ow) =
                                make_uint2(src[2 * g], src[2 * g + 1]);
                        ow += 8;
                        if (ow == pg.Wo) {
                            ow = 0;
                            if (++oh * pg.Wo == pg.HoWo) {
                                oh = 0;
                                ++n;
                            }
                        }
                    }
                } else if (mm + 32 <= M) {
                    *reinterpret_cast<uint4*>(q_t + c * ld_t + mm) = lo;
                    *reinterpret_cast<uint4*>(q_t + c * ld_t + mm + 16) = hi;
                } else {
                    for (int r = 0; r < (int)(M - mm); ++r)
                        q_t[c * ld_t + mm + r] = (int8_t)(src[r / 4] >> (8 * (r % 4)));
                }
            }
            __syncthreads();
        }
    }
}

// Transposed codes on the padded pixel grid (PadGrid), any image width.  A
// tile is 64 channels x up to 128 pixels whose grid positions are whole rows
// of the grid (rows = 128 / Wo image rows) or, for Wo > 128, 128 aligned
// positions of one row.  Grid rows start at multiples of 16 (Wp and the row
// part of the offset are), so every aligned 16-byte chunk of a channel's grid
// that holds codes belongs to one tile: it is written whole, its bytes outside
// the image as the zeros they are.  A chunk's 16 codes are a run of the tile's
// pixels in LDS, moved into place with v_alignbyte.  Bound by memory (4 B read
// and 1 or 2 B written per code).  Against byte stores per pixel (k_quantize):
// 64 x 28 x 28 x 128 input 24.5 -> 9.8 us, 6-bit stochastic gradient 29.5 ->
// 15.6 us; 64 x 14 x 14 x 256 15.2 -> 7.9 and 17.2 -> 8.6 us.  Against 8-byte
// stores with the straddling words of an input put together (widths a multiple
// of 8): 64 x 56 x 56 x 64 input 17.6 -> 14.8 us; where 8-byte stores win,
// launch_quantize takes k_quantize8.
struct GridTiles {
    uint32_t rows;             // image rows per tile
    uint32_t segs;             // tiles per image row (1 unless Wo > 128)
    uint32_t chunks;           // 16-byte chunks per image row of a tile
    uint32_t lead;             // grid position of an image row's first pixel
    uint32_t row_off;          // grid offset of an image's first row
    uint32_t H, NH;            // image rows per image, and in all
    uint32_t mul_chunks, mul_per, mul_H;   // ceil(2^32 / d) of chunks, rows * chunks and H (0: d = 1)
};

// a / d with mul = ceil(2^32 / d): exact while a d < 2^32 (the launcher checks)
__device__ __forceinline__ uint32_t div_mul(uint32_t a, uint32_t mul) { return mul ? __umulhi(a, mul) : a; }

template <bool SR>
__global__ __launch_bounds__(kBlock) void k_quantize_grid(const float* __restrict__ x, int64_t M, int64_t C,
                                                          int64_t ld, const uint8_t* __restrict__ group,
                                                          const sq_scale* __restrict__ scale, QuantCfg cfg,
                                                          int8_t* __restrict__ q_fold, int64_t ld_fold,
                                                          int8_t* __restrict__ q_t, int64_t ld_t,
                                                          const int32_t* __restrict__ desc, int64_t ext_base,
                                                          int meta_vec, PadGrid pg, GridTiles gt, TensorMax tm) {
    constexpr int TC = 64, TW = 33, kFront = 4, kBack = 8;   // words; a chunk may start up to 15 pixels before its row
    __shared__ uint32_t tile_w[kFront + TC * TW + kBack];
    uint32_t* tq = tile_w + kFront;
    __shared__ uint32_t sh_max[4];
    sq_scale sc;
    const uint32_t tmax = tm.block_max ? tensor_max_load(tm) : 0u;
    const int tid = threadIdx.x, g8 = tid & 7, rq = tid >> 3;
    const uint32_t ctiles = (uint32_t)((C + TC - 1) / TC);
    const uint32_t tiles = (gt.NH + gt.rows - 1) / gt.rows * gt.segs;
    const uint32_t per = gt.rows * gt.chunks;

    for (uint64_t tile = blockIdx.x; tile < (uint64_t)tiles * ctiles; tile += gridDim.x) {
        const uint32_t pt = (uint32_t)(tile / ctiles), ct = (uint32_t)(tile - (uint64_t)pt * ctiles);
        const uint32_t yt = pt / gt.segs, seg = pt - yt * gt.segs, y0 = yt * gt.rows;
        // pixel p of the tile is pixel m_base + p of the tensor, p_lo <= p < p_hi
        const int w0 = gt.segs > 1 ? (int)(128 * seg) - (int)gt.lead : 0;
        const int p_lo = max(0, -w0);
        const int p_hi = gt.segs > 1 ? min(128, (int)pg.Wo - w0) : (int)(min(gt.rows, gt.NH - y0) * pg.Wo);
        const int64_t m_base = (int64_t)y0 * pg.Wo + w0;
        const int64_t c0 = (int64_t)ct * TC + 8 * g8, m0 = m_base + 4 * rq;
        const bool cin = c0 < C;
        float4 a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = min(max(4 * rq + i, p_lo), p_hi - 1);
            const float* src = x + (m_base + p) * ld + (cin ? c0 : C - 8);
            a[i] = *reinterpret_cast<const float4*>(src);
            b[i] = *reinterpret_cast<const float4*>(src + 4);
        }
        if (tile == blockIdx.x) sc = tm.block_max ? tensor_scale(tm, tmax, (float)cfg.Q, sh_max) : *scale;
        const Chan8 ch = load_chan8(group, desc, c0, cin, meta_vec, sc.inv);
        bool in[4], ok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = 4 * rq + i;
            in[i] = cin && p >= p_lo && p < p_hi;
            ok[i] = in[i] && sc.flags == 0u;
        }
        uint32_t colw[8];
        uint2 fold[4];
        quant8<SR>(a, b, ok, m0 * C + c0, C, ch, cfg, colw, fold);
#pragma unroll
        for (int j = 0; j < 8; ++j) tq[(8 * g8 + j) * TW + rq] = colw[j];
        if (q_fold) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!in[i]) continue;
                int8_t* row = q_fold + (m0 + i) * ld_fold;
                if (ch.any_ext) store_ext8(ch, colw, i, [&](int pos) { return row + ext_base + pos; });
                *reinterpret_cast<uint2*>(row + c0) = fold[i];
            }
        }
        __syncthreads();
        // chunk k of image row r of channel row cr
        const uint32_t n0 = y0 / gt.H, h0 = y0 - n0 * gt.H;
        for (uint32_t id = tid; id < TC * per; id += kBlock) {
            const uint32_t cr = div_mul(id, gt.mul_per), j = id - cr * per;
            const uint32_t r = div_mul(j, gt.mul_chunks), k = j - r * gt.chunks;
            const int64_t c = (int64_t)ct * TC + cr;
            if (c >= C || y0 + r >= gt.NH) continue;
            // the chunk's byte e is pixel s0 + e of the tile; codes at e_lo <= e < e_hi
            const int lead = gt.segs > 1 ? 0 : (int)gt.lead;
            const int first = 16 * (int)k - lead, s0 = (int)(r * pg.Wo) + first;
            const int e_lo = max(0, (gt.segs > 1 ? p_lo : 0) - first);
            const int e_hi = min(16, (gt.segs > 1 ? p_hi : (int)pg.Wo) - first);
            if (e_lo >= e_hi) continue;
            const uint32_t* src = &tq[(int)cr * TW + (s0 >> 2)];
            const uint32_t w[5] = {src[0], src[1], src[2], src[3], src[4]};
            uint32_t o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int lo_i = min(4, max(0, e_lo - 4 * i)), hi_i = min(4, max(0, e_hi - 4 * i));
                const uint32_t mask = hi_i > lo_i ? (0xFFFFFFFFu >> (32 - 8 * (hi_i - lo_i))) << (8 * lo_i) : 0u;
                o[i] = __builtin_amdgcn_alignbyte(w[i + 1], w[i], (uint32_t)s0 & 3u) & mask;
            }
            const uint32_t dn = div_mul(h0 + r, gt.mul_H), h = h0 + r - dn * gt.H;
            const int64_t d = (int64_t)(n0 + dn) * pg.HpWp + gt.row_off + (int64_t)h * pg.Wp + 128 * seg + 16 * k;
            *reinterpret_cast<uint4*>(q_t + c * ld_t + d) = make_uint4(o[0], o[1], o[2], o[3]);
        }
        __syncthreads();
    }
}

// Gradient codes of an L1BNQ layer together with the channel sums its backward
// needs of them: codes q [M, ldc] (no fold) and, per row block and channel,
// part[0][block][c] = sum q and part[1][block][c] = sum q (x - mu) with the
// layer's input codes x.  A block of 512 threads takes 64 channels of its
// rows, 256 at a time: quant8 leaves a thread the codes of 4 rows of a channel
// in one word, so with x moved to the same order (byte permutes) each channel's
// products are one 4-way dot.  Bound by memory (4 + 1 B read, 1 B written per
// element).  200704 x 64: 17.4 us; as a quantize pass and
// a pass over both codes 13.8 + 10.2 us.
constexpr int kBnQThreads = 512, kBnQRows = kBnQThreads / 8 * 4;

// bytes of 4 row words (columns 0 .. 3 each) to 4 column words (rows 0 .. 3 each)
__device__ __forceinline__ void transpose4x4(const uint32_t (&r)[4], uint32_t (&c)[4]) {
    const uint32_t a = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u);   // r0.0 r1.0 r0.1 r1.1
    const uint32_t b = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);   // r0.2 r1.2 r0.3 r1.3
    const uint32_t d = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u);
    const uint32_t e = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
    c[0] = __builtin_amdgcn_perm(d, a, 0x05040100u);
    c[1] = __builtin_amdgcn_perm(d, a, 0x07060302u);
    c[2] = __builtin_amdgcn_perm(e, b, 0x05040100u);
    c[3] = __builtin_amdgcn_perm(e, b, 0x07060302u);
}

template <bool SR>
__global__ __launch_bounds__(kBnQThreads) void k_quantize_bn(const float* __restrict__ dy, int64_t M, int64_t C,
                                                             int64_t ld, const uint8_t* __restrict__ group,
                                                             const sq_scale* __restrict__ scale, QuantCfg cfg,
                                                             int8_t* __restrict__ q, int64_t ldc,
                                                             const int8_t* __restrict__ xq, int64_t ld_x,
                                                             const sq_l1bn_channel* __restrict__ chan,
                                                             int64_t rows_per_block, int32_t* __restrict__ part) {
    __shared__ int32_t red[2][kBnQThreads / 64][64];
    const int tid = threadIdx.x, g8 = tid & 7, rq = tid >> 3;
    const int64_t c0 = (int64_t)blockIdx.y * 64 + 8 * g8;
    const bool cin = c0 < C;
    const int64_t cs = cin ? c0 : C - 8;
    const int64_t r_end = min(M, ((int64_t)blockIdx.x + 1) * rows_per_block);
    int g1[8], g2[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) g1[j] = g2[j] = 0;
    for (int64_t r0 = (int64_t)blockIdx.x * rows_per_block; r0 < r_end; r0 += kBnQRows) {
        const int64_t m0 = r0 + 4 * rq;
        float4 a[4], b[4];
        uint2 xw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t m = min(m0 + i, M - 1);
            const float* src = dy + m * ld + cs;
            a[i] = *reinterpret_cast<const float4*>(src);
            b[i] = *reinterpret_cast<const float4*>(src + 4);
            xw[i] = *reinterpret_cast<const uint2*>(xq + m * ld_x + cs);
        }
        const sq_scale sc = *scale;
        const Chan8 ch = load_chan8(group, nullptr, c0, cin, (reinterpret_cast<uintptr_t>(group) & 7) == 0, sc.inv);
        bool ok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ok[i] = cin && sc.flags == 0u && m0 + i < r_end;
        uint32_t colw[8];
        uint2 fold[4];
        quant8<SR>(a, b, ok, m0 * C + c0, C, ch, cfg, colw, fold);
        if (cin) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (m0 + i < r_end) *reinterpret_cast<uint2*>(q + (m0 + i) * ldc + c0) = fold[i];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t rows[4] = {h ? xw[0].y : xw[0].x, h ? xw[1].y : xw[1].x, h ? xw[2].y : xw[2].x,
                                      h ? xw[3].y : xw[3].x};
            uint32_t cols[4];
            transpose4x4(rows, cols);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                g1[4 * h + j] = __builtin_amdgcn_sdot4((int)colw[4 * h + j], 0x01010101, g1[4 * h + j], false);
                g2[4 * h + j] = __builtin_amdgcn_sdot4((int)colw[4 * h + j], (int)cols[j], g2[4 * h + j], false);
            }
        }
    }
    // the 8 row lanes of a wave, then the waves through LDS
#pragma unroll
    for (int j = 0; j < 8; ++j) {
#pragma unroll
        for (int o = 8; o < 64; o <<= 1) {
            g1[j] += __shfl_xor(g1[j], o, 64);
            g2[j] += __shfl_xor(g2[j], o, 64);
        }
        if ((tid & 63) < 8) {
            red[0][tid >> 6][8 * g8 + j] = g1[j];
            red[1][tid >> 6][8 * g8 + j] = g2[j];
        }
    }
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.y * 64 + tid;
    if (tid < 64 && c < C) {
        int32_t s1 = 0, s2 = 0;
#pragma unroll
        for (int w = 0; w < kBnQThreads / 64; ++w) {
            s1 += red[0][w][tid];
            s2 += red[1][w][tid];
        }
        part[(int64_t)blockIdx.x * C + c] = s1;
        part[((int64_t)gridDim.x + blockIdx.x) * C + c] = s2 - chan[c].mu * s1;
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Per-channel quantization of a weight matrix (one scale per row or per
// column; the forward pass quantizes weights per output channel and loss
// propagation per input channel, Sec. 5.1).  The forward's row-major codes per
// row have a kernel of their own (k_quantize_rows); the other forms, off the
// training step's path, are plain.
// ---------------------------------------------------------------------------
// column scales from the colmax slab maxima
__global__ void k_channel_scales_cols(const uint32_t* __restrict__ partial, int64_t S, int64_t C, int Q,
                                      sq_scale* __restrict__ scales) {
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < C; c += (int64_t)gridDim.x * blockDim.x)
        scales[c] = make_scale(reduce_slabs(partial, S, C, c), (float)Q);
}

// row scales: one wave per row
__global__ void k_channel_scales_rows(const float* __restrict__ x, int64_t rows, int64_t cols, int64_t ld, int Q,
                                      sq_scale* __restrict__ scales) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t r = wave; r < rows; r += nwaves) {
        uint32_t m = 0u;
        for (int64_t c = lane; c < cols; c += 64) m = max(m, absbits(x[r * ld + c]));
        m = wave_max(m);
        if (lane == 0) scales[r] = make_scale(m, (float)Q);
    }
}

// Row scales and row-major codes in one pass: the row's second read comes from
// the caches.  LPR lanes take a row (4 to 64, its quads of columns, so that
// short rows fill the wave; fixed at compile time, the loops of long rows were
// 15 to 20 % slower otherwise).  Bound by latency (a row of a few thousand
// floats); scales and codes as two launches took 6.2 + 9.9 us on 3072 x 768,
// this one 6.6 us; 100000 x 16 two launches 18.5 us, a wave per row 22.7, four
// lanes per row 4.5.  VEC: 16-byte aligned rows.
template <bool VEC, int LPR>
__global__ __launch_bounds__(256) void k_quantize_rows(const float* __restrict__ x, int64_t rows, int64_t cols, int64_t ld,
                                                       int Q, sq_scale* __restrict__ scales, int8_t* __restrict__ q,
                                                       int64_t ld_q) {
    const int lane = threadIdx.x % LPR;
    const float Qf = (float)Q;
    constexpr int kRows = 256 / LPR;   // rows per block and step
    const int64_t quads = cols >> 2;
    for (int64_t r = (int64_t)blockIdx.x * kRows + threadIdx.x / LPR; r < rows; r += (int64_t)gridDim.x * kRows) {
        const float* row = x + r * ld;
        auto load4 = [&](int64_t i) {
            if constexpr (VEC) return *reinterpret_cast<const float4*>(row + 4 * i);
            else return make_float4(row[4 * i], row[4 * i + 1], row[4 * i + 2], row[4 * i + 3]);
        };
        const int64_t tail = 4 * quads + lane;   // the last cols % 4 columns
        uint32_t m = tail < cols ? absbits(row[tail]) : 0u;
#pragma unroll 4
        for (int64_t i = lane; i < quads; i += LPR) {
            const float4 v = load4(i);
            m = max(max(m, max(absbits(v.x), absbits(v.y))), max(absbits(v.z), absbits(v.w)));
        }
        // the lanes of a row enter and leave this loop together
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
        const sq_scale sc = make_scale(m, Qf);
        if (lane == 0) scales[r] = sc;
        auto code = [&](float v) {
            return sc.flags ? 0u : (uint32_t)(uint8_t)(int)fminf(fmaxf(rintf(__fmul_rn(v, sc.inv)), -Qf), Qf);
        };
        int8_t* out = q + r * ld_q;   // ld_q a multiple of 16, 16-byte aligned
#pragma unroll 4
        for (int64_t i = lane; i < quads; i += LPR) {
            const float4 v = load4(i);
            reinterpret_cast<uint32_t*>(out)[i] = code(v.x) | code(v.y) << 8 | code(v.z) << 16 | code(v.w) << 24;
        }
        if (tail < cols) out[tail] = (int8_t)code(row[tail]);
    }
}

// code = clamp(rint(fl(x * inv_ch)), -Q, Q), 0 in a flagged channel
__global__ void k_quantize_channels(const float* __restrict__ x, int64_t rows, int64_t cols, int64_t ld, int axis,
                                    const sq_scale* __restrict__ scales, int Q, int8_t* __restrict__ q, int64_t ld_q,
                                    int transpose) {
    const float Qf = (float)Q;
    const int64_t n = rows * cols;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = transpose ? e % rows : e / cols, j = transpose ? e / rows : e % cols;
        const sq_scale sc = scales[axis == 0 ? i : j];
        int code = 0;
        if (sc.flags == 0u) code = (int)fminf(fmaxf(rintf(__fmul_rn(x[i * ld + j], sc.inv)), -Qf), Qf);
        if (transpose) q[j * ld_q + i] = (int8_t)code;
        else q[i * ld_q + j] = (int8_t)code;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
ColmaxPlan colmax_plan(int64_t M, int64_t C, bool vec) {
    ColmaxPlan p{};
    const int VEC = vec ? 4 : 1;
    const int64_t units = (C + VEC - 1) / VEC;
    int tpr = 1;
    while (tpr < units && tpr < 64) tpr <<= 1;
    const int nrl = kColThreads / tpr;
    p.vec = VEC;
    p.tpr = tpr;
    p.chunks = std::max<int64_t>(1, (units + tpr - 1) / tpr);
    // about 512 blocks (two per CU), each slab at least 8 row passes deep:
    // fewer slab maxima for the finalize to reduce (1024 blocks cost the
    // 64-channel conv gradient 3 us more, measured)
    int64_t slabs = std::max<int64_t>(1, 512 / p.chunks);
    const int64_t min_rows = 8 * (int64_t)nrl;
    slabs = std::min<int64_t>(slabs, std::max<int64_t>(1, (M + min_rows - 1) / min_rows));
    slabs = std::min<int64_t>(slabs, 65535);
    p.rows_per_slab = std::max<int64_t>(1, (M + slabs - 1) / slabs);
    p.slabs = M > 0 ? (M + p.rows_per_slab - 1) / p.rows_per_slab : 0;
    return p;
}

// 64-channel groups of the finalize (at least one: the scale and header of an
// empty tensor are written too)
static int64_t fin_blocks(int64_t C) { return std::max<int64_t>(1, (C + kFinCh - 1) / kFinCh); }

int64_t colmax_workspace_words(int64_t M, int64_t C) {
    // with ranges from the producer: channel ranges and group maxima; else,
    // worst case over both vector widths, the shift counts and the abs-max
    // outputs (slab maxima, block maxima).  Never more than the finalize in
    // blocks of 256 channels took for C >= 1024, so that the tensors a fixed
    // scratch holds stay the same.
    const int64_t nb = fin_blocks(C);
    int64_t w = C + kMaxRegions + nb;
    for (const bool vec : {true, false}) {
        const ColmaxPlan p = colmax_plan(M, C, vec);
        const int64_t fin = std::max(kMaxRegions * nb, C + (C >= 1024 ? (1 + kMaxRegions) * ((C + 255) / 256) : 0));
        w = std::max(w, p.slabs * C + fin + p.chunks * p.slabs);
    }
    return w;
}

// float4 loads of whole rows need 16-byte aligned rows
static bool colmax_vec(const float* x, int64_t ld) {
    return ((ld & 3) == 0) && ((reinterpret_cast<uintptr_t>(x) & 15) == 0);
}

hipError_t launch_colmax(const float* x, int64_t M, int64_t C, int64_t ld, uint32_t* partial, int64_t* slabs,
                         hipStream_t s, uint32_t* block_max, int64_t* n_block_max) {
    *slabs = 0;
    if (n_block_max) *n_block_max = 0;
    if (M <= 0 || C <= 0) return hipSuccess;
    const bool vec = colmax_vec(x, ld);
    const ColmaxPlan p = colmax_plan(M, C, vec);
    *slabs = p.slabs;
    if (n_block_max) *n_block_max = p.chunks * p.slabs;
    dim3 grid((unsigned)p.chunks, (unsigned)p.slabs);
    // A tensor larger than the 256 MB last-level cache cannot stay there for
    // the quantize pass's second read; streaming it through without
    // allocating leaves other lines in place, in particular dirty ones, which
    // would otherwise be written back during this read (large linear layer,
    // 360 MB: this pass 78.7 -> 55.6 us, the step 741 -> 730 us).  Smaller
    // tensors keep ordinary loads (their second read hits the cache).
    const bool nt = (uint64_t)M * (uint64_t)ld * sizeof(float) > kLastLevelCacheBytes;
    if (vec && nt)
        hipLaunchKernelGGL((k_colmax<4, true>), grid, dim3(kColThreads), 0, s, x, M, C, ld, p.tpr, p.rows_per_slab,
                           partial, block_max);
    else if (vec)
        hipLaunchKernelGGL((k_colmax<4, false>), grid, dim3(kColThreads), 0, s, x, M, C, ld, p.tpr, p.rows_per_slab,
                           partial, block_max);
    else
        hipLaunchKernelGGL((k_colmax<1, false>), grid, dim3(kColThreads), 0, s, x, M, C, ld, p.tpr, p.rows_per_slab,
                           partial, block_max);
    return hipGetLastError();
}

constexpr int64_t kDirectRanges = 16384;   // ranges that a block of 16 waves reads in two batches of loads
// Second-level blocks: 16 waves for 64 channels; 4 where those read the slabs
// and the block maxima in a batch of loads or two; a wave for 64 channels where
// there are many in few slabs (8 x 262144, 6 bits: 83.8 us with 16 waves, 55.4
// with 4, 52.6 with one; below 32768 channels 4 and one are equal).
enum class Fin { kBlock16, kBlock4, kWide };
static Fin fin_kind(int64_t slabs, int64_t nbm, int64_t nb) {
    if (slabs <= 8 && nb >= 512) return Fin::kWide;
    return slabs <= 32 && nbm <= 2048 ? Fin::kBlock4 : Fin::kBlock16;
}

static hipError_t launch_groups_place(const uint32_t* partial, int64_t slabs, const uint32_t* block_max, int64_t nbm,
                                      int64_t C, const QuantCfg& cfg, uint8_t* group, sq_scale* scale, int32_t* layout,
                                      int64_t ext_max, int32_t* hist, int hist_ld, hipStream_t s) {
    const int64_t nb = fin_blocks(C);
    auto groups = [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        const int64_t blocks = NW ? nb : (nb + kWideWaves - 1) / kWideWaves;
        hipLaunchKernelGGL(k_final_groups<NW>, dim3((unsigned)blocks), dim3(kFinThreadsOf<NW>), 0, s, partial, slabs,
                           block_max, nbm, C, cfg, group, scale, layout, ext_max, hist, hist_ld);
    };
    switch (fin_kind(slabs, nbm, nb)) {
        case Fin::kWide: groups(std::integral_constant<int, 0>()); break;
        case Fin::kBlock4: groups(std::integral_constant<int, 4>()); break;
        case Fin::kBlock16: groups(std::integral_constant<int, kFinWaves>()); break;
    }
    if (ext_max > 0)
        hipLaunchKernelGGL(k_final_place, dim3((unsigned)((nb + 3) / 4)), dim3(kPlaceThreads), 0, s, group, hist,
                           hist_ld, nb, C, cfg, layout, ext_max);
    return hipGetLastError();
}

// ws, `words` long: at least channel ranges, kMaxRegions words, group maxima.
hipError_t launch_finalize_ranges(const uint32_t* ranges, int64_t slabs, int64_t C, const QuantCfg& cfg, uint32_t* ws,
                                  int64_t words, uint8_t* group, sq_scale* scale, int32_t* layout, int64_t ext_max,
                                  hipStream_t s) {
    const int64_t nb = fin_blocks(C);
    int32_t* hist = reinterpret_cast<int32_t*>(ws);
    // few ranges: the group kernel takes r_max from all of them (one launch
    // fewer: 256 x 256 in one window 10.0 -> 7.9 us)
    if (slabs * C <= kDirectRanges || (nb == 1 && slabs <= kFinRows))
        return launch_groups_place(ranges, slabs, ranges, slabs * C, C, cfg, group, scale, layout, ext_max, hist,
                                   kMaxRegions, s);
    // Otherwise a reduction before it, over gy parts of the slabs where they
    // are many for their channels and the scratch holds the parts (200704 x 64,
    // 6272 slabs, the call: 35.8 us with one block for all of them, 23.2).
    int64_t gy = std::min({slabs / (C % 4 ? kFinRows / 4 : kFinRows), 512 / nb, (int64_t)64, (words - kMaxRegions * nb) / (C + nb)});
    gy = std::max<int64_t>(gy, 1);
    const int64_t per = (slabs + gy - 1) / gy;
    gy = (slabs + per - 1) / per;
    // ws: shift counts, part ranges, group maxima of the parts; or, with one
    // part, channel ranges, group maxima: a group's shift counts then take the
    // place of its own channel ranges, which its block has read by then
    uint32_t* parts = gy > 1 ? ws + kMaxRegions * nb : ws;
    uint32_t* bmax = gy > 1 ? parts + gy * C : ws + C + kMaxRegions;
    auto reduce = [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        const int64_t blocks = NW ? nb : (nb + kWideWaves - 1) / kWideWaves;
        hipLaunchKernelGGL(k_colmax_reduce<NW>, dim3((unsigned)blocks, (unsigned)gy), dim3(kFinThreadsOf<NW>), 0, s,
                           ranges, slabs, per, C, parts, bmax, nb);
    };
    switch (fin_kind(per, 0, nb)) {
        case Fin::kWide: reduce(std::integral_constant<int, 0>()); break;
        case Fin::kBlock4: reduce(std::integral_constant<int, 4>()); break;
        case Fin::kBlock16: reduce(std::integral_constant<int, kFinWaves>()); break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_groups_place(parts, gy, bmax, gy * nb, C, cfg, group, scale, layout, ext_max, hist,
                               gy > 1 ? kMaxRegions : kFinCh, s);
}

hipError_t launch_colmax_finalize_grad(const float* x, int64_t M, int64_t C, int64_t ld, const QuantCfg& cfg,
                                       uint32_t* ws, uint8_t* group, sq_scale* scale, int32_t* layout,
                                       int64_t ext_max, hipStream_t s) {
    // ws: shift counts, slab maxima, block maxima
    int32_t* hist = reinterpret_cast<int32_t*>(ws);
    uint32_t* partial = ws + kMaxRegions * fin_blocks(C);
    int64_t slabs = 0, nbm = 0;
    uint32_t* bm = partial + colmax_plan(M, C, colmax_vec(x, ld)).slabs * C;
    const hipError_t e = launch_colmax(x, M, C, ld, partial, &slabs, s, bm, &nbm);
    if (e != hipSuccess) return e;
    return launch_groups_place(partial, slabs, bm, nbm, C, cfg, group, scale, layout, ext_max, hist, kMaxRegions, s);
}

hipError_t launch_quantize_tensor(const float* x, int64_t M, int64_t C, int64_t ld, const QuantCfg& cfg, uint32_t* ws,
                                  sq_scale* scale, int8_t* q, int64_t ld_q, int8_t* q_t, int64_t ld_t, hipStream_t s,
                                  PadGrid pg, bool tiled) {
    if (M <= 0 || C <= 0) {
        hipLaunchKernelGGL(k_empty_scale, dim3(1), dim3(1), 0, s, cfg.Q, scale);
        return hipGetLastError();
    }
    int64_t slabs = 0;
    TensorMax tm;
    uint32_t* bm = ws + colmax_plan(M, C, colmax_vec(x, ld)).slabs * C;
    const hipError_t e = launch_colmax(x, M, C, ld, ws, &slabs, s, bm, &tm.n);
    if (e != hipSuccess) return e;
    // 4 x 1000003 (15,626 maxima): 81.9 us without the launch, 57.5 with it; 4 x
    // 300001 (4688): 26.7, 24.1
    constexpr int64_t kManyMaxima = 4096;
    if (tm.n > kManyMaxima) {
        hipLaunchKernelGGL(k_block_max, dim3(1), dim3(1024), 0, s, bm, tm.n);
        tm.n = 1;
    }
    tm.block_max = bm;
    tm.scale = scale;
    return launch_quantize(x, M, C, ld, nullptr, scale, cfg, q, ld_q, q_t, ld_t, nullptr, s, pg, tiled, tm);
}

constexpr int64_t kQuantMaxBlocks = 4096;   // grid-stride beyond this
constexpr int64_t kQuantMinTiles = 1024;    // four blocks per CU

// Tiles of k_quantize_grid (false: outside what it takes).  pg.off is the grid
// position of pixel 0: its row part is a multiple of 16, the rest the lead.
static bool grid_tiles(int64_t M, const PadGrid& pg, GridTiles& gt) {
    if (pg.Wo == 0 || pg.HoWo % pg.Wo || pg.Wp % 16 || pg.HpWp % 16 || M % pg.Wo) return false;
    gt.lead = pg.off % pg.Wp;
    gt.row_off = pg.off - gt.lead;
    gt.H = pg.HoWo / pg.Wo;
    const int64_t NH = M / pg.Wo;
    // lead < 16 (the words before a tile's first), and div_mul's range
    if (gt.lead > 15 || gt.lead + pg.Wo > pg.Wp || gt.H >= 32768 || NH >= ((int64_t)1 << 31)) return false;
    gt.NH = (uint32_t)NH;
    if (pg.Wo <= 128) {
        gt.rows = std::min<uint32_t>(128 / pg.Wo, gt.NH);
        gt.segs = 1;
        gt.chunks = (gt.lead + pg.Wo + 15) / 16;
    } else {
        gt.rows = 1;
        gt.segs = (gt.lead + pg.Wo + 127) / 128;
        gt.chunks = 8;
    }
    auto mul = [](uint32_t d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
    gt.mul_chunks = mul(gt.chunks);
    gt.mul_per = mul(gt.rows * gt.chunks);
    gt.mul_H = mul(gt.H);
    return true;
}

hipError_t launch_quantize(const float* x, int64_t M, int64_t C, int64_t ld, const uint8_t* group,
                           const sq_scale* scale, const QuantCfg& cfg, int8_t* q_fold, int64_t ld_fold,
                           int8_t* q_t, int64_t ld_t, const int32_t* desc, hipStream_t s, PadGrid pg, bool tiled,
                           TensorMax tm) {
    if (M <= 0 || C <= 0) return hipSuccess;
    if (tiled && (pg.Wo || (q_fold && ld_fold % 64) || (q_t && ld_t % 64))) return hipErrorInvalidValue;
    const bool vec = ((ld & 3) == 0) && ((reinterpret_cast<uintptr_t>(x) & 15) == 0);
    const bool sr = cfg.round_mode == SQ_ROUND_STOCHASTIC;
    // 128 x 128 tiles where the tensor gives enough of them to fill the chip
    auto n_tiles = [&](int64_t tc, int64_t tr) { return ((C + tc - 1) / tc) * ((M + tr - 1) / tr); };
    // stochastic rounding keeps the 64-channel tile: the Philox words of a
    // 128-channel tile's passes need about 180 registers (2 waves per SIMD)
    int tc = (C <= 64 || sr) ? 64 : 128, tr = 128;
    if (n_tiles(tc, tr) < kQuantMinTiles) tr = 64;
    if (n_tiles(tc, tr) < kQuantMinTiles) tc = 64;
    const int64_t eb = fold_ext_base(C);
    // groups (8 bytes) and descriptors (2 x 16 bytes) of 8 channels load as
    // vectors when aligned
    const int mv = ((reinterpret_cast<uintptr_t>(group) & 7) == 0 && (reinterpret_cast<uintptr_t>(desc) & 15) == 0);
    // Padded grid: tiles of whole grid rows (k_quantize_grid), or, where image
    // rows and their places are multiples of 8 pixels, k_quantize8's 128
    // consecutive pixels with 8-byte stores.  The latter where whole rows fill
    // too little of a tile, and for stochastic codes (bound by their Philox
    // words) without appended fold windows.  us, whole-row tiles -> pixels, 200704
    // pixels: 32 channels 144 wide, 4 bits 43.5 -> 33.9, stochastic 57.0 -> 40.6;
    // 64 channels 48 wide, 4 bits 33.8 -> 33.3, 6 bits (windows) 40.0 -> 41.9;
    // 56 wide, stochastic, 4 bits 36.4 -> 35.3, 6 bits 42.1 -> 43.1.
    GridTiles gt{};
    const bool on_grid = vec && C % 8 == 0 && pg.Wo && q_t && grid_tiles(M, pg, gt);
    const bool windows = group && cfg.num_groups - 1 > cfg.T;
    const uint64_t used = (uint64_t)gt.rows * pg.Wo * 100, slots = (uint64_t)128 * gt.segs;
    const bool grid8 = on_grid && pg.Wo % 8 == 0 && pg.off % 8 == 0 &&
                       (windows ? used < 70 * slots : sr || used < 80 * slots);
    if (on_grid && !grid8) {
        const int64_t tiles = (int64_t)((gt.NH + gt.rows - 1) / gt.rows) * gt.segs * ((C + 63) / 64);
        const dim3 gg((unsigned)std::min<int64_t>(tiles, kQuantMaxBlocks));
        if (sr) hipLaunchKernelGGL(k_quantize_grid<true>, gg, dim3(kBlock), 0, s, x, M, C, ld, group, scale, cfg, q_fold,
                                   ld_fold, q_t, ld_t, desc, eb, mv, pg, gt, tm);
        else hipLaunchKernelGGL(k_quantize_grid<false>, gg, dim3(kBlock), 0, s, x, M, C, ld, group, scale, cfg, q_fold,
                                ld_fold, q_t, ld_t, desc, eb, mv, pg, gt, tm);
        return hipGetLastError();
    }
    if (grid8 || (vec && C % 8 == 0 && !pg.Wo)) {
        const dim3 g8((unsigned)std::min<int64_t>(((C + 63) / 64) * ((M + 127) / 128), kQuantMaxBlocks));
        auto run = [&](auto k) {
            hipLaunchKernelGGL(k, g8, dim3(kBlock), 0, s, x, M, C, ld, group, scale, cfg, q_fold, ld_fold, q_t, ld_t, desc,
                               eb, mv, tm, pg);
        };
        // Row by row or loads ahead (see k_quantize8), us, ahead / by row: small
        // tensors are a round of blocks or less, where the loads' latency is all
        // there is (197 x 768, 6 bits 17.5 / 19.0); near and beyond the last-level
        // cache the accesses are the bound (16384 x 3072, 6 bits, tile-major 113.3 /
        // 119.6, stochastic 112.4 / 120.7); between them the registers are (200704 x
        // 64 30.2 / 28.6, stochastic 31.2 / 29.6; 1376 x 4864 21.4 / 20.0).
        // Per-tensor codes, one layout only: ahead (12544 x 1024 22.9 / 23.8).
        // Stochastic codes without appended windows: by row (8192 x 11008 182.3 /
        // 176.6; 256 x 256 13.8 / 13.8).
        const uint64_t bytes = (uint64_t)M * (uint64_t)ld * sizeof(float);
        const bool ahead = sr ? windows && bytes > kLastLevelCacheBytes / 4 * 3
                              : grid8 || !group || bytes < (16ull << 20) || bytes > kLastLevelCacheBytes * 3 / 8;
        if (grid8) run(!sr ? k_quantize8<false, false, true, true>
                       : ahead ? k_quantize8<true, false, true, true> : k_quantize8<true, false, true, false>);
        else if (tiled && sr) run(ahead ? k_quantize8<true, true, false, true> : k_quantize8<true, true, false, false>);
        else if (tiled) run(ahead ? k_quantize8<false, true, false, true> : k_quantize8<false, true, false, false>);
        else if (sr) run(ahead ? k_quantize8<true, false, false, true> : k_quantize8<true, false, false, false>);
        else run(ahead ? k_quantize8<false, false, false, true> : k_quantize8<false, false, false, false>);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)std::min<int64_t>(n_tiles(tc, tr), kQuantMaxBlocks));
#define SQ_LAUNCH_QUANT(TC, TR)                                                                                  \
    do {                                                                                                         \
        if (vec && sr) hipLaunchKernelGGL((k_quantize<TC, TR, 4, true>), grid, dim3(kBlock), 0, s, x, M, C, ld,  \
                                          group, scale, cfg, q_fold, ld_fold, q_t, ld_t, desc, eb, pg, (int)tiled, tm);          \
        else if (vec) hipLaunchKernelGGL((k_quantize<TC, TR, 4, false>), grid, dim3(kBlock), 0, s, x, M, C, ld,  \
                                         group, scale, cfg, q_fold, ld_fold, q_t, ld_t, desc, eb, pg, (int)tiled, tm);           \
        else if (sr) hipLaunchKernelGGL((k_quantize<TC, TR, 1, true>), grid, dim3(kBlock), 0, s, x, M, C, ld,    \
                                        group, scale, cfg, q_fold, ld_fold, q_t, ld_t, desc, eb, pg, (int)tiled, tm);            \
        else hipLaunchKernelGGL((k_quantize<TC, TR, 1, false>), grid, dim3(kBlock), 0, s, x, M, C, ld, group,    \
                                scale, cfg, q_fold, ld_fold, q_t, ld_t, desc, eb, pg, (int)tiled, tm);                           \
    } while (0)
    if (tc == 64 && tr == 64) SQ_LAUNCH_QUANT(64, 64);
    else if (tc == 64) SQ_LAUNCH_QUANT(64, 128);
    else if (tr == 64) SQ_LAUNCH_QUANT(128, 64);
    else SQ_LAUNCH_QUANT(128, 128);
#undef SQ_LAUNCH_QUANT
    return hipGetLastError();
}

// At most kBnQBlocks row blocks of whole 256-row steps: with M <= 2^24 a block
// holds at most 16384 rows, and its int32 sums stay below 2^30.
constexpr int64_t kBnQBlocks = 1024;
static int64_t bn_rows_per_block(int64_t M) {
    return round_up((M + kBnQBlocks - 1) / kBnQBlocks, kBnQRows);
}
int64_t quantize_bn_blocks(int64_t M) {
    const int64_t rows = bn_rows_per_block(std::max<int64_t>(M, 1));
    return (M + rows - 1) / rows;
}

bool quantize_bn_ok(const float* dy, int64_t C, int64_t ld) { return C % 8 == 0 && C <= 64 * 65535 && colmax_vec(dy, ld); }

hipError_t launch_quantize_bn(const float* dy, int64_t M, int64_t C, int64_t ld, const uint8_t* group,
                              const sq_scale* scale, const QuantCfg& cfg, int8_t* q, int64_t ldc, const int8_t* xq,
                              int64_t ld_x, const sq_l1bn_channel* chan, int32_t* part, hipStream_t s) {
    if (M <= 0 || C <= 0) return hipSuccess;
    if (!quantize_bn_ok(dy, C, ld) || ldc % 8 || ld_x % 8) return hipErrorInvalidValue;
    const dim3 grid((unsigned)quantize_bn_blocks(M), (unsigned)((C + 63) / 64));
    if (cfg.round_mode == SQ_ROUND_STOCHASTIC)
        hipLaunchKernelGGL(k_quantize_bn<true>, grid, dim3(kBnQThreads), 0, s, dy, M, C, ld, group, scale, cfg, q, ldc, xq,
                           ld_x, chan, bn_rows_per_block(M), part);
    else
        hipLaunchKernelGGL(k_quantize_bn<false>, grid, dim3(kBnQThreads), 0, s, dy, M, C, ld, group, scale, cfg, q, ldc,
                           xq, ld_x, chan, bn_rows_per_block(M), part);
    return hipGetLastError();
}

hipError_t launch_quantize_channels(const float* x, int64_t rows, int64_t cols, int64_t ld, int bits, int axis,
                                   int transpose, int8_t* q, int64_t ld_q, sq_scale* scales, uint32_t* partial,
                                   hipStream_t s) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int Q = (1 << (bits - 1)) - 1;
    if (axis == 0 && !transpose) {
        auto run = [&](auto lpr) {
            constexpr int LPR = decltype(lpr)::value, kRows = 256 / LPR;
            const dim3 grid((unsigned)std::min<int64_t>((rows + kRows - 1) / kRows, 8192));
            if (colmax_vec(x, ld))
                hipLaunchKernelGGL((k_quantize_rows<true, LPR>), grid, dim3(256), 0, s, x, rows, cols, ld, Q, scales, q, ld_q);
            else
                hipLaunchKernelGGL((k_quantize_rows<false, LPR>), grid, dim3(256), 0, s, x, rows, cols, ld, Q, scales, q, ld_q);
        };
        if (cols <= 16) run(std::integral_constant<int, 4>());
        else if (cols <= 32) run(std::integral_constant<int, 8>());
        else if (cols <= 64) run(std::integral_constant<int, 16>());
        else if (cols <= 128) run(std::integral_constant<int, 32>());
        else run(std::integral_constant<int, 64>());
        return hipGetLastError();
    }
    if (axis == 1) {
        int64_t slabs = 0;
        const hipError_t e = launch_colmax(x, rows, cols, ld, partial, &slabs, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_channel_scales_cols, dim3((unsigned)std::min<int64_t>((cols + 255) / 256, 4096)), dim3(256),
                           0, s, partial, slabs, cols, Q, scales);
    } else {
        hipLaunchKernelGGL(k_channel_scales_rows, dim3((unsigned)std::min<int64_t>((rows + 3) / 4, 8192)), dim3(256), 0,
                           s, x, rows, cols, ld, Q, scales);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_quantize_channels, dim3((unsigned)std::min<int64_t>((rows * cols + 255) / 256, 16384)),
                       dim3(256), 0, s, x, rows, cols, ld, axis, scales, Q, q, ld_q, transpose);
    return hipGetLastError();
}

}  // namespace sq
