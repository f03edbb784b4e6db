// Decode attention over the packed cache, portable vector-ALU version (gfx950), and the
// cross-split merge.
//
// One workgroup handles one (sequence, kv head) and one contiguous range of blocks ("split") and
// serves all g = Hq/Hkv query heads of that kv head.  Per block it evaluates, without ever
// materialising the reconstructed keys and values (arxiv 2506.04642 Eq. 5-8):
//   score_t = ( sum_c (q_c s_c) code_tc + sum_c q_c (z_c + m_c) ) / sqrt(d)         keys, Eq. 5, 7
//   o_c     = sum_t (p_t s_tg) code_tc + sum_t p_t z_tg + m_c sum_t p_t             values, Eq. 6, 8
// with an online softmax across blocks (flash decoding, App. A).  Raw residual tokens (Sec. 3.3,
// Eq. 9-10) and 16-bit layers go through the same code with scale 1, zero 0.
// The split's running (max, sum, output) goes to the workspace; join_kernel or merge_kernel combines the splits
// with the log-sum-exp identity, in a fixed order (no atomics), so results are reproducible.
#include "join.h"
#include <hip/hip_fp16.h>

namespace tadakv {
namespace {

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float widen16(uint16_t v, int dtype)
{
    if (dtype == 1) return __uint_as_float((uint32_t)v << 16);
    return __half2float(__ushort_as_half(v));
}
__device__ __forceinline__ float f16_val(uint16_t h) { return __half2float(__ushort_as_half(h)); }
// binary32 -> the 16-bit type, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t narrow16_rne(float f, int dtype)
{
    if (dtype == 1) {
        const uint32_t u = __float_as_uint(f);
        return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
    }
    return __half_as_ushort(__float2half_rn(f));
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// index of the 32-bit word that holds key codes (t, c0 .. c0 + 32/B - 1)
template <int B> __device__ __forceinline__ int k_word(int t, int c0)
{
    const int tt = t >> 4, n = t & 15, cg = c0 >> 4;
    if (B == 8) return ((((tt * 2 + (cg & 1)) * 4 + (cg >> 1)) * 16 + n) << 2) + ((c0 & 15) >> 2);
    if (B == 4) return (((tt * 4 + (cg >> 1)) * 16 + n) << 2) + (cg & 1) * 2 + ((c0 & 15) >> 3);
    if (B == 2) return ((((tt >> 1) * 4 + (cg >> 1)) * 16 + n) << 2) + (tt & 1) * 2 + (cg & 1);
    return t * 64 + (c0 >> 1); // raw 16-bit rows
}
// index of the word that holds value codes (t0 .. t0 + 32/B - 1, c)
template <int B> __device__ __forceinline__ int v_word(int t0, int c, int nt)
{
    const int tt = t0 >> 4, ct = c >> 4, n = c & 15;
    if (B == 8) return (((ct * nt + tt) * 16 + n) << 2) + ((t0 & 15) >> 2);
    if (B == 4) return ((((ct >> 1) * nt + tt) * 16 + n) << 2) + (ct & 1) * 2 + ((t0 & 15) >> 3);
    return ((((ct >> 2) * nt + tt) * 16 + n) << 2) + (ct & 3);
}

struct Smem {
    float *qf, *qs, *part, *ps, *pz, *psum, *alpha, *mrun, *lrun, *bpart, *vmean, *pp;
    uint32_t *kc, *vc, *vmeta;
    uint16_t *xk, *xv; // cross-head mean tiles [G][128] of the block (keys, values)
};

// One block (or one chunk of raw tokens) of one unit.  KB/VB = 16 means raw rows.
template <int KB, int VB>
__device__ __forceinline__ void process_block(const DecodeArgs &a, const Smem &sm, int ntok,
                                              const unsigned char *kcodes, const unsigned char *kscale,
                                              const unsigned char *kzero, const unsigned char *kmean,
                                              const unsigned char *vcodes, const unsigned char *vmeta,
                                              const unsigned char *vmean, const unsigned char *xmean_k,
                                              const unsigned char *xmean_v, float (&acc)[kMaxGroupQ / 2])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = a.g;
    const int G = (KB == 16) ? 32 : a.geom.G;     // row stride of the LDS score arrays
    const int ng = (VB == 16) ? 1 : kHeadDim / a.geom.Gc;
    const int nt = a.geom.G >> 4;

    __syncthreads(); // the previous block's readers are done with the staging buffers

    // ---- stage codes and value metadata
    {
        const int kbytes = (KB == 16) ? ntok * 256 : a.geom.G * kHeadDim * KB / 8;
        for (int i = tid; i < kbytes / 16; i += kThreads) ((uint4 *)sm.kc)[i] = ((const uint4 *)kcodes)[i];
        const int vbytes = (VB == 16) ? ntok * 256 : a.geom.G * kHeadDim * VB / 8;
        for (int i = tid; i < vbytes / 16; i += kThreads) ((uint4 *)sm.vc)[i] = ((const uint4 *)vcodes)[i];
        if (xmean_k) {
            // cross-head mean (Eq. 1-2): one binary16 row per token, shared by all kv heads
            for (int i = tid; i < a.geom.G * 16; i += kThreads) {
                ((uint4 *)sm.xk)[i] = ((const uint4 *)xmean_k)[i];
                ((uint4 *)sm.xv)[i] = ((const uint4 *)xmean_v)[i];
            }
        }
        if (VB != 16) {
            for (int i = tid; i < a.geom.G * ng; i += kThreads) sm.vmeta[i] = ((const uint32_t *)vmeta)[i];
            if (tid < kHeadDim) sm.vmean[tid] = vmean ? f16_val(((const uint16_t *)vmean)[tid]) : 0.0f;
        }
    }
    // ---- fold the key scale into q, and the zero / mean terms into one number per head
    {
        const int c = tid & 127, hsel = tid >> 7;
        float s = 1.0f, zm = 0.0f;
        if (KB != 16) {
            s = f16_val(((const uint16_t *)kscale)[c]);
            zm = f16_val(((const uint16_t *)kzero)[c]);
            if (kmean) zm += f16_val(((const uint16_t *)kmean)[c]);
        }
        for (int i = hsel; i < g; i += 2) {
            const float qv = sm.qf[i * kHeadDim + c];
            sm.qs[i * kHeadDim + c] = qv * s;
            const float bsum = wave_sum(qv * zm);
            if (lane == 0) sm.bpart[i * 2 + (wave & 1)] = bsum;
        }
    }
    __syncthreads();

    // ---- scores: each work item is (token, head, channel half)
    for (int idx = tid; idx < ntok * g * 2; idx += kThreads) {
        const int t = idx % ntok, rest = idx / ntok;
        const int i = rest % g, half = rest / g;
        const float *qrow = sm.qs + i * kHeadDim;
        float s = 0.0f;
        constexpr int per = (KB == 16) ? 2 : 32 / KB;
        for (int c0 = half * 64; c0 < half * 64 + 64; c0 += per) {
            const uint32_t w = sm.kc[k_word<KB>(t, c0)];
            if (KB == 16) {
                s += qrow[c0] * widen16((uint16_t)(w & 0xFFFFu), a.geom.dtype);
                s += qrow[c0 + 1] * widen16((uint16_t)(w >> 16), a.geom.dtype);
            } else {
#pragma unroll
                for (int e = 0; e < per; e++)
                    s += qrow[c0 + e] *
                         (float)((w >> (8 * (e & 3) + (KB & 15) * (e >> 2))) & ((1u << (KB & 15)) - 1u));
            }
        }
        if (KB != 16 && xmean_k) {
            const float *qraw = sm.qf + i * kHeadDim;
            const uint16_t *mrow = sm.xk + t * kHeadDim;
            for (int c = half * 64; c < half * 64 + 64; c++) s += qraw[c] * f16_val(mrow[c]);
        }
        sm.part[(half * g + i) * G + t] = s;
    }
    __syncthreads();

    // ---- online softmax: wave w owns heads w, w+4
    const float sc_scale = 0.08838834764831845f * kLog2e; // 1/sqrt(128) in the exp2 domain
    for (int i = wave; i < g; i += 4) {
        const float beta = sm.bpart[i * 2] + sm.bpart[i * 2 + 1];
        float sv[2];
        float bmax = -INFINITY;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int t = lane + 64 * k;
            sv[k] = -INFINITY;
            if (t < ntok) sv[k] = (sm.part[i * G + t] + sm.part[(g + i) * G + t] + beta) * sc_scale;
            bmax = fmaxf(bmax, sv[k]);
        }
        bmax = wave_max(bmax);
        const float m_old = sm.mrun[i];
        const float m_new = fmaxf(m_old, bmax);
        const float alpha = exp2f(m_old - m_new);
        float psum = 0.0f;
        float pz[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int t = lane + 64 * k;
            if (t < ntok) {
                const float p = exp2f(sv[k] - m_new);
                psum += p;
                sm.pp[i * G + t] = p;
                if (VB == 16) {
                    sm.ps[i * G + t] = p;
                } else {
                    for (int gam = 0; gam < ng; gam++) {
                        const uint32_t mz = sm.vmeta[t * ng + gam];
                        sm.ps[(i * G + t) * ng + gam] = p * f16_val((uint16_t)(mz & 0xFFFFu));
                        pz[gam] += p * f16_val((uint16_t)(mz >> 16));
                    }
                }
            }
        }
        psum = wave_sum(psum);
        if (VB != 16)
            for (int gam = 0; gam < ng; gam++) pz[gam] = wave_sum(pz[gam]);
        if (lane == 0) {
            sm.alpha[i] = alpha;
            sm.mrun[i] = m_new;
            sm.lrun[i] = sm.lrun[i] * alpha + psum;
            sm.psum[i] = psum;
            for (int gam = 0; gam < ng; gam++) sm.pz[i * 4 + gam] = pz[gam];
        }
    }
    __syncthreads();

    // ---- output: thread owns channel c for heads hsel, hsel+2, ...
    {
        const int c = tid & 127, hsel = tid >> 7;
        const int gam = (VB == 16) ? 0 : c / a.geom.Gc;
        float add[kMaxGroupQ / 2];
#pragma unroll
        for (int k = 0; k < kMaxGroupQ / 2; k++) add[k] = 0.0f;
        if (VB == 16) {
            const uint16_t *vr = (const uint16_t *)sm.vc;
            for (int t = 0; t < ntok; t++) {
                const float v = widen16(vr[t * kHeadDim + c], a.geom.dtype);
#pragma unroll
                for (int k = 0; k < kMaxGroupQ / 2; k++) {
                    const int i = hsel + 2 * k;
                    if (i < g) add[k] += sm.ps[i * G + t] * v;
                }
            }
        } else {
            constexpr int per = 32 / (VB & 15 ? VB & 15 : 16);
            for (int t0 = 0; t0 < ntok; t0 += per) {
                const uint32_t w = sm.vc[v_word<VB == 16 ? 8 : VB>(t0, c, nt)];
#pragma unroll
                for (int e = 0; e < per; e++) {
                    const float code =
                        (float)((w >> (8 * (e & 3) + (VB & 15) * (e >> 2))) & ((1u << (VB & 15)) - 1u));
#pragma unroll
                    for (int k = 0; k < kMaxGroupQ / 2; k++) {
                        const int i = hsel + 2 * k;
                        if (i < g) add[k] += sm.ps[(i * G + t0 + e) * ng + gam] * code;
                    }
                }
            }
        }
        if (VB != 16 && xmean_v) {
            for (int t = 0; t < ntok; t++) {
                const float mv = f16_val(sm.xv[t * kHeadDim + c]);
#pragma unroll
                for (int k = 0; k < kMaxGroupQ / 2; k++) {
                    const int i = hsel + 2 * k;
                    if (i < g) add[k] += sm.pp[i * G + t] * mv;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kMaxGroupQ / 2; k++) {
            const int i = hsel + 2 * k;
            if (i < g) {
                float extra = 0.0f;
                if (VB != 16) extra = sm.pz[i * 4 + gam] + sm.vmean[c] * sm.psum[i];
                acc[k] = acc[k] * sm.alpha[i] + add[k] + extra;
            }
        }
    }
}

template <int KB, int VB> __global__ __launch_bounds__(kThreads) void decode_split_valu_kernel(DecodeArgs a)
{
    extern __shared__ float lds[];
    const LayerGeom &gm = a.geom;
    const int g = a.g, G = gm.G;
    Smem sm;
    float *p = lds;
    sm.qf = p;     p += kMaxGroupQ * kHeadDim;
    sm.qs = p;     p += kMaxGroupQ * kHeadDim;
    sm.part = p;   p += 2 * g * G;
    sm.ps = p;     p += g * G * 4;
    sm.pz = p;     p += kMaxGroupQ * 4;
    sm.psum = p;   p += kMaxGroupQ;
    sm.alpha = p;  p += kMaxGroupQ;
    sm.mrun = p;   p += kMaxGroupQ;
    sm.lrun = p;   p += kMaxGroupQ;
    sm.bpart = p;  p += kMaxGroupQ * 2;
    sm.vmean = p;  p += kHeadDim;
    sm.pp = p;     p += g * G;
    sm.vmeta = (uint32_t *)p; p += G * 4;
    // staging sized for the widest case: 8-bit codes of a block, or 32 raw 16-bit rows
    const int code_words = G * kHeadDim * 8 / 32 > 32 * 64 ? G * kHeadDim * 8 / 32 : 32 * 64;
    sm.kc = (uint32_t *)p; p += code_words;
    sm.vc = (uint32_t *)p; p += code_words;
    sm.xk = (uint16_t *)p; p += (gm.mean_mode == 1 ? G * kHeadDim / 2 : 0);
    sm.xv = (uint16_t *)p;

    const int sp = blockIdx.x, u = blockIdx.y;
    const int b = u / a.n_kv_heads, h = u % a.n_kv_heads;
    const int tid = threadIdx.x;

    // q of this kv head's g query heads, widened
    for (int i = tid; i < g * kHeadDim; i += kThreads)
        sm.qf[i] = widen16(a.q[((long long)b * a.n_q_heads + h * g) * kHeadDim + i], gm.dtype);
    if (tid < kMaxGroupQ) {
        sm.mrun[tid] = -INFINITY;
        sm.lrun[tid] = 0.0f;
    }
    float acc[kMaxGroupQ / 2];
#pragma unroll
    for (int k = 0; k < kMaxGroupQ / 2; k++) acc[k] = 0.0f;

    const int nb_seq = seq_blocks(a, b), r_seq = seq_resid(a, b); // this sequence's packed blocks and raw tokens
    const int work = nb_seq + (r_seq > 0 ? 1 : 0);
    const int w0 = sp * a.blocks_per_split;
    int w1 = w0 + a.blocks_per_split;
    if (w1 > work) w1 = work;
    const int b_end = w1 < nb_seq ? w1 : nb_seq;

    for (int j = w0; j < b_end; j++) {
        const unsigned char *rec = a.layer + record_offset(gm, a.n_kv_heads, b, u % a.n_kv_heads, j);
        if (KB == 16) {
            for (int t0 = 0; t0 < G; t0 += 32)
                process_block<16, 16>(a, sm, 32, rec + gm.k_codes + t0 * 256, nullptr, nullptr, nullptr,
                                      rec + gm.v_codes + t0 * 256, nullptr, nullptr, nullptr, nullptr, acc);
        } else {
            const unsigned char *xm = gm.mean_mode == 1
                                          ? a.layer + xmean_offset(gm, b, j, 0)
                                          : nullptr;
            process_block<KB, VB>(a, sm, G, rec + gm.k_codes, rec + gm.k_scale, rec + gm.k_zero,
                                  gm.k_mean >= 0 ? rec + gm.k_mean : nullptr, rec + gm.v_codes,
                                  rec + gm.v_meta, gm.v_mean >= 0 ? rec + gm.v_mean : nullptr, xm,
                                  xm ? xm + G * kHeadDim * 2 : nullptr, acc);
        }
    }
    if (w0 < w1 && w1 > nb_seq && r_seq > 0) {
        const unsigned char *kr = a.layer + gm.k_resid_off + (long long)u * gm.R * 256;
        const unsigned char *vr = a.layer + gm.v_resid_off + (long long)u * gm.R * 256;
        for (int t0 = 0; t0 < r_seq; t0 += 32) {
            const int n = r_seq - t0 < 32 ? r_seq - t0 : 32;
            process_block<16, 16>(a, sm, n, kr + t0 * 256, nullptr, nullptr, nullptr, vr + t0 * 256,
                                  nullptr, nullptr, nullptr, nullptr, acc);
        }
    }
    __syncthreads();

    // partial result of this split
    const int c = tid & 127, hsel = tid >> 7;
#pragma unroll
    for (int k = 0; k < kMaxGroupQ / 2; k++) {
        const int i = hsel + 2 * k;
        if (i < g) {
            float *dst = a.ws + (((long long)u * g + i) * a.n_splits + sp) * kPartialStride;
            dst[c] = acc[k];
            if (c == 0) {
                dst[kHeadDim] = sm.mrun[i];
                dst[kHeadDim + 1] = sm.lrun[i];
            }
        }
    }
}

// Cross-split merge (flash decoding, App. A):
//   out[b, head] = sum_j o_j 2^(m_j - M) / sum_j l_j 2^(m_j - M),  M = max_j m_j.
// One workgroup of NW waves per query head, a lane owns two channels; wave w takes the splits w, w + NW, ... in
// rising order, NB at a time, with a running maximum of its own, and the waves' states are joined in wave order,
// so the result does not depend on timing.  Bound by latency: what the split kernel has just written comes from
// memory, and with NW x NB at least the number of splits all of it is requested at once (launch_decode_merge).
// Against two passes over the splits, the maxima first, with four waves (us a call): 4 x 16461 with the mean over the
// heads, 64 splits, two layers, 65.2 -> 64.4.  More splits a wave (16) or
// one count for all were slower: a wave's loads are then issued in two groups, or the unused ones cost.
template <int NB, int NW> __global__ __launch_bounds__(64 * NW) void merge_kernel(DecodeArgs a)
{
    __shared__ float red[NW][3][64];
    __shared__ float mx[NW];
    asm volatile("" : : "s"(a.g), "s"(a.n_kv_heads), "s"(a.n_q_heads), "s"(a.n_splits), "s"(a.uneven), "s"(a.ws), "s"(a.out), "s"(a.out16),
                 "s"(a.len_dev), "s"(a.xo), "s"(a.n_blocks), "s"(a.n_xr)); // (see decode_args_here)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int uq = blockIdx.x; // (unit, head-in-group)
    const int u = uq / a.g, i = uq % a.g;
    int ns;
    const float *base = a.ws + partial_row(a, u, i, ns) * kPartialStride;
    float M = -INFINITY, n0 = 0.0f, n1 = 0.0f, den = 0.0f;
    for (int j0 = wave; j0 < ns; j0 += NW * NB) {
        float2 ml[NB], o[NB];
#pragma unroll
        for (int k = 0; k < NB; k++) {
            ml[k] = float2{-INFINITY, 0.0f};
            o[k] = float2{0.0f, 0.0f};
            if (j0 + NW * k < ns) { // (nothing is read in the place of a split that does not exist: 0 x inf is NaN)
                const float *pj = base + (j0 + NW * k) * kPartialStride;
                ml[k] = *(const float2 *)(pj + kHeadDim);
                o[k] = *(const float2 *)(pj + 2 * lane);
            }
        }
        float m_new = M;
#pragma unroll
        for (int k = 0; k < NB; k++) m_new = fmaxf(m_new, ml[k].x);
        const float alpha = M == -INFINITY ? 0.0f : exp2f(M - m_new);
        n0 *= alpha;
        n1 *= alpha;
        den *= alpha;
#pragma unroll
        for (int k = 0; k < NB; k++) {
            const float w = ml[k].x == -INFINITY ? 0.0f : exp2f(ml[k].x - m_new);
            n0 += o[k].x * w;
            n1 += o[k].y * w;
            den += ml[k].y * w;
        }
        M = m_new;
    }
    red[wave][0][lane] = n0;
    red[wave][1][lane] = n1;
    red[wave][2][lane] = den;
    if (lane == 0) mx[wave] = M;
    __syncthreads();
    M = mx[0];
#pragma unroll
    for (int w = 1; w < NW; w++) M = fmaxf(M, mx[w]);
    n0 = n1 = den = 0.0f;
    if (a.xo && a.n_blocks > 0) {
        // cross-head mean in kernels of its own: the value mean plane's share, already relative to the largest
        // split maximum (one term per range)
        const float *xb = a.xo + (long long)uq * a.n_xr * kHeadDim;
#pragma unroll 8
        for (int r = wave; r < a.n_xr; r += NW) {
            const float2 o = *(const float2 *)(xb + r * kHeadDim + 2 * lane);
            n0 += o.x;
            n1 += o.y;
        }
        __shared__ float xr[NW][2][64];
        xr[wave][0][lane] = n0;
        xr[wave][1][lane] = n1;
        __syncthreads();
        n0 = n1 = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; w++) {
            n0 += xr[w][0][lane];
            n1 += xr[w][1][lane];
        }
    }
    if (wave != 0) return;
#pragma unroll
    for (int w = 0; w < NW; w++) {
        const float s = mx[w] == -INFINITY ? 0.0f : exp2f(mx[w] - M);
        n0 += red[w][0][lane] * s;
        n1 += red[w][1][lane] * s;
        den += red[w][2][lane] * s;
    }
    const int b = u / a.n_kv_heads, h = u % a.n_kv_heads;
    float2 r;
    // a sequence that holds no token (every split empty, M == -inf) gives zeros
    r.x = M == -INFINITY ? 0.0f : n0 / den;
    r.y = M == -INFINITY ? 0.0f : n1 / den;
    const long long o = ((long long)b * a.n_q_heads + h * a.g + i) * kHeadDim + 2 * lane;
    if (a.out16) *(uint32_t *)(a.out16 + o) = (uint32_t)narrow16_rne(r.x, a.geom.dtype) | ((uint32_t)narrow16_rne(r.y, a.geom.dtype) << 16);
    else *(float2 *)(a.out + o) = r;
    // a decode step on device-resident lengths ends here: the state after the step becomes the current
    // one (no workgroup of this kernel reads the lengths)
    if (a.len_dev && blockIdx.x == 0 && lane == 0) a.len_dev[4 * a.batch] = (a.len_dev[4 * a.batch] & 1) ^ 1;
}

// The same for up to kJoinSplits splits, by a wave per query head (join.h): no LDS and no barrier.  The kernel alone (us, a
// workgroup of four waves per head -> this): 4 splits 3.0 -> 2.9, 7 2.7 -> 2.4, 33 3.7 -> 3.3, 128 units x 4 heads of 2 to 8 splits 2.6 -> 2.2.
__global__ __launch_bounds__(64) void join_kernel(DecodeArgs a)
{
    // (see decode_args_here)
    asm volatile("" : : "s"(a.g), "s"(a.n_kv_heads), "s"(a.n_splits), "s"(a.uneven), "s"(a.ws), "s"(a.out), "s"(a.out16), "s"(a.len_dev));
    const int uq = blockIdx.x, lane = threadIdx.x;
    int ns;
    const float *base = a.ws + partial_row(a, uq / a.g, uq % a.g, ns) * kPartialStride;
    join_f32x4 joined[1];
    if (ns <= kJoinFew) join_rows<kJoinFew / 2, 1, 0>(base, ns, 1, joined);
    else join_rows<kJoinSplits / 2, 1, 0>(base, ns, 1, joined);
    const join_f32x4 &r = joined[0];
    if (lane < 32) {
        const long long o = (long long)uq * kHeadDim + 4 * lane; // (n_q_heads = n_kv_heads g)
        if (a.out16)
            *(uint2 *)(a.out16 + o) = uint2{(uint32_t)narrow16_rne(r.x, a.geom.dtype) | ((uint32_t)narrow16_rne(r.y, a.geom.dtype) << 16),
                                            (uint32_t)narrow16_rne(r.z, a.geom.dtype) | ((uint32_t)narrow16_rne(r.w, a.geom.dtype) << 16)};
        else *(join_f32x4 *)(a.out + o) = r;
    }
    if (a.len_dev && uq == 0 && lane == 0) a.len_dev[4 * a.batch] = (a.len_dev[4 * a.batch] & 1) ^ 1; // (see merge_kernel)
}

// Four codes of a word's field f (consecutive channels of a key word, consecutive tokens of a value
// word), code y in byte y.
template <int B> __device__ __forceinline__ uint32_t field_of(uint32_t w, int f)
{
    return B == 8 ? w : (w >> (B * f)) & (B == 4 ? 0x0F0F0F0Fu : 0x03030303u);
}
// mean + (zero + scale * code), one rounding per operation (the product of an 11-bit significand and a
// code of at most 8 bits is exact)
__device__ __forceinline__ float rebuilt(float m, float z, float s, uint32_t four, int y)
{
    return __fadd_rn(m, __fadd_rn(z, __fmul_rn(s, (float)((four >> (8 * y)) & 0xFFu))));
}
// four consecutive 16-bit values
__device__ __forceinline__ float4 widen4(uint2 w, int dtype)
{
    return float4{widen16((uint16_t)(w.x & 0xFFFFu), dtype), widen16((uint16_t)(w.x >> 16), dtype),
                  widen16((uint16_t)(w.y & 0xFFFFu), dtype), widen16((uint16_t)(w.y >> 16), dtype)};
}
__device__ __forceinline__ float4 half4(const unsigned char *p) { return widen4(*(const uint2 *)p, 0); }

// Tokens t0 .. t0 + 3, channels c0 .. c0 + 3 of a packed block: a key word holds codes of one token
// (one word per token), a value word those of one channel (one word per channel); either way the
// sixteen codes are one field of four words.
template <int B> __device__ __forceinline__ void rebuild_keys(const LayerGeom &gm, const unsigned char *rec, const uint16_t *xm, int t0, int c0, float4 (&x)[4])
{
    constexpr int PW = 32 / B; // codes per word
    const uint32_t *w = (const uint32_t *)(rec + gm.k_codes);
    const float4 s = half4(rec + gm.k_scale + c0 * 2), z = half4(rec + gm.k_zero + c0 * 2);
    const float4 m = gm.k_mean >= 0 ? half4(rec + gm.k_mean + c0 * 2) : float4{0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t four[4];
#pragma unroll
    for (int i = 0; i < 4; i++) four[i] = field_of<B>(w[k_word<B>(t0 + i, c0 - c0 % PW)], c0 % PW / 4);
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float4 mt = xm ? half4((const unsigned char *)(xm + (t0 + i) * kHeadDim + c0)) : m;
        x[i] = float4{rebuilt(mt.x, z.x, s.x, four[i], 0), rebuilt(mt.y, z.y, s.y, four[i], 1),
                      rebuilt(mt.z, z.z, s.z, four[i], 2), rebuilt(mt.w, z.w, s.w, four[i], 3)};
    }
}
template <int B> __device__ __forceinline__ void rebuild_values(const LayerGeom &gm, const unsigned char *rec, const uint16_t *xm, int t0, int c0, float4 (&x)[4])
{
    constexpr int PW = 32 / B;
    const uint32_t *w = (const uint32_t *)(rec + gm.v_codes);
    const int ng = kHeadDim / gm.Gc, nt = gm.G / 16;
    const float4 m = gm.v_mean >= 0 ? half4(rec + gm.v_mean + c0 * 2) : float4{0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t four[4];
#pragma unroll
    for (int e = 0; e < 4; e++) four[e] = field_of<B>(w[v_word<B>(t0 - t0 % PW, c0 + e, nt)], t0 % PW / 4);
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const uint32_t sz = *(const uint32_t *)(rec + gm.v_meta + ((t0 + i) * ng + c0 / gm.Gc) * 4);
        const float s = f16_val((uint16_t)(sz & 0xFFFFu)), z = f16_val((uint16_t)(sz >> 16));
        const float4 mt = xm ? half4((const unsigned char *)(xm + (t0 + i) * kHeadDim + c0)) : m;
        x[i] = float4{rebuilt(mt.x, z, s, four[0], i), rebuilt(mt.y, z, s, four[1], i), rebuilt(mt.z, z, s, four[2], i),
                      rebuilt(mt.w, z, s, four[3], i)};
    }
}

// Reconstruction (Eq. 7-8): x^ = mean + (zero + scale * code) in binary32, one rounding per
// operation, in that order; raw rows (16-bit layers, the residual buffer) are widened.
// out [batch][t_cap][n_kv_heads][128] binary32.  Bound by writing it: 512 bytes per row against the
// 70 to 150 it is made from.  A workgroup takes G consecutive tokens of one unit and one side, a thread
// four tokens x four channels of them -- the square that is one field of four words, of keys and of
// values alike --, so a word is read by the lanes that use it only and a store of the wave covers two
// whole rows.  The units of a block are adjacent in launch order: together they write whole tokens.
// With `pad` the rows past a sequence's length are written too, as zeros.
// Measured (2 sequences of 8197 tokens, 8 kv heads, 4 bits: 134 MB out): 27.7 us, 4.8 TB/s of output (one
// element per thread and step: 63 us); into buffers that no cache holds, the whole call with the padding
// written here 43.5 us, 105 us with two clearing launches before it.  Stores that bypass the caches: 38.6 us
// into such buffers, but 40 instead of 27.7 us where the outputs stay cached for their reader.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5, 8))) void dequant_kernel(DequantArgs q, long long n_items)
{
    const DecodeArgs &a = q.d;
    const LayerGeom &gm = a.geom;
    const int G = gm.G, U = a.batch * a.n_kv_heads, which = blockIdx.y;
    float *out = which == 0 ? q.k_out : q.v_out;
    if (!out) return;
    const int bits = which == 0 ? gm.k_bits : gm.v_bits;
    const long long tstride = (long long)a.n_kv_heads * kHeadDim;
    const int c0 = (threadIdx.x & 31) * 4;
    for (long long it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int u = (int)(it % U), j = (int)(it / U);
        const int b = u / a.n_kv_heads, h = u % a.n_kv_heads;
        const int nb = seq_blocks(a, b), r = seq_resid(a, b);
        float *dst = out + (((long long)b * q.t_cap + (long long)j * G) * a.n_kv_heads + h) * kHeadDim + c0;
        const unsigned char *rec = a.layer + (j < nb ? record_offset(gm, a.n_kv_heads, b, h, j) : 0);
        if (j < nb && bits != 16) {
            const uint16_t *xm = gm.mean_mode == 1 ? (const uint16_t *)(a.layer + xmean_offset(gm, b, j, which)) : nullptr;
            for (int t0 = (threadIdx.x >> 5) * 4; t0 < G; t0 += kThreads / 32 * 4) {
                float4 x[4];
                if (which == 0) {
                    if (bits == 2) rebuild_keys<2>(gm, rec, xm, t0, c0, x);
                    else if (bits == 4) rebuild_keys<4>(gm, rec, xm, t0, c0, x);
                    else rebuild_keys<8>(gm, rec, xm, t0, c0, x);
                } else {
                    if (bits == 2) rebuild_values<2>(gm, rec, xm, t0, c0, x);
                    else if (bits == 4) rebuild_values<4>(gm, rec, xm, t0, c0, x);
                    else rebuild_values<8>(gm, rec, xm, t0, c0, x);
                }
#pragma unroll
                for (int i = 0; i < 4; i++) *(float4 *)(dst + (t0 + i) * tstride) = x[i];
            }
            continue;
        }
        // raw rows: a block of a 16-bit layer, or what lies in the residual buffer behind the last block
        const unsigned char *raw = j < nb ? rec + (which == 0 ? gm.k_codes : gm.v_codes)
                                          : a.layer + (which == 0 ? gm.k_resid_off : gm.v_resid_off) +
                                                ((long long)u * gm.R + (long long)(j - nb) * G) * 256;
        const int n_raw = j < nb ? G : r - (j - nb) * G; // (tokens from here on; may be negative or exceed G)
        const long long room = q.t_cap - (long long)j * G;
        const int n_out = q.pad && room < G ? (int)room : G;
        for (int t = threadIdx.x >> 5; t < n_out; t += kThreads / 32) {
            if (t < n_raw) *(float4 *)(dst + t * tstride) = widen4(*(const uint2 *)(raw + t * 256 + c0 * 2), gm.dtype);
            else if (q.pad) *(float4 *)(dst + t * tstride) = float4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
}

template <int KB, int VB> hipError_t launch_one(const DecodeArgs &a, hipStream_t s)
{
    const int g = a.g, G = a.geom.G;
    size_t floats = 2 * kMaxGroupQ * kHeadDim + 2 * g * G + g * G * 4 + kMaxGroupQ * 4 + 4 * kMaxGroupQ +
                    kMaxGroupQ * 2 + kHeadDim + g * G + G * 4;
    if (a.geom.mean_mode == 1) floats += G * kHeadDim; // two binary16 mean tiles
    const size_t code_words = (size_t)G * kHeadDim * 8 / 32 > 32 * 64 ? (size_t)G * kHeadDim * 8 / 32 : 32 * 64;
    const size_t lds = (floats + 2 * code_words) * 4;
    static size_t granted = 0;
    if (lds > 64 * 1024 && lds > granted) {
        hipError_t e = hipFuncSetAttribute((const void *)decode_split_valu_kernel<KB, VB>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        granted = lds;
    }
    dim3 grid(a.n_splits, a.batch * a.n_kv_heads);
    (void)hipGetLastError(); // drop any stale error left by earlier runtime calls of this thread
    hipLaunchKernelGGL((decode_split_valu_kernel<KB, VB>), grid, dim3(kThreads), lds, s, a);
    return note_launch(hipGetLastError());
}

} // namespace

hipError_t launch_decode_split_valu(const DecodeArgs &a, hipStream_t s)
{
    if (a.uneven) return hipErrorInvalidValue; // (this kernel takes one split count for all)
    if (a.batch * a.n_kv_heads > 65535) return hipErrorInvalidValue;
    const int kb = a.geom.k_bits, vb = a.geom.v_bits;
    if ((kb == 16) != (vb == 16)) return hipErrorInvalidValue; // mixed raw / packed sides: not built
    if (kb == 16) return launch_one<16, 16>(a, s);
#define TADAKV_CASE(K_, V_) if (kb == K_ && vb == V_) return launch_one<K_, V_>(a, s);
    TADAKV_CASE(2, 2) TADAKV_CASE(2, 4) TADAKV_CASE(2, 8)
    TADAKV_CASE(4, 2) TADAKV_CASE(4, 4) TADAKV_CASE(4, 8)
    TADAKV_CASE(8, 2) TADAKV_CASE(8, 4) TADAKV_CASE(8, 8)
#undef TADAKV_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_dequant(const DequantArgs &q, hipStream_t s)
{
    const DecodeArgs &a = q.d;
    const int U = a.batch * a.n_kv_heads, G = a.geom.G;
    if (U > 65535) return hipErrorInvalidValue;
    // groups of G tokens per unit: the longest sequence's blocks and raw rows, or all that the outputs hold
    const long long per = q.pad ? ((long long)q.t_cap + G - 1) / G : (long long)a.n_blocks + (a.r + G - 1) / G;
    const long long items = per * U;
    const int grid = (int)(items < (1 << 22) ? items : 1 << 22); // (a workgroup takes several items beyond that)
    (void)hipGetLastError(); // drop any stale error left by earlier runtime calls of this thread
    hipLaunchKernelGGL(dequant_kernel, dim3(grid, 2), dim3(kThreads), 0, s, q, items);
    return note_launch(hipGetLastError());
}

hipError_t launch_decode_merge(const DecodeArgs &a, hipStream_t s)
{
    dim3 grid(a.batch * a.n_q_heads);
    (void)hipGetLastError(); // drop any stale error left by earlier runtime calls of this thread
    // everything requested at once: up to 34 splits by one wave per query head, else 8 or 9 splits a wave, 4 to 16 waves (up to
    // 36, 72, 128 splits: 32 or 64 for the chunks and a few for the raw tokens).  Where the value mean plane's share waits
    // to be added (xo: 1, 2, 3, ... kv heads with the mean over the heads) up to 8 splits by 2 a wave: with 9, most of them not
    // there, one kv head of 300 tokens takes 23.56 instead of 23.32 us a call, two of 4 x 200 20.88 instead of 20.63.
    const int ns = a.uneven ? a.uneven_most : a.n_splits;
    if (ns <= kJoinSplits && !a.xo) hipLaunchKernelGGL(join_kernel, grid, dim3(64), 0, s, a);
    else if (ns <= 8) hipLaunchKernelGGL((merge_kernel<2, 4>), grid, dim3(256), 0, s, a);
    else if (ns <= 36) hipLaunchKernelGGL((merge_kernel<9, 4>), grid, dim3(256), 0, s, a);
    else if (ns <= 72) hipLaunchKernelGGL((merge_kernel<9, 8>), grid, dim3(512), 0, s, a);
    else hipLaunchKernelGGL((merge_kernel<8, 16>), grid, dim3(1024), 0, s, a);
    return note_launch(hipGetLastError());
}

} // namespace tadakv
