// Decode attention over a layer that is stored in 16 bits (k_bits == v_bits == 16) on the matrix cores
// (gfx950): softmax attention of one query per sequence over raw rows (arxiv 2506.04642 Eq. 5-6 with
// K^ = K, V^ = V; Sec. 3.3 "residual tokens" take the same path), flash decoding over splits (App. A).
//
// Bound: reading the cache, 512 bytes per (unit, token); per such token 4 g x 128 multiply-adds, which
// the vector ALUs could only just keep up with at 4 query heads and not at 8, while the matrix cores do
// both products in a third of the time the bytes take:
//   scores  S^T[token][head] = K Q^T    v_mfma_f32_16x16x32_{bf16,f16}: products of 16-bit values are exact
//   output  O^T[channel][head] += V^T P^T  v_mfma_f32_16x16x4_f32: the weights stay in binary32, no limbs
// The lane layouts fit without any exchange: S^T leaves a lane (row = lane / 16, n = lane % 16) with the
// scores of head n for tokens 4 row + i of a 16-token tile, and that is where the B operand of the second
// product wants the weights if its k-slot `row` of step (tile, i) stands for that token; the A operand's
// value rows are then loaded as 16-byte pieces, whole rows of 256 bytes per quarter of the wave (operand
// row n of step ct is channel 8 n + ct).  A head's softmax state and its output live in one lane column,
// so rescaling needs no exchange either.
//
// Work split: one workgroup (kRawWaves waves) per (sequence, kv head, split); a wave takes chunks of 32 tokens,
// the splits and their waves interleaved chunk by chunk; the unit's raw buffer follows the packed rows as
// further chunks (short ones masked).  A chunk's key rows are requested as soon as the chunk before has
// gone through the score product, its value rows as soon as that chunk has gone through the output
// product: 16 KiB per wave on their way, straight into registers, no LDS before the final merge.
//
// Sums: a score is two sums of 64 channels, a chunk's product is summed from zero before it joins the output.
// Error against 64 bits (2-norm, relative; 4 sequences of 8213 tokens, bfloat16, four seeds): 3.04e-7, with one split 3.3e-7,
// one sequence of 40000 in one split 4.5e-7 (vector-ALU kernel 3.55e-7, 5.1e-7, 9.2e-7; one chain for the scores
// and the output: 3.9e-7, 8.8e-7, 18e-7).  It costs nothing in large calls and 0.1 to 0.35 us in small ones (one sequence
// of 1040 tokens 9.7 -> 10.05 us, of 8213 17.4 -> 17.75), whose last chunk waits for all its values.
//
// Measured (4 sequences of 8213 tokens, 8 kv heads x 4 query heads, 134 MB, the whole attention call with
// the merge launch): 36.5 us, 3.7 TB/s; the vector-ALU kernel, which such layers ran on before and still do
// where path 1 is asked for: 221 us.
#include "join.h"
#include <hip/hip_fp16.h>

namespace tadakv {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

constexpr int kRawWaves = kSplitWaves;
constexpr int kChunk = 32;       // tokens a wave takes at a time
constexpr int kRowBytes = 256;   // one token's row
constexpr float kScoreScale = 0.08838834764831845f * 1.4426950408889634f; // log2(e) / sqrt(128)

template <int DT> __device__ __forceinline__ v4f mfma_scores(const uint4 &k, const uint4 &q, v4f c)
{
    if (DT == 1) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, k), __builtin_bit_cast(v8bf, q), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, k), __builtin_bit_cast(v8h, q), c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma_output(float v, float p, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(v, p, c, 0, 0, 0); }
template <int DT> __device__ __forceinline__ float widen_lo(uint32_t w)
{
    if (DT == 1) return __uint_as_float(w << 16);
    return __half2float(__ushort_as_half((uint16_t)(w & 0xFFFFu)));
}
template <int DT> __device__ __forceinline__ float widen_hi(uint32_t w)
{
    if (DT == 1) return __uint_as_float(w & 0xFFFF0000u);
    return __half2float(__ushort_as_half((uint16_t)(w >> 16)));
}

// NT: a large launch (a.stream) requests its value rows past the caches.  The key rows stay ordinary reads: a request covers half of a
// cache line of every row, and past the caches each half is fetched by itself (16 x 3000 tokens, 8 kv heads: ordinary 41.7 us, values past the
// caches 35.2, both 38.4; 2 x 25000 45.4 / 39.2 / 41.4).
template <bool NT> __device__ __forceinline__ uint4 load_past(const unsigned char *p)
{
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    if (NT) return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4 *)p));
    return *(const uint4 *)p;
}
// JOIN: as in the kernel of the packed layers (decode_mfma.hip).  One sequence of 12016 tokens, whose splits are too many for it: 16.85 -> 16.73 us.
template <int DT, bool PG, bool JOIN, bool NT> __global__ __launch_bounds__(64 * kRawWaves) __attribute__((amdgpu_waves_per_eu(3, 8))) void decode_split_raw_kernel(DecodeArgs a)
{
    constexpr int NW = kRawWaves;
    constexpr int ST = 33; // floats per row of the state exchange (32 lanes of live columns, padded)
    __shared__ float state[NW][34 * ST];
    decode_args_here(a);
    const LayerGeom &gm = a.geom;
    const int lane = threadIdx.x & 63, row = lane >> 4, n = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int sp, u, ns, row0;
    unit_and_split(a, u, sp, ns, row0);
    const int g = a.g;
    const int b = u / a.n_kv_heads, h = u % a.n_kv_heads;
    const int sh = gm.G >> 6; // log2 of the chunks per block of the cache (32, 64, 128 tokens: 1, 2, 4)
    const int nb = seq_blocks(a, b), r = seq_resid(a, b);
    const int n_packed = nb << sh, n_items = n_packed + (r + kChunk - 1) / kChunk;
    const int first = sp + ns * wave, step = ns * NW; // this wave's chunks: first, first + step, ...

    // B operand of the scores: column n = query head n (columns g .. 15 are zero), channels 32 ks + 8 row .. + 7
    uint4 q[4];
    {
        const uint16_t *qp = a.q + ((long long)b * a.n_q_heads + h * g + (n < g ? n : 0)) * kHeadDim + 8 * row;
#pragma unroll
        for (int ks = 0; ks < 4; ks++) q[ks] = *(const uint4 *)(qp + 32 * ks);
    }
    const unsigned char *kres = a.layer + gm.k_resid_off + (long long)u * gm.R * kRowBytes;
    const unsigned char *vres = a.layer + gm.v_resid_off + (long long)u * gm.R * kRowBytes;

    // Paged placement: lane l keeps the block slot of this wave's chunk number 64 * (it / 64) + l, so
    // that no fetch waits for a lookup of its own.
    int slotv = 0;
    auto load_slots = [&](int it0) {
        int c = first + step * (it0 + lane);
        c = c < n_packed ? c : n_packed - 1; // (chunks of the raw buffer or past the end: not used)
        slotv = c < 0 ? 0 : (int)block_slot(gm, b, c >> sh);
    };
    // Rows of this wave's chunk number it: the first key row and the first value row, and the chunk's
    // last token (a short last chunk of the raw buffer reads its last row in the place of the missing
    // ones, whose scores and values are masked: nothing out of range).  Past the last chunk: the
    // first row of the one before, so that every pass of the loop issues the same loads and the
    // waits count them.
    struct Rows {
        const unsigned char *k, *v;
        int lim;
    };
    auto rows_of = [&](int it, bool there) {
        const int ci = first + step * (there ? it : it - 1);
        Rows w;
        if (ci >= n_packed) {
            const int t0 = (ci - n_packed) * kChunk;
            w.k = kres + t0 * kRowBytes;
            w.v = vres + t0 * kRowBytes;
            w.lim = r - t0 < kChunk ? r - t0 - 1 : kChunk - 1;
        } else {
            long long rec;
            if (PG) rec = (long long)__builtin_amdgcn_readlane(slotv, (there ? it : it - 1) & 63) * a.n_kv_heads + h;
            else rec = (long long)u * gm.NB + (ci >> sh);
            const unsigned char *p = a.layer + rec * gm.rec_bytes + (ci & ((1 << sh) - 1)) * (kChunk * kRowBytes);
            w.k = p + gm.k_codes;
            w.v = p + gm.v_codes;
            w.lim = kChunk - 1;
        }
        if (!there) w.lim = 0;
        return w;
    };
    // key rows: piece j holds tile j / 4 (token 16 (j / 4) + n), channels 32 (j % 4) + 8 row .. + 7
    auto load_keys = [&](const Rows &w, uint4 (&x)[8]) {
#pragma unroll
        for (int tt = 0; tt < 2; tt++) {
            const int t = min(16 * tt + n, w.lim);
            const unsigned char *p = w.k + (t * kRowBytes + row * 16);
#pragma unroll
            for (int ks = 0; ks < 4; ks++) x[4 * tt + ks] = *(const uint4 *)(p + 64 * ks);
        }
    };
    // value rows: piece j holds token 16 (j / 4) + 4 row + j % 4, channels 8 n .. + 7
    auto load_values = [&](const Rows &w, uint4 (&x)[8]) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int t = min(16 * (j >> 2) + 4 * row + (j & 3), w.lim);
            x[j] = load_past<NT>(w.v + (t * kRowBytes + n * 16));
        }
    };

    float M = -INFINITY, l = 0.0f; // head n: running maximum (exp2 domain), this lane's share of the sum of weights
    v4f O[8];                      // head n, channels 8 (4 row + i) + ct
#pragma unroll
    for (int ct = 0; ct < 8; ct++) O[ct] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    uint4 k[8], v[8];
    const int my_items = first < n_items ? (n_items - first + step - 1) / step : 0;
    if (my_items > 0) { // (one region with the loop: the compiler's wait counts are those of a single path)
        if (PG) load_slots(0);
        const Rows w = rows_of(0, true);
        // (the order of the requests is part of the pipeline: a wait for the key rows leaves the value rows out)
        __builtin_amdgcn_sched_barrier(0);
        load_keys(w, k);
        __builtin_amdgcn_sched_barrier(0);
        load_values(w, v);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            q[ks].x = n < g ? q[ks].x : 0u;
            q[ks].y = n < g ? q[ks].y : 0u;
            q[ks].z = n < g ? q[ks].z : 0u;
            q[ks].w = n < g ? q[ks].w : 0u;
        }
    for (int it = 0; it < my_items; it++) {
        const int ci = first + step * it;
        if (PG && ((it + 1) & 63) == 0) load_slots(it + 1);
        const Rows next = rows_of(it + 1, it + 1 < my_items);
        float s[8]; // token 16 (j / 4) + 4 row + j % 4
#pragma unroll
        for (int tt = 0; tt < 2; tt++) {
            // (two sums of 64 channels, as short a chain as the vector-ALU kernel's)
            v4f lo = v4f{0.0f, 0.0f, 0.0f, 0.0f}, hi = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 2; ks++) {
                lo = mfma_scores<DT>(k[4 * tt + ks], q[ks], lo);
                hi = mfma_scores<DT>(k[4 * tt + 2 + ks], q[2 + ks], hi);
            }
#pragma unroll
            for (int i = 0; i < 4; i++) s[4 * tt + i] = (lo[i] + hi[i]) * kScoreScale;
        }
        load_keys(next, k);
        const int left = ci >= n_packed ? r - (ci - n_packed) * kChunk : kChunk; // tokens of this chunk
#pragma unroll
        for (int j = 0; j < 8; j++) s[j] = 16 * (j >> 2) + 4 * row + (j & 3) < left ? s[j] : -INFINITY;
        float mc = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
        mc = fmaxf(mc, __shfl_xor(mc, 16));
        mc = fmaxf(mc, __shfl_xor(mc, 32));
        if (__builtin_amdgcn_ballot_w64(mc > M) != 0) { // (rare once the largest score has been seen)
            const float m_new = fmaxf(M, mc);
            const float alpha = __builtin_amdgcn_exp2f(M - m_new);
            M = m_new;
            l *= alpha;
#pragma unroll
            for (int ct = 0; ct < 8; ct++) O[ct] *= alpha;
        }
        float p[8];
#pragma unroll
        for (int j = 0; j < 8; j++) p[j] = __builtin_amdgcn_exp2f(s[j] - M);
        l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        // (a short chunk's missing rows hold its last row, which may not be finite: 0 x inf)
        if (left < kChunk) {
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (16 * (j >> 2) + 4 * row + (j & 3) >= left) v[j] = uint4{0u, 0u, 0u, 0u};
        }
        // The chunk's product is summed from zero and then added to the output: a chain of one addition per chunk instead
        // of eight, or the error grows with the tokens a wave takes.  Four channel tiles at a time, as registers
        // allow (a last chunk that goes straight into the output, row by row as it arrives: 50 spilled registers).
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
            v4f t[4];
#pragma unroll
            for (int x = 0; x < 4; x++) t[x] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const uint32_t w0 = e == 0 ? v[j].x : v[j].z, w1 = e == 0 ? v[j].y : v[j].w;
                t[0] = mfma_output(widen_lo<DT>(w0), p[j], t[0]);
                t[1] = mfma_output(widen_hi<DT>(w0), p[j], t[1]);
                t[2] = mfma_output(widen_lo<DT>(w1), p[j], t[2]);
                t[3] = mfma_output(widen_hi<DT>(w1), p[j], t[3]);
            }
#pragma unroll
            for (int x = 0; x < 4; x++) O[2 * e + x] += t[x];
        }
        load_values(next, v);
    }
    }

    // ---- merge of the waves: state row 4 ct + i, lane column row * 8 + head (heads 0 .. 7)
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (n < kMaxGroupQ) {
        float *mine = state[wave] + row * 8 + n;
#pragma unroll
        for (int ct = 0; ct < 8; ct++)
#pragma unroll
            for (int i = 0; i < 4; i++) mine[(4 * ct + i) * ST] = O[ct][i];
        mine[32 * ST] = M;
        mine[33 * ST] = l;
    }
    __syncthreads();
    for (int o = threadIdx.x; o < g * kHeadDim; o += 64 * NW) {
        const int head = o >> 7, c = o & 127;
        const int at = (4 * (c & 7) + ((c >> 3) & 3)) * ST + (c >> 5) * 8 + head;
        float Mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; w++) Mx = fmaxf(Mx, state[w][32 * ST + head]);
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const float Mw = state[w][32 * ST + head];
            const float wt = Mw == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(Mw - Mx); // a wave that saw no token
            num += state[w][at] * wt;
            den += state[w][33 * ST + head] * wt;
        }
        if (!JOIN && a.direct) {
            put_output(a, u, head, c, num, den, Mx);
            continue;
        }
        float *dst = a.ws + ((long long)row0 + head * ns + sp) * kPartialStride;
        put_partial(dst + c, num, JOIN);
        if (c == 0) {
            put_partial(dst + kHeadDim, Mx, JOIN);
            put_partial(dst + kHeadDim + 1, den, JOIN);
        }
    }
    if constexpr (JOIN) {
        __shared__ uint32_t done;
        if (!last_of_unit<NW>(a, u, ns, &done)) return;
        if (g <= NW) join_heads<1, false>(a, u, wave, row0, ns);
        else join_heads<2, false>(a, u, 2 * wave, row0, ns);
    }
}

template <int DT, bool PG> int resident_blocks()
{
    static const int n = [] {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_split_raw_kernel<DT, PG, false, false>, 64 * kRawWaves, 0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        return per_cu * cus;
    }();
    return n;
}

} // namespace

bool decode_raw_supported(const DecodeArgs &a)
{
    const LayerGeom &g = a.geom;
    return g.k_bits == 16 && g.v_bits == 16 && a.g <= kMaxGroupQ && a.batch * a.n_kv_heads <= 65535;
}

int decode_raw_slots(const DecodeArgs &a)
{
    const bool pg = a.geom.table != nullptr;
    return a.geom.dtype == 1 ? (pg ? resident_blocks<1, true>() : resident_blocks<1, false>())
                             : (pg ? resident_blocks<0, true>() : resident_blocks<0, false>());
}

// One resident round of workgroups, at least four chunks per wave unless the device cannot be filled even
// so (a launch that small is bound by latency: one chunk per wave); never more splits than `cap`.
int decode_raw_splits(const DecodeArgs &a, int cap)
{
    const int slots = decode_raw_slots(a);
    const int U = a.batch * a.n_kv_heads;
    const int chunks = a.n_blocks * (a.geom.G / kChunk) + (a.r + kChunk - 1) / kChunk;
    int ns = slots / U;
    const bool small = (long long)U * chunks < (long long)slots * kRawWaves * 4;
    const int most = small ? (chunks + kRawWaves - 1) / kRawWaves : chunks / (kRawWaves * 4);
    if (ns > most) ns = most;
    if (ns > cap) ns = cap;
    return ns < 1 ? 1 : ns;
}

hipError_t launch_decode_split_raw(const DecodeArgs &a, hipStream_t s)
{
    if (!decode_raw_supported(a) || (a.direct == 1 && (a.uneven || a.n_splits != 1))) return hipErrorInvalidValue;
    if (a.direct == 2 && (!a.sync || (a.uneven ? a.uneven_most : a.n_splits) > kJoinFew)) return hipErrorInvalidValue;
    const dim3 grid = a.uneven ? dim3(a.uneven_total, a.n_kv_heads) : dim3(a.n_splits, a.batch * a.n_kv_heads), block(64 * kRawWaves);
    (void)hipGetLastError(); // drop any stale error left by earlier runtime calls of this thread
    const bool pg = a.geom.table != nullptr, bf16 = a.geom.dtype == 1;
    auto go = [&](auto plain, auto joined, auto stream, auto stream_joined) {
        hipLaunchKernelGGL(a.stream ? (a.direct == 2 ? stream_joined : stream) : (a.direct == 2 ? joined : plain), grid, block, 0, s, a);
    };
#define TADAKV_RAW(DT, PG)                                                                                                      \
    go(decode_split_raw_kernel<DT, PG, false, false>, decode_split_raw_kernel<DT, PG, true, false>, decode_split_raw_kernel<DT, PG, false, true>, \
       decode_split_raw_kernel<DT, PG, true, true>)
    if (bf16 && pg) TADAKV_RAW(1, true);
    else if (bf16) TADAKV_RAW(1, false);
    else if (pg) TADAKV_RAW(0, true);
    else TADAKV_RAW(0, false);
#undef TADAKV_RAW
    return note_launch(hipGetLastError());
}

} // namespace tadakv
