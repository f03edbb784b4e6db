// Joining the splits of a unit (flash decoding, App. A of arxiv 2506.04642):
//   out[b, head] = sum_j o_j 2^(m_j - M) / sum_j l_j 2^(m_j - M),  M = max_j m_j
// for up to kJoinSplits splits, by one wavefront per query head: in a kernel of its own behind the split kernel
// (join_kernel), or inside the split kernel, by the workgroup of a unit that is the last to
// have stored its partial results.  One function does the arithmetic for both, in one order, so the two agree bit for bit.
#pragma once
#include "tadakv_internal.h"

namespace tadakv {

typedef unsigned int join_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int join_u32x2 __attribute__((ext_vector_type(2)));
typedef float join_f32x4 __attribute__((ext_vector_type(4)));

// Partial results that are joined inside the launch cross from the workgroup that stores them to the one that joins
// them, on any of the eight dies, each with an L2 of its own: stores at the device's scope go through to memory, loads at
// the device's scope come from there.  (What a kernel of its own will read is stored plainly: 768 workgroups of eight
// heads each, 96 splits, were 1 us slower with stores at the device's scope.)
constexpr int kDeviceScope = 16; // cache policy of a buffer access: sc1
__device__ __forceinline__ void put_partial(float *p, float v, bool joined)
{
    if (joined) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}
template <int CTRL> __device__ __forceinline__ uint32_t dpp_u(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL> __device__ __forceinline__ float dpp_f(float x)
{
    return __uint_as_float(dpp_u<CTRL>(__float_as_uint(x)));
}
// quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E, row_half_mirror = 0x141, row_mirror = 0x140:
// after the four steps every lane of a row of 16 holds the row's total
__device__ __forceinline__ float row_sum(float x)
{
    x += dpp_f<0xB1>(x);
    x += dpp_f<0x4E>(x);
    x += dpp_f<0x141>(x);
    x += dpp_f<0x140>(x);
    return x;
}
__device__ __forceinline__ float row_max(float x)
{
    x = fmaxf(x, dpp_f<0xB1>(x));
    x = fmaxf(x, dpp_f<0x4E>(x));
    x = fmaxf(x, dpp_f<0x141>(x));
    x = fmaxf(x, dpp_f<0x140>(x));
    return x;
}
__device__ __forceinline__ float lane_f(float x, int lane) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane)); }

// NH query heads: ns rows of kPartialStride floats at base + h * ns rows each (wave-uniform), ns <= 2 NB.  Lane l takes
// channels 4 (l & 31) .. + 3 of the splits 2 k + l / 32 and lane j the maximum and the sum of split j, every load requested
// before any is waited for (rows past the last read as zero, by the range of the buffer).  r: the four
// channels' quotients, in both halves of the wave; a sequence without tokens gives zeros.
// Order of a sum: the even splits in rising order, the odd ones, then the two.
template <int NB, int NH, int POLICY> __device__ __forceinline__ void join_rows(const float *base, int ns, int heads, join_f32x4 (&r)[NH])
{
    static_assert(2 * NB <= 48, "the weights are in the first three rows of lanes");
    const int lane = threadIdx.x & 63, half = lane >> 5, at = (lane & 31) * 16;
    constexpr int ROW = kPartialStride * 4;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, heads * ns * ROW, 0x00020000);
    join_u32x2 ml[NH];
    join_u32x4 o[NH][NB];
#pragma unroll
    for (int h = 0; h < NH; h++) {
        const int row0 = h * ns * ROW, past = lane < ns ? 0 : 1 << 30; // (out of the buffer's range)
        ml[h] = __builtin_amdgcn_raw_buffer_load_b64(rs, lane * ROW + kHeadDim * 4 + past, row0, POLICY);
#pragma unroll
        for (int k = 0; k < NB; k++)
            o[h][k] = __builtin_amdgcn_raw_buffer_load_b128(rs, (2 * k + half) * ROW + at + (2 * k + half < ns ? 0 : 1 << 30), row0, POLICY);
    }
#pragma unroll
    for (int h = 0; h < NH; h++) {
        const float m = lane < ns ? __uint_as_float(ml[h].x) : -INFINITY;
        const float rm = row_max(m);
        const float M = fmaxf(fmaxf(lane_f(rm, 0), lane_f(rm, 16)), lane_f(rm, 32));
        const float w = m == -INFINITY ? 0.0f : exp2f(m - M);
        const float rd = row_sum(lane < ns ? __uint_as_float(ml[h].y) * w : 0.0f);
        const float den = (lane_f(rd, 0) + lane_f(rd, 16)) + lane_f(rd, 32);
        join_f32x4 num = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < NB; k++) {
            const float w0 = lane_f(w, 2 * k), w1 = lane_f(w, 2 * k + 1), wk = half ? w1 : w0;
#pragma unroll
            for (int c = 0; c < 4; c++) num[c] += __uint_as_float(o[h][k][c]) * wk;
        }
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const uint32_t x = __float_as_uint(num[c]);
            const join_u32x2 two = __builtin_amdgcn_permlane32_swap(x, x, false, false); // the lower half's, the upper half's
            r[h][c] = M == -INFINITY ? 0.0f : (__uint_as_float(two.x) + __uint_as_float(two.y)) / den;
        }
    }
}
// Counts a workgroup in at *c: true for the last of n, which leaves the count zero.  From zero a call counts down from
// base + n - 1 to its base, and every call of a cache has a base of its own, kSyncCalls below that of the call before.  So whatever
// calls that overlapped have left there is above what a later call counts, and starts over like zero (the
// instruction's own rule: a value that is zero or larger than its operand is replaced by it).
__device__ __forceinline__ bool count_in(unsigned long long *c, unsigned long long base, uint32_t n)
{
    const unsigned long long first = base + (n - 1);
    const unsigned long long was = __builtin_amdgcn_atomic_dec64((unsigned long *)c, first, __ATOMIC_RELAXED, "agent");
    if ((was - 1 < first ? was - 1 : first) != base) return false;
    __hip_atomic_store(c, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}
// The end of a split kernel that joins the splits itself: called by every wave of a workgroup once it has stored its part
// of the partial results (put_partial).  The workgroups of a unit count themselves in; the last of the ns finds
// everybody's results in memory and joins them (true), the others are through.  Nobody waits for another workgroup.
// The count is then zero again, as the next launch on the stream expects it.  flag: a word of LDS that nobody reads
// any more.
// What it costs, of a launch with one chunk a wave (one head of 1024 tokens, 4 splits; the device's clock): 0.7 us from the
// stores to the count, 0.9 us for the join, against a second launch's 2.0 us on the device and 3.5 us of the host's time:
// attention in us, two launches -> one: that one 8.2 -> 7.1, 8205 tokens, 8 kv heads x 4 (33 splits) 9.4 -> 8.6,
// 4 x 1523 (7) 7.9 -> 7.2, 24 sequences up to 8011 paged (4) 45 -> 43.
template <int NW> __device__ __forceinline__ bool last_of_unit(const DecodeArgs &a, int u, int ns, uint32_t *flag)
{
    unsigned long long *c = a.sync + u * kSyncStride;
    asm volatile("s_waitcnt vmcnt(0)" : : "s"(c), "s"(a.sync_base) : "memory"); // this wave's partial results are in memory (the arguments: requested before)
    __syncthreads();                                          // everybody's are
    if (threadIdx.x == 0) *flag = count_in(c, a.sync_base, ns);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane((int)*flag) != 0;
}
// Heads i0 .. i0 + NH - 1 (those below a.g) of unit u, whose first partial result (head 0) is row `row`, to the output.
// MANY: more than kJoinFew splits, too (see join_in_kernel).
template <int NH, bool MANY> __device__ __forceinline__ void join_heads(const DecodeArgs &a, int u, int i0, long long row, int ns)
{
    const int heads = a.g - i0 < NH ? a.g - i0 : NH;
    if (heads <= 0) return;
    const float *base = a.ws + (row + (long long)i0 * ns) * kPartialStride;
    join_f32x4 r[NH];
    if (MANY && ns > kJoinFew) join_rows<kJoinSplits / 2, NH, kDeviceScope>(base, ns, heads, r);
    else join_rows<kJoinFew / 2, NH, kDeviceScope>(base, ns, heads, r);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 0; h < NH; h++) // (n_q_heads = n_kv_heads g)
        if (h < heads && lane < 32) *(join_f32x4 *)(a.out + ((long long)u * a.g + i0 + h) * kHeadDim + 4 * lane) = r[h];
}
// A launch on device-resident lengths: the last unit to be joined makes the state after the step the current one (every
// workgroup has read the lengths before its unit is joined).
__device__ __forceinline__ void step_is_done(const DecodeArgs &a)
{
    if (threadIdx.x != 0 || !a.len_dev) return;
    const int units = a.batch * a.n_kv_heads;
    if (!count_in(a.sync + units * kSyncStride, a.sync_base, units)) return; // (behind the units' counts)
    a.len_dev[4 * a.batch] = (a.len_dev[4 * a.batch] & 1) ^ 1;
}

} // namespace tadakv
