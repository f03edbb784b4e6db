// Value projection fused with the compression of the values (gfx950): Algorithm 1 step 3 of
// arxiv 2506.04642, "CompressV(X, W_V)" (Sec. 3.4; App. A "Compressing value activations": the
// linear projection that produces the values is the only operator in front of their mean-centring
// and quantisation, so the two are one kernel and the projected values never travel through memory
// as a tensor of their own).
//
//   V[t][o] = sum_k X[t][k] * W_V[o][k]      16-bit operands, binary32 accumulation on the matrix
//                                            cores, the sum rounded (nearest even) to the 16-bit type
// followed, for every whole block of 32 tokens of one (sequence, kv head), by the value side of the
// quantiser (block mean per channel, deviation, one (scale, zero) per token and group of Gc
// channels, codes, packed words: quant_wave.h) on the accumulator tile, or, for tokens that stay
// in the raw residual buffer (Sec. 3.3), by a store of the rounded rows into that buffer.
//
// compressv_gemm_kernel: in bulk a workgroup owns 256 tokens (eight groups of 32) x NH kv heads (128
// channels each); wave (wm, wn) owns tokens 64 wm .. + 63 of head wn: 4 x 8 tiles of
// v_mfma_f32_16x16x32 accumulators, i.e. two quantiser items, two waves per SIMD.  X and W_V tiles
// of 64 k-values (rows of 128 bytes, whole cache lines) are fetched straight into LDS
// (global_load_lds_dwordx4), 16-byte pieces of a row XOR-swizzled by the row so that
// the operand reads (16 rows x one piece) hit distinct banks (4.1 cycles a read instruction; rows of 64 bytes: 8).
// LDS holds three stages of X, which comes from HBM, and two of W_V, which the L2 and the cache behind it serve: all of the
// 160 KiB.  With two of each (a stage's 64 KiB requested one stage ahead) the fetches alone, without a matrix
// instruction, took 1.27 us a stage: 0.55 of transfer and the latency; the matrix instructions alone take 0.85.
// A call of up to 2048 (group, kv head) items would leave half of the device idle that way: there a workgroup owns 128 tokens x one
// head, two waves of 64 tokens (three stages of X and two of W_V); up to 512 items 64 tokens x one head, two waves of 32, with four stages of
// both.  (Large tiles of one head, where their number is odd: three of both.)
// Every output element is one chain of model_dim / 32 matrix instructions in ascending k, the same
// chain in project_rows_kernel below, so a token's projected value does not depend on which of
// the two kernels, or which tile, produced it.
//
// project_rows_kernel: the decode step's shape (a handful of rows against the whole of W_V): one
// wave per 16 output channels and 16 rows, its operands streamed with sixteen steps in flight.
#include "quant_wave.h"
#include <type_traits>

namespace tadakv {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4))); // one matrix operand: eight 16-bit values
typedef const __attribute__((address_space(1))) void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

constexpr int kStepK = 64;       // k-values per stage: rows of 128 bytes, whole cache lines
constexpr int kEpiBytes = 16384; // per wave after the main loop: transposed 16-bit tile + record image
// (32 tokens x one head) items up to which the small and the middle tile are the faster: one round of them on 256 compute
// units, one or two workgroups each
constexpr int kSmallTileItems = 512, kMiddleTileItems = 2048;
constexpr int kTTStride = 80;    // bytes per channel column of the transposed tile (32 tokens + pad)

template <int DT> __device__ __forceinline__ v4f mfma16(const u32x4 &a, const u32x4 &b, v4f c)
{
    if (DT == 1) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}
template <int DT> __device__ __forceinline__ v4f mfma16(const uint4 &a, const uint4 &b, v4f c)
{
    return mfma16<DT>(u32x4{a.x, a.y, a.z, a.w}, u32x4{b.x, b.y, b.z, b.w}, c);
}

// LDS operand read issued by hand.  The compiler makes every LDS read it knows of wait for all
// outstanding direct-to-LDS fetches (it cannot tell which buffer they fill), which would undo the
// fetch-ahead of the main loop; these reads are invisible to that rule.  The result must not be used
// before lds_reads_done has been given the same registers.
template <int OFF> __device__ __forceinline__ void lds_read16(u32x4 &dst, uint32_t addr)
{
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
__device__ __forceinline__ void lds_reads_done(u32x4 (&a)[2], u32x4 (&b)[8])
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5]), "+v"(b[6]), "+v"(b[7]));
}
__device__ __forceinline__ void lds_reads_done(u32x4 (&a)[4], u32x4 (&b)[8])
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]),
                   "+v"(b[4]), "+v"(b[5]), "+v"(b[6]), "+v"(b[7]));
}

// the 16-bit pattern of a binary32 value that is exactly representable in the type
template <int DT> __device__ __forceinline__ uint32_t bits16_exact(float f)
{
    if (DT == 1) return __float_as_uint(f) >> 16;
    return (uint32_t)f16_rne(f);
}

// Group f of the launch: sequence (of the run), group inside the sequence, valid tokens.
struct GroupId {
    int b, gi, nv;
};
__device__ __forceinline__ GroupId group_of(const ProjectArgs &p, int f)
{
    GroupId g;
    g.b = f / p.n_groups;
    g.gi = f % p.n_groups;
    const int left = p.n_tok - 32 * g.gi;
    g.nv = left < 32 ? left : 32;
    return g;
}

// The rounded 32-token x 128-channel tile of one (group, kv head), held by a wave in the
// quantiser's lane layout x[token j][channel e] (tokens 8 tg + j, channels 8 c8 + e), goes where
// the launch says: into the record of block first_block + gi (values' part: codes, metadata,
// mean), or as raw rows into the residual buffer; and, if asked for, into the caller's tensor.
template <int DT, int GC, int BITS>
__device__ __forceinline__ void tile_out(const ProjectArgs &p, float (&x)[8][8], const GroupId &g, int h, int lane,
                                         unsigned char *img, uint32_t mean_pair)
{
    constexpr int G = 32, NGV = kHeadDim / GC;
    const LayerGeom &gm = p.geom;
    const int tg = lane & 3, c8 = lane >> 2;
    if (p.v_out || p.mode == 1) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int t = 8 * tg + j;
            uint4 row;
            row.x = bits16_exact<DT>(x[j][0]) | (bits16_exact<DT>(x[j][1]) << 16);
            row.y = bits16_exact<DT>(x[j][2]) | (bits16_exact<DT>(x[j][3]) << 16);
            row.z = bits16_exact<DT>(x[j][4]) | (bits16_exact<DT>(x[j][5]) << 16);
            row.w = bits16_exact<DT>(x[j][6]) | (bits16_exact<DT>(x[j][7]) << 16);
            if (t < g.nv) {
                const int tn = p.t0 + 32 * g.gi + t; // token of the call
                if (p.v_out)
                    *(uint4 *)(p.v_out + (long long)g.b * p.vo_stride_b + (long long)tn * p.vo_stride_t +
                               (long long)h * p.vo_stride_h + c8 * 8) = row;
                if (p.mode == 1) {
                    const long long u = (long long)(p.b0 + g.b) * p.n_kv_heads + h;
                    *(uint4 *)(p.layer + gm.v_resid_off + (u * gm.R + p.dst_row + 32 * g.gi + t) * (kHeadDim * 2) + c8 * 16) = row;
                }
            }
        }
    }
    if (p.mode == 1) return;

    // ---- the quantiser's value side on the tile (Eq. 1-4 with the per-channel block mean, or no mean)
    const int base_off = gm.v_codes;
    if (gm.mean_mode == 0) {
        // mean_pair: the binary16 means of channels 2 lane and 2 lane + 1 (the caller formed the sums over
        // the block's tokens, in token order, with a channel's 32 tokens in one lane); the record's mean
        // row is the lanes' words in order, and channels 8 c8 + 2 k and + 2 k + 1 are quad lane k's
        *(uint32_t *)(img + (gm.v_mean - base_off) + lane * 4) = mean_pair;
        const uint32_t q0 = quad_bcast_u<0>(mean_pair), q1 = quad_bcast_u<1>(mean_pair), q2 = quad_bcast_u<2>(mean_pair),
                       q3 = quad_bcast_u<3>(mean_pair);
        float m[8];
        m[0] = f16_val((uint16_t)(q0 & 0xFFFFu)); m[1] = f16_val((uint16_t)(q0 >> 16));
        m[2] = f16_val((uint16_t)(q1 & 0xFFFFu)); m[3] = f16_val((uint16_t)(q1 >> 16));
        m[4] = f16_val((uint16_t)(q2 & 0xFFFFu)); m[5] = f16_val((uint16_t)(q2 >> 16));
        m[6] = f16_val((uint16_t)(q3 & 0xFFFFu)); m[7] = f16_val((uint16_t)(q3 >> 16));
#pragma unroll
        for (int j = 0; j < 8; j++)
#pragma unroll
            for (int e = 0; e < 8; e++) x[j][e] = x[j][e] - m[e];
    } else {
#pragma unroll
        for (int j = 0; j < 8; j++)
#pragma unroll
            for (int e = 0; e < 8; e++) x[j][e] = x[j][e] - 0.0f;
    }
    emit_value_half<GC, BITS, 2>(x, 0, lane, img, img + (gm.v_meta - base_off));
    const int part_bytes = (gm.mean_mode == 0 ? gm.v_mean + 256 : gm.v_meta + G * NGV * 4) - base_off;
    unsigned char *rec = p.layer + record_offset(gm, p.n_kv_heads, p.b0 + g.b, h, p.first_block + g.gi);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // this wave's LDS writes have landed
    for (int off = lane * 16; off < part_bytes; off += 64 * 16) put_record((uint4 *)(rec + base_off + off), *(const uint4 *)(img + off));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the image is in registers before the next group overwrites it
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>)
template <int N, int I = 0, class F> __device__ __forceinline__ void static_for(const F &f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        static_for<N, I + 1>(f);
    }
}

template <int N> __device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// WT: tokens of a wave's tile (64 or 32); MW: such tiles per workgroup; SA, SB: stages of X and of W_V in LDS (SA >= SB >= 2).
template <int DT, int NH, int GC, int BITS, int WT, int MW, int SA, int SB>
__global__ __launch_bounds__(64 * MW * NH) void compressv_gemm_kernel(ProjectArgs p)
{
    constexpr int TT = WT * MW, NF = TT / 32;       // tokens per workgroup, groups of 32 of them
    constexpr int MT = WT / 16, NI = WT / 32;       // a wave's row tiles, its items
    constexpr int NW = MW * NH;                     // waves: MW token parts x NH heads
    constexpr int A_BYTES = TT * 128;               // X tile of a stage: 64 k-values, rows of 128 bytes
    constexpr int B_BYTES = NH * kHeadDim * 128;    // W_V tile of a stage
    constexpr int PA = A_BYTES / 1024 / NW, PB = B_BYTES / 1024 / NW; // fetch instructions (1 KiB each) per wave and stage
    static_assert(A_BYTES / 1024 % NW == 0 && B_BYTES / 1024 % NW == 0, "a stage divides among the waves");
    static_assert(SA >= SB && SB >= 2 && NW * kEpiBytes <= SA * A_BYTES + SB * B_BYTES, "the epilogue fits the staging buffers");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[]; // SA stages of X, behind them SB of W_V

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave % MW, wn = wave / MW;
    // Workgroups are dealt to the eight dies in turn: the ones that share a token tile (the head
    // groups of that tile) get ids a multiple of eight apart, so they run on one die and find the
    // tile's rows of X in its cache.
    const int HG = p.n_kv_heads / NH;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int tile = (slot / HG) * 8 + xcd, hg = slot % HG;
    const int n_f = p.batch * p.n_groups;
    if (tile * NF >= n_f) return; // (the grid is padded to whole rounds of eight tiles)

    // ---- where this lane's pieces of a stage come from: instruction q of a tile fills rows
    // 8 q .. 8 q + 7 (128 bytes each: whole cache lines), lane l the piece (l & 7) ^ (row & 7) of row 8 q + (l >> 3)
    const uint16_t *src_a[PA], *src_b[PB];
    {
        const int r8 = lane >> 3, pc = (lane & 7) ^ r8;
#pragma unroll
        for (int i = 0; i < PA; i++) {
            const int row = 8 * (wave * PA + i) + r8;
            int f = tile * NF + (row >> 5);
            f = f < n_f ? f : n_f - 1; // past the end: any valid row, the result is not stored
            const GroupId g = group_of(p, f);
            int t = row & 31;
            t = t < g.nv ? t : g.nv - 1;
            src_a[i] = p.x + (long long)g.b * p.x_stride_b + (long long)(p.t0 + 32 * g.gi + t) * p.x_stride_t + pc * 8;
        }
#pragma unroll
        for (int i = 0; i < PB; i++) // (output channel within the workgroup's heads)
            src_b[i] = p.w + ((long long)hg * NH * kHeadDim + 8 * (wave * PB + i) + r8) * p.model_dim + pc * 8;
    }
    const int stages = p.model_dim / kStepK;
    // this wave's piece i of a tile of stage sg (k-values 64 sg .. + 63; the last stage again beyond it) into the buffer at byte `at`
    auto issue_a = [&](int sg, uint32_t at, int i) {
        const int sk = sg < stages ? sg : stages - 1;
        __builtin_amdgcn_global_load_lds((gptr_t)(src_a[i] + (long long)sk * kStepK), (lptr_t)(lds + at + (wave * PA + i) * 1024), 16, 0, 0);
    };
    auto issue_b = [&](int sg, uint32_t at, int i) {
        const int sk = sg < stages ? sg : stages - 1;
        __builtin_amdgcn_global_load_lds((gptr_t)(src_b[i] + (long long)sk * kStepK), (lptr_t)(lds + at + (wave * PB + i) * 1024), 16, 0, 0);
    };

    v4f acc[MT][8];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int nt = 0; nt < 8; nt++) acc[mt][nt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    const int n = lane & 15, kg = lane >> 4;
    // this lane's operand piece inside a 16-row tile (2 KiB) for the low and the high 32 k-values of
    // a stage: row n, piece 4 half + kg, swizzled by the row
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds;
    const uint32_t a_base = lds0 + wm * (WT * 128) + n * 128, b_base = lds0 + wn * (kHeadDim * 128) + n * 128;
    const uint32_t sw_lo = (uint32_t)((kg ^ (n & 7)) << 4), sw_hi = (uint32_t)(((4 + kg) ^ (n & 7)) << 4);
    u32x4 fa[2][MT], fb[2][8]; // operands of the current half step and of the next one
    // operand r of a half step: a wave's row tile r, or its column tile r - MT
    auto read_frag = [&](auto rc, uint32_t ra, uint32_t rb, u32x4(&a)[MT], u32x4(&b)[8]) {
        constexpr int r = decltype(rc)::value;
        if constexpr (r < MT) lds_read16<r * 2048>(a[r], ra);
        else lds_read16<(r - MT) * 2048>(b[r - MT], rb);
    };
    // 8 MT matrix instructions on one half step's operands, four at a time, and between the fours the reads of the half
    // step after it (from ra and rb) and, with FETCH, this wave's fetches of W_V stage sg + SB and X stage sg + SA (to
    // the buffers of stage sg at wa and wb).
    constexpr int NG = 2 * MT, NR = MT + 8;
    auto half_step = [&](auto fetch, int sg, uint32_t wa, uint32_t wb, uint32_t ra, uint32_t rb, u32x4(&a)[MT], u32x4(&b)[8], u32x4(&na)[MT], u32x4(&nb)[8]) {
        static_for<NG>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            static_for<NR>([&](auto rc) {
                if constexpr (decltype(rc)::value * (3 * NG / 4) / NR == g) read_frag(rc, ra, rb, na, nb);
            });
            if constexpr (decltype(fetch)::value) {
#pragma unroll
                for (int i = 0; i < PA + PB; i++)
                    if (i * NG / (PA + PB) == g) {
                        if (i < PB) issue_b(sg + SB, wb, i);
                        else issue_a(sg + SA, wa, i - PB);
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nt = 0; nt < 4; nt++) {
                constexpr int mt = g / 2, n0 = 4 * (g & 1);
                acc[mt][n0 + nt] = mfma16<DT>(a[mt], b[n0 + nt], acc[mt][n0 + nt]);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    constexpr uint32_t B0 = SA * A_BYTES; // the W_V buffers lie behind the X buffers
    auto after_a = [](uint32_t at) { return at + A_BYTES == B0 ? 0u : at + A_BYTES; };
    auto after_b = [](uint32_t at) { return at + B_BYTES == B0 + SB * B_BYTES ? B0 : at + B_BYTES; };

    // (Requested in one burst behind the barrier, a stage's 64 fetches and 96 reads keep every wave from its matrix instructions
    // until the memory pipe has taken them, up to a thousand cycles: 65536 tokens, 8 heads, model_dim 4096: 503 us a call; spread
    // out 471, with the third stage of X 445.  What is left above the matrix instructions is mostly the clock: the same call on
    // zeros, which cost the matrix cores less power, takes 378; the epilogue 28, the keys' side 38.)
    // A stage is consumed in two half steps of 32 k-values (32 matrix instructions per wave each);
    // the operands of a half step are read from LDS while the matrix instructions of the half step
    // before it run.  Once a wave holds the high half's operands it is done with the stage's buffer;
    // at the one barrier of a stage everybody is, and everybody's part of the next stage (fetched one
    // stage earlier, or two) has landed; then later stages are fetched into the freed buffers and
    // the next stage's low operands are read.  Past the last stage the fetch repeats the last one into
    // a buffer nobody reads any more and the operand read returns unused data, so that every stage is
    // the same straight line of code.
    // (in the order of the loop: W_V of stage sg + SB, then X of stage sg + SA.  The waits count on it, and to the compiler the
    // buffers are unrelated: the barriers keep it from exchanging requests, and the build reads the order that came out)
#pragma unroll
    for (int sg = -SA; sg < 0; sg++) {
        if (sg + SB >= 0)
#pragma unroll
            for (int i = 0; i < PB; i++) issue_b(sg + SB, B0 + (sg + SB) * B_BYTES, i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < PA; i++) issue_a(sg + SA, (sg + SA) * A_BYTES, i);
        __builtin_amdgcn_sched_barrier(0);
    }
    // fetches that may be on their way when the next stage's two tiles have to be there
    constexpr int LATER = (SB - 2) * (PA + PB) + (SA > SB ? PA : 0);
    wait_vm<LATER + PA + PB>(); // stage 0 has landed
    __builtin_amdgcn_s_barrier();
    uint32_t at_a = 0, at_b = B0;
    static_for<NR>([&](auto rc) { read_frag(rc, a_base + sw_lo, b_base + B0 + sw_lo, fa[0], fb[0]); });
    for (int sg = 0; sg < stages; sg++) {
        const uint32_t na = after_a(at_a), nb = after_b(at_b);
        lds_reads_done(fa[0], fb[0]);
        half_step(std::false_type(), 0, 0u, 0u, a_base + at_a + sw_hi, b_base + at_b + sw_hi, fa[0], fb[0], fa[1], fb[1]);
        lds_reads_done(fa[1], fb[1]);
        wait_vm<LATER>();
        __builtin_amdgcn_s_barrier();
        half_step(std::true_type(), sg, at_a, at_b, a_base + na + sw_lo, b_base + nb + sw_lo, fa[1], fb[1], fa[0], fb[0]);
        at_a = na;
        at_b = nb;
    }
    lds_reads_done(fa[0], fb[0]); // (of the stage past the last)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads(); // the staging buffers are free: each wave takes 16 KiB of them for its epilogue
    unsigned char *tt = lds + wave * kEpiBytes;  // [128 channels][32 tokens] 16-bit, kTTStride bytes per channel
    unsigned char *img = tt + kHeadDim * kTTStride; // the values' part of a record
    const int tg = lane & 3, c8 = lane >> 2;
    const int h = hg * NH + wn;
#pragma unroll
    for (int blk = 0; blk < NI; blk++) {
        const int f = tile * NF + NI * wm + blk;
        if (f >= n_f) break;
        const GroupId g = group_of(p, f);
        // accumulators (lane: tokens 16 mt + 4 kg .. + 3 of channel 16 nt + n), rounded, into the
        // transposed tile: the four tokens are 8 contiguous bytes
#pragma unroll
        for (int m2 = 0; m2 < 2; m2++)
#pragma unroll
            for (int nt = 0; nt < 8; nt++) {
                const v4f c = acc[2 * blk + m2][nt];
                *(uint2 *)(tt + (16 * nt + n) * kTTStride + (16 * m2 + 4 * kg) * 2) = uint2{narrow2<DT>(c[0], c[1]), narrow2<DT>(c[2], c[3])};
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // back in the quantiser's layout: tokens 8 tg .. + 7 of channel 8 c8 + e are 16 contiguous bytes
        float x[8][8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const uint4 pcs = *(const uint4 *)(tt + (8 * c8 + e) * kTTStride + tg * 16);
            const uint32_t wv[4] = {pcs.x, pcs.y, pcs.z, pcs.w};
#pragma unroll
            for (int k = 0; k < 4; k++) {
                x[2 * k][e] = widen16((uint16_t)(wv[k] & 0xFFFFu), DT);
                x[2 * k + 1][e] = widen16((uint16_t)(wv[k] >> 16), DT);
            }
        }
        // the per-channel sums of the block mean, over the tokens in order: a channel's 32 tokens are
        // 64 contiguous bytes of the transposed tile, so lane l adds up channels 2 l and 2 l + 1 (every
        // lane adds; in the quantiser's layout three quarters of a quad's adds would be masked)
        uint32_t mean_pair = 0u;
        if (p.geom.mean_mode == 0 && p.mode != 1) {
            float sm[2];
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const unsigned char *col = tt + (2 * lane + c) * kTTStride;
                float sacc = 0.0f;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const uint4 pcs = *(const uint4 *)(col + 16 * q);
                    const uint32_t wv[4] = {pcs.x, pcs.y, pcs.z, pcs.w};
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        sacc = sacc + widen16((uint16_t)(wv[k] & 0xFFFFu), DT);
                        sacc = sacc + widen16((uint16_t)(wv[k] >> 16), DT);
                    }
                }
                sm[c] = sacc;
            }
            mean_pair = (uint32_t)f16_rne(sm[0] / 32.0f) | ((uint32_t)f16_rne(sm[1] / 32.0f) << 16);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the tile is in registers before the next group overwrites it
        tile_out<DT, GC, BITS>(p, x, g, h, lane, img, mean_pair);
    }
}

// A few rows (a decode step: one token per sequence) against all of W_V.  One wave per (16 output
// channels, 16 rows): B operand = its 16 rows of W_V, 16 bytes per lane and matrix instruction
// (k-values 32 s + 8 (l >> 4) .. + 7 of channel l & 15); A operand = its rows of X.  Sixteen steps
// of loads are in flight per lane: each step's registers are loaded again as soon as its matrix
// instruction has consumed them.  Same accumulation chain as the tiled kernel.
// Row r of the launch is token t0 + r % n_tok of sequence r / n_tok (of the run).
template <int DT>
__global__ __launch_bounds__(64) void project_rows_kernel(ProjectArgs p)
{
    const int lane = threadIdx.x, n = lane & 15, kg = lane >> 4;
    const int o0 = blockIdx.x * 16, r0 = blockIdx.y * 16; // first output channel, first row of the wave
    const int rows = p.batch * p.n_tok;
    const uint16_t *wrow = p.w + (long long)(o0 + n) * p.model_dim + 8 * kg;
    int ra = r0 + n;
    ra = ra < rows ? ra : rows - 1;
    const uint16_t *xrow = p.x + (long long)(ra / p.n_tok) * p.x_stride_b + (long long)(p.t0 + ra % p.n_tok) * p.x_stride_t + 8 * kg;
    v4f acc = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int D = 16; // steps in flight
    const int steps = p.model_dim / 32;
    uint4 a[D], b[D];
#pragma unroll
    for (int i = 0; i < D; i++) {
        const int s = i < steps ? i : steps - 1;
        b[i] = *(const uint4 *)(wrow + 32 * s);
        a[i] = *(const uint4 *)(xrow + 32 * s);
    }
    for (int s0 = 0; s0 < steps; s0 += D) {
#pragma unroll
        for (int i = 0; i < D; i++) {
            if (s0 + i < steps) acc = mfma16<DT>(a[i], b[i], acc);
            const int s = s0 + i + D < steps ? s0 + i + D : steps - 1;
            b[i] = *(const uint4 *)(wrow + 32 * s);
            a[i] = *(const uint4 *)(xrow + 32 * s);
        }
    }
    // lane: rows r0 + 4 kg .. + 3 of channel o0 + n
    const int o = o0 + n, h = o / kHeadDim, c = o % kHeadDim;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int r = r0 + 4 * kg + j;
        if (r >= rows) continue;
        const int bb = r / p.n_tok, t = r % p.n_tok;
        const uint16_t v = (uint16_t)(narrow2<DT>(acc[j], 0.0f) & 0xFFFFu);
        if (p.v_out)
            p.v_out[(long long)bb * p.vo_stride_b + (long long)(p.t0 + t) * p.vo_stride_t + (long long)h * p.vo_stride_h + c] = v;
        const long long u = (long long)(p.b0 + bb) * p.n_kv_heads + h;
        *(uint16_t *)(p.layer + p.geom.v_resid_off + (u * p.geom.R + p.dst_row + t) * (kHeadDim * 2) + c * 2) = v;
    }
}

template <int DT, int NH, int GC, int BITS, int WT, int MW, int SA, int SB> hipError_t launch_gemm(const ProjectArgs &p, hipStream_t s)
{
    constexpr int NF = WT * MW / 32;
    constexpr size_t lds = SA * (size_t)(WT * MW * 128) + SB * (size_t)(NH * kHeadDim * 128);
    static const bool ready = hipFuncSetAttribute((const void *)compressv_gemm_kernel<DT, NH, GC, BITS, WT, MW, SA, SB>,
                                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
    if (!ready) return note_launch(hipErrorInvalidValue);
    const long long n_f = (long long)p.batch * p.n_groups;
    const long long tiles = (n_f + NF - 1) / NF, rounds = (tiles + 7) / 8;
    const long long grid = rounds * 8 * (p.n_kv_heads / NH);
    if (grid > 0x7FFFFFFF) return note_launch(hipErrorInvalidValue);
    hipLaunchKernelGGL((compressv_gemm_kernel<DT, NH, GC, BITS, WT, MW, SA, SB>), dim3((unsigned)grid), dim3(64 * MW * NH), lds, s, p);
    return note_launch(hipGetLastError());
}
// The tile by the number of tokens: 256 x NH heads where that fills the device; up to 2048 items 128 tokens x one head (two
// waves of the same 64 x 128 tile, two such workgroups per compute unit); up to 512 items 64 tokens x one head with
// four stages on their way (a small workgroup's stage is through in a fifth of the time that its fetch takes; six are 2 % slower).  Same
// chain per element, same bytes.  Beyond its one round a tile that is smaller than another only reads the operands more often.
// Measured (us a call with the keys' side, bf16, 4 bits, calls in a row; small / middle / large): 8 kv heads, model_dim 4096: 1024 tokens
// 35 / 55 / 81, 2048 (512 items) 37 / 55 / 81, 3072 65 / 56 / 82, 4096 65 / 56 / 81, 8192 (2048 items) 122 / 70 / 86, 12288 177 / 118 / 93,
// 24576 365 / 202 / 194; 2 heads, model_dim 2048: 8192 tokens (512 items) 24 / 34 / 49, 16384 40 / 35 / 49, 32768 (2048) 75 / 44 / 54.
template <int DT, int GC, int BITS> hipError_t launch_gemm_tile(const ProjectArgs &p, hipStream_t s)
{
    const long long items = (long long)p.batch * p.n_groups * p.n_kv_heads;
    if (items <= kSmallTileItems) return launch_gemm<DT, 1, GC, BITS, 32, 2, 4, 4>(p, s);
    if (items <= kMiddleTileItems) return launch_gemm<DT, 1, GC, BITS, 64, 2, 3, 2>(p, s);
    if (p.n_kv_heads % 2 == 0) return launch_gemm<DT, 2, GC, BITS, 64, 4, 3, 2>(p, s);
    return launch_gemm<DT, 1, GC, BITS, 64, 4, 3, 3>(p, s);
}
template <int DT> hipError_t launch_gemm_fmt(const ProjectArgs &p, hipStream_t s)
{
    const int gc = p.geom.Gc, b = p.geom.v_bits;
#define TADAKV_CV(GCV) (b == 2 ? launch_gemm_tile<DT, GCV, 2>(p, s) : b == 4 ? launch_gemm_tile<DT, GCV, 4>(p, s) : launch_gemm_tile<DT, GCV, 8>(p, s))
    return gc == 32 ? TADAKV_CV(32) : gc == 64 ? TADAKV_CV(64) : TADAKV_CV(128);
#undef TADAKV_CV
}

template <int DT> hipError_t launch_rows(const ProjectArgs &p, hipStream_t s)
{
    const int rows = p.batch * p.n_tok;
    const dim3 grid(p.n_kv_heads * kHeadDim / 16, (rows + 15) / 16), block(64);
    hipLaunchKernelGGL((project_rows_kernel<DT>), grid, block, 0, s, p);
    return note_launch(hipGetLastError());
}

} // namespace

bool compressv_supported(const LayerGeom &g)
{
    return g.G == 32 && g.k_bits == g.v_bits && (g.v_bits == 2 || g.v_bits == 4 || g.v_bits == 8) && g.mean_mode != 1;
}

hipError_t launch_compressv(const ProjectArgs &p, hipStream_t s)
{
    if (!compressv_supported(p.geom) || p.model_dim % kStepK || p.n_groups < 1 || p.n_tok < 1 || p.batch < 1)
        return note_launch(hipErrorInvalidValue);
    (void)hipGetLastError(); // drop any stale error left by earlier runtime calls of this thread
    // raw rows of a decode step: the streaming kernel
    if (p.mode == 1 && (long long)p.batch * p.n_tok <= 256)
        return p.geom.dtype == 1 ? launch_rows<1>(p, s) : launch_rows<0>(p, s);
    return p.geom.dtype == 1 ? launch_gemm_fmt<1>(p, s) : launch_gemm_fmt<0>(p, s);
}

} // namespace tadakv
