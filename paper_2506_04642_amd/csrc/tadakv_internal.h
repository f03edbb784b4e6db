// Internal declarations shared by the host-side ABI and the HIP kernels of libtadakv.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tadakv {

constexpr int kHeadDim = 128;
constexpr int kMaxGroupQ = 8;       // query heads per kv head the kernels are sized for
constexpr int kPartialStride = 132; // floats per (unit, q head, split): O[128], max, sum, pad
constexpr int kMaxSplits = 256;
constexpr int kJoinSplits = 34;     // splits that one wavefront joins at once (join.h; the line: join_in_kernel)
constexpr int kJoinFew = 8;         // splits of which it joins several query heads at once
constexpr int kSyncStride = 8;      // 64-bit words from one count of finished workgroups to the next
constexpr uint64_t kSyncCalls = 1 << 20; // what a call may count (units, workgroups of a unit), with room to spare (count_in)
constexpr int kMaxRaggedBatch = 256; // sequences whose lengths may differ from one another

// Geometry of one layer's buffer; byte offsets, -1 where a field is absent.
struct LayerGeom {
    int k_bits, v_bits;
    int G, Gc, R, NB;     // group_tokens, group_channels, resid_cap, blocks per sequence
    int mean_mode, dtype;
    long long rec_bytes;
    int k_codes, k_scale, k_zero, k_mean;
    int v_codes, v_meta, v_mean;
    long long xmean_off, k_resid_off, v_resid_off, layer_bytes;
    // paged placement: block slots shared through a device table [batch][table_stride] (null: dense)
    const int32_t *table;
    int table_stride, pool;
};

// Block slot of logical block blk of sequence b.  Entries outside the pool are clamped into it.
__device__ __forceinline__ long long block_slot(const LayerGeom &g, int b, int blk)
{
    if (!g.table) return (long long)b * g.NB + blk;
    int p = g.table[(long long)b * g.table_stride + blk];
    p = p < 0 ? 0 : (p >= g.pool ? g.pool - 1 : p);
    return p;
}
// Byte offset of the record of (sequence b, kv head h, block blk) in the layer buffer.
__device__ __forceinline__ long long record_offset(const LayerGeom &g, int n_kv_heads, int b, int h, int blk)
{
    if (!g.table) return ((long long)(b * n_kv_heads + h) * g.NB + blk) * g.rec_bytes;
    return (block_slot(g, b, blk) * n_kv_heads + h) * g.rec_bytes;
}
// Byte offset of the cross-head mean tile [G][128] binary16 of (sequence b, block blk, K | V).
__device__ __forceinline__ long long xmean_offset(const LayerGeom &g, int b, int blk, int which)
{
    return g.xmean_off + ((block_slot(g, b, blk) * 2 + which) * g.G * kHeadDim) * 2;
}

// Device-resident lengths of one layer (for decode steps replayed from a HIP graph, whose kernel
// arguments cannot follow a growing cache): ints st[p * 2B + 2b] = packed blocks and st[p * 2B + 2b + 1]
// = raw tokens of sequence b in state p (0 or 1), st[4B] = which state is the current one; B = batch.
// A step's first kernel writes the state after the step into the other slot, its last one makes that
// slot the current one.  Counts are clamped to the layer's capacity, so stale or foreign contents
// cannot take an access out of the layer's buffers.
constexpr int kDevLenPad = 4;
__host__ __device__ inline int dev_len_ints(int batch) { return 4 * batch + kDevLenPad; }
__device__ __forceinline__ void dev_len(const int *st, int batch, int b, int after, int nb_cap, int r_cap, int &nb, int &r)
{
    const int p = (st[4 * batch] & 1) ^ after;
    nb = st[p * 2 * batch + 2 * b];
    r = st[p * 2 * batch + 2 * b + 1];
    nb = nb < 0 ? 0 : (nb > nb_cap ? nb_cap : nb);
    r = r < 0 ? 0 : (r > r_cap ? r_cap : r);
}

struct AppendArgs {
    LayerGeom geom;
    unsigned char *layer;   // device base of the layer buffer
    const uint16_t *k_new;  // device
    const uint16_t *v_new;
    long long stride_b, stride_t, stride_h; // elements
    int n_kv_heads, batch; // batch: sequences of this launch (a run b0 .. b0 + batch - 1 of the cache's)
    int b0;             // first sequence of the run in the cache; the input pointers already point at it
    int r_old;          // residual tokens before the call
    int first_block;    // index of the first block this call writes
    int n_flush_blocks; // blocks to compress
    int copy_src, copy_dst, copy_n; // raw tail: input tokens [copy_src, copy_src+copy_n) -> residual[copy_dst..]
    int tail_too;       // the quantiser's launch stores the raw tail as well (no block of it comes from the
                        // residual buffer; not with len_dev)
    // rotary embedding applied to the new keys on their way in (0: none, 1: pairs (i, i + 64),
    // 2: pairs (2i, 2i + 1)); tables [n_new][64] binary32, device
    int rope;
    const float *rope_cos, *rope_sin;
    // 0: keys and values; 1: keys only; 2: values only (the other side of the call is handled by
    // another kernel: the value projection fused with the compression, Alg. 1 step 3).  Only the
    // one-wavefront-per-item quantiser (blocks of 32 tokens, one width) and the raw copy take 1 or 2.
    int sides;
    // not null: a decode step on device-resident lengths (dev_len).  The quantiser's launch first
    // stores one token per sequence at the sequence's own position in the raw buffer and writes the
    // state after the step; then it compresses a sequence's raw buffer only if that token fills it
    // (r_old = R - 1: the last row from the caller), as block number "packed blocks" of the state before.
    int *len_dev;
};

// Value projection fused with the compression (Alg. 1 step 3): one launch covers, for each sequence
// of a run, n_groups groups of up to 32 consecutive tokens of the call's input.
struct ProjectArgs {
    LayerGeom geom;
    unsigned char *layer;    // device base of the layer buffer
    const uint16_t *x;       // layer input rows, [sequence of the run][token of the call][model_dim]
    long long x_stride_b, x_stride_t; // elements
    const uint16_t *w;       // value projection weights [n_kv_heads * 128][model_dim], one row per output channel
    int model_dim;
    int n_kv_heads, batch, b0; // sequences of this launch and the first one's index in the cache
    int t0;                  // token of the call's input that group 0 starts at
    int n_groups, n_tok;     // groups per sequence; tokens per sequence they cover (the last group may be short)
    int mode;                // 0: group gi is compressed into block first_block + gi; 1: raw rows into the
                             // residual buffer, token i of the launch at row dst_row + i
    int first_block, dst_row;
    uint16_t *v_out;         // if not null: the projected values as a tensor [sequence][token][kv head][128]
    long long vo_stride_b, vo_stride_t, vo_stride_h;
};

struct DecodeArgs {
    LayerGeom geom;
    const unsigned char *layer;
    const uint16_t *q;   // [batch][Hq][128]
    float *ws;           // partials [U][g][n_splits][kPartialStride] (uneven: see partial_row)
    float *out;          // [batch][Hq][128]
    uint16_t *out16;     // the same in the cache's 16-bit type, if not null (then `out` is not written)
    int n_kv_heads, n_q_heads, batch, g;
    int n_blocks;        // packed blocks in the layer
    int r;               // residual tokens
    int n_splits;
    // not 0: a split count per sequence in place of n_splits, for the kernels without a mean over the heads and
    // the kernel of the 16-bit layers: as many as its chunks need for `uneven` rounds of a workgroup's waves
    // (uneven_count); grid (uneven_total, n_kv_heads), a sequence's splits behind those of the one before
    int uneven;
    int uneven_chunk;  // tokens of such a chunk (32, 64 or 128), uneven_tails: the raw tokens are chunks, too
    int uneven_tails, uneven_total, uneven_most; // (most: of any sequence)
    // of a unit's splits the last resid_splits take its raw tokens (tiles of 32 in turn) and no chunks; 0: the raw
    // tokens are dealt to all splits behind their chunks (matrix-core kernel without a mean over the heads)
    int resid_splits;
    // 1: one split per unit, and the split kernel writes the output itself (binary32, to out; no merge).  2: the split
    // kernel joins the splits itself (join.h) and counts the finished workgroups of each unit at `sync`
    int direct;
    int blocks_per_split;
    // the launch's records are fetched past the caches (matrix-core kernel and the kernel of the 16-bit layers; read by the host, which
    // launches another instance)
    int stream;
    // matrix-core kernel only: the newest residual token (index r - 1) is not in the cache yet;
    // the kernel takes it from these rows and stores it (null: every token is in the cache)
    const uint16_t *k_fresh, *v_fresh;
    long long fresh_stride_b, fresh_stride_h; // elements
    // cross-head mean on the matrix-core path: the dense mean terms go through three arrays in the
    // workspace (null otherwise).  xs [batch][Hq][tcap]: q . mean_K of every packed token;
    // xp [batch][Hq][tcap]: softmax weight of every packed token relative to its chunk's maximum;
    // xmc [batch][Hq][tcap / 64 + 1]: that maximum (exp2 domain) per 64-token chunk.
    float *xs, *xp, *xmc;
    int tcap;
    // xo [batch][Hq][n_xr][128]: the value mean plane's share of the output, per range of chunks,
    // relative to the head's largest split maximum; the merge adds the ranges up
    float *xo;
    int n_xr;
    // sequences of different lengths: n_blocks and r above are the maxima, the kernels take each
    // sequence's own counts from these (ragged == 0: every sequence has n_blocks and r)
    int ragged;
    // not null: the kernels take every sequence's counts from these device-resident lengths (the state
    // after the step's append, dev_len) instead; n_blocks and r only size the launch.  The call's last kernel
    // makes that state the current one: the merge, or the split kernel where it joins the splits (step_is_done).
    int *len_dev;
    unsigned long long *sync, sync_base; // counts, zero after the launch; what this call counts down to (count_in)
    uint16_t nb_seq[kMaxRaggedBatch], r_seq[kMaxRaggedBatch]; // 1 KiB of the kernel arguments
};

// packed blocks / raw tokens of sequence b
__host__ __device__ inline int seq_blocks(const DecodeArgs &a, int b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if (a.len_dev) {
        int nb, r;
        dev_len(a.len_dev, a.batch, b, 1, a.geom.NB, a.geom.R, nb, r);
        return nb;
    }
#endif
    return a.ragged ? a.nb_seq[b] : a.n_blocks;
}
__host__ __device__ inline int seq_resid(const DecodeArgs &a, int b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if (a.len_dev) {
        int nb, r;
        dev_len(a.len_dev, a.batch, b, 1, a.geom.NB, a.geom.R, nb, r);
        return r;
    }
#endif
    return a.ragged ? a.r_seq[b] : a.r;
}

constexpr int kSplitWaves = 4; // wavefronts of a workgroup that share a unit's chunks (kernels that take uneven splits)
// chunks and splits of a sequence that holds nb packed blocks and r raw tokens
__host__ __device__ inline int uneven_chunks(const DecodeArgs &a, int nb, int r)
{
    return (nb * a.geom.G + a.uneven_chunk - 1) / a.uneven_chunk + (a.uneven_tails ? (r + a.uneven_chunk - 1) / a.uneven_chunk : 0);
}
__host__ __device__ inline int uneven_count(const DecodeArgs &a, int nb, int r)
{
    const int chunks = uneven_chunks(a, nb, r);
    const int per = kSplitWaves * a.uneven, n = (chunks + per - 1) / per;
    return n > 0 ? n + a.resid_splits : (r > 0 ? 1 + a.resid_splits : 0);
}
// channel c of query head `head` (of unit u's group) of a launch with one split per unit: the sums num and den
// relative to the maximum M, divided as the merge does (a sequence without tokens, M == -inf, gives zero)
__device__ __forceinline__ void put_output(const DecodeArgs &a, int u, int head, int c, float num, float den, float M)
{
    a.out[((long long)u * a.g + head) * kHeadDim + c] = M == -INFINITY ? 0.0f : num / den; // (n_q_heads = n_kv_heads g)
}
// Where sequence b's splits begin, and how many there are: every lane counts those of up to four sequences and
// the lanes add up (a table of the offsets in the arguments is one more dependent load from
// memory and made every launch 0.3 us longer, also those that do not use it).  b < 0: the sequence that split x
// belongs to.
__device__ __forceinline__ void uneven_find(const DecodeArgs &a, int x, int &b, int &first, int &ns)
{
    const int lane = threadIdx.x & 63;
    int before = 0;
    for (int b0 = 0;; b0 += 64) {
        const int i = b0 + lane;
        const int n = i < a.batch ? uneven_count(a, a.nb_seq[i], a.r_seq[i]) : 0;
        int end = n;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(end, o);
            end += lane >= o ? t : 0;
        }
        end += before;
        // (split x: behind the sequences that end at or before it)
        const int at = b >= 0 ? b : b0 + (int)__popcll(__builtin_amdgcn_ballot_w64(i < a.batch && end <= x));
        if (at < b0 + 64 || b0 + 64 >= a.batch) {
            b = at < a.batch ? at : a.batch - 1;
            ns = __builtin_amdgcn_readlane(n, b - b0);
            first = __builtin_amdgcn_readlane(end, b - b0) - ns;
            return;
        }
        before = __builtin_amdgcn_readlane(end, 63);
    }
}
// The arguments that a decode kernel's first steps depend on, requested together at its start.  Left to itself the
// compiler loads an argument behind the branch that needs it, and every such load is a round trip to memory (nothing
// of a launch's arguments is in a cache yet) that the next one waits for: five of them stood in front of the
// split kernel's first fetch.  With this, and the operand scratch cleared behind that fetch:
// one sequence of 8205 tokens 11.4 -> 10.5 us a call, 16 sequences of 32781 tokens at 2, 4 and 8 bits 458 -> 453 us, one of
// 131079 tokens with 64 query heads 141 -> 134 us.
__device__ __forceinline__ void decode_args_here(const DecodeArgs &a)
{
    const LayerGeom &g = a.geom;
    asm volatile("" : : "s"(a.n_kv_heads), "s"(a.n_q_heads), "s"(a.batch), "s"(a.g), "s"(a.n_blocks), "s"(a.r), "s"(a.n_splits),
                 "s"(a.uneven), "s"(a.resid_splits), "s"(a.direct), "s"(a.out), "s"(a.ragged), "s"(a.len_dev), "s"(a.layer), "s"(a.q), "s"(a.ws),
                 "s"(g.NB), "s"(g.R), "s"(g.dtype), "s"(g.k_resid_off), "s"(g.v_resid_off), "s"(a.k_fresh), "s"(g.table),
                 "s"(g.table_stride), "s"(g.pool));
}
// first partial result of (unit u, query head i of its group) and the number of its splits
__device__ __forceinline__ long long partial_row(const DecodeArgs &a, int u, int i, int &ns)
{
    if (__builtin_expect(!a.uneven, 1)) {
        ns = a.n_splits;
        return ((long long)u * a.g + i) * ns;
    }
    int b = u / a.n_kv_heads, first;
    uneven_find(a, 0, b, first, ns);
    return ((long long)first * a.n_kv_heads + (long long)(u % a.n_kv_heads) * ns) * a.g + (long long)i * ns;
}
// unit and split of this workgroup, the number of the unit's splits and its first partial result (query head 0;
// head i: i * ns further).  Grid: see DecodeArgs::uneven; otherwise (n_splits, units).
__device__ __forceinline__ void unit_and_split(const DecodeArgs &a, int &u, int &sp, int &ns, int &row)
{
    if (__builtin_expect(!a.uneven, 1)) {
        sp = blockIdx.x;
        u = blockIdx.y;
        ns = a.n_splits;
        row = u * a.g * ns;
        return;
    }
    int b = -1, first;
    uneven_find(a, blockIdx.x, b, first, ns);
    b = __builtin_amdgcn_readfirstlane(b);
    sp = (int)blockIdx.x - first;
    u = b * a.n_kv_heads + (int)blockIdx.y;
    row = (first * a.n_kv_heads + (int)blockIdx.y * ns) * a.g;
}

// reconstruction of a layer's contents: lengths and geometry as for a decode launch
struct DequantArgs {
    DecodeArgs d;
    float *k_out, *v_out; // [batch][t_cap][n_kv_heads][128] binary32, either may be null
    int t_cap;
    int pad; // not 0: zeros go to the rows past a sequence's length
};

// records the outcome of a launch for kv_last_hip_error and passes it through
hipError_t note_launch(hipError_t e);

hipError_t launch_flush(const AppendArgs &a, hipStream_t s);
hipError_t launch_resid_copy(const AppendArgs &a, hipStream_t s);
bool step_store_supported(const LayerGeom &g); // formats the device-length decode step serves (launch_flush with len_dev)
bool compressv_supported(const LayerGeom &g); // formats the fused value projection serves
hipError_t launch_compressv(const ProjectArgs &p, hipStream_t s);
hipError_t launch_decode_split_valu(const DecodeArgs &a, hipStream_t s);
hipError_t launch_decode_split_mfma(const DecodeArgs &a, hipStream_t s);
// layers stored in 16 bits
bool decode_raw_supported(const DecodeArgs &a);
int decode_raw_splits(const DecodeArgs &a, int cap); // preferred split count, at most cap
int decode_raw_slots(const DecodeArgs &a);           // workgroups the device holds at once
hipError_t launch_decode_split_raw(const DecodeArgs &a, hipStream_t s);
// the calling thread's next matrix-core split launch records its begin and end into these (one-shot; null cancels)
void set_split_timing_events(hipEvent_t begin, hipEvent_t end);
bool decode_mfma_supported(const DecodeArgs &a);
// the matrix-core split kernel for keys of one width (decode_mfma.hip)
struct SplitTiming { hipEvent_t begin, end; };
struct MfmaWidth {
    bool (*matches)(const DecodeArgs &a); // is the layer's record laid out as its instance takes it to be
    int (*splits)(const DecodeArgs &a);
    int (*slots)(const DecodeArgs &a);
    hipError_t (*launch)(const DecodeArgs &a, hipStream_t s, SplitTiming &ev); // ev: recorded into, then cleared
    hipError_t (*launch_stream)(const DecodeArgs &a, hipStream_t s, SplitTiming &ev); // with DecodeArgs::stream
};
MfmaWidth mfma_width_2(), mfma_width_4(), mfma_width_8();
hipError_t mfma_stream_2(const DecodeArgs &a, hipStream_t s, SplitTiming &ev), mfma_stream_4(const DecodeArgs &a, hipStream_t s, SplitTiming &ev),
    mfma_stream_8(const DecodeArgs &a, hipStream_t s, SplitTiming &ev);
// Does the layer get the fused cross-head form (both mean terms inside the split kernel)?  It takes a
// wave per kv head, a multiple of 4 kv heads.
inline bool xhead_fused_fmt(const DecodeArgs &a) { return a.geom.mean_mode == 1 && a.n_kv_heads % 4 == 0; }
bool xhead_fused(const DecodeArgs &a); // cross-head mean: both mean terms inside the matrix-core split kernel
int decode_mfma_splits(const DecodeArgs &a); // preferred split count of the matrix-core kernel
int decode_mfma_slots(const DecodeArgs &a);  // workgroups of it the device holds at once
hipError_t launch_decode_merge(const DecodeArgs &a, hipStream_t s);
hipError_t launch_dequant(const DequantArgs &q, hipStream_t s);
// cross-head mean, matrix-core path: scores of the queries against the key mean plane (before the
// split kernel) and the value mean plane's contribution to the partial outputs (before the merge)
hipError_t launch_xhead_scores(const DecodeArgs &a, hipStream_t s);
hipError_t launch_xhead_values(const DecodeArgs &a, hipStream_t s);
int xhead_values_resident(int n_q_heads);
// read-only streaming pass over a buffer (the benchmark's measured bandwidth ceiling)
hipError_t launch_stream_read(const void *buf, size_t bytes, unsigned long long *sink, hipStream_t s); // workgroups of the value-mean kernel the device holds at once

} // namespace tadakv
