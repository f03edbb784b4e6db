// The matrix-core split kernel's host side: which layers it serves, and which of its six units, two per width of the
// keys, a launch's instance is in (decode_mfma.hip).
#include "tadakv_internal.h"

namespace tadakv {
namespace {

// Events that the calling thread's next split launch records its own begin and end into (set_split_timing_events)
thread_local SplitTiming t_ev = {};

MfmaWidth width(const DecodeArgs &a) { return a.geom.k_bits == 2 ? mfma_width_2() : a.geom.k_bits == 4 ? mfma_width_4() : mfma_width_8(); }

} // namespace

bool xhead_fused(const DecodeArgs &a) { return decode_mfma_supported(a) && xhead_fused_fmt(a); }

bool decode_mfma_supported(const DecodeArgs &a)
{
    const LayerGeom &g = a.geom;
    if (!(g.k_bits == 2 || g.k_bits == 4 || g.k_bits == 8) || !(g.v_bits == 2 || g.v_bits == 4 || g.v_bits == 8)) return false;
    if (g.k_bits != g.v_bits && !(g.G == 32 && g.Gc == 32 && g.mean_mode != 1 && g.table == nullptr)) return false; // different widths: one format, dense
    const bool sizes = (g.G == 32 || g.G == 64 || g.G == 128) && (g.Gc == 32 || g.Gc == 64 || g.Gc == 128);
    if (!sizes) return false;
    if (g.G != g.Gc && g.mean_mode == 1) return false; // the cross-head forms take equal sizes only
    if (a.g > 8) return false;
    if (g.mean_mode == 1 && a.n_q_heads > 64) return false; // the dense mean terms keep all query heads of a sequence in LDS
    if (a.batch * a.n_kv_heads > 65535) return false;
    // the kernels address record fields with compile-time offsets
    return width(a).matches(a);
}

int decode_mfma_splits(const DecodeArgs &a) { return decode_mfma_supported(a) ? width(a).splits(a) : 1; }

int decode_mfma_slots(const DecodeArgs &a) { return decode_mfma_supported(a) ? width(a).slots(a) : 0; }

void set_split_timing_events(hipEvent_t begin, hipEvent_t end) { t_ev = SplitTiming{begin, end}; }

hipError_t launch_decode_split_mfma(const DecodeArgs &a, hipStream_t s)
{
    if (!decode_mfma_supported(a)) return hipErrorInvalidValue;
    if (a.geom.mean_mode == 1 && !xhead_fused_fmt(a)) {
        if (!a.xs || !a.xp || !a.xmc) return hipErrorInvalidValue;
        const hipError_t e = launch_xhead_scores(a, s);
        if (e != hipSuccess) return e;
    }
    const MfmaWidth w = width(a);
    return a.stream ? w.launch_stream(a, s, t_ev) : w.launch(a, s, t_ev);
}

} // namespace tadakv
