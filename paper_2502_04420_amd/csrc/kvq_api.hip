// Host side of the C ABI declared in include/kvq.h: argument validation, workspace
// planning, the per-layer token bookkeeping of the full-precision window, and the
// kernel launches.  No device memory is allocated here and nothing synchronises.
#include "../../include/kvq.h"

#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "kvq_internal.h"

namespace {

constexpr int kMaxSplits = 128;
constexpr int kPrefillChunk = 16;   // caches dequantized per prefill-attention pass (two per XCD)
constexpr size_t kPrefillSlots = 512;  // partial results of prefill attention: two pieces of a query tile per compute unit (68 MB)
constexpr int kWindowWeight = 6;   // cost of a chunk (<= 32 tokens) of the fp16 window in a split's share, in packed blocks
using kvq::kCUs;
constexpr size_t kAlign = 256;

thread_local char g_last_error[256] = "";

// Built-in scratch of kvq_decode_attention_noalloc: the partial results of the token-range splits, which the other
// decode calls keep in the caller's workspace.  One record per (query row, split): 128 un-normalised outputs, then
// (further back) the pair (maximum, sum).  Every GPU the library runs on holds its own copy until the process ends.
constexpr size_t kStaticRecords = 16384;                                   // 2048 groups x 8 grouped query heads
constexpr size_t kStaticOutBytes = kStaticRecords * kvq::kD * sizeof(float);
constexpr size_t kStaticBytes = kStaticOutBytes + kStaticRecords * 2 * sizeof(float);      // 8.1 MiB
constexpr int kMaxDevices = 64;
}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticBytes];

namespace {
// device address of `scratch` on each GPU (the array's name is only a host-side handle), looked up once per device
std::atomic<unsigned char *> g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mutex;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool bits_ok(int b) { return b == 2 || b == 4 || b == 8 || b == 16; }

bool config_ok(const kvq_config *c)
{
    if (!c || !c->kbits || !c->vbits) return false;
    if (c->n_layers < 1 || c->batch < 1 || c->n_kv_heads < 1 || c->n_q_heads < 1) return false;
    if (c->n_q_heads % c->n_kv_heads) return false;
    if (c->head_dim != kvq::kD || c->group != kvq::kG) return false;
    if (c->max_tokens < 1 || c->residual < 0 || c->residual > (1 << 20)) return false;
    if ((int64_t)c->batch * c->n_q_heads > (1 << 24)) return false;
    if ((int64_t)c->batch * c->n_kv_heads > 65535) return false;        // one grid row per (batch, kv head)
    for (int l = 0; l < c->n_layers; l++)
        if (!bits_ok(c->kbits[l]) || !bits_ok(c->vbits[l])) return false;
    if (c->meta_dtype != KVQ_META_FP32 && c->meta_dtype != KVQ_META_FP16) return false;
    if (c->key_mode != KVQ_KEYS_PER_CHANNEL && c->key_mode != KVQ_KEYS_PER_TOKEN) return false;
    return true;
}

struct LayerPlan {
    size_t kcode, kmeta, vcode, vmeta, bexp, kres, vres;   // byte offsets into the workspace
};

struct Plan {
    std::vector<LayerPlan> layer;
    size_t part_o, part_ml, prefill_scratch, prefill_select, total;
    int prefill_slots;      // pieces of query tiles whose partial results the prefill attention may keep (at part_o)
    int NB, RC;
    int prefill_chunk;      // (batch, kv head) caches whose dequantized units the prefill scratch holds at a time
};

// bytes: what the caller's workspace holds
Plan make_plan(const kvq_config *c, size_t bytes = SIZE_MAX)
{
    Plan p;
    const size_t BH = (size_t)c->batch * c->n_kv_heads;
    p.NB = c->max_tokens / kvq::kG;                 // N_p never exceeds G * floor(max_tokens / G)
    p.RC = c->residual + kvq::kG;                   // the fp16 window never holds R + G tokens or more
    const bool narrow = c->meta_dtype == KVQ_META_FP16;
    size_t off = 0;
    p.layer.resize(c->n_layers);
    for (int l = 0; l < c->n_layers; l++) {
        LayerPlan &y = p.layer[l];
        const int kb = c->kbits[l], vb = c->vbits[l];
        y.kcode = off; off = align_up(off + BH * p.NB * kvq::block_code_bytes(kb));
        y.kmeta = off; off = align_up(off + BH * p.NB * kvq::block_meta_bytes(kb, narrow));
        y.vcode = off; off = align_up(off + BH * p.NB * kvq::block_code_bytes(vb));
        y.vmeta = off; off = align_up(off + BH * p.NB * kvq::block_meta_bytes(vb, narrow));
        y.bexp = off; off = align_up(off + BH * p.NB * sizeof(uint32_t));
        y.kres = off; off = align_up(off + BH * p.RC * kvq::kD * 2);
        y.vres = off; off = align_up(off + BH * p.RC * kvq::kD * 2);
    }
    const size_t rows = (size_t)c->batch * c->n_q_heads;
    p.part_o = off; off = align_up(off + rows * kMaxSplits * kvq::kD * sizeof(float));
    p.part_ml = off; off = align_up(off + rows * kMaxSplits * 2 * sizeof(float));
    // The prefill attention's partial results share that area with the decode splits': the two kinds of calls follow each
    // other on the context's stream.  They belong to pieces of query tiles (tiles are cut where they are too few to fill the
    // GPU, into pieces of 12 units or more, so only where there are 24).  A piece per compute unit is enough for most
    // launches; where the splits' area does not hold that many, it grows to hold two, or as many as the workspace has
    // room for: with fewer slots the tiles are cut less, or not at all.
    p.prefill_chunk = BH < (size_t)kPrefillChunk ? (int)BH : kPrefillChunk;
    const size_t scratch = align_up((size_t)p.prefill_chunk * p.NB * kvq::prefill_unit_bytes());
    const size_t select = align_up(BH * kvq::prefill_select_bytes());                     // (a pass may take all caches)
    const size_t least = off + scratch + select, piece = kvq::prefill_piece_bytes();
    const size_t tiles = ((size_t)c->max_tokens + kvq::kQueryTile - 1) / kvq::kQueryTile;
    const size_t most = p.NB < 24 ? 0 : rows * tiles * (p.NB / 12);
    size_t slots = (off - p.part_o) / piece;
    if (slots < kPrefillSlots / 2) slots = kPrefillSlots;
    if (slots > most) slots = most;
    if (slots > kPrefillSlots) slots = kPrefillSlots;
    const size_t room = (off - p.part_o + (bytes > least ? bytes - least : 0)) / piece;   // (piece: a multiple of kAlign)
    if (slots > room) slots = room;
    p.prefill_slots = (int)slots;
    if (off < p.part_o + slots * piece) off = p.part_o + slots * piece;
    p.prefill_scratch = off; off += scratch;
    p.prefill_select = off; off += select;
    p.total = off;
    return p;
}

}  // namespace

struct kvq_ctx {
    kvq_config cfg;
    std::vector<uint8_t> kbits, vbits;
    std::vector<int> tokens;        // T per layer
    Plan plan;
    uint8_t *ws;
    hipStream_t stream;
    int variant;                    // 0 auto, 1 vector ALU, 2 matrix core
    int splits;                     // 0 auto
    int prefill_low_parts;          // 0: chosen per cache, 1: every key channel keeps its low part
    hipEvent_t ev_begin, ev_end;    // recorded around the main decode kernel when both are set
};

namespace {

int decode_variant(const kvq_ctx *c) { return c->variant == 0 ? 2 : c->variant; }     // the matrix-core kernel is the default

int packed_tokens(const kvq_ctx *c, int T)
{
    const int over = T - c->cfg.residual;
    return over > 0 ? kvq::kG * (over / kvq::kG) : 0;
}

kvq::LayerView view(const kvq_ctx *c, int l)
{
    const LayerPlan &y = c->plan.layer[l];
    kvq::LayerView v;
    v.kcode = c->ws + y.kcode;
    v.kmeta = reinterpret_cast<float *>(c->ws + y.kmeta);
    v.vcode = c->ws + y.vcode;
    v.vmeta = reinterpret_cast<float *>(c->ws + y.vmeta);
    v.bexp = reinterpret_cast<uint32_t *>(c->ws + y.bexp);
    v.kres = reinterpret_cast<uint16_t *>(c->ws + y.kres);
    v.vres = reinterpret_cast<uint16_t *>(c->ws + y.vres);
    v.kbits = c->kbits[l];
    v.vbits = c->vbits[l];
    v.narrow = c->cfg.meta_dtype == KVQ_META_FP16 ? 1 : 0;
    v.kpt = c->cfg.key_mode == KVQ_KEYS_PER_TOKEN ? 1 : 0;
    return v;
}

float *ws_part_o(const kvq_ctx *c) { return reinterpret_cast<float *>(c->ws + c->plan.part_o); }
float *ws_part_ml(const kvq_ctx *c) { return reinterpret_cast<float *>(c->ws + c->plan.part_ml); }
size_t ws_part_records(const kvq_ctx *c) { return (size_t)c->cfg.batch * c->cfg.n_q_heads * kMaxSplits; }

// Arrival counters of the decode and the channel selection kernels: in the selection records of the prefill attention, one record per
// cache, shared by all layers.  A cache's counters start at zero when a layer's first block is quantized (only calls with packed
// blocks count) and are zero again after every call.
uint32_t *ws_tickets(const kvq_ctx *c) { return reinterpret_cast<uint32_t *>(c->ws + c->plan.prefill_select + kvq::prefill_ticket_offset()); }
int ticket_stride() { return (int)(kvq::prefill_select_bytes() / sizeof(uint32_t)); }
int tickets_per_cache(const kvq_ctx *c) { return (c->cfg.n_q_heads / c->cfg.n_kv_heads + 7) / 8; }

int launch_failed(const char *what, hipError_t e)
{
    snprintf(g_last_error, sizeof g_last_error, "%s: %s", what, hipGetErrorString(e));
    return KVQ_ELAUNCH;
}

}  // namespace

extern "C" {

size_t kvq_workspace_bytes(const kvq_config *cfg)
{
    if (!config_ok(cfg)) return 0;
    return make_plan(cfg).total;
}

int kvq_configure(kvq_ctx **out, const kvq_config *cfg, void *workspace_device, size_t workspace_bytes,
                  void *hip_stream)
{
    if (!out) return KVQ_EINVAL;
    *out = nullptr;
    if (!config_ok(cfg)) return KVQ_EINVAL;
    Plan plan = make_plan(cfg, workspace_bytes);
    if (!workspace_device || (reinterpret_cast<uintptr_t>(workspace_device) % kAlign) || workspace_bytes < plan.total)
        return KVQ_EWORKSPACE;
    kvq_ctx *c = new (std::nothrow) kvq_ctx();
    if (!c) return KVQ_EINVAL;
    c->cfg = *cfg;
    c->kbits.assign(cfg->kbits, cfg->kbits + cfg->n_layers);
    c->vbits.assign(cfg->vbits, cfg->vbits + cfg->n_layers);
    c->cfg.kbits = c->kbits.data();
    c->cfg.vbits = c->vbits.data();
    c->tokens.assign(cfg->n_layers, 0);
    c->plan = plan;
    c->ws = static_cast<uint8_t *>(workspace_device);
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->variant = 0;
    c->splits = 0;
    c->prefill_low_parts = 0;
    c->ev_begin = c->ev_end = nullptr;
    *out = c;
    return KVQ_OK;
}

namespace {

// Append n_tokens to a layer: quantize the groups that leave the fp16 window, then (unless the caller's decode
// launch takes the single new token along) copy the tokens that stay in the window into the ring.
int append_tokens(kvq_ctx *c, int layer, const void *k_device, const void *v_device, int n_tokens, bool copy_window)
{
    const int t_old = c->tokens[layer];
    if ((int64_t)t_old + n_tokens > c->cfg.max_tokens) return KVQ_ECAPACITY;
    const int t_new = t_old + n_tokens;
    const int np_old = packed_tokens(c, t_old), np_new = packed_tokens(c, t_new);
    const int BH = c->cfg.batch * c->cfg.n_kv_heads;

    // new tokens that stay in the window go to the ring
    const int pos0 = np_new > t_old ? np_new : t_old;
    bool copy = copy_window && t_new > pos0;

    // 1. quantize the groups that leave the fp16 window: positions [np_old, np_new)
    if (np_new > np_old) {
        kvq::QuantArgs a;
        a.lv = view(c, layer);
        a.k_in = static_cast<const uint16_t *>(k_device);
        a.v_in = static_cast<const uint16_t *>(v_device);
        a.n_in = n_tokens;
        a.t_old = t_old;
        a.first_block = np_old / kvq::kG;
        a.n_blocks = (np_new - np_old) / kvq::kG;
        a.BH = BH;
        a.NB = c->plan.NB;
        a.RC = c->plan.RC;
        a.copy_pos0 = a.copy_pos1 = 0;
        a.tickets = ws_tickets(c);
        a.ticket_stride = ticket_stride();
        // The same launch fills the ring, unless a new token's slot still holds a token that this launch quantizes: slots are
        // positions modulo RC, so the first such token would be RC behind the last new one.  (Never the case in a prompt's
        // first append, which quantizes nothing from the ring, or when one token is appended.)
        if (copy && (np_old >= t_old || t_new - 1 < np_old + c->plan.RC) && kvq::quantize_takes_window(a.n_blocks, BH, t_new - pos0)) {
            a.copy_pos0 = pos0;
            a.copy_pos1 = t_new;
            copy = false;
        }
        hipError_t e = kvq::launch_quantize(a, c->stream);
        if (e != hipSuccess) return launch_failed("quantize kernel", e);
    }
    // 2. the ring, if step 1 has not filled it: after it has read the old slots
    if (copy) {
        kvq::ResidualCopyArgs a;
        a.lv = view(c, layer);
        a.k_in = static_cast<const uint16_t *>(k_device);
        a.v_in = static_cast<const uint16_t *>(v_device);
        a.n_in = n_tokens;
        a.t_old = t_old;
        a.pos0 = pos0;
        a.pos1 = t_new;
        a.BH = BH;
        a.RC = c->plan.RC;
        hipError_t e = kvq::launch_residual_copy(a, c->stream);
        if (e != hipSuccess) return launch_failed("window copy kernel", e);
    }
    c->tokens[layer] = t_new;
    return KVQ_OK;
}

// How a decode launch divides the tokens of a (batch, kv head) cache among its groups.
struct SplitPlan { int splits, units_per_split, split_rem; };

// BH caches of gq query heads, code width = key bits + value bits, n_blocks packed blocks and n_res fp16 window tokens per cache;
// forced: the caller's split count (0 = choose); variant: 1 vector-ALU kernel, 2 matrix-core kernel.
SplitPlan plan_splits(int BH, int gq, int width, int n_blocks, int n_res, int forced, int variant)
{
    int splits = forced;
    if (splits <= 0) {
        // 16 waves per compute unit (4 on every SIMD) over 256 compute units: 2048 two-wave groups of the
        // matrix-core kernel or 1024 four-wave groups of the vector kernel.  More splits only add per-group
        // set-up and merge work, so split no further and keep at least 4 (8) blocks per group.
        // The wider a layer's codes, the more bytes every group keeps in flight and the fewer groups serve it
        // best (measured at batch 8..64, 8K and 32K tokens: K8V8 4-7 % faster with 1024 groups than with 2048,
        // K8V4 and K4V8 5 %; K4V4 and narrower are fastest with 2048).  K8V2 and K2V8 are as fast with 1024 as with
        // 2048 and 2-6 % slower with 1536 (3 waves per SIMD: the key and value roles cannot be even on every SIMD).
        const int groups = variant != 2 ? 1024 : width <= 8 ? 2048 : 1024;
        const int min_units = variant == 2 ? 4 : 8;
        splits = (groups + BH - 1) / BH;
        // most splits where each takes `blocks` blocks and one the window, and the work-groups they make (one per split, cache and 8 query heads)
        auto cap_at = [&](int blocks) { return (n_blocks + blocks - 1) / blocks + (n_res > 0 ? 1 : 0); };
        const long long per_split = (long long)BH * ((gq + 7) / 8);
        const int chunks = (n_res + 31) / 32;
        int cap = cap_at(min_units);
        if (variant == 2) {
            // Few groups leave every compute unit one group or none, and a call takes as long as its longest group.  The lines were drawn with one
            // pair of waves per group.  With the kernels as they stand (two pairs up to kvq::paired_groups; K4V2 and K8V8 within 1 % of
            // each other unless said), us a call, blocks per group / the other:
            // - 4 / 5, where 4 make more groups than there are compute units and 5 do not: one sequence, 8 kv heads, a window of two chunks,
            //   272..320 groups 7.8..8.1 / 7.4, 4 kv heads 8.1 / 7.4; a window of one chunk 8.0 / 7.4 at 272 groups, 7.7 / 7.4 at 312 (below 32 groups
            //   over, the line still takes 4 there).  Where 5 still make more (328 / 264 groups) 7.7 / 8.2.  With a window of five chunks (24 caches of
            //   47 blocks, 312 / 264 groups) K4V2 7.7 / 7.7, K8V8 7.9 / 7.7.  (6 blocks where 5 make more: 7.5, 12 x 2 kv heads 7.5.)
            // - 4 / 2, up to 64 groups, where the window is one chunk at most: 6.4 / 6.0 (2 kv heads, 512 tokens).  With two chunks, where the line
            //   keeps 4, 6.5 / 6.1 now (2 kv heads, 512 and 900 tokens), and tiles of 8 heads 7.3 / 6.6 (513 tokens), 7.3 / 6.7 (900), 8.4 / 8.2 (2000).
            const long long with4 = per_split * cap_at(4), with5 = per_split * cap_at(5);
            if (with4 >= kCUs + (chunks > 1 ? 1 : 32) && (with5 <= kCUs || (chunks > 2 && with4 <= kCUs + kCUs / 4))) cap = cap_at(5);
            else if (chunks <= 1 && per_split * (n_blocks / 2 + 1) <= kCUs / 4) cap = cap_at(2);
        }
        if (splits > cap) splits = cap;
    }
    if (splits > kMaxSplits) splits = kMaxSplits;
    if (splits < 1) splits = 1;
    // The fp16 window rides on the last split, behind the split's blocks and chunk by chunk: a chunk's key and value rows are
    // each asked for at once.  The window counts as kWindowWeight units per chunk behind
    // the blocks, and the units are dealt out evenly (the last split gets that many blocks fewer, none at all when its share
    // is smaller than that).  A chunk takes about as long as a block (0.48 us, a block 0.54 or, of 8 heads, 0.69), but its rows come behind the
    // split's blocks, and the weight was set when it took two or three times that.  Measured, us a call, weights 2 / 3 / 4 / 6: batch 16,
    // 8192 tokens K4V2 31.0 / 30.4 / 31.2 / 30.8, K4V4 35.6 / 35.1 / 35.4 / 35.5; 16 x 4096 tokens K8V8 29.2 / 29.0 / 29.6 / 29.9; 64 x 1000 tokens 18.7 / 18.6 /
    // 19.0 / 19.2; 15 others, one sequence to 64, within 2 % but for one.
    int window = kWindowWeight * ((n_res + 31) / 32);
    if (n_blocks == 0) splits = 1;
    const int most = n_blocks + (window ? 1 : 0);                // no more splits than blocks (+ one for the window)
    if (splits > most) splits = most;
    if (splits < 1) splits = 1;
    // (never more than the share of a split in front of the window's: with many small splits the window's split takes no
    // blocks, not even the odd one that is left over.  With one pair of waves per group and an earlier kernel, one sequence, 23 blocks: 11.1 us a call
    // with a block in front of the window in the same group, 9.1 without)
    if (splits > 1) {
        const int share = (n_blocks + splits - 2) / (splits - 1);
        if (window > share) window = share;
    } else if (window > n_blocks) {
        window = n_blocks;
    }
    if (n_res > 0 && window < 1) window = 1;
    SplitPlan p;
    for (;;) {
        const int total = n_blocks + window;
        p.units_per_split = total / splits;
        p.split_rem = total % splits;
        if (splits <= 1) break;
        // No empty split: every split but the last must start inside the blocks (look at the one before the last), and
        // without a window so must the last.
        auto first_unit = [&](int sidx) { return sidx * p.units_per_split + (sidx > splits - p.split_rem ? sidx - (splits - p.split_rem) : 0); };
        if (first_unit(splits - 2) < n_blocks && (window || first_unit(splits - 1) < n_blocks)) break;
        splits--;
    }
    p.splits = splits;
    return p;
}

// How the matrix-core kernel is launched: pairs of waves per work-group; whether it writes the outputs itself (no combine launch).
struct DecodeForm { int pairs; bool merges; };

// Two pairs of waves per work-group (launch_decode_short) where the work-groups are few.  Such work-groups hold twice the waves and more
// registers, so fewer are resident at once (kvq::paired_groups), and beyond that the second half of them waits for the first.  Measured over 432 calls (32 / 8,
// 28 / 4 and 8 / 2 heads, K4V2, K8V8, K16V16, windows of two chunks and of three or four, 1 to 512 sequences of 60 to 7000 tokens) with the lines as they
// are: 392 take the fastest form or one within 3 % of it, the mean is 0.8 % over the fastest.  Below: the time with one pair over that with two.
// - Several splits, as long as all are resident: up to one work-group per compute unit 1.06..1.37 (median 1.2), beyond K4V2 1.01..1.13, K8V8 1.02..1.13,
//   K16V16 1.01..1.06.  More work-groups: up to half as many again K4V2 0.76..0.80, K8V8 1.00..1.09, K16V16 0.96..1.01; then 0.65..0.9.
//   (The lines for splits of 2 or 3 units and windows of one chunk were drawn where calls of either kind gained and lost up to 8 %.)
// - A single split saves the merge launch.  Up to three work-groups per compute unit 1.27..2.1, at any length and width.  Four, of packed blocks
//   0.85..1.0 (the line still takes two pairs of 4 heads with narrow codes and fp16 there: 8 / 2 heads, 512 sequences of 500 fp16 tokens 44.6 / 52.3).  Beyond:
//   - blocks are streamed faster by one pair (2048 groups of 500 tokens, K4V2 0.80..0.92) except by tiles of 4 heads where both tensors are as wide
//     (K8V8 1.03, K16V16 1.16);
//   - a window alone: tiles of 4 heads 1.01..1.06, K16V16 1.10..1.15, and of 8 heads, for which the line keeps one pair, 1.04..1.06, K16V16 1.16..1.20.
// The last work-group merges up to 48 splits of 4 heads, 32 records at a time, or 16 of 8 heads, in one go.  The launch's time over the merge's: 4 heads, 2 to 18
// splits 1.00..1.42, 27 to 48 splits 1.01..1.13, 55 and 56 splits, which the limit leaves to the launch, 1.00..1.13; 8 heads, 2 to 16 splits 0.99..1.37,
// 18 splits 1.03..1.18 (one sequence of 2200 tokens, K4V2 8.3 / 7.95, K16V16 8.0 / 6.9), 33 splits 1.00..1.03 (more are not merged: 32 lanes per head).
DecodeForm decode_form(const SplitPlan &sp, int BH, int gq, int kbits, int vbits, int n_blocks, int n_res)
{
    const int tiles = (gq + 7) / 8, chunks = (n_res + 31) / 32;
    const long long groups = (long long)BH * tiles * sp.splits;
    const bool four = gq <= 4, light = four && (kbits + vbits <= 8 || kbits == 16 || vbits == 16);
    bool paired;
    if (sp.splits > 1) {
        const int longest = sp.units_per_split + (sp.split_rem > 0 ? 1 : 0), resident = kvq::paired_groups(kbits + vbits);
        paired = groups <= (chunks > 1 ? resident : longest < (four ? 3 : 4) ? 1 : four ? resident : 2) * kCUs;
    } else if (groups <= (light ? 4 : 3) * kCUs) {
        paired = true;
    } else if (n_blocks > 0) {
        paired = four && kbits == vbits && (kbits == 16 || (kbits == 8 && n_blocks >= 16 && groups >= 6 * kCUs));
    } else {
        paired = (light && chunks >= 2) || (chunks >= 4 && groups >= 6 * kCUs);
    }
    if (!paired) return {1, false};
    return {2, sp.splits == 1 || (sp.splits <= (four ? kvq::kMergeSplits : 16) && tiles < kvq::kMaxTickets)};      // (the last counter is not the decode kernel's)
}

// Decode attention over the layer's tokens.  k_new / v_new: rows of a token that append_tokens() left out of the
// window ring (fused append), or NULL.
// part_o / part_ml: where the splits' partial results go, room for part_records (query row, split) records.
int decode_layer(kvq_ctx *c, int layer, const void *q_device, void *out_device, const void *k_new, const void *v_new,
                 float *part_o, float *part_ml, size_t part_records)
{
    const int T = c->tokens[layer];
    if (T < 1) return KVQ_ESTATE;
    const int np = packed_tokens(c, T);
    kvq::ShortDecodeArgs a;
    a.lv = view(c, layer);
    a.q = static_cast<const uint16_t *>(q_device);
    a.out = static_cast<uint16_t *>(out_device);
    a.part_o = part_o;
    a.part_ml = part_ml;
    a.B = c->cfg.batch;
    a.Hq = c->cfg.n_q_heads;
    a.Hkv = c->cfg.n_kv_heads;
    a.n_blocks = np / kvq::kG;
    a.n_res = T - np;
    a.NB = c->plan.NB;
    a.RC = c->plan.RC;
    a.scale_log2e = (float)(1.4426950408889634 / std::sqrt((double)kvq::kD));
    a.k_new = static_cast<const uint16_t *>(k_new);
    a.v_new = static_cast<const uint16_t *>(v_new);
    a.new_pos = T - 1;
    a.gq = a.Hq / a.Hkv;
    a.win_slot = np % a.RC;
    const int variant = decode_variant(c);
    const SplitPlan sp = plan_splits(a.B * a.Hkv, a.Hq / a.Hkv, a.lv.kbits + a.lv.vbits, a.n_blocks, a.n_res, c->splits, variant);
    const int splits = sp.splits;
    a.units_per_split = sp.units_per_split;
    a.split_rem = sp.split_rem;
    a.splits = splits;
    if ((size_t)a.B * a.Hq * (size_t)splits > part_records) {
        snprintf(g_last_error, sizeof g_last_error,
                 "decode needs %zu partial records (%d query rows x %d splits), the scratch holds %zu",
                 (size_t)a.B * a.Hq * (size_t)splits, a.B * a.Hq, splits, part_records);
        return KVQ_ESCRATCH;
    }
    const DecodeForm form = variant == 2 ? decode_form(sp, a.B * a.Hkv, a.Hq / a.Hkv, a.lv.kbits, a.lv.vbits, a.n_blocks, a.n_res) : DecodeForm{1, false};
    const bool paired = form.pairs > 1, merged = form.merges;
    a.tickets = merged ? ws_tickets(c) : nullptr;
    a.ticket_stride = ticket_stride();
    const bool timed = c->ev_begin && c->ev_end;
    hipError_t e;
    if (variant == 2) {
        // the matrix-core kernel's dispatch stamps the two events itself (its own start and end, no marker in between)
        const hipEvent_t begin = timed ? c->ev_begin : nullptr, end = timed ? c->ev_end : nullptr;
        e = paired ? kvq::launch_decode_short(a, c->stream, begin, end) : kvq::launch_decode_mfma(a, c->stream, begin, end);
    } else {
        if (timed && hipEventRecord(c->ev_begin, c->stream) != hipSuccess) return launch_failed("event record", hipGetLastError());
        e = kvq::launch_decode_valu(a, c->stream);
        if (e == hipSuccess && timed && hipEventRecord(c->ev_end, c->stream) != hipSuccess) return launch_failed("event record", hipGetLastError());
    }
    if (e != hipSuccess) return launch_failed("decode kernel", e);
    if (merged) return KVQ_OK;
    e = kvq::launch_combine(a, c->stream);
    if (e != hipSuccess) return launch_failed("combine kernel", e);
    return KVQ_OK;
}

}  // namespace

int kvq_quantize_append(kvq_ctx *c, int32_t layer, const void *k_device, const void *v_device, int32_t n_tokens)
{
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !k_device || !v_device || n_tokens < 1) return KVQ_EINVAL;
    return append_tokens(c, layer, k_device, v_device, n_tokens, true);
}

int kvq_decode_attention(kvq_ctx *c, int32_t layer, const void *q_device, void *out_device)
{
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !q_device || !out_device) return KVQ_EINVAL;
    return decode_layer(c, layer, q_device, out_device, nullptr, nullptr, ws_part_o(c), ws_part_ml(c), ws_part_records(c));
}

int kvq_decode_attention_noalloc(kvq_ctx *c, int32_t layer, const void *q_device, void *out_device)
{
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !q_device || !out_device) return KVQ_EINVAL;
    // the device address of the built-in scratch array, looked up once per GPU with that GPU current
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return launch_failed("hipGetDevice", e);
    if (dev < 0 || dev >= kMaxDevices) {
        snprintf(g_last_error, sizeof g_last_error, "device ordinal %d beyond the %d this build keeps scratch addresses for", dev, kMaxDevices);
        return KVQ_ESCRATCH;
    }
    unsigned char *ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        ptr = g_scratch_ptr[dev].load(std::memory_order_relaxed);
        if (!ptr) {
            e = hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr) return launch_failed("hipGetSymbolAddress(scratch)", e);
            g_scratch_ptr[dev].store(ptr, std::memory_order_release);
        }
    }
    // every record the merge reads is written by this call's decode kernel first: nothing has to start at zero
    return decode_layer(c, layer, q_device, out_device, nullptr, nullptr, reinterpret_cast<float *>(ptr),
                        reinterpret_cast<float *>(ptr + kStaticOutBytes), kStaticRecords);
}

int kvq_append_decode_attention(kvq_ctx *c, int32_t layer, const void *k_device, const void *v_device, const void *q_device,
                                void *out_device)
{
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !k_device || !v_device || !q_device || !out_device) return KVQ_EINVAL;
    // the matrix-core kernel takes the new token along (if it stays in the fp16 window); otherwise copy it first
    const int t_old = c->tokens[layer], t_new = t_old + 1;
    const bool fused = decode_variant(c) == 2 && t_new <= c->cfg.max_tokens && t_new > packed_tokens(c, t_new);
    int rc = append_tokens(c, layer, k_device, v_device, 1, !fused);
    if (rc != KVQ_OK) return rc;
    rc = decode_layer(c, layer, q_device, out_device, fused ? k_device : nullptr, fused ? v_device : nullptr,
                      ws_part_o(c), ws_part_ml(c), ws_part_records(c));
    // A refused decode launch must not leave a token counted whose window rows the decode kernel was to store: the
    // layer goes back to its length before the call.  What was enqueued before the refusal (a flush of the oldest
    // window group, a window copy) only writes what a repeat of the call writes again, identically.
    if (rc != KVQ_OK) c->tokens[layer] = t_old;
    return rc;
}

namespace {

// The caches are taken a chunk at a time: dequantize the chunk's packed units into the scratch area, attend.
// The scratch area holds prefill_chunk caches of NB units; a shorter prompt leaves room for more caches per
// pass (kept a multiple of the 8 XCDs, which the attention kernel's placement wants): fewer, larger launches.
int prefill_pass_caches(const Plan &plan, int BH, int n_blocks)
{
    int chunk = plan.prefill_chunk;
    if (n_blocks > 0 && chunk < BH) {
        const long long fit = (long long)plan.prefill_chunk * plan.NB / n_blocks;
        if (fit >= BH) chunk = BH;
        else if (fit / 8 * 8 > chunk) chunk = (int)(fit / 8 * 8);
    } else if (n_blocks == 0) {
        chunk = BH;                                             // window only: nothing goes through the scratch area
    }
    return chunk;
}

}  // namespace

int kvq_prefill_attention(kvq_ctx *c, int32_t layer, const void *q_device, int32_t n_q, void *out_device)
{
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !q_device || !out_device) return KVQ_EINVAL;
    const int T = c->tokens[layer];
    if (T < 1) return KVQ_ESTATE;
    if (n_q < 1 || n_q > T) {
        snprintf(g_last_error, sizeof g_last_error, "kvq_prefill_attention: n_q = %d queries, the layer holds %d tokens", n_q, T);
        return KVQ_EINVAL;
    }
    const int np = packed_tokens(c, T);
    kvq::PrefillArgs a;
    a.lv = view(c, layer);
    a.q = static_cast<const uint16_t *>(q_device);
    a.out = static_cast<uint16_t *>(out_device);
    a.Hq = c->cfg.n_q_heads;
    a.Hkv = c->cfg.n_kv_heads;
    a.n_blocks = np / kvq::kG;
    a.n_res = T - np;
    a.NB = c->plan.NB;
    a.RC = c->plan.RC;
    a.n_q = n_q;
    a.scale_log2e = (float)(1.4426950408889634 / std::sqrt((double)kvq::kD));
    a.scratch = c->ws + c->plan.prefill_scratch;
    a.select = nullptr;
    a.part_o = ws_part_o(c);
    a.part_ml = a.part_o + (size_t)c->plan.prefill_slots * kvq::kQueryTile * kvq::kD;
    const bool timed = c->ev_begin && c->ev_end;
    const int BH = c->cfg.batch * a.Hkv;
    const int chunk = prefill_pass_caches(c->plan, BH, a.n_blocks);
    // Keys quantized per channel: one kernel in front decides for every cache which channels keep the low parts of
    // their keys (one record per cache), unless the caller wants them kept for all.
    uint8_t *select = nullptr;
    bool begun = false;                                         // the first kernel of the call has taken ev_begin
    if (c->prefill_low_parts == 0 && a.lv.kbits < 16 && !a.lv.kpt && a.n_blocks > 0) {
        select = c->ws + c->plan.prefill_select;
        a.bh0 = 0;
        a.n_bh = BH;
        a.select = select;
        const hipError_t e = kvq::launch_prefill_select(a, c->stream, timed ? c->ev_begin : nullptr);
        if (e != hipSuccess) return launch_failed("prefill channel selection kernel", e);
        begun = true;
    }
    for (int bh0 = 0; bh0 < BH; bh0 += chunk) {
        a.bh0 = bh0;
        a.n_bh = BH - bh0 < chunk ? BH - bh0 : chunk;
        a.select = select ? select + (size_t)bh0 * kvq::prefill_select_bytes() : nullptr;
        const bool first = bh0 == 0 && !begun, last = bh0 + chunk >= BH;
        const hipError_t e = kvq::launch_prefill_attention(a, c->plan.prefill_slots, c->stream, timed && first ? c->ev_begin : nullptr,
                                                           timed && last ? c->ev_end : nullptr);
        if (e != hipSuccess) return launch_failed("prefill attention kernels", e);
    }
    return KVQ_OK;
}

int kvq_layer_tokens(const kvq_ctx *c, int32_t layer, int32_t *n_packed, int32_t *n_residual)
{
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !n_packed || !n_residual) return KVQ_EINVAL;
    const int T = c->tokens[layer];
    *n_packed = packed_tokens(c, T);
    *n_residual = T - *n_packed;
    return KVQ_OK;
}

int kvq_reset(kvq_ctx *c, int32_t layer)
{
    if (!c || layer < -1 || layer >= c->cfg.n_layers) return KVQ_EINVAL;
    for (int l = 0; l < c->cfg.n_layers; l++)
        if (layer < 0 || l == layer) c->tokens[l] = 0;
    return KVQ_OK;
}

int kvq_debug_export(kvq_ctx *c, int32_t layer, void *k_codes, void *k_scale, void *k_zero, void *v_codes,
                     void *v_scale, void *v_zero, void *k_res, void *v_res)
{
    if (!c || layer < 0 || layer >= c->cfg.n_layers) return KVQ_EINVAL;
    const int T = c->tokens[layer];
    kvq::ExportArgs a;
    a.lv = view(c, layer);
    a.k_codes = static_cast<uint8_t *>(k_codes);
    a.v_codes = static_cast<uint8_t *>(v_codes);
    a.k_scale = static_cast<float *>(k_scale);
    a.k_zero = static_cast<float *>(k_zero);
    a.v_scale = static_cast<float *>(v_scale);
    a.v_zero = static_cast<float *>(v_zero);
    a.k_res = static_cast<uint16_t *>(k_res);
    a.v_res = static_cast<uint16_t *>(v_res);
    a.n_packed = packed_tokens(c, T);
    a.n_res = T - a.n_packed;
    a.BH = c->cfg.batch * c->cfg.n_kv_heads;
    a.NB = c->plan.NB;
    a.RC = c->plan.RC;
    if (T == 0) return KVQ_OK;
    hipError_t e = kvq::launch_export(a, c->stream);
    if (e != hipSuccess) return launch_failed("export kernel", e);
    return KVQ_OK;
}

int kvq_debug_split_plan(const kvq_config *cfg, int32_t layer, int32_t n_tokens, int32_t variant, int32_t forced_splits,
                         int32_t *splits, int32_t *units_per_split, int32_t *split_rem)
{
    if (!config_ok(cfg) || layer < 0 || layer >= cfg->n_layers || n_tokens < 1 || n_tokens > cfg->max_tokens || variant < 0 ||
        variant > 2 || forced_splits < 0 || forced_splits > kMaxSplits || !splits || !units_per_split || !split_rem)
        return KVQ_EINVAL;
    const int over = n_tokens - cfg->residual;
    const int np = over > 0 ? kvq::kG * (over / kvq::kG) : 0;
    const SplitPlan p = plan_splits(cfg->batch * cfg->n_kv_heads, cfg->n_q_heads / cfg->n_kv_heads, cfg->kbits[layer] + cfg->vbits[layer], np / kvq::kG, n_tokens - np,
                                    forced_splits, variant == 0 ? 2 : variant);
    *splits = p.splits;
    *units_per_split = p.units_per_split;
    *split_rem = p.split_rem;
    return KVQ_OK;
}

int kvq_debug_decode_form(const kvq_config *cfg, int32_t layer, int32_t n_tokens, int32_t forced_splits, int32_t *pairs, int32_t *merges)
{
    if (!config_ok(cfg) || layer < 0 || layer >= cfg->n_layers || n_tokens < 1 || n_tokens > cfg->max_tokens || forced_splits < 0 ||
        forced_splits > kMaxSplits || !pairs || !merges)
        return KVQ_EINVAL;
    const int over = n_tokens - cfg->residual, np = over > 0 ? kvq::kG * (over / kvq::kG) : 0;
    const int BH = cfg->batch * cfg->n_kv_heads, gq = cfg->n_q_heads / cfg->n_kv_heads, kb = cfg->kbits[layer], vb = cfg->vbits[layer];
    const SplitPlan p = plan_splits(BH, gq, kb + vb, np / kvq::kG, n_tokens - np, forced_splits, 2);
    const DecodeForm f = decode_form(p, BH, gq, kb, vb, np / kvq::kG, n_tokens - np);
    *pairs = f.pairs;
    *merges = f.merges ? 1 : 0;
    return KVQ_OK;
}

namespace {

// Pass `pass` of a prefill-attention call, as kvq_debug_prefill_plan and _form look at it (a.n_bh = 0: there is no such pass).
int debug_prefill_pass(const kvq_config *cfg, size_t workspace_bytes, int32_t n_tokens, int32_t n_q, int32_t pass, kvq::PrefillArgs &a, int &slots)
{
    if (!config_ok(cfg) || n_tokens < 1 || n_tokens > cfg->max_tokens || n_q < 1 || n_q > n_tokens || pass < 0) return KVQ_EINVAL;
    const Plan plan = make_plan(cfg, workspace_bytes);
    if (workspace_bytes < plan.total) return KVQ_EWORKSPACE;
    const int over = n_tokens - cfg->residual, np = over > 0 ? kvq::kG * (over / kvq::kG) : 0, BH = cfg->batch * cfg->n_kv_heads;
    const int chunk = prefill_pass_caches(plan, BH, np / kvq::kG);
    const long long bh0 = (long long)pass * chunk;
    a = {};
    a.Hq = cfg->n_q_heads;
    a.Hkv = cfg->n_kv_heads;
    a.n_blocks = np / kvq::kG;
    a.n_res = n_tokens - np;
    a.n_q = n_q;
    a.n_bh = bh0 >= BH ? 0 : BH - bh0 < chunk ? (int)(BH - bh0) : chunk;
    slots = plan.prefill_slots;
    return KVQ_OK;
}

}  // namespace

int kvq_debug_prefill_plan(const kvq_config *cfg, size_t workspace_bytes, int32_t n_tokens, int32_t n_q, int32_t pass, int32_t tile,
                           int32_t *caches, int32_t *pieces)
{
    if (tile < 0 || tile > (n_q - 1) / kvq::kQueryTile || !caches || !pieces) return KVQ_EINVAL;
    kvq::PrefillArgs a;
    int slots;
    const int rc = debug_prefill_pass(cfg, workspace_bytes, n_tokens, n_q, pass, a, slots);
    if (rc != KVQ_OK) return rc;
    *caches = a.n_bh;
    *pieces = a.n_bh > 0 ? kvq::prefill_tile_pieces(a, slots, tile) : 0;
    return KVQ_OK;
}

int kvq_debug_prefill_form(const kvq_config *cfg, size_t workspace_bytes, int32_t n_tokens, int32_t n_q, int32_t pass, int32_t *waves,
                           int32_t *row_heads, int32_t *order)
{
    if (!waves || !row_heads || !order) return KVQ_EINVAL;
    kvq::PrefillArgs a;
    int slots;
    const int rc = debug_prefill_pass(cfg, workspace_bytes, n_tokens, n_q, pass, a, slots);
    if (rc != KVQ_OK) return rc;
    const kvq::PrefillForm f = a.n_bh > 0 ? kvq::prefill_form(a, slots) : kvq::PrefillForm{0, 0, 0};
    *waves = f.waves;
    *row_heads = f.row_heads;
    *order = f.order;
    return KVQ_OK;
}

int kvq_set_decode_options(kvq_ctx *c, int32_t variant, int32_t splits)
{
    if (!c || variant < 0 || variant > 2 || splits < 0 || splits > kMaxSplits) return KVQ_EINVAL;
    c->variant = variant;
    c->splits = splits;
    return KVQ_OK;
}

int kvq_set_prefill_options(kvq_ctx *c, int32_t low_parts)
{
    if (!c || low_parts < 0 || low_parts > 1) return KVQ_EINVAL;
    c->prefill_low_parts = low_parts;
    return KVQ_OK;
}

int kvq_set_kernel_events(kvq_ctx *c, void *begin_event, void *end_event)
{
    if (!c || (begin_event == nullptr) != (end_event == nullptr)) return KVQ_EINVAL;
    c->ev_begin = static_cast<hipEvent_t>(begin_event);
    c->ev_end = static_cast<hipEvent_t>(end_event);
    return KVQ_OK;
}

void kvq_destroy(kvq_ctx *c) { delete c; }

const char *kvq_strerror(int status)
{
    switch (status) {
    case KVQ_OK: return "ok";
    case KVQ_EINVAL: return "invalid argument (null pointer, layer index, bits, shape or group)";
    case KVQ_ECAPACITY: return "append exceeds max_tokens";
    case KVQ_ESTATE: return "layer holds no token";
    case KVQ_EWORKSPACE: return "workspace missing, misaligned or too small";
    case KVQ_ELAUNCH: return "HIP launch failed";
    case KVQ_ESCRATCH: return "the call needs more scratch than the library's built-in array holds";
    default: return "unknown status";
    }
}

const char *kvq_last_error(void) { return g_last_error; }

}  // extern "C"
