// Prefill-stage attention over the cache as it stands (gfx950, wave64): the last n_q tokens are the queries, the
// query at absolute position p attends causally to positions 0..p (Eq. 1 under the causal mask).  The paper quantizes
// the cache in the prefill stage too and lets the prompt's own attention read the dequantized K and V (calibration
// design of Section 5.3): quantized tokens enter as X^ = Q(X) s + z (Eq. 2), window tokens as their fp16 values.
//
// This is a dense contraction (4 * D flops per query-token pair), so it runs on the matrix cores, in two passes over a
// chunk of (batch, kv head) caches at a time, behind one small kernel per call:
//   0. prefill_select (keys quantized per channel): the low parts of the keys (below) cost a third of the matrix
//      instructions, and they matter in the channels where keys and queries are large.  Per cache, from the stored
//      scales and zero-points and a sample of the queries, the kernel (a) finds every channel's centre, which pass 1
//      takes off the dequantized keys: a constant per channel moves all scores of a query alike and the softmax does
//      not see it, so an offset that a channel's keys share no longer costs fp16 precision (the window's fp16 rows keep
//      theirs; their scores are lowered by q . centre instead); (b) picks the 32 channels where one fp16 rounding of
//      the centred keys moves the logits most and checks that in all the others together it moves them by less than
//      the fp16 softmax weights are rounded by anyway; then only those 32 keep their low parts (one batch of score
//      products instead of four), otherwise all 128 do.
//   1. prefill_dequantize: every packed unit (32 tokens) of the chunk is dequantized once, X^ = fma(code, s, z) in
//      fp32, into a scratch area as fp16, in the layout the attention kernel keeps a unit in LDS: K^ as
//      [token][channel], V^ transposed as [channel][token].  Dequantized keys are multiplied by the softmax constant
//      log2(e) / sqrt(D) in fp32 (the score products then come out in the exponent's units) and kept as two fp16
//      numbers (the rounded value and the remainder), which are multiplied twice: keys have a few channels of large
//      magnitude, and one fp16 rounding of those, times a large query entry, moves a logit by several 1e-3.
//      Dequantizing inside the attention
//      kernel instead repeats this work for every query head of the group and every query tile (256 times per unit at
//      8192 queries) and made that kernel bound by its vector instructions.
//   2. prefill_attention: a work-group of 8 or 4 waves owns 256 or 128 rows (queries of one query head or of several of the
//      group's), 32 per wave (two 16-row tiles).  The units are fetched from the scratch area straight into LDS (fp16 window chunks:
//      from the ring, through registers), five or three tile buffers, so that the score products of the next
//      unit can be issued next to the softmax weights of the current one.  Scores are computed transposed, S^T = K^ Q^T
//      (16x16x32 f16 instructions, tokens along the rows): a lane then holds, for its query, the scores of tokens
//      {4 rq .. 4 rq + 3} and {16 + 4 rq ..}, which is exactly a B operand of O^T += V^T P^T when the A operand (V^T
//      from LDS) lists its tokens in the same order.  The softmax weights therefore go from the accumulator of one
//      product into the operand of the next without leaving the registers.  Online softmax in base 2 per query (the
//      reference is shared by the four lanes that hold a query and only moves when a score exceeds it by more than 8
//      in the exponent; the score products of quantized keys start from minus the reference, so that in the common
//      case their results are the exponents themselves), fp32 accumulation, one division at the end.
//   3. prefill_merge, only where a launch has too few query tiles for the GPU: the units of a tile are then attended in pieces by
//      several work-groups (plan_pieces), and this kernel merges their un-normalised results.
#include <hip/hip_ext.h>

#include <cstddef>
#include <type_traits>

#include "kvq_internal.h"

namespace kvq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kStagers = 4;              // waves that turn a unit into tiles (256 threads: the thread -> code maps below)
constexpr int kQT = 2;                   // tiles of 16 queries per wave
constexpr int kQW = 16 * kQT;            // queries per wave
constexpr int kQB = kQueryTile;         // rows of a query tile
constexpr int kKStride = kD + 16;       // halves per K^ row: 288 bytes.  Measured with a probe kernel: the 16-byte operand reads of a wave
                                        // (16 rows x 4 pieces) take 3.9 LDS cycles at this stride, like a linear read; 7.8 + 3.9 conflict cycles at 272

struct Tiles {
    _Float16 K[32][kKStride];           // K^[token][channel], rounded to fp16
    _Float16 Klo[32][kKStride];         // what the rounding left over (quantized keys only)
    _Float16 Vt[kD][32];                // V^[channel][value_place(channel, token)]
};

// Rows of 64 bytes without padding (the V^ rows, the rows of the compact low parts): the four pieces of 16 bytes of a row are rotated by row / 2.  An operand
// read takes the same piece of 16 neighbouring rows for 16 lanes; a 16-byte read of a wave is served 16 lanes at a time, but not in the order of
// the lanes.  Measured with a probe kernel, eight waves reading, bytes per cycle: rotated by row / 2 256, like a linear read and rows of 288 bytes;
// by row / 4, by row and not at all 160, rows of 80 bytes 160.
__host__ __device__ constexpr int rotated_piece(int row, int piece, int shift = 1) { return (piece + (row >> shift)) & 3; }

// Place of a token in the V^ row of a channel, rotated by channel >> shift.  A lane's operand of the output product (tokens 4 rq .. + 3 and 16 + 4 rq .. + 3, the
// rows of the scores' result tile that it holds) is one piece of 16 bytes.
__host__ __device__ constexpr int value_place(int channel, int t, int shift) { return 8 * rotated_piece(channel, (t >> 2) & 3, shift) + 4 * (t >> 4) + (t & 3); }

// fp16 keys in work-groups of 4 waves: rotated by channel / 4, and a step's fetches go out at its top.  The step is short there (no low parts, four
// batches) and ends with a wait for the unit that it fetches, and the transposed stores of a value row meet two piece addresses per lane instead
// of four.  us a pass, K16V16, rotated by / 2 and fetched between the products / so: 32 / 8 heads, four prompts of 2000 tokens 209.6 / 201.6, one
// of 190 15.25 / 15.10, four of 4000 631 / 650, last 300 of 8000 85.3 / 83.6; 28 / 4 heads, one of 1000 35.4 / 34.8; 8 / 2 heads, one of 6000 118.4 / 112.9, of
// 2500 39.9 / 38.6; 99 such calls lie between 0.97 and 1.05, without a line between them.  Work-groups of 8 waves wait once in two units and gain: last 512 of
// 24576 240.5 / 246, 8 / 2 heads, one prompt of 9000 tokens 215.5 / 220.
constexpr bool half_keys_of_4(bool quantized, int waves) { return !quantized && waves == 4; }
constexpr int value_shift(bool quantized, int waves) { return half_keys_of_4(quantized, waves) ? 2 : 1; }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Which key channels of a (batch, kv head) cache keep the remainders of their fp16 rounding (prefill_select).  In the
// compact form only the 32 selected channels do, and their remainders are stored as a tile [token][slot] of
// kLoStride halves per row at the place of Tiles::Klo (the first 2 KiB of it): one batch of the score products
// instead of four.
struct Select {
    uint8_t pos[kD];          // slot (0..31) of a channel's remainders in the compact tile, 255 = none kept
    uint8_t chan[32];         // the channel of a slot
    uint32_t compact;         // 0: every channel keeps its remainder (Tiles::Klo as declared)
    uint32_t tickets[kMaxTickets];      // arrival counters of this cache: the decode kernel's, the last one prefill_select's
    float centre[kD];         // per channel: subtracted from every dequantized key of the cache before it is rounded
};
static_assert(sizeof(Select) == 768, "one record per cache");
constexpr int kLoStride = 32;           // halves per row of the compact tile
constexpr int kLoPieces = 2;            // KiB of it
__host__ __device__ constexpr int low_place(int t, int slot) { return 8 * rotated_piece(t, slot >> 3) + (slot & 7); }
// how the keys' low parts enter the attention kernel
constexpr int kLoNone = 0, kLoAll = 1, kLoCompact = 2;

// Metadata of the unit being dequantized (in LDS), one slab per wave (wave w dequantizes channel group w of the keys and of the
// values, so it needs 32 scales and 32 zero-points of each tensor and nobody else's): written and read by the same
// wave, no work-group barrier in between.
struct MetaSlab {
    uint32_t ks[32];     // key scales (fp32, or 32 fp16 numbers in the first 16 dwords)
    uint16_t kz[32];     // key zero-points
    uint32_t vs[32];     // value scales
    uint16_t vz[32];     // value zero-points
};

// Registers of a unit on its way from the packed cache to the tiles.  Quantized tensor: k0 / v0 = the dwords of the thread's two code
// groups; fp16 rows (16-bit tensor or window): k0, k1 / v0, v1 = two 16-byte row pieces.  m = this lane's 16-byte
// piece of the wave's metadata (lanes 0..23).
// c, pos, compact: what the thread needs of the cache's selection record (keys quantized per channel): the centres and slots of its 8 channels.
struct Stage { u32x4 k0, k1, v0, v1, m, c0, c1; u32x2 pos; uint32_t compact; };

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float half_bits(uint32_t h) { return (float)__builtin_bit_cast(_Float16, (uint16_t)h); }
__device__ __forceinline__ u32x4 ld16(const void *p) { return *reinterpret_cast<const u32x4 *>(p); }
__device__ __forceinline__ u32x4 zero4() { return u32x4{0u, 0u, 0u, 0u}; }

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    const uint32_t lo = __builtin_bit_cast(uint16_t, (_Float16)a), hi = __builtin_bit_cast(uint16_t, (_Float16)b);
    return lo | (hi << 16);
}
__device__ __forceinline__ u32x4 pack8(const float *x)
{
    return u32x4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7])};
}

// ---- fp16 rows: thread tid takes 16-byte piece c16 of token t for idx = tid and tid + 256.  A token past the end reads
// the last one instead; it is zeroed on its way to LDS (an operation on the loaded value right here would make the
// wave wait for the load where it is issued).
__device__ __forceinline__ u32x4 load_row_piece(const uint16_t *base, int ring, int pos0, int T, int idx)
{
    const int t = idx >> 4, c16 = idx & 15, pos = pos0 + t, pc = pos < T ? pos : T - 1;
    return ld16(base + (size_t)(ring ? pc % ring : pc) * kD + 8 * c16);
}

// tokens past the end count as zero (their weights are zero)
__device__ __forceinline__ u32x4 live_piece(u32x4 x, int pos0, int T, int idx)
{
    const bool live = pos0 + (idx >> 4) < T;
    return u32x4{live ? x[0] : 0u, live ? x[1] : 0u, live ? x[2] : 0u, live ? x[3] : 0u};
}

__device__ __forceinline__ void store_key_rows(Tiles &L, int tid, u32x4 r0, u32x4 r1)
{
    *reinterpret_cast<u32x4 *>(&L.K[tid >> 4][8 * (tid & 15)]) = r0;
    *reinterpret_cast<u32x4 *>(&L.K[16 + (tid >> 4)][8 * (tid & 15)]) = r1;
}

// value rows are staged with the token index fastest across the lanes (piece idx: token idx & 31, 16-byte piece
// idx >> 5): the transposed 2-byte writes of a wave then fall on consecutive addresses instead of on two banks
__device__ __forceinline__ u32x4 load_value_row_piece(const uint16_t *base, int ring, int pos0, int T, int idx)
{
    const int t = idx & 31, c16 = idx >> 5, pos = pos0 + t, pc = pos < T ? pos : T - 1;
    return ld16(base + (size_t)(ring ? pc % ring : pc) * kD + 8 * c16);
}

template <int SHIFT>
__device__ __forceinline__ void store_value_piece(Tiles &L, int idx, u32x4 x, int pos0, int T)
{
    const int t = idx & 31, c16 = idx >> 5;
    const bool live = pos0 + t < T;                        // tokens past the end count as zero
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const uint32_t w = x[e >> 1];
        L.Vt[8 * c16 + e][value_place(8 * c16 + e, t, SHIFT)] = __builtin_bit_cast(_Float16, (uint16_t)(live ? ((e & 1) ? w >> 16 : w & 0xffffu) : 0u));
    }
}

// code e (0..7) of the group of eight codes numbered m, from the dwords w0, w1 that hold it
template <int BITS>
__device__ __forceinline__ float code_of(uint32_t w0, uint32_t w1, int m, int e)
{
    if constexpr (BITS == 8) return (float)(((e < 4 ? w0 : w1) >> (8 * (e & 3))) & 255u);
    else if constexpr (BITS == 4) return (float)((w0 >> (4 * ((e >> 1) + 4 * (e & 1)))) & 15u);
    else return (float)((w0 >> (2 * (4 * (m & 1) + (e >> 1) + 8 * (e & 1)))) & 3u);
}

// ---- quantized keys: thread (lane l, channel group cb = tid >> 6) takes the code groups m = cb (token n) and
// m = 4 + cb (token 16 + n), channels 32 cb + 8 kq .. + 7.  Returned: [0], [1] dwords of the first group, [2], [3] of
// the second.  Always four loads (codes narrower than 8 bits load their one dword twice): the number of loads in
// flight does not depend on the bit width.
__device__ __forceinline__ u32x4 load_key_codes(const LayerView &lv, size_t blk, int tid)
{
    const int l = tid & 63, cb = tid >> 6, kb = lv.kbits;
    const uint8_t *block = lv.kcode + blk * (size_t)block_code_bytes(kb);
    // first dword of the two groups: 8 bit -> dwords 2 m, 2 m + 1 (same 16-byte chunk); 4 bit -> dword m; 2 bit -> dword m / 2
    const int d0 = kb == 8 ? 2 * cb : kb == 4 ? cb : cb >> 1;
    const int d1 = kb == 8 ? 8 + 2 * cb : kb == 4 ? 4 + cb : 2 + (cb >> 1);
    const uint32_t *p0 = reinterpret_cast<const uint32_t *>(block + dword_offset(l, d0));
    const uint32_t *p1 = reinterpret_cast<const uint32_t *>(block + dword_offset(l, d1));
    const int odd = kb == 8 ? 1 : 0;
    return u32x4{p0[0], p0[odd], p1[0], p1[odd]};
}

// ---- quantized values: thread (lane l, channel group g = tid >> 6) takes the code groups m = 2 g, 2 g + 1
// (channels 16 m + n), tokens 8 kq .. + 7.  8 bit: dwords 4 g .. 4 g + 3 (one chunk); 4 bit: dwords 2 g, 2 g + 1;
// 2 bit: dword g; dwords beyond the width's own are loaded from the first again.
__device__ __forceinline__ u32x4 load_value_codes(const LayerView &lv, size_t blk, int tid)
{
    const int l = tid & 63, g = tid >> 6, vb = lv.vbits;
    const uint8_t *block = lv.vcode + blk * (size_t)block_code_bytes(vb);
    const uint32_t *p = reinterpret_cast<const uint32_t *>(block + dword_offset(l, vb == 8 ? 4 * g : vb == 4 ? 2 * g : g));
    return u32x4{p[0], p[vb >= 4 ? 1 : 0], p[vb == 8 ? 2 : 0], p[vb == 8 ? 3 : 0]};
}

// ---- this lane's piece of the wave's metadata: lanes 0..11 keys, 12..23 values; of each, pieces 0..7 are the 32
// scales of channel group w (fp16 scales: pieces 0..3 only) and 8..11 the 32 zero-points
__device__ __forceinline__ u32x4 load_meta_piece(const LayerView &lv, size_t blk, int wave, int lane, bool kq, bool vq)
{
    const bool narrow = lv.narrow != 0;
    const int tensor = lane >= 12 ? 1 : 0, j = lane - 12 * tensor;
    const float *meta = (tensor ? lv.vmeta : lv.kmeta) + blk * (size_t)meta_words(narrow);
    const bool wanted = lane < 24 && (tensor ? vq : kq) && !(narrow && j >= 4 && j < 8);
    const uint8_t *src = j < 8 ? reinterpret_cast<const uint8_t *>(meta) + (narrow ? 64 : 128) * wave + 16 * j
                               : reinterpret_cast<const uint8_t *>(meta_zeros(meta, narrow)) + 64 * wave + 16 * (j - 8);
    // lanes with nothing to fetch read the start of the key codes instead (the result is not used): one load per unit
    // on every path
    return ld16(wanted ? src : lv.kcode);
}

__device__ __forceinline__ void store_meta_piece(MetaSlab &M, int lane, u32x4 x)
{
    if (lane < 24) {
        const int tensor = lane >= 12 ? 1 : 0, j = lane - 12 * tensor;
        uint32_t *dst = j < 8 ? (tensor ? M.vs : M.ks) + 4 * j : reinterpret_cast<uint32_t *>(tensor ? M.vz : M.kz) + 4 * (j - 8);
        *reinterpret_cast<u32x4 *>(dst) = x;
    }
}

// eight consecutive scales / zero-points of a slab, starting at index i0 (a multiple of 8), as fp32
__device__ __forceinline__ void slab_meta8(const uint32_t *scales, const uint16_t *zeros, bool narrow, int i0, float *s, float *z)
{
    if (narrow) {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const uint16_t *>(scales) + i0);
#pragma unroll
        for (int e = 0; e < 8; e++) s[e] = half_bits((e & 1) ? a[e >> 1] >> 16 : a[e >> 1] & 0xffffu);
    } else {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(scales + i0), b = *reinterpret_cast<const u32x4 *>(scales + i0 + 4);
#pragma unroll
        for (int e = 0; e < 8; e++) s[e] = __builtin_bit_cast(float, e < 4 ? a[e & 3] : b[e & 3]);
    }
    const u32x4 c = *reinterpret_cast<const u32x4 *>(zeros + i0);
#pragma unroll
    for (int e = 0; e < 8; e++) z[e] = half_bits((e & 1) ? c[e >> 1] >> 16 : c[e >> 1] & 0xffffu);
}

// kscale: the softmax constant log2(e) / sqrt(D), multiplied into the dequantized keys in fp32 before they are split
// into two fp16 numbers: the attention kernel's score products then come out in the exponent's units.
// st.c0, c1: the channels' centres (zero without a selection record); compact: the low parts go into the compact tile
template <int BITS, bool KPT>
__device__ __forceinline__ void store_key_codes(const LayerView &lv, Tiles &L, const MetaSlab &M, int tid, const Stage &st, float kscale, bool compact)
{
    const u32x4 c = st.k0;
    const int l = tid & 63, cb = tid >> 6, n = l & 15, kq = l >> 4;
    const bool narrow = lv.narrow != 0;
    float s[8], z[8];
    if constexpr (!KPT) {
        slab_meta8(M.ks, M.kz, narrow, 8 * kq, s, z);                          // one (s, z) per channel
        // the channel's centre goes off with the zero-point: a constant per channel moves every score of a query
        // alike, which the softmax does not see (window tokens: see attend)
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const uint32_t w = e < 4 ? st.c0[e & 3] : st.c1[e & 3];
            z[e] -= __builtin_bit_cast(float, w);
        }
    }
#pragma unroll
    for (int th = 0; th < 2; th++) {
        const int t = 16 * th + n;
        if constexpr (KPT) {
            // grouped per token: one (s, z) for this token and channel group
            const float st_ = narrow ? half_bits(reinterpret_cast<const uint16_t *>(M.ks)[t]) : __builtin_bit_cast(float, M.ks[t]);
            const float zt_ = half_bits(M.kz[t]);
#pragma unroll
            for (int e = 0; e < 8; e++) { s[e] = st_; z[e] = zt_; }
        }
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; e++)      // m = 4 th + cb: m & 1 == cb & 1
            x[e] = fmaf(code_of<BITS>(th == 0 ? c[0] : c[2], th == 0 ? c[1] : c[3], cb, e), s[e], z[e]) * kscale;
        *reinterpret_cast<u32x4 *>(&L.K[t][32 * cb + 8 * kq]) = pack8(x);
#pragma unroll
        for (int e = 0; e < 8; e++) x[e] -= (float)(_Float16)x[e];
        if (compact) {
            // (channels without a slot write behind the compact tile, where nothing is read: a branch per element costs more)
            static_assert(sizeof(L.Klo) >= kLoPieces * 1024 + 256 * 2, "a place per thread behind the compact tile");
            _Float16 *tile = &L.Klo[0][0];
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const uint32_t pw = e < 4 ? st.pos[0] : st.pos[1], slot = (pw >> (8 * (e & 3))) & 255u;
                tile[slot < 32u ? t * kLoStride + low_place(t, (int)slot) : 32 * kLoStride + tid] = (_Float16)x[e];
            }
        } else {
            *reinterpret_cast<u32x4 *>(&L.Klo[t][32 * cb + 8 * kq]) = pack8(x);
        }
    }
}

template <int BITS, int SHIFT>
__device__ __forceinline__ void store_value_codes(const LayerView &lv, Tiles &L, const MetaSlab &M, int tid, u32x4 c)
{
    const int l = tid & 63, g = tid >> 6, n = l & 15, kq = l >> 4;
    float s[8], z[8];
    slab_meta8(M.vs, M.vz, lv.narrow != 0, 8 * kq, s, z);
#pragma unroll
    for (int mm = 0; mm < 2; mm++) {
        const uint32_t w0 = BITS == 8 ? (mm == 0 ? c[0] : c[2]) : BITS == 4 ? (mm == 0 ? c[0] : c[1]) : c[0];
        const uint32_t w1 = mm == 0 ? c[1] : c[3];
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; e++) x[e] = fmaf(code_of<BITS>(w0, w1, mm, e), s[e], z[e]);
        const u32x4 h = pack8(x);
        const int ch = 16 * (2 * g + mm) + n;
        *reinterpret_cast<uint2 *>(&L.Vt[ch][value_place(ch, 8 * kq, SHIFT)]) = make_uint2(h[0], h[1]);
        *reinterpret_cast<uint2 *>(&L.Vt[ch][value_place(ch, 8 * kq + 4, SHIFT)]) = make_uint2(h[2], h[3]);
    }
}

// ---- one packed unit: packed cache -> registers, registers -> tiles (LDS or the scratch area: the stores below only
// see a reference).  KQ / VQ: the layer's keys / values are quantized (else fp16 rows in the code area).
template <bool KQ, bool VQ>
__device__ __forceinline__ void load_packed(const PrefillArgs &a, int bh, int u, int T, int tid, const Select *rec, Stage &st)
{
    st.c0 = st.c1 = zero4();
    st.pos = u32x2{0u, 0u};
    st.compact = 0;
    if constexpr (KQ) {
        if (rec) {
            const int ch = 32 * (tid >> 6) + 8 * ((tid & 63) >> 4);
            st.compact = rec->compact;
            st.c0 = ld16(&rec->centre[ch]);
            st.c1 = ld16(&rec->centre[ch + 4]);
            st.pos = *reinterpret_cast<const u32x2 *>(&rec->pos[ch]);
        }
    }
    const size_t blk = (size_t)bh * a.NB + u;
    if constexpr (KQ) {
        st.k0 = load_key_codes(a.lv, blk, tid);
        st.k1 = zero4();
    } else {
        const uint16_t *rows = reinterpret_cast<const uint16_t *>(a.lv.kcode) + (size_t)bh * a.NB * kG * kD;
        st.k0 = load_row_piece(rows, 0, 32 * u, T, tid);
        st.k1 = load_row_piece(rows, 0, 32 * u, T, tid + 256);
    }
    if constexpr (VQ) {
        st.v0 = load_value_codes(a.lv, blk, tid);
        st.v1 = zero4();
    } else {
        const uint16_t *rows = reinterpret_cast<const uint16_t *>(a.lv.vcode) + (size_t)bh * a.NB * kG * kD;
        st.v0 = load_value_row_piece(rows, 0, 32 * u, T, tid);
        st.v1 = load_value_row_piece(rows, 0, 32 * u, T, tid + 256);
    }
    if constexpr (KQ || VQ) st.m = load_meta_piece(a.lv, blk, tid >> 6, tid & 63, KQ, VQ);
    else st.m = zero4();
}

template <bool KQ, bool VQ, int SHIFT>
__device__ __forceinline__ void store_packed(const PrefillArgs &a, int tid, const Stage &st, Tiles &L, MetaSlab &M, bool compact)
{
    if constexpr (KQ || VQ) {
        wave_lds_sync();                                   // the slab's readers of the unit before are done
        store_meta_piece(M, tid & 63, st.m);
        wave_lds_sync();
    }
    if constexpr (KQ) {
        if (a.lv.kpt) {
            if (a.lv.kbits == 8) store_key_codes<8, true>(a.lv, L, M, tid, st, a.scale_log2e, compact);
            else if (a.lv.kbits == 4) store_key_codes<4, true>(a.lv, L, M, tid, st, a.scale_log2e, compact);
            else store_key_codes<2, true>(a.lv, L, M, tid, st, a.scale_log2e, compact);
        } else {
            if (a.lv.kbits == 8) store_key_codes<8, false>(a.lv, L, M, tid, st, a.scale_log2e, compact);
            else if (a.lv.kbits == 4) store_key_codes<4, false>(a.lv, L, M, tid, st, a.scale_log2e, compact);
            else store_key_codes<2, false>(a.lv, L, M, tid, st, a.scale_log2e, compact);
        }
    } else {
        store_key_rows(L, tid, st.k0, st.k1);
    }
    if constexpr (VQ) {
        if (a.lv.vbits == 8) store_value_codes<8, SHIFT>(a.lv, L, M, tid, st.v0);
        else if (a.lv.vbits == 4) store_value_codes<4, SHIFT>(a.lv, L, M, tid, st.v0);
        else store_value_codes<2, SHIFT>(a.lv, L, M, tid, st.v0);
    } else {
        store_value_piece<SHIFT>(L, tid, st.v0, 0, 32);
        store_value_piece<SHIFT>(L, tid + 256, st.v1, 0, 32);
    }
}

// ---- one chunk of the fp16 window, ring -> LDS tiles (at most two chunks per work-group: staged without overlap)
template <int SHIFT>
__device__ __forceinline__ void stage_window(const PrefillArgs &a, int bh, int u, int T, int tid, Tiles &L)
{
    const uint16_t *krows = a.lv.kres + (size_t)bh * a.RC * kD, *vrows = a.lv.vres + (size_t)bh * a.RC * kD;
    const u32x4 k0 = load_row_piece(krows, a.RC, 32 * u, T, tid), k1 = load_row_piece(krows, a.RC, 32 * u, T, tid + 256);
    const u32x4 v0 = load_value_row_piece(vrows, a.RC, 32 * u, T, tid), v1 = load_value_row_piece(vrows, a.RC, 32 * u, T, tid + 256);
    store_key_rows(L, tid, live_piece(k0, 32 * u, T, tid), live_piece(k1, 32 * u, T, tid + 256));
    store_value_piece<SHIFT>(L, tid, v0, 32 * u, T);
    store_value_piece<SHIFT>(L, tid + 256, v1, 32 * u, T);
}

__device__ __forceinline__ float xor_lanes(float x, int mask) { return __shfl_xor(x, mask, 64); }

// ---- the three phases of one unit (32 tokens, in X) against the 32 queries of a wave

// S^T = K^ Q^T: rows = tokens 16 tt + 4 rq + r, column = query n of tile qt.  KLO: quantized keys, whose fp16 rounding
// remainders are multiplied as well.
// the A operand of the output product for channel tile ct: V^T rows 16 ct + n, tokens {4 rq .. + 3, 16 + 4 rq .. + 3}
template <int SHIFT>
__device__ __forceinline__ half8 value_operand(const Tiles &X, int ct, int n, int rq)
{
    return *reinterpret_cast<const half8 *>(&X.Vt[16 * ct + n][8 * rotated_piece(n, rq, SHIFT)]);            // (16 ct: whole turns)
}

struct NoSlice { __device__ __forceinline__ void operator()(int) const {} };

// batches of score products per unit: four for the keys' 128 channels, then those of the low parts
template <int LO> constexpr int score_batches() { return LO == kLoAll ? 8 : LO == kLoCompact ? 5 : 4; }

// LO: how the low parts of quantized keys come (none: fp16 rows; all channels: Tiles::Klo; compact: the tile of the 32
// selected channels, against Qlo = the queries' values at those channels).
template <int LO, int SHIFT, class Slice = NoSlice>
__device__ __forceinline__ void score_unit(const Tiles &X, const half8 (&Qf)[kQT][4], const half8 (&Qlo)[kQT], float4v (&S)[2][kQT],
                                           int n, int rq, const float4v (&init)[kQT], const Tiles *Xv = nullptr, half8 *Av = nullptr,
                                           Slice slice = Slice())
{
    constexpr bool KLO = LO != kLoNone;
    // KLO: the keys carry the softmax constant (see prefill_dequantize) and the accumulators start from init[qt] = minus
    // the query's reference maximum, four times: the products come out in the exponent's units, relative to the
    // reference, and the common case of the softmax has neither a multiplication nor a subtraction left to do.
    // Otherwise (fp16 rows: window chunks, 16-bit keys) they start from zero and the scores are raw.
    // Operands come from LDS one batch (two rows x 8 channels per lane = 8 registers) at a time, two batches ahead of the
    // products that use them; a compiler barrier per batch keeps the order (left alone, the compiler either fetches all
    // 64 registers of a unit up front or waits for every batch right after asking for it).  With Xv: the value
    // operands of the output product that follows (unit Xv) are asked for during the last batches, so that they are
    // there when the softmax is done.
    // slice(bt): vector work of another unit (a share of its softmax) that is to be issued between the products of batch
    // bt and those of the next; with one, nothing is moved across the end of a batch (left alone, the compiler puts all
    // of it behind the last products, where the matrix cores then idle).
    constexpr int kBatches = score_batches<LO>();
    auto fetch = [&](int bt, half8 &A0, half8 &A1) {
        const int step = bt & 3;
        if (LO == kLoCompact && bt >= 4) {
            const _Float16 *lo = &X.Klo[0][0];
            A0 = *reinterpret_cast<const half8 *>(lo + n * kLoStride + 8 * rotated_piece(n, rq));
            A1 = *reinterpret_cast<const half8 *>(lo + (16 + n) * kLoStride + 8 * rotated_piece(n, rq));
        } else if (KLO && bt >= 4) {
            A0 = *reinterpret_cast<const half8 *>(&X.Klo[n][32 * step + 8 * rq]);
            A1 = *reinterpret_cast<const half8 *>(&X.Klo[16 + n][32 * step + 8 * rq]);
        } else {
            A0 = *reinterpret_cast<const half8 *>(&X.K[n][32 * step + 8 * rq]);
            A1 = *reinterpret_cast<const half8 *>(&X.K[16 + n][32 * step + 8 * rq]);
        }
    };
    half8 A0[kBatches], A1[kBatches];
    constexpr int kAhead = 2;                                   // batches in flight (2..4 measured alike)
#pragma unroll
    for (int bt = 0; bt < kAhead && bt < kBatches; bt++) fetch(bt, A0[bt], A1[bt]);
    constexpr int kVFirst = kBatches - 2;                       // the value operands ride with the last two batches
#pragma unroll
    for (int bt = 0; bt < kBatches; bt++) {
        if (bt + kAhead < kBatches) fetch(bt + kAhead, A0[bt + kAhead], A1[bt + kAhead]);
        if (Xv && bt >= kVFirst && bt < kVFirst + 2) {
#pragma unroll
            for (int k = 0; k < 4; k++) Av[4 * (bt - kVFirst) + k] = value_operand<SHIFT>(*Xv, 4 * (bt - kVFirst) + k, n, rq);
        }
        asm volatile("" ::: "memory");
        const int step = bt & 3;
#pragma unroll
        for (int qt = 0; qt < kQT; qt++) {
            const float4v start = KLO ? init[qt] : float4v{0.0f, 0.0f, 0.0f, 0.0f};
            const half8 B = LO == kLoCompact && bt >= 4 ? Qlo[qt] : Qf[qt][step];
            S[0][qt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A0[bt], B, bt == 0 ? start : S[0][qt], 0, 0, 0);
            S[1][qt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A1[bt], B, bt == 0 ? start : S[1][qt], 0, 0, 0);
        }
        if constexpr (!std::is_same<Slice, NoSlice>::value) {
            slice(bt);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// acc + the sum of the eight weights as they enter the output product (rounded to fp16), in fp32: four two-element dot
// products.  The denominator then matches the numerators exactly.
__device__ __forceinline__ float add_weights(float acc, half8 P)
{
    typedef _Float16 half2 __attribute__((ext_vector_type(2)));
    const half2 ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
    for (int k = 0; k < 4; k++) acc = __builtin_amdgcn_fdot2(half2{P[2 * k], P[2 * k + 1]}, ones, acc, false);
    return acc;
}

// The reference m of a query (in the exponent's units: score * log2(e) / sqrt(D)) only has to keep the weights in range,
// it need not be the exact maximum: as long as no score exceeds it by more than kCalm, it stays (no rescaling, weights
// <= 2^kCalm: fp16 holds them, the accumulators are fp32).
constexpr float kCalm = 8.0f;

// Online softmax in base 2 of the unit's scores, exact form: weights P (fp16, already in the operand order of the output
// product), reference m, partial sums lsum, and the factors alpha by which the accumulators shrink.  Returns whether
// some reference moved (in any lane).
// PRE: the scores are in the exponent's units and relative to base[qt] (score_unit with KLO); otherwise raw: the
// exponent is score * c + base[qt].
// MASK: the unit reaches beyond some query's position.
template <bool MASK, bool PRE>
__device__ __forceinline__ bool softmax_unit(const float4v (&S)[2][kQT], float c, int u, const int (&qpos)[kQT], const float (&base)[kQT],
                                             float (&m)[kQT], float (&lsum)[kQT], half8 (&P)[kQT], float (&alpha)[kQT], int rq)
{
    bool moved = false;
#pragma unroll
    for (int qt = 0; qt < kQT; qt++) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; e++) x[e] = S[e >> 2][qt][e & 3];
        if constexpr (MASK) {
#pragma unroll
            for (int e = 0; e < 8; e++)
                if (32 * u + 16 * (e >> 2) + 4 * rq + (e & 3) > qpos[qt]) x[e] = -INFINITY;
        }
        float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
        mx = fmaxf(mx, xor_lanes(mx, 16));
        mx = fmaxf(mx, xor_lanes(mx, 32));
        // a tile's first unit holds token 0, and a piece starts with a unit that lies before all of its tile's queries:
        // every query sees a token of it, so the reference is finite from the start
        const float top = PRE ? mx + base[qt] : fmaf(mx, c, base[qt]);
        const float mn = top > m[qt] + kCalm ? top : m[qt];              // m = -inf at the start: moves
        moved |= mn != m[qt];
        alpha[qt] = __builtin_amdgcn_exp2f(m[qt] - mn);
        m[qt] = mn;
        const float shift = base[qt] - mn;
#pragma unroll
        for (int e = 0; e < 8; e++) x[e] = __builtin_amdgcn_exp2f(PRE ? x[e] + shift : fmaf(x[e], c, shift));
        P[qt] = half8{(_Float16)x[0], (_Float16)x[1], (_Float16)x[2], (_Float16)x[3],
                      (_Float16)x[4], (_Float16)x[5], (_Float16)x[6], (_Float16)x[7]};
        lsum[qt] = add_weights(lsum[qt] * alpha[qt], P[qt]);
    }
    return __any(moved);
}

// true if some score of the unit (no mask) exceeds its query's reference by more than kCalm, in any lane of the wave.
// PRE: the scores are relative to the reference already; otherwise raw (compared against (m + kCalm) / c).
template <bool PRE>
__device__ __forceinline__ bool unit_exceeds(const float4v (&S)[2][kQT], float inv_c, const float (&m)[kQT])
{
    bool over = false;
#pragma unroll
    for (int qt = 0; qt < kQT; qt++) {
        const float4v a = S[0][qt], b = S[1][qt];
        float mx = fmaxf(fmaxf(a[0], a[1]), a[2]);          // chains of three-operand maxima
        mx = fmaxf(fmaxf(mx, a[3]), b[0]);
        mx = fmaxf(fmaxf(mx, b[1]), b[2]);
        mx = fmaxf(mx, b[3]);
        over |= PRE ? mx > kCalm : mx > (m[qt] + kCalm) * inv_c;
    }
    return __any(over);
}

// Softmax weights of a unit against the unchanged reference (no mask), dealt out in kBatches shares so that a share
// can be issued between two batches of another unit's score products.  PRE: the scores are the exponents themselves.
template <bool PRE, int SHARES, class Fetch>
struct CalmSoftmax {
    const float4v (&S)[2][kQT];
    float c;
    const float (&m)[kQT];
    float (&lsum)[kQT];
    half8 (&P)[kQT];
    const Fetch &fetch;                                         // fetch(i): the wave's i-th load of a unit to come, of Fetch::kSlots
    static constexpr int kShares = SHARES;                      // = the batches of the score products it rides with
    __device__ __forceinline__ void operator()(int share) const
    {
        typedef _Float16 half2 __attribute__((ext_vector_type(2)));
        const half2 ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
        for (int i = Fetch::kSlots * share / kShares; i < Fetch::kSlots * (share + 1) / kShares; i++) fetch(i);
#pragma unroll
        for (int pair = 8 * share / kShares; pair < 8 * (share + 1) / kShares; pair++) {
            const int qt = pair >> 2, e = 2 * (pair & 3);                                       // elements e, e + 1 of query tile qt
            const float s0 = S[e >> 2][qt][e & 3], s1 = S[e >> 2][qt][(e & 3) + 1];
            const float x0 = __builtin_amdgcn_exp2f(PRE ? s0 : fmaf(s0, c, -m[qt]));
            const float x1 = __builtin_amdgcn_exp2f(PRE ? s1 : fmaf(s1, c, -m[qt]));
            const half2 h = {(_Float16)x0, (_Float16)x1};
            P[qt][e] = h[0];
            P[qt][e + 1] = h[1];
            // the denominator is summed from the rounded weights, as they enter the output product
            lsum[qt] = __builtin_amdgcn_fdot2(h, ones, lsum[qt], false);
        }
    }
};

// O^T += V^T P^T: rows = channels 16 ct + 4 rq + r; both operands list the tokens as
// {4 rq .. 4 rq + 3, 16 + 4 rq .. 16 + 4 rq + 3}.
__device__ __forceinline__ void output_add(const half8 (&Av)[8], const half8 (&P)[kQT], float4v (&O)[8][kQT])
{
#pragma unroll
    for (int ct = 0; ct < 8; ct++)
#pragma unroll
        for (int qt = 0; qt < kQT; qt++) O[ct][qt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Av[ct], P[qt], O[ct][qt], 0, 0, 0);
}

// O^T *= alpha per query, before the unit's product is added (on the exact path only, which is the rare one).
__device__ __forceinline__ void output_rescale(const float (&alpha)[kQT], float4v (&O)[8][kQT])
{
#pragma unroll
    for (int qt = 0; qt < kQT; qt++)
#pragma unroll
        for (int ct = 0; ct < 8; ct++) O[ct][qt] *= alpha[qt];
}

// ---- pass 0 (per-channel quantized keys only): which channels of each cache keep the low parts of their keys.
// A key rounded once to fp16 is off by up to 2^-11 of itself, and the logit by the sum over the channels of that times
// the query's entry.  Per channel d this kernel estimates the centre of the dequantized keys (the mean of the blocks'
// midpoints, rounded to fp16) and w_d = (mean square of the keys about that centre) x (mean square of the queries):
// the keys' from the block metadata alone (a block's values of a channel lie in [z, z + s (2^bits - 1)],
// taken as spread evenly), the queries' from up to 64 positions of every query head of the group.  The 32 channels of
// largest w_d keep their low parts; if the w_d of all others add up to less than kSelectBudget, i.e. one fp16 rounding
// of those channels moves a logit by less than 2^-11 / sqrt(3) * log2(e) / sqrt(D) * sqrt(kSelectBudget) = 6e-4 (root
// mean square, in the exponent's units: below the 2^-11 by which the fp16 softmax weights are rounded anyway), the
// cache takes the compact form; otherwise every channel keeps its low part.  Keys whose large channels are few
// (the case the per-channel grouping is made for, Section 3.2) qualify, and so do keys with a large offset on every
// channel (the offsets are centred away); keys that are large and widely spread on many channels do not.
constexpr float kSelectBudget = 300.0f;
// One work-group per cache, or several (below).  Bound by the latency of its loads: a wave takes a block's metadata (a query's row) at a time,
// lane = two neighbouring channels, 16 query rows and kSelectAhead blocks outstanding.  Four blocks per wave (64 per work-group) do: with 16,
// whose code is twice as long and read from memory by every launch, and with the blocks asked for in front of the queries, a launch took 7.8 instead
// of 7.2 us at 2027 tokens, 9.3 instead of 8.6 at 8275 (113 queries, which then waited for the blocks); a call of 4 layers of 2290 tokens
// 181.7 -> 176.3 us, of 2027 350.8 -> 343.8.
constexpr int kSelectWaves = 16;
constexpr int kSelectAhead = 4;
// Long caches: up to kSelectParts work-groups share a cache's blocks; each leaves its sums in the scratch area (prefill_dequantize
// comes later), written through to memory, and counts itself; the last one adds them up, in their order, and does the rest.
constexpr int kSelectParts = 8;
constexpr int kSelectWhole = 256;        // units of a cache that one work-group takes

__device__ __forceinline__ void store_through(float *p, float v) { asm volatile("global_store_dword %0, %1, off sc0 sc1" ::"v"(p), "v"(v) : "memory"); }

template <bool NARROW>
__global__ __launch_bounds__(64 * kSelectWaves) void prefill_select(PrefillArgs a, int parts)
{
    const int tid = threadIdx.x, lane = tid & 63, local = blockIdx.y, bh = a.bh0 + local;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: so are the addresses of a wave's rows
    asm volatile("" ::"s"(a.lv.kmeta), "s"(a.n_blocks), "s"(a.n_res), "s"(parts));      // the argument record's lines are asked for at once
    __shared__ __attribute__((aligned(16))) float k1[kSelectWaves][kD], k2[kSelectWaves][kD], q2[kSelectWaves][kD], w[kD];
    __shared__ int above[8][kD];
    __shared__ float rest[2];
    const float top = (float)((1 << a.lv.kbits) - 1);
    const int gq = a.Hq / a.Hkv, stride = (a.n_q + 63) / 64;
    const int head0 = (bh / a.Hkv) * a.Hq + (bh % a.Hkv) * gq;
    const int per_head = (a.n_q + stride - 1) / stride, samples = gq * per_head;
    float sq[2] = {0.0f, 0.0f}, sk[2] = {0.0f, 0.0f}, sm[2] = {0.0f, 0.0f};
    // Queries of four heads, four samples of each per wave: at most 64 samples per head (numbering the samples of all heads through instead
    // costs a division per load: 10.6 instead of 8.6 us a launch).
    static_assert(4 * kSelectWaves == 64, "four samples of a head per wave");
    uint32_t x[4][4];
    auto ask = [&](int j0) {
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int jc = j0 + j < gq ? j0 + j : gq - 1, i = wave + kSelectWaves * k < per_head ? wave + kSelectWaves * k : 0;
                x[j][k] = *reinterpret_cast<const uint32_t *>(a.q + ((size_t)(head0 + jc) * a.n_q + (size_t)i * stride) * kD + 2 * lane);
            }
    };
    auto take = [&](int j0) {
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (j0 + j < gq && wave + kSelectWaves * k < per_head) {
                    const float v0 = half_bits(x[j][k] & 0xffffu), v1 = half_bits(x[j][k] >> 16);
                    sq[0] = fmaf(v0, v0, sq[0]);
                    sq[1] = fmaf(v1, v1, sq[1]);
                }
    };
    const int across = kSelectWaves * parts, first = blockIdx.x * kSelectWaves + wave;      // waves of the cache, this one's number
    u32x2 sc[kSelectAhead];                                      // (fp16 scales: one word, the other one is not used)
    uint32_t zp[kSelectAhead];
    auto fetch = [&](int u0) {                                   // (past the end: block 0)
#pragma unroll
        for (int k = 0; k < kSelectAhead; k++) {
            const int u = u0 + across * k < a.n_blocks ? u0 + across * k : 0;
            const float *meta = a.lv.kmeta + ((size_t)bh * a.NB + u) * meta_words(NARROW);
            if constexpr (NARROW) sc[k][0] = *reinterpret_cast<const uint32_t *>(meta_scales16(meta) + 2 * lane);
            else sc[k] = *reinterpret_cast<const u32x2 *>(meta + 2 * lane);
            zp[k] = *reinterpret_cast<const uint32_t *>(meta_zeros(meta, NARROW) + 2 * lane);
        }
    };
    // The first part takes the queries.  Their loads go out first and those of the first blocks right behind, so that both share a round trip
    // and the queries are waited for without the blocks.
    if (blockIdx.x == 0) ask(0);
    fetch(first);
    if (blockIdx.x == 0) {
        take(0);
        for (int j0 = 4; j0 < gq; j0 += 4) {
            ask(j0);
            take(j0);
        }
    }
    for (int u0 = first; u0 < a.n_blocks; u0 += kSelectAhead * across) {
        if (u0 != first) fetch(u0);
#pragma unroll
        for (int k = 0; k < kSelectAhead; k++) {
            if (u0 + across * k < a.n_blocks) {
                const uint32_t s0 = sc[k][0], s1 = sc[k][1];
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    const float s = NARROW ? half_bits(e ? s0 >> 16 : s0 & 0xffffu) : __builtin_bit_cast(float, e ? s1 : s0);
                    const float lo = half_bits(e ? zp[k] >> 16 : zp[k] & 0xffffu), hi = fmaf(s, top, lo);
                    sk[e] += (lo * lo + lo * hi + hi * hi) * (1.0f / 3.0f);      // mean of x^2 over [lo, hi]
                    sm[e] += 0.5f * (lo + hi);
                }
            }
        }
    }
    *reinterpret_cast<float2 *>(&k1[wave][2 * lane]) = make_float2(sm[0], sm[1]);
    *reinterpret_cast<float2 *>(&k2[wave][2 * lane]) = make_float2(sk[0], sk[1]);
    *reinterpret_cast<float2 *>(&q2[wave][2 * lane]) = make_float2(sq[0], sq[1]);
    __syncthreads();
    Select *sel = reinterpret_cast<Select *>(a.select) + local;
    const int d = tid & (kD - 1), slice = tid >> 7;              // 8 slices of 16 channels for the ranks
    float tm = 0.0f, tk = 0.0f, tq = 0.0f;
    if (tid < kD) {
#pragma unroll
        for (int k = 0; k < kSelectWaves; k++) { tm += k1[k][d]; tk += k2[k][d]; tq += q2[k][d]; }
    }
    if (parts > 1) {
        static_assert(8 * kD == 64 * kSelectWaves && kSelectParts == 8, "a slice of threads per part");
        float *sums = reinterpret_cast<float *>(a.scratch) + (size_t)local * parts * 3 * kD;
        if (tid < kD) {
            float *mine = sums + (size_t)blockIdx.x * 3 * kD + d;
            store_through(mine, tm);
            store_through(mine + kD, tk);
            store_through(mine + 2 * kD, tq);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t *t = &sel->tickets[kMaxTickets - 1];
            const bool last = (int)__hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
            if (last) __hip_atomic_store(t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            above[0][0] = last ? 1 : 0;
        }
        __syncthreads();
        if (above[0][0] == 0) return;
        const __amdgpu_buffer_rsrc_t all = __builtin_amdgcn_make_buffer_rsrc(sums, 0, parts * 3 * kD * (int)sizeof(float), 0x00020000);
        if (slice < parts) {                                     // (read past the caches, as they were written)
            const int off = (slice * 3 * kD + d) * (int)sizeof(float), row = kD * (int)sizeof(float);
            const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(all, off, 0, 17), y = __builtin_amdgcn_raw_buffer_load_b32(all, off + row, 0, 17),
                           z = __builtin_amdgcn_raw_buffer_load_b32(all, off + 2 * row, 0, 17);
            k1[slice][d] = __builtin_bit_cast(float, x);
            k2[slice][d] = __builtin_bit_cast(float, y);
            q2[slice][d] = __builtin_bit_cast(float, z);
        }
        __syncthreads();
        if (tid < kD) {
            tm = tk = tq = 0.0f;
            for (int k = 0; k < parts; k++) { tm += k1[k][d]; tk += k2[k][d]; tq += q2[k][d]; }
        }
    }
    if (tid < kD) {
        // the channel's centre: the mean of its blocks' midpoints, as an fp16 number (the zero-points are fp16 numbers, so
        // zero-point minus centre is exact in fp32).  What counts from here on is the keys' spread about it.
        const float centre = (float)(_Float16)(tm / (float)a.n_blocks);
        const float centre_ok = fabsf(centre) < 65504.0f ? centre : 0.0f;
        sel->centre[d] = centre_ok;
        const float spread = fmaxf(tk / (float)a.n_blocks - centre_ok * (2.0f * tm / (float)a.n_blocks - centre_ok), 0.0f);
        w[d] = spread * (tq / (float)samples);
    }
    __syncthreads();
    const float mine = w[d];
    int over = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const float4 o4 = *reinterpret_cast<const float4 *>(&w[16 * slice + 4 * k]);
        const float o[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
        for (int e = 0; e < 4; e++) over += (o[e] > mine || (o[e] == mine && 16 * slice + 4 * k + e < d)) ? 1 : 0;
    }
    above[slice][d] = over;
    __syncthreads();
    if (tid < kD) {
        int rank = 0;
#pragma unroll
        for (int k = 0; k < 8; k++) rank += above[k][d];
        sel->pos[d] = rank < 32 ? (uint8_t)rank : (uint8_t)255;
        if (rank < 32) sel->chan[rank] = (uint8_t)d;
        float r = rank < 32 && mine == mine ? 0.0f : mine;       // (not a number: stays one, and the sum below with it)
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) r += xor_lanes(r, m);
        if (lane == 0) rest[wave] = r;
    }
    __syncthreads();
    if (tid == 0) sel->compact = rest[0] + rest[1] < kSelectBudget ? 1u : 0u;    // (a sum that is not a number compares false: all channels)
}

// ---- pass 1: every packed unit of the (batch, kv head) caches [bh0, bh0 + n_bh) is dequantized once into the scratch
// area, in the very layout the attention kernel keeps a unit in LDS (struct Tiles), so that pass 2 fetches plain copies.
// KQ / VQ: the layer's keys / values are quantized (else fp16 rows in the code area).
//
// The unit is put together in LDS and goes out as whole KiB, 16 bytes per lane at consecutive addresses: bound by the writes
// (26 KiB per unit, 19 in the compact form; its code and metadata reads are a tenth of that).  Stored to the scratch area
// straight from the registers that hold the values (64-byte pieces of rows, 8-byte pieces of the transposed values, 2-byte
// low parts, row padding left out) the lines were written in parts.  Measured (K4V2, compact): 16 caches of 255 units
// 40 -> 31.5 us, 8 caches of 767 units 60 -> 45 us; with 2 KiB of low parts and the selection record asked for early 28.5 and 37.5 us.
constexpr int kTileKiB = 9, kValuesKiB = 8;
static_assert(sizeof(_Float16) * 32 * kKStride == kTileKiB * 1024 && sizeof(_Float16) * kD * 32 == kValuesKiB * 1024 &&
              sizeof(Tiles) == (2 * kTileKiB + kValuesKiB) * 1024, "tiles of a unit are whole KiB");

// SHIFT: the value rows' rotation that the attention kernel behind it reads (value_shift).
template <bool KQ, bool VQ, int SHIFT>
__device__ __forceinline__ void dequantize_unit(const PrefillArgs &a)
{
    const int tid = threadIdx.x, u = blockIdx.x, local = blockIdx.y;
    // The argument record's lines are asked for at once (RC: read along with NB, and its register is free for the next load only then).
    // Short caches, us a launch, one line behind the other / at once: 48 work-groups 4.44 / 4.29, 80 work-groups 5.56 / 5.38.
    asm volatile("" ::"s"(a.lv.kcode), "s"(a.lv.kbits), "s"(a.n_blocks), "s"(a.NB), "s"(a.RC), "s"(a.bh0), "s"(a.scratch));
    const int T = 32 * a.n_blocks + a.n_res;
    __shared__ __attribute__((aligned(16))) MetaSlab M[kStagers];
    __shared__ __attribute__((aligned(16))) Tiles tile;
    Stage st;
    // The selection record's share is asked for with the unit's codes: field by field where it is needed, it cost three more round trips.
    const Select *rec = KQ && a.select ? reinterpret_cast<const Select *>(a.select) + local : nullptr;
    load_packed<KQ, VQ>(a, a.bh0 + local, u, T, tid, rec, st);
    const bool compact = KQ && __builtin_amdgcn_readfirstlane((int)st.compact) != 0;
    store_packed<KQ, VQ, SHIFT>(a, tid, st, tile, M[tid >> 6], compact);
    __syncthreads();
    const int lo_pieces = !KQ ? 0 : compact ? kLoPieces : kTileKiB;
    uint8_t *dst = a.scratch + ((size_t)local * a.n_blocks + u) * sizeof(Tiles);
    const uint8_t *src = reinterpret_cast<const uint8_t *>(&tile);
    for (int p = tid >> 6; p < kTileKiB + lo_pieces + kValuesKiB; p += kStagers) {
        const int off = 1024 * (p < kTileKiB + lo_pieces ? p : p - lo_pieces + kTileKiB) + 16 * (tid & 63);      // K^, low parts, then V^
        *reinterpret_cast<u32x4 *>(dst + off) = *reinterpret_cast<const u32x4 *>(src + off);
    }
}

template <bool KQ, bool VQ>
__global__ __launch_bounds__(64 * kStagers) void prefill_dequantize(PrefillArgs a) { dequantize_unit<KQ, VQ, value_shift(KQ, 8)>(a); }

// the same in front of half_keys_of_4
template <bool VQ>
__global__ __launch_bounds__(64 * kStagers) void units_of_half_keys(PrefillArgs a) { dequantize_unit<false, VQ, value_shift(false, 4)>(a); }

// A unit goes from the scratch area into an LDS buffer without passing through registers: a wave issues
// global-to-LDS loads of 1 KiB each (64 lanes x 16 bytes, which land at consecutive LDS addresses from the base
// that M0 holds).  The tiles of a unit are whole KiB, so a piece never straddles two of them.

__device__ __forceinline__ void fetch_piece(const uint8_t *piece, uint32_t lane_offset, uint32_t lds_base)
{
    // The compiler does not see this load: the waits for it are written out below (wait_fetches).  Loads it does not
    // know of can only make its own waits longer, never too short.  M0 is declared as clobbered, so a use of its own the compiler
    // might make of M0 (it sets M0 right before an instruction that reads it) stays correct.
    // Address = a wave-uniform one (scalar registers) + a 32-bit offset per lane that is the same for every unit.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(lane_offset), "s"(piece) : "memory", "m0");
}

// Pieces of a unit that come with the keys' low parts: none, the whole tile, or the first kLoPieces KiB of it (the compact tile).
template <int LO> constexpr int low_pieces() { return LO == kLoAll ? kTileKiB : LO == kLoCompact ? kLoPieces : 0; }
template <int LO> constexpr int unit_pieces() { return kTileKiB + low_pieces<LO>() + kValuesKiB; }
// loads per wave and unit, at most
template <int LO, int WAVES> constexpr int fetch_slots() { return (unit_pieces<LO>() + WAVES - 1) / WAVES; }

// The i-th of them: wave `wave` of WAVES fetches the pieces wave, wave + WAVES, ... of a unit.
template <int LO, int WAVES>
__device__ __forceinline__ void fetch_slot(const uint8_t *unit, Tiles &L, int wave, int lane, int i)
{
    const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)reinterpret_cast<uint8_t *>(&L);
    const int p = wave + WAVES * i;                               // the same for all lanes of the wave
    if (p < unit_pieces<LO>()) {
        const int off = 1024 * (p < kTileKiB + low_pieces<LO>() ? p : p - low_pieces<LO>() + kTileKiB);     // K^, low parts, then V^
        // (eight waves have registers for a lane offset per piece, four add the piece's to the scalar address)
        if constexpr (WAVES == 8) fetch_piece(unit, (uint32_t)(off + 16 * lane), lds + off);
        else fetch_piece(unit + off, (uint32_t)(16 * lane), lds + off);
    }
}

template <int LO, int WAVES>
__device__ __forceinline__ void fetch_unit(const uint8_t *unit, Tiles &L, int wave, int lane)
{
#pragma unroll
    for (int i = 0; i < fetch_slots<LO, WAVES>(); i++) fetch_slot<LO, WAVES>(unit, L, wave, lane, i);
}

// what a step fetches on its way, or nothing
struct NoFetch {
    static constexpr int kSlots = 0;
    __device__ __forceinline__ void operator()(int) const {}
};
template <int LO, int WAVES>
struct UnitFetch {
    const uint8_t *unit;
    Tiles &to;
    int wave, lane;
    bool real;
    static constexpr int kSlots = fetch_slots<LO, WAVES>();
    __device__ __forceinline__ void operator()(int i) const { if (real) fetch_slot<LO, WAVES>(unit, to, wave, lane, i); }
};

// Returns once all fetches of this wave have landed in LDS.
__device__ __forceinline__ void wait_fetches() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Order in which an XCD's work-groups of whole tiles start: cache by cache, the longest of each first; all of them by length; those that
// find a compute unit for themselves by length, then the shortest of the others first (two per compute unit: long and short together).
enum { kByCache, kByLength, kPaired };

// Which queries the rows of a work-group are: row r is query r / heads of head r % heads of a group of `heads` query heads.
struct Rows {
    int heads;                           // query heads that share a work-group's rows
    int groups;                          // of a cache's query heads
    uint32_t magic;                      // for divisions by heads
    int order;                           // in which the work-groups start
};

// r / heads, exactly: magic = ceil(2^32 / heads), and r * heads < 2^32 (plan_launch sees to it).  Divided by the compiler's
// sequence instead a window-only prompt of packed rows takes 0.5 us longer.
__device__ __forceinline__ int row_query(const Rows &rw, int r) { return rw.heads == 1 ? r : (int)__umulhi((uint32_t)r, rw.magic); }

// ---- pass 2: the attention itself.  A work-group has 8 waves and 256 rows or 4 waves and 128 (see plan_launch), a row being a query of
// one of Rows::heads query heads; every wave attends 32 rows and fetches its share of each unit from the scratch area into LDS.  KLO: the
// keys are quantized (they come as two fp16 numbers).
//
// 8 waves, alone on their compute unit: five LDS buffers and two units per trip: while units u and u + 1 are being used, unit u + 2 is already there and units
// u + 3 and u + 4 are on their way; one barrier per trip.  With the next unit present, a wave issues the score products
// of unit u + 1 in the same stretch of code as the softmax of unit u (matrix and vector instructions that do not depend
// on each other), instead of waiting for each product's result in turn.
// 4 waves, two such work-groups per compute unit: three buffers and one unit per trip; while one work-group waits for its unit, the
// other goes on.  (Their 256 registers leave none for the window's offsets, which are kept in LDS over the loop.)
__host__ __device__ constexpr int tile_buffers(int waves) { return waves == 8 ? 5 : 3; }
constexpr size_t attention_lds(int waves) { return tile_buffers(waves) * sizeof(Tiles) + (waves == 4 ? 64 * 4 * kQT * sizeof(float) : 0); }
static_assert(2 * attention_lds(4) <= 160 * 1024, "two work-groups of four waves per compute unit");

// What one work-group attends to: the rows from row0 on of the heads from `head` on, and of the `count` pieces that the packed units of
// their tile (256 rows) are cut into piece `index` (the fp16 window goes with the last one); slot: where the partial results of the
// tile's piece go (count > 1).
struct Piece { int tile, row0, head, index, count, slot; };

// How the tiles of a query head are cut into pieces (plan_pieces).  One word per tile, the tiles with the longest pieces
// first: tile | pieces << 8 | pieces in front of it << 16 (whole words: the kernel reads them through the scalar unit).
// pieces = 0: every tile is one piece.
constexpr int kMaxCutTiles = 128;
constexpr int kMaxPieces = 255;          // of a tile
struct PieceTable : Rows {
    int pieces;                          // of a query head
    int partials;                        // those of tiles with more than one piece: their results go through memory
    uint32_t entry[kMaxCutTiles];
};

// in place of the table where no tile can be cut
struct WholeTiles : Rows {};

__device__ __forceinline__ int piece_partials(uint32_t entry)
{
    const int count = (int)((entry >> 8) & 255u);
    return count > 1 ? count : 0;
}

// LO: how the low parts of the keys come (score_unit); rec: the cache's selection record or null (never null with
// kLoCompact); CUT: the tile may be cut (else pc.tile alone counts).
template <int LO, bool CUT, int WAVES, bool PACKED>
__device__ __forceinline__ void attend(const PrefillArgs &a, const Rows &rows_of, const Select *rec, int local, const Piece &pc)
{
    constexpr bool KLO = LO != kLoNone;
    constexpr int kShift = value_shift(KLO, WAVES);
    constexpr bool kRide = !half_keys_of_4(KLO, WAVES);          // a step's fetches go out between its products
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, rq = lane >> 4;
    const int gq = a.Hq / a.Hkv;
    const int bh = a.bh0 + local;
    const int head0 = (bh / a.Hkv) * a.Hq + (bh % a.Hkv) * gq + pc.head;  // b * Hq + first query head
    const int T = 32 * a.n_blocks + a.n_res;
    const int p0 = T - a.n_q;                                    // absolute position of query 0
    const int hp = PACKED ? rows_of.heads : 1, rows = a.n_q * hp;      // row r: query r / hp of head head0 + r % hp
    auto query_of = [&](int r) { return PACKED ? row_query(rows_of, r) : r; };
    // (The code that the compiler makes of the 8-wave loop depends on how the numbers in front of it are formed.  These forms give that of the kernel without
    // rows of several heads and 4-wave work-groups; with row0 and open_units as one expression for all: 16 x 8192 tokens 9.77 instead of 9.71 ms.)
    const int row0 = WAVES == 8 ? pc.tile * kQB : pc.row0;
    const int rlast = (row0 + kQW * WAVES < rows ? row0 + kQW * WAVES : rows) - 1;
    const int units = (p0 + query_of(rlast)) / 32 + 1;                // units the work-group walks through
    const int rw = row0 + kQW * wave;                            // first row of this wave
    const int wlast = rw < rows ? (p0 + query_of(rw + kQW - 1 < rows ? rw + kQW - 1 : rows - 1)) / 32 : -1;
    const int wmin = p0 + query_of(rw);
    const int open_units = rw < rows ? (wmin + 1) / 32 : 0;   // units [0, open_units) lie before the wave's first query: no mask needed
    const float c = a.scale_log2e;
    const float inv_c = 1.0f / c;

    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    Tiles *L = reinterpret_cast<Tiles *>(lds_raw);

    // rows of this lane: rw + 16 qt + n; past the end the last row is repeated and never stored
    int qpos[kQT];
    half8 Qf[kQT][4], Qlo[kQT];
#pragma unroll
    for (int qt = 0; qt < kQT; qt++) {
        const int r = rw + 16 * qt + n, rc = r < rows ? r : rows - 1, ic = query_of(rc);
        qpos[qt] = p0 + ic;
        const uint16_t *row = a.q + ((size_t)(head0 + rc - ic * hp) * a.n_q + ic) * kD;
#pragma unroll
        for (int step = 0; step < 4; step++) Qf[qt][step] = __builtin_nontemporal_load(reinterpret_cast<const half8 *>(row + 32 * step + 8 * rq));
        Qlo[qt] = half8{};
    }
    if constexpr (LO == kLoCompact) {
        // The queries' values at the channels of slots 8 rq .. 8 rq + 7: the operand that meets the compact tile.  Gathered from the wave's rows in LDS (16 at a
        // time, in buffers that no unit is fetched into before the loop): 2-byte gathers from memory, 64 addresses each, are served
        // line by line, and 16 of them per wave kept a compute unit's memory pipeline busy for microseconds before its first unit.  us a pass, before / after: a
        // 2027-token prompt, 4 layers 326 / 316, 4 x 8192 tokens 2414 / 2356, last 512 of 24576, 4 layers 1070 / 1059.
        constexpr int kRowHalves = kD + 8;
        static_assert(WAVES * 16 * kRowHalves * sizeof(_Float16) <= (WAVES == 8 ? 2 : 1) * sizeof(Tiles), "the rows fit the last buffers");
        _Float16 *rows16 = reinterpret_cast<_Float16 *>(&L[WAVES == 8 ? 3 : 2]) + wave * (16 * kRowHalves) + n * kRowHalves;
        const u32x2 cw = *reinterpret_cast<const u32x2 *>(&rec->chan[8 * rq]);
#pragma unroll
        for (int qt = 0; qt < kQT; qt++) {
            wave_lds_sync();
#pragma unroll
            for (int step = 0; step < 4; step++) *reinterpret_cast<half8 *>(rows16 + 32 * step + 8 * rq) = Qf[qt][step];
            wave_lds_sync();
#pragma unroll
            for (int e = 0; e < 8; e++) Qlo[qt][e] = rows16[((e < 4 ? cw[0] : cw[1]) >> (8 * (e & 3))) & 127u];
        }
    }

    // Packed keys come with their channel's centre taken off (prefill_dequantize), which lowers every packed score of a
    // query by q . centre; the scores of the window's fp16 rows are lowered by the same amount here, so that the softmax
    // sees all of a query's scores moved alike.  woff = minus that amount in the exponent's units.
    // (Four waves keep it in LDS over the loop, which leaves no registers for it.)
    float woff[kQT];
    float *kept = reinterpret_cast<float *>(lds_raw + tile_buffers(WAVES) * sizeof(Tiles)) + tid;
#pragma unroll
    for (int qt = 0; qt < kQT; qt++) woff[qt] = 0.0f;
    if constexpr (KLO) {
        if (rec) {
#pragma unroll
            for (int qt = 0; qt < kQT; qt++) {
                float dot = 0.0f;
#pragma unroll
                for (int step = 0; step < 4; step++) {
                    const float4 c0 = *reinterpret_cast<const float4 *>(&rec->centre[32 * step + 8 * rq]);
                    const float4 c1 = *reinterpret_cast<const float4 *>(&rec->centre[32 * step + 8 * rq + 4]);
                    const float cen[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
                    for (int e = 0; e < 8; e++) dot = fmaf((float)Qf[qt][step][e], cen[e], dot);
                }
                dot += xor_lanes(dot, 16);
                dot += xor_lanes(dot, 32);
                woff[qt] = -c * dot;
            }
        }
        if constexpr (WAVES == 4) {
#pragma unroll
            for (int qt = 0; qt < kQT; qt++) kept[64 * WAVES * qt] = woff[qt];
        }
    }

    float4v O[8][kQT];
    float m[kQT], lsum[kQT];
#pragma unroll
    for (int qt = 0; qt < kQT; qt++) {
        m[qt] = -INFINITY;
        lsum[qt] = 0.0f;
#pragma unroll
        for (int ct = 0; ct < 8; ct++) O[ct][qt] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // ---- packed units [ub, nb): the tile's, or a piece of them.  Unit u lives in buffer (u - ub) % 5.  Per trip: the wave issues its fetches of units u + 3 and
    // u + 4 (into the buffers of units u - 2 and u - 1, which everybody left at the last barrier), uses units u and u + 1
    // (taking the scores of the following unit ahead each time), then waits until its fetches have landed, and the
    // barrier makes everybody's visible.
    const int nbt = a.n_blocks < units ? a.n_blocks : units;     // the work-group's
    int ub = 0, nb = nbt;
    if constexpr (CUT) {
        int all = nbt;
        if constexpr (WAVES == 4) {
            // (the tile's rows may reach further than the work-group's: only its last piece ends earlier here)
            const int tlast = ((pc.tile + 1) * kQB < rows ? (pc.tile + 1) * kQB : rows) - 1, tunits = (p0 + query_of(tlast)) / 32 + 1;
            all = a.n_blocks < tunits ? a.n_blocks : tunits;
        }
        ub = all * pc.index / pc.count;
        nb = all * (pc.index + 1) / pc.count;
        if constexpr (WAVES == 4) nb = nb < nbt ? nb : nbt;
    }
    if (nb > ub) {
        const uint8_t *mine = a.scratch + (size_t)local * a.n_blocks * sizeof(Tiles);
        const int last = nb - 1;
        auto unit_at = [&](int u) { return mine + (size_t)(u < last ? u : last) * sizeof(Tiles); };
        auto fetch = [&](int u, Tiles &to) {
            // 4 waves wait for every unit: none is fetched past the end.  8 waves, whose loop is a little slower with the condition (0.3 %), fetch
            // the last one again, into a buffer nobody reads.
            if (WAVES == 8 || u < nb) fetch_unit<LO, WAVES>(unit_at(u), to, wave, lane);
        };
        fetch(ub, L[0]);
        fetch(ub + 1, L[1]);
        if constexpr (WAVES == 8) fetch(ub + 2, L[2]);
        // The queries are first used under a condition; without this the compiler would keep their loads on its list
        // of pending ones inside the loop and wait there for everything in flight, the fetches just issued included.
#pragma unroll
        for (int qt = 0; qt < kQT; qt++)
#pragma unroll
            for (int step = 0; step < 4; step++) asm volatile("" ::"v"(Qf[qt][step]));
        if constexpr (LO == kLoCompact) {
#pragma unroll
            for (int qt = 0; qt < kQT; qt++) asm volatile("" ::"v"(Qlo[qt]));
        }
        wait_fetches();                                         // the first units are there
        __syncthreads();
        float4v S[2][kQT], Sn[2][kQT];
        // base[qt]: what the scores waiting in S / Sn are relative to (KLO only: the reference as it stood when their
        // products were issued, zero while it is still -inf); init = minus that, as the products' starting value
        float base[kQT];
        float4v init[kQT];
        auto set_base = [&]() {
#pragma unroll
            for (int qt = 0; qt < kQT; qt++) {
                base[qt] = KLO && m[qt] > -INFINITY ? m[qt] : 0.0f;
                init[qt] = float4v{-base[qt], -base[qt], -base[qt], -base[qt]};
            }
        };
        set_base();
        if (ub <= wlast) score_unit<LO, kShift>(L[0], Qf, Qlo, S, n, rq, init);
        // one unit: its scores come in Sin, those of the next unit leave in Sout (the two arrays swap roles from unit to
        // unit).  Whether a unit may take the calm form is decided one unit ahead, right after its scores were issued:
        // the test then sits next to the output products of the unit before, which need nothing from it.
        bool calm = false;                                       // the first unit never is: the references start at -inf
        // The wave's loads of unit uf go out on the way (into Xf, which everybody left at the last barrier), one or two behind each batch of products: issued
        // all at once behind the barrier, by all waves, they wait for each other (80 to 100 cycles each, 200..245 a unit and wave) while the matrix cores idle.
        // (Half-precision keys in 4 waves: see half_keys_of_4.)  us a pass, so / on the way: a 2027-token prompt, 4 layers 342 / 330, 4 x 8192 tokens 2482 / 2437, last 512 of 24576, 4 layers 1088 / 1074.
        auto step = [&](int u, const Tiles &X0, const Tiles &X1, const float4v (&Sin)[2][kQT], float4v (&Sout)[2][kQT], int uf, Tiles &Xf) {
            const UnitFetch<LO, WAVES> ride = {unit_at(uf), Xf, wave, lane, WAVES == 8 || uf < nb};
            if (kRide && !(u <= wlast && calm)) {
#pragma unroll
                for (int i = 0; i < ride.kSlots; i++) ride(i);
            }
            if (u <= wlast) {
                const bool ahead = u + 1 < nb && u + 1 <= wlast;
                half8 P[kQT];
                float alpha[kQT];
                const bool was_calm = calm;
                bool moved = false;                              // some reference moved after the next unit's scores were issued
                half8 Av[8];
                if (calm) {
                    // the common case, one stretch of straight-line code: score products of the next unit next to the
                    // weights of this one against the unchanged reference (calm implies that there is a next unit, and
                    // that this unit's scores are relative to the reference as it stands: base, init are up to date)
                    if constexpr (kRide) score_unit<LO, kShift>(X1, Qf, Qlo, Sout, n, rq, init, &X0, Av, CalmSoftmax<KLO, score_batches<LO>(), UnitFetch<LO, WAVES>>{Sin, c, m, lsum, P, ride});
                    else score_unit<LO, kShift>(X1, Qf, Qlo, Sout, n, rq, init, &X0, Av, CalmSoftmax<KLO, score_batches<LO>(), NoFetch>{Sin, c, m, lsum, P, NoFetch()});
                } else {
                    float bin[kQT];
#pragma unroll
                    for (int qt = 0; qt < kQT; qt++) bin[qt] = base[qt];
                    if (ahead) {
                        set_base();
                        score_unit<LO, kShift>(X1, Qf, Qlo, Sout, n, rq, init, &X0, Av);
                    } else {
#pragma unroll
                        for (int ct = 0; ct < 8; ct++) Av[ct] = value_operand<kShift>(X0, ct, n, rq);
                    }
                    if (u < open_units) moved = softmax_unit<false, KLO>(Sin, c, u, qpos, bin, m, lsum, P, alpha, rq);
                    else moved = softmax_unit<true, KLO>(Sin, c, u, qpos, bin, m, lsum, P, alpha, rq);
                }
                // The accumulators are touched under a condition of their own, not inside the two-sided one above: there
                // the compiler's merge block sits in front of the calm side, and the calm side then copied all 64
                // accumulator registers, every unit, to meet the rescaled ones.
                if (!was_calm) output_rescale(alpha, O);
                // one place adds to the accumulators on every path: they stay in the same registers (with a product
                // on each path the compiler copied all 64 of them after every unit)
                output_add(Av, P, O);
                // the next unit is calm if it needs no mask, has a unit after it to look ahead to, its scores are
                // relative to the reference as it stands now, and none of them exceeds it by more than kCalm
                calm = ahead && u + 2 < nb && u + 2 <= wlast && u + 1 < open_units && !(KLO && moved) && !unit_exceeds<KLO>(Sout, inv_c, m);
            }
        };
        auto after = [](int x) { return x + 1 < tile_buffers(WAVES) ? x + 1 : 0; };
        int b0 = 0;                                              // buffer of unit u
        if constexpr (WAVES == 8) {
            for (int u = ub; u < nb; u += 2) {
                const int b1 = after(b0), b2 = after(b1), b3 = after(b2), b4 = after(b3);
                step(u, L[b0], L[b1], S, Sn, u + 3, L[b3]);     // buffers of units u - 2 and u - 1: all are done with them
                if (u + 1 < nb) step(u + 1, L[b1], L[b2], Sn, S, u + 4, L[b4]);
                wait_fetches();                                 // units u + 3 and u + 4 are there
                __syncthreads();
                b0 = b2;
            }
        } else {
            for (int u = ub; u < nb; u += 2) {
                const int b1 = after(b0), b2 = after(b1);
                if (!kRide) fetch(u + 2, L[b2]);
                step(u, L[b0], L[b1], S, Sn, u + 2, L[b2]);     // buffer of unit u - 1
                wait_fetches();                                 // unit u + 2 is there
                __syncthreads();
                if (!kRide) fetch(u + 3, L[b0]);
                if (u + 1 < nb) step(u + 1, L[b1], L[b2], Sn, S, u + 3, L[b0]);
                wait_fetches();
                __syncthreads();
                b0 = b2;
            }
        }
    }
    // ---- chunks of the fp16 window (with the tile's last piece), staged by the first four waves straight from the ring
    const int uend = !CUT || pc.index + 1 == pc.count ? units : nbt;
    if constexpr (KLO && WAVES == 4) {
#pragma unroll
        for (int qt = 0; qt < kQT; qt++) woff[qt] = kept[64 * WAVES * qt];
    }
    for (int u = nbt; u < uend; u++) {
        if (WAVES == kStagers || wave < kStagers) stage_window<kShift>(a, bh, u, T, tid, L[0]);
        __syncthreads();
        if (u <= wlast) {
            float4v S[2][kQT];
            half8 P[kQT];
            float alpha[kQT];
            const float4v none[kQT] = {};
            score_unit<kLoNone, kShift>(L[0], Qf, Qlo, S, n, rq, none);                 // fp16 rows: raw scores
            softmax_unit<true, false>(S, c, u, qpos, woff, m, lsum, P, alpha, rq);
            output_rescale(alpha, O);
            half8 Av[8];
#pragma unroll
            for (int ct = 0; ct < 8; ct++) Av[ct] = value_operand<kShift>(L[0], ct, n, rq);
            output_add(Av, P, O);
        }
        __syncthreads();
    }

#pragma unroll
    for (int qt = 0; qt < kQT; qt++) {
        float l = lsum[qt];
        l += xor_lanes(l, 16);
        l += xor_lanes(l, 32);
        const int r = rw + 16 * qt + n;
        if (CUT && r < rows && pc.count > 1) {
            // a piece: un-normalised outputs and (reference, sum) of the row, for prefill_merge
            const size_t at = (size_t)pc.slot * kQB + (r - pc.tile * kQB);
            float *o = a.part_o + at * kD;
            if (rq == 0) *reinterpret_cast<float2 *>(a.part_ml + at * 2) = make_float2(m[qt], l);
#pragma unroll
            for (int ct = 0; ct < 8; ct++) *reinterpret_cast<float4v *>(o + 16 * ct + 4 * rq) = O[ct][qt];
        } else if (r < rows) {
            const float inv = 1.0f / l;
            const int i = query_of(r);
            uint16_t *row = a.out + ((size_t)(head0 + r - i * hp) * a.n_q + i) * kD;
#pragma unroll
            for (int ct = 0; ct < 8; ct++)
                __builtin_nontemporal_store(u32x2{pack2(O[ct][qt][0] * inv, O[ct][qt][1] * inv), pack2(O[ct][qt][2] * inv, O[ct][qt][3] * inv)},
                                            reinterpret_cast<u32x2 *>(row + 16 * ct + 4 * rq));
        }
    }
}

// KQ: the layer's keys are quantized.  Each cache of such a layer is attended in the form its selection record names
// (without records: low parts of all channels).
//
// PT: PieceTable, or WholeTiles (whole tiles, 4 waves): reading the table and dividing by piece counts that are all 1
// costs a work-group about 0.14 us, which shows in short prompts (call of one layer with / without: 32 sequences of 22
// tokens, 32 / 8 heads 15.6 / 15.1 us, of 33 tokens, 28 / 4 heads 21.0 / 20.4 us).  Long prompts of whole tiles keep the kernel
// that knows the table: its loop is compiled a little better (4 x 8192 tokens 2436 us; without 2454).
// PACKED: rows of several query heads (Rows::heads).
template <bool KQ, class PT, int WAVES, bool PACKED>
__device__ __forceinline__ void attend_group(const PrefillArgs &a, const PT &pt)
{
    constexpr bool CUT = std::is_same<PT, PieceTable>::value;
    constexpr int kRows = kQW * WAVES;
    // The first three lines of the argument record are asked for at once, instead of one behind the other as they are needed (pieces of 27 queries
    // over 2290 tokens, 28 / 4 heads: 24.0 -> 23.5 us).  (In the 4-wave kernels it moves registers about and costs 0.5..1 %.)
    if constexpr (WAVES == 8) asm volatile("" ::"s"(a.lv.kres), "s"(a.Hq), "s"(a.n_bh), "s"(pt.pieces));
    const int hp = PACKED ? pt.heads : 1;                        // a cache's query heads are taken hp at a time
    const int rows = a.n_q * hp, heads = PACKED ? pt.groups : a.Hq / a.Hkv;
    const int tiles = CUT ? (rows + kQB - 1) / kQB : 0;
    const int parts = CUT && rows > kRows ? kQB / kRows : 1;     // work-groups of a piece
    int groups = WAVES == 8 ? tiles : (rows + kRows - 1) / kRows;      // work-groups per cache and `heads`
    if constexpr (CUT) groups = pt.pieces ? pt.pieces * parts : groups;
    // Work-groups go to the 8 XCDs in turn by their index, and each XCD has an L2 of its own: all query heads and
    // query tiles that read one (batch, kv head) cache are given to one XCD (when the count divides), so that its
    // units are fetched from memory once and then served by that L2.  Otherwise the pieces of all heads start in the order
    // of their length, and as many neighbouring heads as possible share an XCD.
    int local, jh, rank;                                         // cache within this launch, heads within its group, order
    const bool across = WAVES == 4 && !CUT && pt.order != kByCache, paired = WAVES == 4 && !CUT && pt.order == kPaired;
    if (a.n_bh % 8 == 0) {
        const int xcd = blockIdx.x & 7, per = heads * groups;
        int k = blockIdx.x >> 3;
        if (across) {
            const int caches = a.n_bh >> 3, first = kCUs / 8;
            if (paired && k >= first) k = per * caches - 1 - (k - first);
            rank = k / (heads * caches);
            local = 8 * ((k % (heads * caches)) / heads) + xcd;
            jh = k % heads;
        } else {
            local = 8 * (k / per) + xcd;
            jh = (k % per) % heads;
            rank = (k % per) / heads;
        }
    } else {
        const int all = a.n_bh * heads;
        int k = blockIdx.x;
        if (paired && k >= kCUs) k = all * groups - 1 - (k - kCUs);
        int head = k % all;
        rank = k / all;
        if (all % 8 == 0) head = (head & 7) * (all >> 3) + (head >> 3);
        local = head / heads;
        jh = head % heads;
    }
    Piece pc = {WAVES == 8 ? tiles - 1 - rank : kRows * (groups - 1 - rank) / kQB, kRows * (groups - 1 - rank), jh * hp, 0, 1, 0};      // the longest rows start first
    if constexpr (CUT) if (pt.pieces) {
        const int order = rank / parts;
        uint32_t w = pt.entry[0];
        int before = 0;                                          // partial results of the tiles in front of this one
        for (int r = 1; r < tiles && (int)(pt.entry[r] >> 16) <= order; r++) {
            before += piece_partials(w);
            w = pt.entry[r];
        }
        pc.tile = (int)(w & 255u);
        pc.row0 = pc.tile * kQB + (rank % parts) * kRows;
        if (WAVES == 4 && pc.row0 >= rows) return;               // the tile's second half is empty
        pc.index = order - (int)(w >> 16);
        pc.count = (int)((w >> 8) & 255u);
        pc.slot = (local * heads + jh) * pt.partials + before + pc.index;
    }
    if constexpr (KQ) {
        const Select *rec = a.select ? reinterpret_cast<const Select *>(a.select) + local : nullptr;
        if (rec && __builtin_amdgcn_readfirstlane((int)rec->compact) != 0) attend<kLoCompact, CUT, WAVES, PACKED>(a, pt, rec, local, pc);
        else attend<kLoAll, CUT, WAVES, PACKED>(a, pt, rec, local, pc);
    } else {
        attend<kLoNone, CUT, WAVES, PACKED>(a, pt, nullptr, local, pc);
    }
}

template <bool KQ, class PT>
__global__ __launch_bounds__(64 * 4, 2) void prefill_attention(PrefillArgs a, PT pt) { attend_group<KQ, PT, 4, true>(a, pt); }

template <bool KQ, bool PACKED>
__global__ __launch_bounds__(64 * 8, 1) void prefill_attend_long(PrefillArgs a, PieceTable pt) { attend_group<KQ, PieceTable, 8, PACKED>(a, pt); }

// ---- pass 3, only behind a pass 2 whose tiles were cut: merges the pieces of every tile that has more than one.  32 lanes
// per query row, 16 bytes per lane and piece, up to eight pieces in flight.  Bound by the traffic of the partial results.
constexpr int kMergeRows = 8;

__global__ __launch_bounds__(32 * kMergeRows) void prefill_merge(PrefillArgs a, PieceTable pt)
{
    const uint32_t w = pt.entry[blockIdx.y];
    const int tile = (int)(w & 255u), count = (int)((w >> 8) & 255u);
    const int row = blockIdx.x * kMergeRows + (threadIdx.x >> 5), lane = threadIdx.x & 31;
    const int r = tile * kQB + row, hp = pt.heads, i = row_query(pt, r);
    if (count < 2 || i >= a.n_q) return;
    int before = 0;
    for (int k = 0; k < (int)blockIdx.y; k++) before += piece_partials(pt.entry[k]);
    const int head = blockIdx.z;                                 // local * (heads of the group / row_heads) + which of them
    const int gq = a.Hq / a.Hkv, heads = pt.groups, local = head / heads, bh = a.bh0 + local;
    const size_t row0 = ((size_t)head * pt.partials + before) * kQB + row;
    const float *po = a.part_o + row0 * kD + 4 * lane, *pm = a.part_ml + row0 * 2;
    float M = -INFINITY, Lsum = 0.0f;
    float4v O = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = 0; k0 < count; k0 += 8) {
        float2 ml[8];
        float4v o[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int kk = k0 + k < count ? k0 + k : k0;         // past the end: a valid record again, weight zero
            ml[k] = *reinterpret_cast<const float2 *>(pm + (size_t)kk * kQB * 2);
            o[k] = *reinterpret_cast<const float4v *>(po + (size_t)kk * kQB * kD);
        }
        float Mn = M;
#pragma unroll
        for (int k = 0; k < 8; k++) Mn = fmaxf(Mn, ml[k].x);
        const float f0 = __builtin_amdgcn_exp2f(M - Mn);         // M = -inf on the first pass: factor 0 on empty sums
        Lsum *= f0;
        O *= f0;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const float f = k0 + k < count ? __builtin_amdgcn_exp2f(ml[k].x - Mn) : 0.0f;
            Lsum = fmaf(ml[k].y, f, Lsum);
            O += o[k] * f;
        }
        M = Mn;
    }
    const float inv = 1.0f / Lsum;
    uint16_t *out = a.out + ((size_t)((bh / a.Hkv) * a.Hq + (bh % a.Hkv) * gq + (head - local * heads) * hp + r - i * hp) * a.n_q + i) * kD + 4 * lane;
    __builtin_nontemporal_store(u32x2{pack2(O[0] * inv, O[1] * inv), pack2(O[2] * inv, O[3] * inv)}, reinterpret_cast<u32x2 *>(out));
}

// ---- how many pieces each tile is cut into (host).
//
// A compute unit holds one attention work-group of 8 waves (its five tile buffers fill the LDS) or two of 4, so a launch of few tiles leaves the
// chip idle, and one whose longest tiles take longer than an even share of all units waits for them.  The plan compares
// the uncut launch with cuts of the one to four longest tiles only and with cuts into pieces of 1/2, 1/3 .. 1/16 of the
// longest tile, each by the time its pieces take when the compute units pick them up longest first.  In units of 32 tokens:
// kPieceCost more per piece for its queries, first fetches and results; behind a cut kMergeCost for the launch that merges, and
// one per kPartialsPerUnit partial results (130 KiB each, written and read once).  Measured on the Llama shape (K4V2, whole call in us, uncut / cut as
// planned): 512 queries over 24576 tokens 833 / 292, 300 over 8000 297 / 129, a 2000-token prompt of 2 kv heads
// 92 / 63, of 8 kv heads 106 / 100 (finer cuts 106..122: the partial results outweigh the even load).  The constants are those
// of compact units (36 products); units with all low parts (48) or fp16 keys (32) count the same.  Of 163 calls of all forms,
// 17 to 30000 tokens, 8 queries and more, none takes longer than with whole tiles.  (A piece's start has become 2.5 us shorter since the two costs were set.  With
// kPieceCost 2, 3, 4 and 5, 27 calls of 8 to 9000 queries over 1500 to 32000 tokens are within 1.5 % of each other and no value is ahead: 512 over 24576 tokens
// 250.8 / 247.5 / 248.5 / 250.1, 512 over 8000 106.0 / 104.4 / 105.2 / 104.5, 8 / 2 heads, prompts of 4000 and 9000 tokens 75.2 / 75.5 / 74.7 / 73.9 and 229 / 230 / 230 / 231.)
constexpr int kPieceCost = 4;
constexpr int kMergeCost = 4;
constexpr int kPartialsPerUnit = 20;
constexpr int kMinPiece = 12;            // units: more than a tile's diagonal and one unit in front of it (9 + 1), so that every query of the
                                         // tile sees the whole first unit of its last piece (softmax_unit relies on it)
constexpr int kLeastCut = 2 * kMinPiece; // units of a cache that can be cut

struct Tiling { int tiles, n_blocks, p0, n_q, hp, waves; };

int tile_units(const Tiling &g, int tile)
{
    const int rows = g.n_q * g.hp, last = (tile + 1) * kQB < rows ? (tile + 1) * kQB - 1 : rows - 1;
    const int units = (g.p0 + last / g.hp) / 32 + 1;
    return g.n_blocks < units ? g.n_blocks : units;
}

int tile_pieces(int units, int length)
{
    const int most = units / kMinPiece < kMaxPieces ? units / kMinPiece : kMaxPieces, want = (units + length - 1) / length;
    return want < 1 || most < 1 ? 1 : want < most ? want : most;
}

// What a unit takes a work-group, in percent of the unit above: fewer rows than fill a work-group of 8 waves take less, down to the latency
// of its chain; one of 4 waves has 128 rows and shares its compute unit, unless there are no more of them than compute units.
int unit_cost(int waves, int rows, bool alone)
{
    if (waves == 8) return rows <= 64 ? 50 : rows <= 128 ? 65 : rows <= 192 ? 85 : 100;
    return !alone ? 100 : rows <= 64 ? 55 : 75;
}

// Behind a cut: the launch that merges and the partial results of `partials` pieces of up to `rows` rows.
long long merge_time(int partials, int heads, int rows)
{
    return partials ? 100 * kMergeCost + 100LL * partials * heads * rows / (kQB * kPartialsPerUnit) : 0;
}

// Fills t for pieces of at most `length` units of several tiles; returns the time by the rule above for `heads` query heads, in percent of a unit.
long long cut(const Tiling &g, int heads, int length, PieceTable &t)
{
    // tiles by falling length of their pieces
    int len[kMaxCutTiles], num[kMaxCutTiles], id[kMaxCutTiles];
    for (int i = 0; i < g.tiles; i++) {
        const int tile = g.tiles - 1 - i, units = tile_units(g, tile), count = tile_pieces(units, length);
        const int each = (units + count - 1) / count;
        int at = i;
        for (; at > 0 && len[at - 1] < each; at--) { len[at] = len[at - 1]; num[at] = num[at - 1]; id[at] = id[at - 1]; }
        len[at] = each; num[at] = count; id[at] = tile;
    }
    int pieces = 0, partials = 0;
    for (int r = 0; r < g.tiles; r++) {
        t.entry[r] = (uint32_t)(id[r] | num[r] << 8 | pieces << 16);
        pieces += num[r];
        partials += num[r] > 1 ? num[r] : 0;
    }
    t.pieces = pieces;
    t.partials = partials;
    // compute units grouped by when they are free, soonest first; equal pieces go to whole groups at a time
    struct { long long free; int count; } cu[kMaxCutTiles + 2];
    int groups = 1;
    cu[0] = {0, kCUs};
    for (int r = 0; r < g.tiles; r++) {
        long long left = (long long)num[r] * heads;
        const int cost = 100 * (len[r] + kPieceCost);
        const long long rounds = left / kCUs;                    // whole rounds over all compute units
        for (int i = 0; i < groups; i++) cu[i].free += rounds * cost;
        left -= rounds * kCUs;
        while (left > 0) {
            const int take = left < cu[0].count ? (int)left : cu[0].count;
            const long long until = cu[0].free + cost;
            left -= take;
            if (take < cu[0].count) cu[0].count -= take;
            else { for (int i = 1; i < groups; i++) cu[i - 1] = cu[i]; groups--; }
            int at = groups;
            while (at > 0 && cu[at - 1].free > until) { cu[at] = cu[at - 1]; at--; }
            if (at > 0 && cu[at - 1].free == until) {            // joins a group: close the gap again
                cu[at - 1].count += take;
                for (int i = at; i < groups; i++) cu[i] = cu[i + 1];
            } else {
                cu[at] = {until, take};
                groups++;
            }
        }
    }
    return cu[groups - 1].free + merge_time(partials, heads, kQB);
}

// Time of a single tile of `units` units in `count` pieces, which may have fewer rows than a work-group has room for (unit_cost, and that
// much less of partial results): its pieces are all alike, so the compute units take them in rounds.
long long single_tile_time(const Tiling &g, int heads, int units, int count)
{
    const int rows = g.n_q * g.hp, places = g.waves == 4 && rows <= kQB / 2 ? 2 * kCUs : kCUs, each = (units + count - 1) / count;
    const unsigned pieces = (unsigned)(count * heads);           // (fewer than 255 * 3 * kCUs)
    const int unit = unit_cost(g.waves, rows, pieces * (rows <= kQB / 2 ? 1 : 2) <= (unsigned)kCUs);
    return (long long)((pieces + places - 1) / places) * (each * unit + 100 * kPieceCost) + merge_time(count > 1 ? count : 0, heads, rows);
}

// slots: partial results the scratch area has room for; least: the time by the rule above (0: not a case for pieces)
PieceTable plan_pieces(const Tiling &g, int heads, int slots, long long &least)
{
    PieceTable best;
    best.pieces = best.partials = 0;
    least = 0;
    // (with three work-groups and more for every compute unit the longest tiles start early enough)
    if (g.tiles > kMaxCutTiles || g.n_blocks < kLeastCut || (long long)heads * g.tiles >= 3 * kCUs || slots < 2) return best;
    const int longest = tile_units(g, g.tiles - 1);
    // (so few tiles that 16 pieces of each do not fill the chip: up to 64)
    const int most = (long long)heads * g.tiles * 16 < 2 * kCUs ? 64 : 16;
    if (g.tiles == 1) {
        // Several such searches decide about a launch of a few tens of us (plan_launch), so each count of pieces is looked at once, up
        // to the most there is room for, and by a formula: 120 heads on one cache 29 us a plan with `cut` for every length, 0.8 now.
        int chosen = 1;
        least = single_tile_time(g, heads, longest, 1);
        for (int parts = 2, before = 1; parts <= most && longest / parts >= kMinPiece; parts++) {
            const int count = tile_pieces(longest, (longest + parts - 1) / parts);
            if (count == before) continue;
            before = count;
            if (count * heads > slots) break;
            const long long time = single_tile_time(g, heads, longest, count);
            if (time < least) { least = time; chosen = count; }
        }
        if (chosen > 1) {
            best.entry[0] = (uint32_t)(chosen << 8);
            best.pieces = best.partials = chosen;
        }
        return best;
    }
    PieceTable t;
    least = cut(g, heads, longest, t);
    auto consider = [&](int length) {
        if (length < kMinPiece || length >= longest) return;
        const long long time = cut(g, heads, length, t);
        if ((long long)t.partials * heads <= slots && time < least) { least = time; best = t; }
    };
    for (int k = 1; k <= 4 && k < g.tiles; k++) consider(tile_units(g, g.tiles - 1 - k));
    for (int parts = 2; parts <= most && longest / parts >= kMinPiece; parts++) consider((longest + parts - 1) / parts);
    return best;
}

// How a launch is divided.
struct LaunchPlan {
    PieceTable pt;
    int waves;
};

// The two forms of the attention kernel: work-groups of 8 waves and 256 rows, one per compute unit, or of 4 waves and 128 rows,
// two per compute unit.  The latter fetch every unit twice as often, but have the finer grain: the chip is filled by half as
// many rows, of two work-groups on a compute unit one goes on while the other waits, and a long one that is left alone
// speeds up.  A row of a work-group is a query of one of row_heads query heads.  Taken together, the heads of a group let 128
// rows end on the same or the next unit, so that hardly a wave waits for the others' last units, and few queries fill a work-group.
//
// - Whole tiles, 4 waves, all heads of the group together: caches of up to kShortCache units, unless pieces take less time (whole_time,
//   looked at where the rows are half of what fills the chip).  Up to two work-groups per compute unit start together, the longest
//   with the shortest.  Measured (us a call of one K4V4 or K4V2 layer with selection and dequantization, 8 waves of one head / 4
//   waves of the group): one prompt of 2027 tokens, 32 / 8 heads 87 / 76, 5000 tokens 290 / 269, 6000 tokens 390 / 367, 7000 tokens
//   480 / 483, 8192 tokens 619 / 637; four of 1024 tokens 129 / 114, eight of 500 tokens 165 / 136, four of 6000 tokens 1410 / 1399,
//   one of 300 tokens 37 / 34; 28 / 4 heads, two of 6000 tokens 621 / 602; 8 / 2 heads, one of 4000 tokens: 89 in pieces / 127.
//   (An XCD's L2 holds the 19 KiB units of one cache up to about there.)  Caches without packed units take them at any length, their window
//   comes through registers either way (us a pass with its append): 32 / 8 heads, one prompt of 300 tokens 22.0 / 20.7, 2027 tokens 129 / 104, 4000 tokens 271 / 265, 16000
//   tokens 3732 / 3437, four of 4000 tokens 1075 / 927; 28 / 4 heads, two of 8000 tokens 1710 / 1526; last 33 of 8000 tokens 368 / 362.
// - Tiles cut into pieces: 4 waves where they leave out an empty half of a tile (32 / 8 heads, 300 queries over 8000 tokens 110 / 104, over 24000
//   261 / 254) or many of the units are some query's last ones: prompts and halves of them up to kShortPieces units (8 / 2 heads, prompts of
//   6400, 7500, 8100, 9000, 10500 tokens 146 / 141, 185 / 182, 208 / 199, 248 / 250, 298 / 304; last 3800 of 7500 tokens 148 / 145), else 8 waves
//   (512 queries over 8000 tokens 111 / 114, over 24576 281 / 295; 450 over 8000 111 / 113).  An empty half counts where there are at
//   most two tiles (three, 600 queries: they gain 0..4 %) and the caches divide by the 8 XCDs; with other numbers it goes either way
//   (28 / 4 heads, 300 queries over 24000 tokens 209 / 229, three sequences of 8000 tokens 211 / 228; one of 8000 tokens 102 / 99).
// - Else whole tiles and 8 waves.
constexpr int kShortCache = 192;
constexpr int kShortPieces = 256;
constexpr int kFewUnits = 8;

// Time of whole tiles in work-groups of 4 waves, as `cut` has it (100: a unit of two work-groups on a compute unit); one that has its
// compute unit for itself takes 0.75 per unit.  Of 22 shapes around the line it names the
// faster one or one within 1 % for 21 (us a call, pieces / whole: 32 / 8 heads, prompts of 1300 and 1790 tokens 57.0 / 56.9, 72.1 / 69.8, last 1024 of
// 3000 and 5000 tokens 90 / 99, 125 / 151, last 1700 of 6000 196 / 196; 28 / 4 heads, prompts of 1500 and 2300 tokens 55.8 / 62.2, 86.8 / 82.1;
// 8 / 2 heads, one prompt of 5000 tokens 108 / 148, two of 2100 and 3800 tokens 60.0 / 75.7, 126 / 119, last 2500 of 5500 160 / 169, four
// of 1790 tokens 71.9 / 69.9), and not for four of 1100 tokens (49.8 / 52.3).
long long whole_time(const PrefillArgs &a)
{
    const int gq = a.Hq / a.Hkv, p0 = 32 * a.n_blocks + a.n_res - a.n_q, rows = a.n_q * gq, per = kQB / 2, tiles = (rows + per - 1) / per;
    auto units = [&](long long place) {                          // of the place-th longest work-group
        const int t = tiles - 1 - (int)(place / a.n_bh), last = (t + 1) * per < rows ? (t + 1) * per - 1 : rows - 1, u = (p0 + last / gq) / 32 + 1;
        return (long long)(a.n_blocks < u ? a.n_blocks : u);
    };
    const long long n = (long long)tiles * a.n_bh;
    const long long fixed = 100 * (kPieceCost + (a.n_bh % 8 == 0 ? 2 : 4));
    if (n <= kCUs) return units(0) * 75 + fixed;
    const long long uneven = units(0) * 75 + units(n - 1) * 25, even = 100 * units(kCUs);
    return (uneven > even ? uneven : even) + fixed;
}

long long rows_of(const PrefillArgs &a, int row_heads) { return (long long)a.n_q * row_heads; }

// part_slots: partial results there is room for
LaunchPlan plan_launch(const PrefillArgs &a, int part_slots)
{
    LaunchPlan p;
    const int gq = a.Hq / a.Hkv, heads = a.n_bh * gq, tiles = (a.n_q + kQB - 1) / kQB;
    const bool brief = a.n_blocks <= kShortCache;
    const long long work = (long long)heads * tiles;
    p.pt.pieces = p.pt.partials = 0;
    if (!brief || work < kCUs) {
        // the heads by themselves, or as many together as fit a tile; 8 waves or 4
        const int last = a.n_q - (tiles - 1) * kQB;              // rows of the last tile
        const bool prompt = a.n_blocks <= kShortPieces && 2 * a.n_q >= 32 * a.n_blocks;
        long long least = 0;
        for (int hp = 1; hp <= gq && (hp == 1 || (long long)a.n_q * hp <= kQB); hp++)
            for (int waves = 8; waves >= 4 && gq % hp == 0; waves -= 4) {
                const bool four = hp > 1 || prompt || (a.n_bh % 8 == 0 && tiles <= 2 && last <= kQB / 2);
                if (waves == 4 ? !four : tiles > 1 && four) continue;                 // (several tiles: the one or the other)
                const Tiling tiling = {(a.n_q * hp + kQB - 1) / kQB, a.n_blocks, 32 * a.n_blocks + a.n_res - a.n_q, a.n_q, hp, waves};
                long long time;
                const PieceTable t = plan_pieces(tiling, heads / hp, part_slots / hp, time);   // (as many records as with every head by itself)
                if (!t.pieces || (p.pt.pieces && time >= least)) continue;
                least = time;
                p.pt = t;
                p.waves = waves;
                p.pt.heads = hp;
            }
        if (brief && work >= kCUs / 2 && p.pt.pieces && whole_time(a) < least) p.pt.pieces = p.pt.partials = 0;
    }
    if (p.pt.pieces) {
        p.pt.order = kByCache;
    } else {
        p.waves = brief ? 4 : 8;
        // (Caches of a few units, where the heads by themselves leave no compute unit with two work-groups: those have fewer rows each. Two
        // sequences of 54 tokens, 32 / 8 heads, 4 layers: 96 us, 100 with the heads together; one of 300 tokens, 2 layers 65 / 67, of 500 84 / 82.)
        const bool few = a.n_blocks <= kFewUnits && (long long)heads * ((a.n_q + kQB / 2 - 1) / (kQB / 2)) <= kCUs;
        p.pt.heads = brief && !few && (long long)a.n_q * gq * gq < (1LL << 30) ? gq : 1;    // (row numbers: see row_query)
        for (int hp = 2; !brief && work >= 3 * kCUs && hp <= gq; hp++)
            if (gq % hp == 0 && (long long)a.n_q * hp <= kQB) p.pt.heads = hp;
        // The work-groups of an XCD cache by cache, or all by length while its caches fit its L2: the longest of the last cache
        // would start late (24 caches of 1114 tokens, per-token keys: 4 layers 506 us by cache).
        const long long groups = a.n_bh * ((rows_of(a, p.pt.heads) + kQB / 2 - 1) / (kQB / 2)) * (gq / p.pt.heads);
        p.pt.order = !brief ? kByCache : groups <= 2 * kCUs ? kPaired : (long long)a.n_bh * a.n_blocks <= 8 * kShortCache ? kByLength : kByCache;
    }
    p.pt.groups = gq / p.pt.heads;
    p.pt.magic = (uint32_t)(((1ULL << 32) + p.pt.heads - 1) / p.pt.heads);      // (of one head: not used)
    return p;
}

}  // namespace

int prefill_tile_pieces(const PrefillArgs &a, int part_slots, int tile)
{
    const LaunchPlan p = plan_launch(a, part_slots);
    for (int r = 0; p.pt.pieces && r < (a.n_q * p.pt.heads + kQB - 1) / kQB; r++)
        if ((int)(p.pt.entry[r] & 255u) == tile) return (int)((p.pt.entry[r] >> 8) & 255u);
    return 1;
}

PrefillForm prefill_form(const PrefillArgs &a, int part_slots)
{
    const LaunchPlan p = plan_launch(a, part_slots);
    return {p.waves, p.pt.heads, p.pt.order};
}

size_t prefill_piece_bytes() { return kQB * (kD + 2) * sizeof(float); }

size_t prefill_unit_bytes() { return sizeof(Tiles); }
size_t prefill_select_bytes() { return sizeof(Select); }
size_t prefill_ticket_offset() { return offsetof(Select, tickets); }

// Pass 0 for the caches [bh0, bh0 + n_bh) (a.select = their first record); only for layers whose keys are quantized
// per channel and hold packed blocks.  ev_begin (may be null) receives the kernel's start.
hipError_t launch_prefill_select(const PrefillArgs &a, hipStream_t s, hipEvent_t ev_begin)
{
    if (!a.select || a.lv.kbits >= 16 || a.lv.kpt || a.n_blocks < 1 || a.n_bh < 1) return hipErrorInvalidValue;
    // Several rounds of loads cost more than the parts' way through memory.  us a call of one layer, 8
    // caches, 1 / 2 / 4 / 8 work-groups each: 249 units 51 / 52 / 53 / 52, 499 units 82 / 79 / 78 / 78, 936 units 134 / 127 / 123 / 122.
    int parts = 1;
    if (a.n_blocks > kSelectWhole)
        while (parts < kSelectParts && 2 * parts * a.n_bh <= kCUs) parts *= 2;
    const dim3 grid((unsigned)parts, (unsigned)a.n_bh), block(64 * kSelectWaves);
    auto launch = [&](auto kernel) {
        if (ev_begin) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev_begin, nullptr, 0, a, parts);
        else hipLaunchKernelGGL(kernel, grid, block, 0, s, a, parts);
    };
    if (a.lv.narrow) launch(prefill_select<true>);
    else launch(prefill_select<false>);
    return hipGetLastError();
}

hipError_t launch_prefill_attention(const PrefillArgs &a, int part_slots, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end)
{
    const LaunchPlan plan = plan_launch(a, part_slots);
    const PieceTable &pt = plan.pt;
    const long long rows = (long long)a.n_q * pt.heads;
    const int heads = a.n_bh * pt.groups, per = kQW * plan.waves;
    const int tiles = (int)((rows + kQB - 1) / kQB);
    const long long groups = heads * (pt.pieces ? (long long)pt.pieces * (rows > per ? kQB / per : 1) : (rows + per - 1) / per);
    if (groups < 1 || groups > 0x7fffffffLL || a.n_bh < 1 || a.n_bh > 65535) return hipErrorInvalidConfiguration;
    const bool kq = a.lv.kbits < 16, vq = a.lv.vbits < 16;
    // selection records only exist where launch_prefill_select could write them
    if (a.select && !(kq && !a.lv.kpt && a.n_blocks > 0)) return hipErrorInvalidValue;
    hipEvent_t begin = ev_begin;                                 // stamped by the start of the first kernel launched
    if (a.n_blocks > 0) {
        // pass 1
        const dim3 grid((unsigned)a.n_blocks, (unsigned)a.n_bh), block(64 * kStagers);
        auto launch = [&](auto kernel) {
            if (begin) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, begin, nullptr, 0, a);
            else hipLaunchKernelGGL(kernel, grid, block, 0, s, a);
            begin = nullptr;
        };
        if (half_keys_of_4(kq, plan.waves)) {
            if (vq) launch(units_of_half_keys<true>);
            else launch(units_of_half_keys<false>);
        } else if (kq && vq) launch(prefill_dequantize<true, true>);
        else if (kq) launch(prefill_dequantize<true, false>);
        else if (vq) launch(prefill_dequantize<false, true>);
        else launch(prefill_dequantize<false, false>);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // pass 2 (more LDS than a kernel may declare statically)
    const dim3 grid((unsigned)groups), block(64 * plan.waves);
    const size_t lds = attention_lds(plan.waves);
    auto attend_launch = [&](auto kernel, auto table) -> hipError_t {
        // the larger dynamic LDS size is asked for at every launch of either kernel, on whichever device is current:
        // a host-side setting, negligible next to a launch of milliseconds, and no process-wide state to keep
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipEvent_t end = pt.pieces ? nullptr : ev_end;           // stamped by the end of the last kernel
        if (begin || end) hipExtLaunchKernelGGL(kernel, grid, block, lds, s, begin, end, 0, a, table);
        else hipLaunchKernelGGL(kernel, grid, block, lds, s, a, table);
        return hipGetLastError();
    };
    hipError_t e;
    if (plan.waves == 4 && !pt.pieces)
        e = kq ? attend_launch(prefill_attention<true, WholeTiles>, WholeTiles{pt}) : attend_launch(prefill_attention<false, WholeTiles>, WholeTiles{pt});
    else if (plan.waves == 4) e = kq ? attend_launch(prefill_attention<true, PieceTable>, pt) : attend_launch(prefill_attention<false, PieceTable>, pt);
    else if (pt.heads > 1) e = kq ? attend_launch(prefill_attend_long<true, true>, pt) : attend_launch(prefill_attend_long<false, true>, pt);
    else e = kq ? attend_launch(prefill_attend_long<true, false>, pt) : attend_launch(prefill_attend_long<false, false>, pt);
    if (e != hipSuccess || !pt.pieces) return e;
    // pass 3
    const dim3 mgrid(kQB / kMergeRows, (unsigned)tiles, (unsigned)heads), mblock(32 * kMergeRows);
    if (ev_end) hipExtLaunchKernelGGL(prefill_merge, mgrid, mblock, 0, s, nullptr, ev_end, 0, a, pt);
    else hipLaunchKernelGGL(prefill_merge, mgrid, mblock, 0, s, a, pt);
    return hipGetLastError();
}

}  // namespace kvq
