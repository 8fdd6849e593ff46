// Fused dequantize-and-attend decode kernel, matrix-core version (gfx950 MFMA 16x16x32 f16).
//
// Same computation as the vector-ALU kernel (Section 3.1, Eq. 1 over the dequantized cache
// of Section 3.2), reorganised so that the per-element work is done by the matrix cores:
//
//   scores   sum_d q_d (c_td s_d + z_d) = sum_d (q_d s_d) c_td + sum_d q_d z_d
//   output   sum_t p_t (c_td s_tg + z_tg) = sum_t (p_t s_tg) c_td + sum_t p_t z_tg
//
// The integer codes are the B operand.  Masked into the mantissa of an fp16 with a zero
// exponent field they read as c * 2^-k exactly (k depends on the bit position; differences are
// folded into the A operand), so "conversion" is about one AND per two codes.  The A operand
// carries q_d s_d (scores) or p_t s_tg (output); to keep fp32-class accuracy it is split into a
// high and a low fp16 part held in rows 2j and 2j + 1 of the 16-row tile (j = query head within
// the group, at most 8); a lane of the result tile holds both rows of a head, so the two partial
// results are added in registers after the MFMA.  The zero-point terms: q . z is one more MFMA
// per 32 channels (q and z are exact in fp16), sum_t p_t z_tg is a handful of fp32 FMAs per block.
//
// A work-group owns one (batch, kv head, split) and has two waves: one (the key wave) streams the
// key blocks and produces the softmax numerators of each block, the other (the value wave)
// consumes them one block later and accumulates the output.  The hand-off goes through
// double-buffered LDS tiles and one work-group barrier per block, so score and output work of
// neighbouring blocks overlap on different SIMDs and each wave carries only half of the state
// (which is what lets 4 waves share a SIMD and hide the memory latency).  Each wave writes its
// part of the split's partial result itself; the splits are merged by combine_splits.
//
// Short caches give few work-groups, each of which takes its blocks one after the other, and a call of such work-groups takes as long as that
// chain (0.54 us per block, 0.69 of 8 heads, on two of a compute unit's four SIMDs) and two launches.  There a work-group has two such pairs (KVQ_DECODE_PAIRS 2,
// kvq_decode_short.hip): each takes half of the split's units, or one the blocks and one the window, their results meet in LDS, a
// single split writes the outputs, and of several splits the work-group that finishes last merges the records (merge_pairs).
#include <hip/hip_ext.h>

#include <type_traits>

#include "kvq_internal.h"

#ifndef KVQ_DECODE_PAIRS
#define KVQ_DECODE_PAIRS 1
#endif

namespace kvq {
namespace {

constexpr int kPairs = KVQ_DECODE_PAIRS;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ half8 as_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    u32x4 v = {a, b, c, d};
    return __builtin_bit_cast(half8, v);
}

__device__ __forceinline__ float half_lo(uint32_t w) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu)); }
__device__ __forceinline__ float half_hi(uint32_t w) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16)); }

// B operand of MFMA m (8 codes of this lane) straight from the packed dwords.  Each code is
// masked into the mantissa of an fp16 whose exponent field is zero: a subnormal number, which
// the matrix core takes at face value, so element e of the operand is exactly
// code * 2^-CodeShift<BITS> * code_weight<BITS>(e) and "conversion" costs about one AND per two
// codes.  (The sum of a tile is aligned to the largest nominal exponent and keeps about 24 bits
// below it, the same as for a normal operand 1 + code * 2^-10, without a "1 +" to remove.)

// log2 of the divisor of the code in the base position: operand element = code * 2^-CodeShift
template <int BITS> struct CodeShift { static constexpr int value = 24; };

// one 32-token block of quantized keys / values as loaded by this lane
template <int BITS>
struct CodeRegs {
    u32x4 q[BITS < 16 ? BITS / 2 : 1];       // the lane's 64 codes, 16 bytes per load
    u32x2 s2;                                // two fp32 scales.  keys: channels 2*lane, +1; values: group lane>>4, tokens 2*(lane&15), +1
    uint32_t s1;                             // the same two scales as an fp16 pair (narrow metadata)
    uint32_t z;                              // zero-points of the same two elements, fp16 pair
    __device__ __forceinline__ uint32_t dw(int k) const { return q[k >> 2][k & 3]; }
};

template <int BITS>
__device__ __forceinline__ half8 codes_operand(const CodeRegs<BITS> &r, int m)
{
    if constexpr (BITS == 8) {
        // bytes (b0, b1), (b2, b3) -> halves 0x0000 | b : b * 2^-24
        const uint32_t w0 = r.dw(2 * m), w1 = r.dw(2 * m + 1);
        return as_half8(__builtin_amdgcn_perm(0u, w0, 0x0C010C00u), __builtin_amdgcn_perm(0u, w0, 0x0C030C02u),
                        __builtin_amdgcn_perm(0u, w1, 0x0C010C00u), __builtin_amdgcn_perm(0u, w1, 0x0C030C02u));
    } else if constexpr (BITS == 4) {
        // nibbles (k, k + 4) of the dword form a pair; mantissa bits 3:0 read c * 2^-24, bits 7:4 read 16 c * 2^-24
        const uint32_t x = r.dw(m), y = x >> 8;
        return as_half8(x & 0x000F000Fu, x & 0x00F000F0u, y & 0x000F000Fu, y & 0x00F000F0u);
    } else {
        // the four 2-bit fields of a byte pair are masked where they sit: mantissa bits 1:0, 3:2, 5:4, 7:6 read
        // c, 4 c, 16 c, 64 c (* 2^-24); the upper byte pair of the dword comes down with one shift
        const uint32_t x = (m & 1) ? r.dw(m >> 1) >> 8 : r.dw(m >> 1);
        return as_half8(x & 0x00030003u, x & 0x000C000Cu, x & 0x00300030u, x & 0x00C000C0u);
    }
}

// power of two by which the A operand must be divided for element e (its code sits higher in
// the mantissa than the base position)
template <int BITS>
__device__ __forceinline__ float code_weight_inv(int e)
{
    if (BITS == 4) return ((e >> 1) & 1) ? 0.0625f : 1.0f;
    if (BITS == 2) return 1.0f / (float)(1 << (2 * ((e >> 1) & 3)));
    return 1.0f;
}

// Split two products a0 b0, a1 b1, whose factors are also at hand rounded to fp16 (a16, b16: pairs), into fp16 high parts and fp16 low parts (the
// operands are kept near the top of the fp16 range, so the low parts are normal numbers too).  The
// high parts are the packed fp16 product of the rounded factors (one instruction for both; off the true product by
// less than 2^-9 of it), the low parts what is missing from the true products, each one mixed-precision
// multiply-add.  hi + lo = a b to about 2^-20: four instructions instead of six.
__device__ __forceinline__ void split_products(float a0, float b0, float a1, float b1, uint32_t a16, uint32_t b16,
                                               uint32_t &hi, uint32_t &lo)
{
    const half2v h = __builtin_bit_cast(half2v, a16) * __builtin_bit_cast(half2v, b16);
    const float d0 = __builtin_fmaf(a0, b0, -(float)h[0]), d1 = __builtin_fmaf(a1, b1, -(float)h[1]);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(d0, d1));
}

// The packed blocks of one tensor of one (batch, kv head) cache, addressed through buffer resources: a load's address
// is resource base + scalar byte offset of the block + a per-lane offset that never changes, so no vector register
// holds an address.
//
// The block loads of the streaming loop are issued and awaited by hand (issue_block / await_block).  The loop keeps
// one or two blocks in flight behind the one it works on, and what it must wait for is exactly "all but the loads of
// the younger blocks".  Left to the compiler, the wait counts of a loop whose loads stay in flight across the back
// edge came out far too low (all but one to three loads instead of all but eight to ten), the registers of the stage
// about to be loaded were re-used for address arithmetic, which added waits in front of the issue, and a one-word
// load per block was converted to a scalar where it was issued: every iteration cost one full memory round trip.
// The compiler does not know that these loads exist: its own waits (for loads it knows of) can only come out longer
// than needed, never shorter, and the registers a load writes are tied to the asm statements as read-write operands
// from the issue to the wait, so nothing else is put into them in between.
typedef int i32x4 __attribute__((ext_vector_type(4)));

struct BlockStream {
    i32x4 code, meta;                        // buffer resources: base, no stride, no bounds, 32-bit raw format
    i32x4 bexp;                              // exponent words of this cache only (reads beyond it return zero)
    uint32_t l16, l8, l4;                    // this lane's byte offsets into 16-, 8- and 4-byte-per-lane pieces
};

// The loop issues its loads unconditionally (so that the number of loads behind a block is a constant); past the end of
// the group's range they go through a resource with no bytes in range: every load through it is out of range, touches
// no memory and returns zero.
// (`code` and `meta` are emptied in place, once and for the rest of the sweep: copies would cost four scalar moves per resource and step.)
__device__ __forceinline__ void end_unless(bool real, BlockStream &S)
{
    S.code[2] = real ? S.code[2] : 0;
    S.meta[2] = real ? S.meta[2] : 0;
}
// r, or r with no bytes in range: one scalar select
__device__ __forceinline__ i32x4 pick(bool real, const i32x4 &r)
{
    return i32x4{r[0], r[1], real ? r[2] : 0, r[3]};
}

__device__ __forceinline__ i32x4 buffer_words(const void *base, int bytes = 0x7fffffff)
{
    const uint64_t v = reinterpret_cast<uint64_t>(base);
    return i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)v), __builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32) & 0xffff),
                 bytes, 0x00020000};
}

// streams of the keys (values = false) or values of the cache whose first block is number blk0 of the layer
__device__ __forceinline__ BlockStream block_stream(const LayerView &lv, bool values, size_t blk0, int n_cache_blocks, int lane, bool narrow)
{
    BlockStream S;
    const int bits = values ? lv.vbits : lv.kbits;
    S.code = buffer_words((values ? lv.vcode : lv.kcode) + blk0 * block_code_bytes(bits));
    S.meta = buffer_words((values ? lv.vmeta : lv.kmeta) + blk0 * meta_words(narrow));
    S.bexp = buffer_words(lv.bexp + blk0, n_cache_blocks * 4);
    S.l4 = (uint32_t)lane * 4u; S.l8 = (uint32_t)lane * 8u; S.l16 = (uint32_t)lane * 16u;
    return S;
}

// The exponent words (largest key scale / largest value scale of a block, see the quantize kernel) of the blocks that
// kChunk consecutive steps of the sweep visit, one per lane.  A block's word is read from the register with a lane
// index, so the block pipeline holds no load whose result a scalar computation waits for.  Loaded once per chunk of
// the sweep (issued by hand like the block loads; the first one ahead of the first blocks, later ones with a full
// wait, once per kChunk blocks).  Lanes whose block lies beyond the cache read zero.
constexpr int kChunk = 48;                   // steps per chunk: a multiple of both stage counts and of kZChunk, at most 64
constexpr int kZChunk = 16;                  // steps whose zero-point terms of the scores are formed at once (the columns of one tile)

// voff: byte offset of this lane's word in the cache's exponent array
__device__ __forceinline__ void issue_exponents(uint32_t &words, const BlockStream &S, uint32_t voff)
{
    asm volatile("buffer_load_dword %0, %1, %2, 0 offen" : "+v"(words) : "v"(voff), "s"(S.bexp));
}
template <int N>
__device__ __forceinline__ void await_exponents(uint32_t &words)
{
    asm volatile("s_waitcnt vmcnt(%1)" : "+v"(words) : "n"(N));
}

// loads of one block per lane
template <int BITS, bool LOADZ = true> constexpr int block_loads() { return BITS < 16 ? BITS / 2 + (LOADZ ? 2 : 1) : 0; }

// Issue the loads of block `blk` of the cache (counted from the cache's first block) into r.  NARROW: the block's
// scales are stored as fp16 (and were used that way by the encoder).  Codes and metadata are read once per call and
// never again before the whole cache has streamed by: the loads carry the non-temporal hint, so the lines are not
// kept in the caches at the expense of anything else (measured: 2-7 % shorter calls, most for the 8-bit pair).
// LOADZ = false: without the zero-points (the key wave fetches those of sixteen blocks at a time, issue_zero_points).
template <int BITS, bool NARROW, bool LOADZ = true>
__device__ __forceinline__ void issue_block(const BlockStream &S, int blk, CodeRegs<BITS> &r)
{
    static_assert(BITS < 16, "packed blocks only");
    const int coff = blk * block_code_bytes(BITS), moff = blk * 4 * meta_words(NARROW);
    asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen nt" : "+v"(r.q[0]) : "v"(S.l16), "s"(S.code), "s"(coff));
    if constexpr (BITS >= 4) asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen offset:1024 nt" : "+v"(r.q[BITS >= 4 ? 1 : 0]) : "v"(S.l16), "s"(S.code), "s"(coff));
    if constexpr (BITS == 8) {
        asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen offset:2048 nt" : "+v"(r.q[BITS == 8 ? 2 : 0]) : "v"(S.l16), "s"(S.code), "s"(coff));
        asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen offset:3072 nt" : "+v"(r.q[BITS == 8 ? 3 : 0]) : "v"(S.l16), "s"(S.code), "s"(coff));
    }
    if constexpr (NARROW) {
        asm volatile("buffer_load_dword %0, %1, %2, %3 offen nt" : "+v"(r.s1) : "v"(S.l4), "s"(S.meta), "s"(moff));
        if constexpr (LOADZ) asm volatile("buffer_load_dword %0, %1, %2, %3 offen offset:256 nt" : "+v"(r.z) : "v"(S.l4), "s"(S.meta), "s"(moff));
    } else {
        asm volatile("buffer_load_dwordx2 %0, %1, %2, %3 offen nt" : "+v"(r.s2) : "v"(S.l8), "s"(S.meta), "s"(moff));
        if constexpr (LOADZ) asm volatile("buffer_load_dword %0, %1, %2, %3 offen offset:512 nt" : "+v"(r.z) : "v"(S.l4), "s"(S.meta), "s"(moff));
    }
}

// The zero-points of the keys of kZChunk blocks, fetched as the B operand of one matrix product: lane (n, rq) gets
// channels 32 cb + 8 rq .. + 7 of the n-th of those blocks (16 bytes per load, cb = 0..3).  voff: byte offset, in the
// cache's metadata, of that block's zero-points plus 16 rq.  Issued by hand like the block loads.
__device__ __forceinline__ void issue_zero_points(u32x4 (&zb)[4], const BlockStream &S, bool real, uint32_t voff)
{
    const i32x4 meta = pick(real, S.meta);
    asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen nt" : "+v"(zb[0]) : "v"(voff), "s"(meta));
    asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen offset:64 nt" : "+v"(zb[1]) : "v"(voff), "s"(meta));
    asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen offset:128 nt" : "+v"(zb[2]) : "v"(voff), "s"(meta));
    asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen offset:192 nt" : "+v"(zb[3]) : "v"(voff), "s"(meta));
}
template <int N>
__device__ __forceinline__ void await_zero_points(u32x4 (&zb)[4])
{
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(zb[0]), "+v"(zb[1]), "+v"(zb[2]), "+v"(zb[3]) : "n"(N));
}

// The query rows of a tile, issued by hand like the block loads and ahead of them.  As ordinary loads, and behind branches for the heads that do
// not exist, they cost a round trip each: the compiler waited for them before it let the first blocks be asked for (it
// also took loads of the other role's code path to be pending), and, not knowing of the blocks' loads, waited for those too before
// the queries could be used.  Heads that do not exist read the first head's row.  Together with the arguments asked for at
// once and all divisions but one taken out of the way to the first load (decode_mfma), us a call, before / after: 2 kv heads, 512 tokens 7.0 / 6.5; 8 kv heads,
// 4133 tokens 9.8 / 9.1; 32 kv heads, 760 tokens 8.6 / 8.0; streaming launches 0.4 shorter (batch 16, 8192 tokens 32.5 / 32.0).
// (Two channels of every head per lane.  Only the key wave needs them.)
__device__ __forceinline__ void issue_query(uint32_t &q, const uint8_t *rows, uint32_t voff)
{
    asm volatile("global_load_dword %0, %1, %2" : "+v"(q) : "v"(voff), "s"(rows));
}
// N: loads issued behind the queries.  One statement for all of them: they are in registers when it is done.
template <int N>
__device__ __forceinline__ void await_queries(uint32_t (&q)[4])
{
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]) : "n"(N));
}
template <int N>
__device__ __forceinline__ void await_queries(uint32_t (&q)[8])
{
    asm volatile("s_waitcnt vmcnt(%8)" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(q[4]), "+v"(q[5]), "+v"(q[6]), "+v"(q[7]) : "n"(N));
}
// Wait until at most N vector memory operations of this wave are outstanding; r's registers are operands, so every
// use of the block comes after the wait.
template <int N, int BITS>
__device__ __forceinline__ void await_loads(CodeRegs<BITS> &r)
{
    if constexpr (BITS == 8)
        asm volatile("s_waitcnt vmcnt(%7)" : "+v"(r.q[0]), "+v"(r.q[BITS == 8 ? 1 : 0]), "+v"(r.q[BITS == 8 ? 2 : 0]), "+v"(r.q[BITS == 8 ? 3 : 0]), "+v"(r.s2), "+v"(r.s1), "+v"(r.z) : "n"(N));
    else if constexpr (BITS == 4)
        asm volatile("s_waitcnt vmcnt(%5)" : "+v"(r.q[0]), "+v"(r.q[BITS == 4 ? 1 : 0]), "+v"(r.s2), "+v"(r.s1), "+v"(r.z) : "n"(N));
    else
        asm volatile("s_waitcnt vmcnt(%4)" : "+v"(r.q[0]), "+v"(r.s2), "+v"(r.s1), "+v"(r.z) : "n"(N));
}

// Block r is needed; the loads of DEPTH - 1 blocks were issued after its own (real ones or empty ones).
template <int BITS, int DEPTH>
__device__ __forceinline__ void await_block(CodeRegs<BITS> &r)
{
    await_loads<(DEPTH - 1) * block_loads<BITS>(), BITS>(r);
}

// The same wait with one of two counts, N + EXTRA in step `first` (where EXTRA further loads were issued behind the
// block's own) and N otherwise.  One statement with the branch inside: two statements on two code paths would make
// the compiler merge two versions of registers that loads are still writing.
template <int N, int EXTRA, int BITS>
__device__ __forceinline__ void await_loads_either(CodeRegs<BITS> &r, int step, int first)
{
    static_assert(BITS == 2 || BITS == 4 || BITS == 8, "packed blocks only");
#define KVQ_EITHER "s_cmp_lg_u32 %[at], %[first]\n\ts_cbranch_scc1 1f\n\ts_waitcnt vmcnt(%[hi])\n\ts_branch 2f\n1:\n\ts_waitcnt vmcnt(%[lo])\n2:"
    if constexpr (BITS == 8)
        asm volatile(KVQ_EITHER : "+v"(r.q[0]), "+v"(r.q[BITS == 8 ? 1 : 0]), "+v"(r.q[BITS == 8 ? 2 : 0]), "+v"(r.q[BITS == 8 ? 3 : 0]), "+v"(r.s2), "+v"(r.s1), "+v"(r.z)
                     : [at] "s"(step), [first] "s"(first), [hi] "n"(N + EXTRA), [lo] "n"(N) : "scc");
    else if constexpr (BITS == 4)
        asm volatile(KVQ_EITHER : "+v"(r.q[0]), "+v"(r.q[BITS == 4 ? 1 : 0]), "+v"(r.s2), "+v"(r.s1), "+v"(r.z)
                     : [at] "s"(step), [first] "s"(first), [hi] "n"(N + EXTRA), [lo] "n"(N) : "scc");
    else
        asm volatile(KVQ_EITHER : "+v"(r.q[0]), "+v"(r.s2), "+v"(r.s1), "+v"(r.z)
                     : [at] "s"(step), [first] "s"(first), [hi] "n"(N + EXTRA), [lo] "n"(N) : "scc");
#undef KVQ_EITHER
}

// The (empty) loads of a group without blocks have landed.  The registers are not named: naming them on a second code path
// would make the compiler copy them while the loads are still writing.  That nothing else is put into them on the way here is
// for the build to check (decode_check.py follows this path too).
__device__ __forceinline__ void drain_unused() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// a block outside the streaming loop: issue and wait for everything
template <int BITS, bool NARROW>
__device__ __forceinline__ void load_block_now(const BlockStream &S, int blk, CodeRegs<BITS> &r)
{
    issue_block<BITS, NARROW>(S, blk, r);
    await_loads<0, BITS>(r);
}

// registers that a hand-issued load is going to write: any value will do, so none is moved in
template <typename T>
__device__ __forceinline__ void undefined(T &x) { asm volatile("" : "=v"(x)); }
template <int BITS>
__device__ __forceinline__ void undefined_regs(CodeRegs<BITS> &r)
{
#pragma unroll
    for (int c = 0; c < (BITS < 16 ? BITS / 2 : 1); c++) undefined(r.q[c]);
    undefined(r.s2); undefined(r.s1); undefined(r.z);
}

// the two scales of a loaded block as floats
template <bool NARROW, int BITS>
__device__ __forceinline__ float2 scales_of(const CodeRegs<BITS> &r)
{
    if constexpr (NARROW) return make_float2(half_lo(r.s1), half_hi(r.s1));
    const uint32_t x = r.s2[0], y = r.s2[1];       // (a bit cast applied to a vector element directly reads element 0)
    return make_float2(__builtin_bit_cast(float, x), __builtin_bit_cast(float, y));
}

// Reductions over the 16 lanes of a DPP row (lanes that share lane >> 4), result in every lane: two or four values at once, whose steps fill the two
// wait states between the write of a register and a DPP read of it.  (One at a time and by the compiler a step takes four or
// five instructions instead of one or two, and where few waves share a SIMD a wave issues one in five cycles.)
#define KVQ_ROW_STEP2(OP, CTRL) OP " %0, %0, %0 " CTRL " row_mask:0xf bank_mask:0xf\n\t" OP " %1, %1, %1 " CTRL " row_mask:0xf bank_mask:0xf"
#define KVQ_ROW_STEP4(OP, CTRL) KVQ_ROW_STEP2(OP, CTRL) "\n\t" OP " %2, %2, %2 " CTRL " row_mask:0xf bank_mask:0xf\n\t" OP " %3, %3, %3 " CTRL " row_mask:0xf bank_mask:0xf"
#define KVQ_ROW_REDUCE2(OP) "s_nop 1\n\t" KVQ_ROW_STEP2(OP, "quad_perm:[1,0,3,2]") "\n\ts_nop 0\n\t" KVQ_ROW_STEP2(OP, "quad_perm:[2,3,0,1]") \
                            "\n\ts_nop 0\n\t" KVQ_ROW_STEP2(OP, "row_half_mirror") "\n\ts_nop 0\n\t" KVQ_ROW_STEP2(OP, "row_mirror")
#define KVQ_ROW_REDUCE4(OP) "s_nop 1\n\t" KVQ_ROW_STEP4(OP, "quad_perm:[1,0,3,2]") "\n\t" KVQ_ROW_STEP4(OP, "quad_perm:[2,3,0,1]") \
                            "\n\t" KVQ_ROW_STEP4(OP, "row_half_mirror") "\n\t" KVQ_ROW_STEP4(OP, "row_mirror")
__device__ __forceinline__ void row_max16(float &a, float &b) { asm(KVQ_ROW_REDUCE2("v_max_f32_dpp") : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void row_sum16(float &a, float &b) { asm(KVQ_ROW_REDUCE2("v_add_f32_dpp") : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void row_sum16(float &a, float &b, float &c, float &d) { asm(KVQ_ROW_REDUCE4("v_add_f32_dpp") : "+v"(a), "+v"(b), "+v"(c), "+v"(d)); }
#undef KVQ_ROW_REDUCE4
#undef KVQ_ROW_REDUCE2
#undef KVQ_ROW_STEP4
#undef KVQ_ROW_STEP2
__device__ __forceinline__ float row_max16(float x) { float y = x; row_max16(x, y); return x; }
__device__ __forceinline__ float row_sum16(float x) { float y = x; row_sum16(x, y); return x; }

// A split's partial results are written through to memory as they are stored (system-scope stores): left in the
// write-back cache they would all be written out at once when the kernel ends, in front of the merge kernel that is
// waiting for it (measured: calls 1-3 % shorter, most with many splits per cache).
__device__ __forceinline__ void store_through(float *p, float2 v)
{
    asm volatile("global_store_dwordx2 %0, %1, off sc0 sc1" ::"v"(p), "v"(v) : "memory");
}

// Work-group barrier that waits for this wave's LDS traffic only: __syncthreads() would also wait for
// the global loads of the next block, which are meant to stay in flight across it.
__device__ __forceinline__ void wg_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// LDS of one key-wave / value-wave pair.  A tiles: row 2j = high parts, row 2j + 1 = low parts of head j.
template <int GQ>
struct __attribute__((aligned(16))) PairLds {
    _Float16 Ak[16][kD + 8];       // key wave: score A tiles [row][channel]
    // value wave: output A tiles [channel group][row][token].  A tile is 16 rows of 80 bytes plus 64 bytes: the four
    // lane rows of a wave write the same (row, token pair) of the four tiles at once, and with this distance between
    // the tiles (336 dwords = 16 banks more than a multiple of 64) they fall on four different quarters of the banks
    struct AvTile { _Float16 at[16][32 + 8]; _Float16 pad[32]; } Av[4];
    _Float16 Zk[kD];               // key wave: key zero-points (fp16 as stored); per-token keys: 32 floats of query sums
    float Mk[2][kD];               // key wave, per-token keys: the block's scales and zero-points as [group][token] floats
    // hand-off: softmax numerators of a block per head, double-buffered.  Rows of 40 floats: the four lane rows of
    // the key wave write rows 2 rq + hh at once, 80 dwords apart = four different quarters of the banks
    float P[2][8][32 + 8];
    float Zt[kZChunk][4][2];       // key wave: zero-point terms of the scores of kZChunk blocks, [block][lane row] = heads 2 rq, 2 rq + 1
    float alpha[2][8];             // hand-off: factor by which everything accumulated before the block shrinks
    int rescale[2][2];             // hand-off: non-zero when alpha is not all ones (padded to 16 bytes)
};

template <int GQ>
struct QueryRegs {
    float q2[GQ][2];               // scaled queries for channels 2*lane, 2*lane+1 (for q * s)
    uint32_t q16[GQ];              // the same pair rounded to fp16
    int nvalid;                    // heads of this tile that exist
    // what this lane reads of an A tile: its row (16 rows, high and low parts of 8 heads; where heads are absent, rows of the last one that
    // exists: no row has to be cleared, and the lanes of absent heads see finite values, which nobody reads)
    int row;
    const _Float16 *Aq;            // LDS: exact fp16 queries, the row of this lane's head (rows 2j and 2j + 1 of the A tile are equal: one is stored)
    float c, alpha_h;              // log2(e)/sqrt(D); weight of the partial scores
    float vw0, vw1;                // bit-position weights of tokens 2n, 2n+1 in the value codes
    float kappa;                   // per-token keys: weight of the partial score sums
    float qs[2][4];                // per-token keys: c * sum of q over channel group g, heads 2*rq, 2*rq + 1
    half8 At[4];                   // per-token keys, two pairs: the A operands, the same for every block
};

template <int GQ>
struct KeyState {
    float m[2], l[2];              // heads 2*rq, 2*rq + 1: reference max (log2 units), partial sum over this lane's tokens
};

template <int GQ>
struct ValueState {
    float4v O[8];                  // un-normalised output tile per 16-channel block (scaled by 2^(14 - ev - shift))
    float accz[GQ];                // sum_t p_t z_tg for group rq, tokens 2n, 2n+1
    int ev;                        // largest value-scale exponent so far
};

// Issue priority of this wave for the next block of its sweep: the more blocks it still has in front of it, the higher.
// The arbiter of a SIMD otherwise prefers the wave that was dispatched first, and the waves dispatched later to a SIMD
// ended 4 us behind the first ones (of 28) although all have the same work; with the priority tied to the progress a
// wave that falls behind is served first until it has caught up (the spread between the first and the last tenth of
// the waves to finish went from 6.3 us to 4.3 us).
// The priority is 3 for the first quarter of the sweep (set before it) and drops by one at the steps where another
// quarter of the blocks is done: three scalar compares per step.
struct PrioritySteps { int to2, to1, to0; };
__device__ __forceinline__ PrioritySteps priority_steps(int total)
{
    return PrioritySteps{(total + 3) >> 2, (total + 1) >> 1, (3 * total + 3) >> 2};
}
__device__ __forceinline__ void priority_at_step(int i, const PrioritySteps &t)
{
    if (i == t.to0) __builtin_amdgcn_s_setprio(0);
    else if (i == t.to1) __builtin_amdgcn_s_setprio(1);
    else if (i == t.to2) __builtin_amdgcn_s_setprio(2);
}

// ------------------------------------------------------------------ key wave

// The four A operands of a tile (16 bytes of this lane's row, 64 bytes apart or in four tiles), asked for together: one LDS round trip, where the
// compiler would fetch each behind the products of the one before.  (With the bookkeeping taken out of a block's path - cleared registers, resources
// copied, a barrier, zeroed rows, re-basing of empty sums - us a call: 8 kv heads, 4133 tokens 9.1 / 8.1; a wave alone on its SIMD
// issues one instruction in five cycles, so a hundred instructions are 0.2 us.)  Where four waves share a SIMD it may: they fill the gaps, and
// 4-bit instantiations would spill up to nine registers.
__device__ __forceinline__ void read_operands(half8 (&A)[4], const _Float16 *first, int stride)
{
#pragma unroll
    for (int k = 0; k < 4; k++) A[k] = *reinterpret_cast<const half8 *>(first + k * stride);
    if constexpr (kPairs > 1) asm volatile("" : "+v"(A[0]), "+v"(A[1]), "+v"(A[2]), "+v"(A[3]));
}

// scores of a quantized block: s[th][hh] for head 2*rq + hh, tokens 16*th + n
// ZB: the zero-point terms c * sum_d q_d z_d of heads 2 rq and 2 rq + 1 come ready-made in zc (zero_point_terms) instead
// of from the block's own zero-points.
template <int KB, int GQ, bool NARROW, bool ZB = false>
__device__ __forceinline__ void scores_packed(const CodeRegs<KB> &blk, uint32_t bexp, const QueryRegs<GQ> &Q, PairLds<GQ> &L, int lane,
                                              float (&s)[2][2], float2 zc = make_float2(0.0f, 0.0f))
{
    const int rq = lane >> 4;
    // lift the operand to the top of the fp16 range: the largest q*s of the block lands in [2^12, 2^14)
    const int ek = (int)(bexp & 0xffffu) - 32768;
    const float2 sc = scales_of<NARROW>(blk);
    const float ks0 = ldexpf(sc.x, 14 - ek), ks1 = ldexpf(sc.y, 14 - ek);
    const float ah = ldexpf(Q.alpha_h, ek - 14);
    const uint32_t ks16 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(ks0, ks1));
#pragma unroll
    for (int j = 0; j < GQ; j++) {
        if (j >= 4 && j >= Q.nvalid) continue;           // (a tile of 8 holds at least 5 heads)
        uint32_t hi, lo;
        split_products(Q.q2[j][0], ks0, Q.q2[j][1], ks1, Q.q16[j], ks16, hi, lo);
        *reinterpret_cast<uint32_t *>(&L.Ak[2 * j][2 * lane]) = hi;
        *reinterpret_cast<uint32_t *>(&L.Ak[2 * j + 1][2 * lane]) = lo;
    }
    if constexpr (!ZB) *reinterpret_cast<uint32_t *>(&L.Zk[2 * lane]) = blk.z;
    wave_lds_sync();
    float4v S0 = {0.0f, 0.0f, 0.0f, 0.0f}, S1 = S0, Z = S0;
    half8 Aop[4];
    read_operands(Aop, &L.Ak[Q.row][8 * rq], 32);
#pragma unroll
    for (int cb = 0; cb < 4; cb++) {
        S0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop[cb], codes_operand<KB>(blk, cb), S0, 0, 0, 0);
        S1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop[cb], codes_operand<KB>(blk, 4 + cb), S1, 0, 0, 0);
        if constexpr (!ZB) {
            const half8 Bz = *reinterpret_cast<const half8 *>(&L.Zk[32 * cb + 8 * rq]);
            Z = __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const half8 *>(Q.Aq + 32 * cb), Bz, Z, 0, 0, 0);
        }
    }
    // this lane holds rows 4*rq + i: (high, low) of head 2*rq and (high, low) of head 2*rq + 1
#pragma unroll
    for (int hh = 0; hh < 2; hh++) {
        const float zt = ZB ? (hh ? zc.y : zc.x) : Q.c * Z[2 * hh];
        s[0][hh] = fmaf(ah, S0[2 * hh] + S0[2 * hh + 1], zt);
        s[1][hh] = fmaf(ah, S1[2 * hh] + S1[2 * hh + 1], zt);
    }
}

// The zero-point terms c * sum_d q_d z_d of kZChunk blocks at once: the blocks are the columns of one product whose
// A operand is the exact fp16 query tile (rows 2j = 2j + 1 = head j) and whose B operand came straight from memory
// (issue_zero_points).  Lane (n, rq) ends up with the terms of block n for heads 2 rq and 2 rq + 1 and leaves them in
// L.Zt[n][rq], where the lanes of row rq pick them up block by block.
template <int GQ>
__device__ __forceinline__ void zero_point_terms(const u32x4 (&zb)[4], const QueryRegs<GQ> &Q, PairLds<GQ> &L, int lane)
{
    const int n = lane & 15, rq = lane >> 4;
    float4v Z = {0.0f, 0.0f, 0.0f, 0.0f};
    half8 Aop[4];
    read_operands(Aop, Q.Aq, 32);
#pragma unroll
    for (int cb = 0; cb < 4; cb++)
        Z = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop[cb],
                                                   as_half8(zb[cb][0], zb[cb][1], zb[cb][2], zb[cb][3]), Z, 0, 0, 0);
    *reinterpret_cast<float2 *>(&L.Zt[n][rq][0]) = make_float2(Q.c * Z[0], Q.c * Z[2]);
}

// Scores of a quantized block whose keys are grouped per token (one (s, z) per token and 32-channel group):
//   sum_d q_d (c_td s_tg + z_tg) = sum_g [ s_tg * sum_{d in g} q_d c_td  +  z_tg * sum_{d in g} q_d ].
// A channel group is exactly the depth of one MFMA, so each MFMA yields one inner sum per (head, token); the
// scale is applied to its result.  The A tile holds the exact fp16 queries (times a power of two and the code
// position weight; rows 2j, the odd rows are not used) and is built once per kernel.
template <int KB, int GQ, bool NARROW>
__device__ __forceinline__ void scores_packed_per_token(const CodeRegs<KB> &blk, const QueryRegs<GQ> &Q, PairLds<GQ> &L, int lane,
                                                        float (&s)[2][2])
{
    const int n = lane & 15, rq = lane >> 4;
    const float2 sc = scales_of<NARROW>(blk);
    *reinterpret_cast<float2 *>(&L.Mk[0][2 * lane]) = make_float2(sc.x * Q.kappa, sc.y * Q.kappa);
    *reinterpret_cast<float2 *>(&L.Mk[1][2 * lane]) = make_float2(half_lo(blk.z), half_hi(blk.z));
    wave_lds_sync();
    s[0][0] = s[0][1] = s[1][0] = s[1][1] = 0.0f;
    const float4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    float sv[4][2], zv[4][2];
    if constexpr (kPairs > 1) {
        // (together, like the operands of read_operands)
#pragma unroll
        for (int cb = 0; cb < 4; cb++) {
            sv[cb][0] = L.Mk[0][32 * cb + n]; sv[cb][1] = L.Mk[0][32 * cb + 16 + n];
            zv[cb][0] = L.Mk[1][32 * cb + n]; zv[cb][1] = L.Mk[1][32 * cb + 16 + n];
        }
#pragma unroll
        for (int cb = 0; cb < 4; cb++) asm volatile("" : "+v"(sv[cb][0]), "+v"(sv[cb][1]), "+v"(zv[cb][0]), "+v"(zv[cb][1]));
    }
#pragma unroll
    for (int cb = 0; cb < 4; cb++) {
        const half8 Aop = kPairs > 1 ? Q.At[cb] : *reinterpret_cast<const half8 *>(&L.Ak[Q.row][32 * cb + 8 * rq]);
        const float4v D0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop, codes_operand<KB>(blk, cb), zero, 0, 0, 0);
        const float4v D1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop, codes_operand<KB>(blk, 4 + cb), zero, 0, 0, 0);
        if constexpr (kPairs == 1) {
            sv[cb][0] = L.Mk[0][32 * cb + n]; sv[cb][1] = L.Mk[0][32 * cb + 16 + n];
            zv[cb][0] = L.Mk[1][32 * cb + n]; zv[cb][1] = L.Mk[1][32 * cb + 16 + n];
        }
        const float s0 = sv[cb][0], s1 = sv[cb][1], z0 = zv[cb][0], z1 = zv[cb][1];
#pragma unroll
        for (int hh = 0; hh < 2; hh++) {
            s[0][hh] = fmaf(s0, D0[2 * hh], fmaf(z0, Q.qs[hh][cb], s[0][hh]));
            s[1][hh] = fmaf(s1, D1[2 * hh], fmaf(z1, Q.qs[hh][cb], s[1][hh]));
        }
    }
    wave_lds_sync();          // the metadata tile is rewritten for the next block
}

// ---- fp16 rows (16-bit layers, window chunks): 32 tokens of a wave's tensor in registers
//
// A 16-bit layer is bound by memory, a window chunk by the latency of its rows, so all 32 rows of a tensor (8 KiB) are asked
// for at once, and of a 16-bit layer two units at a time.  Measured against one unit at a time with the value rows in four
// batches of eight: K16V16, batch 8, 4519 tokens (296 MB) 52.6 -> 33.4 us a call = 4.4 TB/s; one layer of 512 tokens
// 11.4 -> 9.2 us; batch 4, 760 tokens 14.4 -> 11.3 us.

// keys: tokens n and 16 + n, channels 32 cb + 8 rq .. + 7
struct KeyRows { u32x4 lo[4], hi[4]; };
// values: tokens 8 rq + i, channels 8 n .. + 7: one load fetches four whole rows
struct ValueRows { u32x4 row[8]; };

// One unit (32 rows of 256 bytes) of a 16-bit layer.  Issued unconditionally, past the end of a range through a resource
// with no bytes in range (no traffic, zeros): the number of loads behind a unit is then the same on every path, and the
// compiler's waits leave the next unit's loads in flight.
typedef __amdgpu_buffer_rsrc_t RowStream;
__device__ __forceinline__ RowStream row_stream(const uint8_t *base, bool real, int unit)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base) + (size_t)unit * block_code_bytes(16), 0, real ? block_code_bytes(16) : 0, 0x00020000);
}
constexpr int kNonTemporal = 2;          // cache policy bit of the buffer loads: 16-bit layers stream by like the packed codes

__device__ __forceinline__ void fetch_unit(const uint8_t *base, bool real, int unit, int lane, KeyRows &x)
{
    const RowStream r = row_stream(base, real, unit);
    const int off = (lane & 15) * (kD * 2) + (lane >> 4) * 16;
#pragma unroll
    for (int cb = 0; cb < 4; cb++) {
        x.lo[cb] = __builtin_amdgcn_raw_buffer_load_b128(r, off + 64 * cb, 0, kNonTemporal);
        x.hi[cb] = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * kD * 2 + 64 * cb, 0, kNonTemporal);
    }
}
__device__ __forceinline__ void fetch_unit(const uint8_t *base, bool real, int unit, int lane, ValueRows &x)
{
    const RowStream r = row_stream(base, real, unit);
    const int off = (lane >> 4) * (8 * kD * 2) + (lane & 15) * 16;
#pragma unroll
    for (int i = 0; i < 8; i++) x.row[i] = __builtin_amdgcn_raw_buffer_load_b128(r, off + i * (kD * 2), 0, kNonTemporal);
}

// A chunk of nt <= 32 window tokens from position pos0 on: rows of the ring of RC >= 32 slots, except for the token of a fused
// append (the chunk's last one: new_row), which is not in the ring yet.  Rows past the end are the last one again.
struct WindowChunk {
    const uint16_t *ring, *new_row;      // new_row: null unless the chunk's last token is the appended one
    int slot0, RC, nt;
    __device__ __forceinline__ const uint16_t *row(int t) const
    {
        const int tc = t < nt ? t : nt - 1;
        int slot = slot0 + tc;
        slot = slot >= RC ? slot - RC : slot;
        const uint16_t *p = ring + (size_t)slot * kD;
        return new_row && tc == nt - 1 ? new_row : p;
    }
};

__device__ __forceinline__ WindowChunk window_chunk(const DecodeArgs &a, bool values, int bh, int chunk)
{
    WindowChunk w;
    const int pos0 = a.n_blocks * kG + chunk * 32, left = a.n_res - chunk * 32;
    const uint16_t *fresh = values ? a.v_new : a.k_new;
    w.nt = left < 32 ? left : 32;
    w.ring = (values ? a.lv.vres : a.lv.kres) + (size_t)bh * a.RC * kD;
    w.RC = a.RC;
    w.slot0 = a.win_slot + chunk * 32;                           // (the window is shorter than the ring)
    w.slot0 = w.slot0 >= a.RC ? w.slot0 - a.RC : w.slot0;
    w.new_row = fresh && a.new_pos == pos0 + w.nt - 1 ? fresh + (size_t)bh * kD : nullptr;
    return w;
}

// the chunk's appended row goes into the ring for later launches (nothing reads that slot in this launch)
__device__ __forceinline__ void keep_new_row(const WindowChunk &w, int lane)
{
    if (w.new_row) {
        int slot = w.slot0 + w.nt - 1;
        slot = slot >= w.RC ? slot - w.RC : slot;
        reinterpret_cast<uint32_t *>(const_cast<uint16_t *>(w.ring) + (size_t)slot * kD)[lane] = reinterpret_cast<const uint32_t *>(w.new_row)[lane];
    }
}

__device__ __forceinline__ void fetch_chunk(const WindowChunk &w, int lane, KeyRows &x)
{
    asm volatile("" : "+v"(lane));                               // (nothing of the addresses is worked out ahead or kept)
    const uint16_t *row0 = w.row(lane & 15) + 8 * (lane >> 4), *row1 = w.row(16 + (lane & 15)) + 8 * (lane >> 4);
#pragma unroll
    for (int cb = 0; cb < 4; cb++) {
        x.lo[cb] = *reinterpret_cast<const u32x4 *>(row0 + 32 * cb);
        x.hi[cb] = *reinterpret_cast<const u32x4 *>(row1 + 32 * cb);
    }
}
// values: the ring's rows by 32-bit offsets; the appended row comes in `fresh` and takes its place in settle_chunk
__device__ __forceinline__ void fetch_chunk(const WindowChunk &w, int lane, ValueRows &x, u32x4 &fresh)
{
    const uint8_t *ring = reinterpret_cast<const uint8_t *>(w.ring);
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int i = 0; i < 8; i++) {
        const int t = 8 * (lane >> 4) + i, tc = t < w.nt ? t : w.nt - 1;
        int slot = w.slot0 + tc;
        slot = slot >= w.RC ? slot - w.RC : slot;
        x.row[i] = *reinterpret_cast<const u32x4 *>(ring + (uint32_t)(slot * (kD * 2) + 16 * (lane & 15)));
    }
    // (the caller's rows: fp16 alignment is all they owe)
    __builtin_memcpy(&fresh, (w.new_row ? w.new_row : w.ring + (size_t)w.slot0 * kD) + 8 * (lane & 15), sizeof fresh);
}
__device__ __forceinline__ void settle_chunk(const WindowChunk &w, int lane, ValueRows &x, u32x4 fresh)
{
    if (w.new_row) {
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int i = 0; i < 8; i++) {                            // (rows past the end too: the ring's may never have been written)
            const bool mine = 8 * (lane >> 4) + i >= w.nt - 1;
            x.row[i] = mine ? fresh : x.row[i];
        }
    }
}

// scores of nt fp16 rows; rows 2j and 2j + 1 of the query tile are equal
template <int GQ>
__device__ __forceinline__ void scores_rows(const KeyRows &x, int nt, const QueryRegs<GQ> &Q, int lane, float (&s)[2][2])
{
    const int n = lane & 15;
    float4v S0 = {0.0f, 0.0f, 0.0f, 0.0f}, S1 = S0;
#pragma unroll
    for (int cb = 0; cb < 4; cb++) {
        const half8 Aop = *reinterpret_cast<const half8 *>(Q.Aq + 32 * cb);
        S0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop, __builtin_bit_cast(half8, x.lo[cb]), S0, 0, 0, 0);
        S1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop, __builtin_bit_cast(half8, x.hi[cb]), S1, 0, 0, 0);
    }
#pragma unroll
    for (int hh = 0; hh < 2; hh++) {
        s[0][hh] = n < nt ? Q.c * S0[2 * hh] : -INFINITY;
        s[1][hh] = 16 + n < nt ? Q.c * S1[2 * hh] : -INFINITY;
    }
}

// Online softmax over the block's 32 scores per head.  Publishes the numerators (L.P[buf]) and the factor
// by which the value wave must shrink what it has accumulated (L.alpha[buf], L.rescale[buf]).
// The reference maximum only has to keep the numerators in range: it is refreshed (exact maximum over
// the block) when some score exceeds it by more than 1, so numerators stay <= 2 and the fp16 output
// operands cannot overflow.  Heads that do not exist see the last one's operands (QueryRegs::row), hence no other values than that head's.
template <int GQ>
__device__ __forceinline__ void softmax_publish(const float (&s)[2][2], KeyState<GQ> &W, PairLds<GQ> &L, int unit, int lane)
{
    const int buf = unit & 1;
    const int n = lane & 15, rq = lane >> 4;
    const float mx0 = fmaxf(s[0][0], s[1][0]), mx1 = fmaxf(s[0][1], s[1][1]);
    const bool grow = __builtin_amdgcn_ballot_w64((mx0 > W.m[0] + 1.0f) || (mx1 > W.m[1] + 1.0f)) != 0;
    if (grow) {
        float rm0 = mx0, rm1 = mx1;
        row_max16(rm0, rm1);
        const float mn0 = fmaxf(W.m[0], rm0), mn1 = fmaxf(W.m[1], rm1);
        const float a0 = __builtin_amdgcn_exp2f(W.m[0] - mn0), a1 = __builtin_amdgcn_exp2f(W.m[1] - mn1);
        W.l[0] *= a0; W.l[1] *= a1;
        W.m[0] = mn0; W.m[1] = mn1;
        L.alpha[buf][2 * rq] = a0;            // the 16 lanes of a row write the same value
        L.alpha[buf][2 * rq + 1] = a1;
    }
    if (lane == 0) L.rescale[buf][0] = grow && unit > 0 ? 1 : 0;       // (in front of the first unit nothing has been accumulated)
#pragma unroll
    for (int hh = 0; hh < 2; hh++) {
        const float p0 = __builtin_amdgcn_exp2f(s[0][hh] - W.m[hh]), p1 = __builtin_amdgcn_exp2f(s[1][hh] - W.m[hh]);
        W.l[hh] += p0 + p1;
        L.P[buf][2 * rq + hh][n] = p0;
        L.P[buf][2 * rq + hh][16 + n] = p1;
    }
}

// ------------------------------------------------------------------ value wave

// shrink everything accumulated so far if the key wave moved the reference maximum for this block
template <int GQ>
__device__ __forceinline__ void apply_rescale(ValueState<GQ> &W, const PairLds<GQ> &L, int buf, int lane)
{
    const int rq = lane >> 4;
    if (__builtin_amdgcn_readfirstlane(L.rescale[buf][0])) {
        const float2 al = *reinterpret_cast<const float2 *>(&L.alpha[buf][2 * rq]);
#pragma unroll
        for (int cblk = 0; cblk < 8; cblk++) {
            W.O[cblk][0] *= al.x; W.O[cblk][1] *= al.x;
            W.O[cblk][2] *= al.y; W.O[cblk][3] *= al.y;
        }
#pragma unroll
        for (int j = 0; j < GQ; j++) {
            const float aj = L.alpha[buf][j];
            W.accz[j] *= aj;
        }
    }
}

// output contribution of a quantized block
template <int VB, int GQ, bool NARROW>
__device__ __forceinline__ void output_packed(const CodeRegs<VB> &blk, uint32_t bexp, const QueryRegs<GQ> &Q, ValueState<GQ> &W,
                                              PairLds<GQ> &L, int buf, int lane)
{
    const int n = lane & 15, rq = lane >> 4;
    // keep p*s at the top of the fp16 range; when a block brings a larger scale, re-base the accumulators (exact)
    const int ev = (int)(bexp >> 16) - 32768;
    if (ev > W.ev) {
#pragma unroll
        for (int cblk = 0; cblk < 8; cblk++)
#pragma unroll
            for (int i = 0; i < 4; i++) W.O[cblk][i] = ldexpf(W.O[cblk][i], W.ev - ev);
        W.ev = ev;
    }
    const float2 sc = scales_of<NARROW>(blk);
    const float sv0 = ldexpf(sc.x * Q.vw0, 14 - W.ev), sv1 = ldexpf(sc.y * Q.vw1, 14 - W.ev);
    const uint32_t sv16 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(sv0, sv1));
#pragma unroll
    for (int j = 0; j < GQ; j++) {
        if (j >= 4 && j >= Q.nvalid) continue;
        const float2 pp = *reinterpret_cast<const float2 *>(&L.P[buf][j][2 * n]);
        uint32_t hi, lo;
        split_products(pp.x, sv0, pp.y, sv1, __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(pp.x, pp.y)), sv16, hi, lo);
        *reinterpret_cast<uint32_t *>(&L.Av[rq].at[2 * j][2 * n]) = hi;
        *reinterpret_cast<uint32_t *>(&L.Av[rq].at[2 * j + 1][2 * n]) = lo;
        W.accz[j] = fmaf(pp.x, half_lo(blk.z), fmaf(pp.y, half_hi(blk.z), W.accz[j]));
    }
    wave_lds_sync();
    half8 Aop[4];
    read_operands(Aop, &L.Av[0].at[Q.row][8 * rq], sizeof(L.Av[0]) / sizeof(_Float16));
#pragma unroll
    for (int gd = 0; gd < 4; gd++) {
#pragma unroll
        for (int c2 = 0; c2 < 2; c2++) {
            const int cblk = 2 * gd + c2;
            W.O[cblk] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop[gd], codes_operand<VB>(blk, cblk), W.O[cblk], 0, 0, 0);
        }
    }
}

// Output contribution of 32 fp16 rows (numerators of rows past the end are zero).  The rows are the B operand as they are, but for the order: a lane
// has 8 channels of 8 tokens, and operand e is the 8 tokens of channel 8 n + e, one byte permutation per pair of tokens.  The numerators are the A
// operand, read from the hand-off tile: 2^12 p as an fp16 number and, 2^14 times as large, what that leaves, the nearest fp16 number too (p <= 2).  Together they
// are p to a unit of its 24th bit (below 2^-12 two) for p >= 2^-22 and to 2^-47 below that.  The high part is the nearest number to 2^12 p + 2^-24 and so never zero (the low
// part makes up for it): an infinite value stays infinite under any weight.
// R[e]: rows 4 rq + i as everywhere (high and low parts of heads 2 rq, 2 rq + 1), channel 8 n + e, times 2^12 (low parts 2^26).
// With vector multiply-adds instead (16 tokens x 4 channels x the heads, 256 instructions for 4 heads against about 75 here) this was the
// longest step of a short call: a chunk took the value wave 1.1 us, 0.35 now.  (Parts cut off instead of rounded, with 2^-12 of the low one's factor: 22 bits
// of p, nothing below 2^-36, and an infinite value under such a weight was lost.  us a call, so / now: one sequence of 1000 fp16 tokens 6.00 / 6.08, 733 tokens
// with a window of five chunks 7.1 / 7.2, 8 x 4519 fp16 tokens 29.7 / 29.75.)
constexpr float kRowLift = 4096.0f, kLowLift = 16384.0f, kLeastHalf = 1.0f / (1 << 24);      // (the last: the smallest fp16 number)
template <int GQ>
__device__ __forceinline__ void output_rows(const ValueRows &x, float4v (&R)[8], const QueryRegs<GQ> &Q, const PairLds<GQ> &L, int buf, int lane)
{
    const int rq = lane >> 4;
    const float *p = &L.P[buf][Q.row >> 1][8 * rq];
    const float4v pa = *reinterpret_cast<const float4v *>(p), pb = *reinterpret_cast<const float4v *>(p + 4);
    const float pp[8] = {pa[0], pa[1], pa[2], pa[3], pb[0], pb[1], pb[2], pb[3]};
    // (even lanes hold rows of high parts, odd lanes of low parts: the same instructions with other factors)
    const float of_high = lane & 1 ? -kLowLift : 1.0f, of_p = lane & 1 ? kRowLift * kLowLift : 0.0f;
    uint32_t a[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const float p0 = pp[2 * k], p1 = pp[2 * k + 1];
        const half2v h = {(_Float16)fmaf(p0, kRowLift, kLeastHalf), (_Float16)fmaf(p1, kRowLift, kLeastHalf)};
        const half2v part = {(_Float16)fmaf((float)h[0], of_high, p0 * of_p), (_Float16)fmaf((float)h[1], of_high, p1 * of_p)};
        a[k] = __builtin_bit_cast(uint32_t, part);
    }
    const half8 Aop = as_half8(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int e = 0; e < 8; e++) {
        uint32_t b[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t w0 = x.row[2 * k][e >> 1], w1 = x.row[2 * k + 1][e >> 1];
            b[k] = __builtin_amdgcn_perm(w1, w0, e & 1 ? 0x07060302u : 0x05040100u);
        }
        R[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Aop, as_half8(b[0], b[1], b[2], b[3]), R[e], 0, 0, 0);
    }
}

// high + low parts.  An infinite value makes the high part infinite and the low part infinite with either sign or, where the numerator has no
// low part, not a number: then the high part is the sum.  (Where a value is no number, both are none.)
__device__ __forceinline__ float join_parts(float hi, float lo)
{
    const float sum = fmaf(lo, 1.0f / kLowLift, hi);
    return sum == sum ? sum : hi;
}

// shrink: what the outputs of the blocks before the rows (already out of the registers) are to be multiplied by, heads 2 rq and 2 rq + 1
template <int GQ>
__device__ __forceinline__ void rescale_rows(float4v (&R)[8], float2 &shrink, const PairLds<GQ> &L, int buf, int lane)
{
    if (__builtin_amdgcn_readfirstlane(L.rescale[buf][0])) {
        const float2 al = *reinterpret_cast<const float2 *>(&L.alpha[buf][2 * (lane >> 4)]);
        shrink = make_float2(shrink.x * al.x, shrink.y * al.y);
#pragma unroll
        for (int e = 0; e < 8; e++) R[e] = float4v{R[e][0] * al.x, R[e][1] * al.x, R[e][2] * al.y, R[e][3] * al.y};
    }
}

// ------------------------------------------------------------------ merge of a work-group's pairs, and of the splits

// reductions over the 32 lanes of a half wave or (LANES = 64) over the wave, in every lane: the rows of 16, then the row's neighbour and the other
// half by the lane swaps (fed the same register twice, every lane gets its own value in one result and its partner's in the other)
__device__ __forceinline__ u32x2 with_row_partner(float x) { const uint32_t v = __builtin_bit_cast(uint32_t, x); return __builtin_amdgcn_permlane16_swap(v, v, false, false); }
__device__ __forceinline__ u32x2 with_half_partner(float x) { const uint32_t v = __builtin_bit_cast(uint32_t, x); return __builtin_amdgcn_permlane32_swap(v, v, false, false); }
__device__ __forceinline__ float swap_sum(u32x2 v) { const uint32_t a = v[0], b = v[1]; return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b); }
__device__ __forceinline__ float swap_max(u32x2 v) { const uint32_t a = v[0], b = v[1]; return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)); }
template <int LANES>
__device__ __forceinline__ float lanes_max(float x)
{
    x = swap_max(with_row_partner(row_max16(x)));
    return LANES == 64 ? swap_max(with_half_partner(x)) : x;
}
template <int LANES>
__device__ __forceinline__ float lanes_sum(float x)
{
    x = swap_sum(with_row_partner(row_sum16(x)));
    return LANES == 64 ? swap_sum(with_half_partner(x)) : x;
}

__device__ __forceinline__ void store_through(float *p, float4v v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1" ::"v"(p), "v"(v) : "memory");
}

__device__ __forceinline__ void store_through(float *p, float2v v) { store_through(p, make_float2(v[0], v[1])); }

// o / l as fp16 to channels of the output row (the caller's tensor: fp16 alignment is all it owes)
__device__ __forceinline__ void store_output(uint16_t *out, float2v o, float l)
{
    const half2v h = {(_Float16)(o[0] / l), (_Float16)(o[1] / l)};
    __builtin_memcpy(out, &h, sizeof h);
}
__device__ __forceinline__ void store_output(uint16_t *out, float4v o, float l)
{
    const half2v h0 = {(_Float16)(o[0] / l), (_Float16)(o[1] / l)}, h1 = {(_Float16)(o[2] / l), (_Float16)(o[3] / l)};
    const u32x2 h = {__builtin_bit_cast(uint32_t, h0), __builtin_bit_cast(uint32_t, h1)};
    __builtin_memcpy(out, &h, sizeof h);
}

// The records of all splits (at most kMergeSplits; of a tile of 8 heads, 16) of a wave's head or, in a tile of 8, two heads -> outputs.  kLanes lanes per
// head hold the splits' maxima and sums, 32 lanes fetch a record's outputs (16 bytes each), two records of a head at a time.  rows: heads of this
// wave that exist, row: the first.  The order of all sums is fixed, whichever work-group comes last.
// Splits and heads that do not exist lie beyond their head's resource and read as zero: a resource per head, since behind one for both the second head's
// records would come in place of the first head's absent ones, and an infinity among them times the weight zero is no number.
// A record's place is in the vector offset, which is checked against the resource as it is (as a scalar offset it would be taken off the resource's
// size first, which is smaller where records are absent).
// The records come from work-groups on all XCDs: they are read past the caches (sc0 sc1), as they were written.
// Bound by the latency of the reads (0.45 us), so up to 32 records of a head (16 of each of two) are asked for at once, without a branch per record.  One
// sequence of 8 kv heads, 4133 tokens (27 splits), us a call, with half as many at once and sums that met in LDS behind a barrier / now: 7.9 / 7.4.
template <int GQ, int PAIRS>
__device__ __forceinline__ void merge_splits(const DecodeArgs &a, PairLds<GQ> (&Ls)[PAIRS], size_t row, int rows, int lane, int wave)
{
    constexpr int kBeyond = 17;                                  // cache policy bits: sc0, sc1
    constexpr int kHeads = GQ / 4, kLanes = 64 / kHeads, kAhead = 16 / kHeads, kList = 32 / kHeads, kRecord = (int)(kD * sizeof(float));
    static_assert(kMergeSplits <= 64 && 2 * PAIRS == 4, "a lane per split of a single head; a wave per head or two");
    // weights by head, half wave and round; the key waves' A tiles are no longer needed
    float *weights = reinterpret_cast<float *>(&Ls[0].Ak[0][0]) + wave * 64;
    static_assert(sizeof(Ls[0].Ak) >= 4 * 64 * sizeof(float), "the weights fit");
    const int half = lane >> 5, sl = lane & (kLanes - 1), head = kHeads == 2 ? half : 0;
    RowStream po[kHeads];
#pragma unroll
    for (int h = 0; h < kHeads; h++) po[h] = __builtin_amdgcn_make_buffer_rsrc(a.part_o + (row + h) * a.splits * kD, 0, h < rows ? a.splits * kRecord : 0, 0x00020000);
    const RowStream pm = __builtin_amdgcn_make_buffer_rsrc(a.part_ml + row * a.splits * 2, 0, rows * a.splits * (int)(2 * sizeof(float)), 0x00020000);
    const u32x2 ml = __builtin_amdgcn_raw_buffer_load_b64(pm, (head * a.splits + sl) * 8, 0, kBeyond);
    u32x4 x[kHeads][kAhead];
    const int off = half * kRecord + 16 * (lane & 31);
    auto fetch = [&](int s0) {
#pragma unroll
        for (int k = 0; k < kAhead; k++)
#pragma unroll
            for (int h = 0; h < kHeads; h++) x[h][k] = __builtin_amdgcn_raw_buffer_load_b128(po[h], off + (s0 + 2 * k) * kRecord, 0, kBeyond);
    };
    fetch(0);
    const uint32_t mw = ml[0], lw = ml[1];
    const float m = sl < a.splits ? __builtin_bit_cast(float, mw) : -INFINITY, l = __builtin_bit_cast(float, lw);
    const float M = lanes_max<kLanes>(m);
    const float f = m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m - M);         // (no such split: weight zero)
    weights[2 * kList * head + kList * (sl & 1) + (sl >> 1)] = f;
    const float sum = lanes_sum<kLanes>(sl < a.splits ? f * l : 0.0f);
    wave_lds_sync();
    float4v O[kHeads] = {};
    const float *w = weights + kList * half;
    for (int s0 = 0; s0 < a.splits; s0 += 2 * kAhead) {
        if (s0 > 0) fetch(s0);
        float4v wk[kHeads][kAhead / 4];
#pragma unroll
        for (int h = 0; h < kHeads; h++)
#pragma unroll
            for (int k = 0; k < kAhead / 4; k++) wk[h][k] = *reinterpret_cast<const float4v *>(w + 2 * kList * h + s0 / 2 + 4 * k);
#pragma unroll
        for (int k = 0; k < kAhead; k++)
#pragma unroll
            for (int h = 0; h < kHeads; h++) {
                const uint32_t w0 = x[h][k][0], w1 = x[h][k][1], w2 = x[h][k][2], w3 = x[h][k][3];
                O[h] += wk[h][k / 4][k % 4] * float4v{__builtin_bit_cast(float, w0), __builtin_bit_cast(float, w1), __builtin_bit_cast(float, w2), __builtin_bit_cast(float, w3)};
            }
    }
    // even and odd splits: of one head in every lane, of two the first's in the lower and the second's in the upper half wave
    float4v sums;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float lower = O[0][i], upper = O[kHeads - 1][i];
        sums[i] = swap_sum(__builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, lower), __builtin_bit_cast(uint32_t, upper), false, false));
    }
    if (head < rows) store_output(a.out + (row + head) * kD + 4 * (lane & 31), sums, sum);
}

// The pairs' results, from LDS, to the record of the split (or, with a single split, to the outputs).  A wave has a head or, in a tile of 8, two, merged here and, by
// the last work-group, in merge_splits.  With arrival counters the
// work-group that is the last of its cache and tile to count itself merges the splits: it waits for nobody.  A record is written
// through to memory and its stores are complete before the work-group counts itself, the counter is in memory too (device
// scope), and the last one reads past the caches, so it sees every record.  It leaves the counter at zero for the next call.
// Stores, count and reads are one memory round trip each (0.4, 0.4, 0.45 us) and take the place of a launch (2.6 us from kernel to
// kernel).  (Every wave counting for itself saves the two barriers and costs more than they do in counts of the same word: 27 splits 8.2 / 8.0.)
template <int GQ, int PAIRS>
__device__ __forceinline__ void merge_pairs(const ShortDecodeArgs &a, PairLds<GQ> (&Ls)[PAIRS], size_t qrow0, int nvalid, int split, int bh, int lane, int wave)
{
    wg_barrier();                                                // all pairs' results are in LDS
    constexpr int kLanes = 256 / GQ, kVec = kD / kLanes;         // lanes per head, channels per lane
    typedef float vec __attribute__((ext_vector_type(kVec)));
    const int first = wave * (64 / kLanes), head = first + (kLanes == 32 ? lane >> 5 : 0), c0 = kVec * (lane & (kLanes - 1));
    const bool any = first < nvalid;                             // of the wave's heads, one exists
    const size_t row = qrow0 + head;
    float m[PAIRS], l[PAIRS], M = -INFINITY, L = 0.0f;
#pragma unroll
    for (int p = 0; p < PAIRS; p++) {
        const float2 ml = *reinterpret_cast<const float2 *>(&Ls[p].Zt[head][0][0]);
        m[p] = ml.x;
        l[p] = ml.y;
        M = fmaxf(M, ml.x);
    }
    vec O = 0.0f;
#pragma unroll
    for (int p = 0; p < PAIRS; p++) {
        if (m[p] == -INFINITY) continue;                         // a pair without units: nothing of it is in LDS
        const float f = __builtin_amdgcn_exp2f(m[p] - M);
        L = fmaf(f, l[p], L);
        O += f * *reinterpret_cast<const vec *>(reinterpret_cast<const float *>(&Ls[p].Av[0].at[0][0]) + head * kD + c0);
    }
    if (head < nvalid) {
        if (a.splits == 1) {
            store_output(a.out + row * kD + c0, O, L);
        } else {
            store_through(a.part_o + (row * a.splits + split) * kD + c0, O);
            if (c0 == 0) store_through(a.part_ml + (row * a.splits + split) * 2, make_float2(M, L));
        }
    }
    if (a.splits == 1 || !a.tickets) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this wave's part of the record has reached memory
    wg_barrier();
    if (threadIdx.x == 0) {
        uint32_t *t = a.tickets + (size_t)bh * a.ticket_stride + blockIdx.z;
        const bool last = (int)__hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.splits - 1;
        if (last) __hip_atomic_store(t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        Ls[0].rescale[0][0] = last ? 1 : 0;
    }
    wg_barrier();
    if (any && __builtin_amdgcn_readfirstlane(Ls[0].rescale[0][0]))
        merge_splits<GQ, PAIRS>(a, Ls, qrow0 + first, kLanes == 32 && first + 1 < nvalid ? 2 : 1, lane, wave);
}

// ------------------------------------------------------------------ kernel

// Waves per SIMD the register allocation must leave room for: the host plans 2048 groups (4 waves per SIMD) for code
// widths up to 8 bits per key + value element and 1024 (2) beyond; the wider instantiations may
// use the registers that fewer resident waves leave free instead of spilling (16-bit layers: two units of rows).
template <int KB, int VB, int PAIRS> constexpr int resident_waves() { return PAIRS > 1 ? paired_groups(KB + VB) : KB + VB <= 8 ? 4 : 2; }

template <int PAIRS> using KernelArgs = std::conditional_t<PAIRS == 1, DecodeArgs, ShortDecodeArgs>;

template <int KB, int VB, int GQ, bool NARROW, bool KPT, int PAIRS>
__global__ __launch_bounds__(128 * PAIRS, (resident_waves<KB, VB, PAIRS>())) void decode_mfma(KernelArgs<PAIRS> a)
{
    static_assert(GQ == 4 || GQ == 8, "rows 2j and 2j + 1 of a 16-row tile");
    constexpr bool kFast = KB < 16 && VB < 16;
    // register stages of the phase-1 pipelines (blocks in flight per wave = stages - 1)
    // One block in flight behind the one being worked on (measured with exact wait counts, batch 16..32, 8K..32K
    // tokens: two or three blocks behind are 3-5 % slower for 4- and 2-bit codes and no faster for 8-bit ones: the
    // memory system is the queue here, more requests in it only wait longer).
    constexpr int DK = 2, DV = 2;
    // A group without blocks asks for its window rows ahead of the branch between the two kinds of group: the value wave at once, the key wave behind its
    // queries (whose wait counts the loads behind them).  In the streaming form of packed layers both ask behind the branch: that path would
    // hold registers of the rows over the loop, which has none to spare.  Launches of such groups alone, us a call, with the rows ahead and
    // their values on the vector units / so: 32 / 8 heads, 200 sequences of 60 tokens K4V2 15.4 / 13.3, K8V8 18.6 / 13.3, 640 of 25 tokens 25.3 / 21.3; 28 / 4
    // heads, 64 of 33 tokens 7.3 / 4.7, 320 of 100 tokens 25.6 / 16.5.
    constexpr bool kEarlyRows = !kFast || PAIRS > 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);     // wave-uniform on purpose: block indices stay scalar
    const int n = lane & 15, rq = lane >> 4;
    // The record's lines are asked for at once, here (each is a read from memory of its own; where the compiler asks for an argument when
    // it is first needed, they follow one another), and of divisions only the one by the blocks of the range is on the way to the first loads.
    asm volatile("" ::"s"(a.lv.kcode), "s"(a.lv.kmeta), "s"(a.lv.vcode), "s"(a.lv.vmeta), "s"(a.lv.bexp), "s"(a.q), "s"(a.gq), "s"(a.n_blocks), "s"(a.n_res),
                 "s"(a.NB), "s"(a.splits), "s"(a.units_per_split), "s"(a.split_rem), "s"(a.scale_log2e), "s"(a.win_slot));
    const int split = blockIdx.x, bh = blockIdx.y;
    const int head0 = blockIdx.z * GQ;
    const int nvalid = a.gq - head0 < GQ ? a.gq - head0 : GQ;
    const size_t qrow0 = (size_t)bh * a.gq + head0;
    // wave 0 / wave 1 take the key / value role in even work-groups and the other way round in odd ones,
    // so that both kinds of wave land on every SIMD
    const int pair = PAIRS > 1 ? wave >> 1 : 0;
    const bool key_wave = ((wave ^ (split + bh)) & 1) == 0;

    __shared__ PairLds<GQ> Ls[PAIRS];
    PairLds<GQ> &L = Ls[pair];
    __shared__ __attribute__((aligned(16))) _Float16 aq_lds[PAIRS][GQ][kD + 8];

    // ---- work of this group: units [u0, u1) = quantized blocks, then chunks of <= 32 fp16 window tokens; of this pair: `blocks`
    // blocks from block u0 on, then `chunks` chunks from first_chunk on.
    // Phase 1 covers the fully quantized blocks (only when both tensors are quantized), phase 2 the rest.
    // Unit number it (counted from the pair's first) is handed over through buffer it & 1.
    int u0, u1;
    split_range(a, split, u0, u1);
    int blocks = (u1 < a.n_blocks ? u1 : a.n_blocks) - u0, first_chunk = 0, chunks = u1 > a.n_blocks ? u1 - a.n_blocks : 0;
    int steps = blocks + chunks;                  // of the pair with most units: every wave meets that many barriers
    if constexpr (PAIRS > 1) {
        // the window's chunks go to the last pairs (to all, where there are no blocks), the blocks to those in front: the window's split has few blocks or
        // none, and a chunk (0.48 us) takes about as long as one
        static_assert(PAIRS == 2, "all units to both pairs, or the window to one and the blocks to the other");
        if (blocks == 0 || chunks == 0) {
            const int units = blocks + chunks, lower = units >> 1, mine = pair ? units - lower : lower, first = pair ? lower : 0;
            steps = units - lower;
            if (chunks == 0) {
                u0 += first;
                blocks = mine;
            } else {
                first_chunk = first;
                chunks = mine;
            }
        } else {
            steps = blocks > chunks ? blocks : chunks;
            if (pair == 0) chunks = 0;
            else blocks = 0;
        }
    }
    const int n1 = kFast ? blocks : 0, n2p = kFast ? 0 : blocks;      // the blocks of phase 1, of phase 2
    const int n2 = n2p + chunks;
    const size_t blk0 = (size_t)bh * a.NB;       // first block of this cache in the layer's arrays
    // cache block number of the i-th phase-1 unit (0 <= i < n1).
    // Every group starts its sweep at a different place of its range and wraps around: groups advance at the
    // same pace, and with equal phases their addresses would keep falling on the same memory channels.
    // (The start decides the order of all sums and how the operands round against the running maximum.  As the upper half of a product with the blocks,
    // without a division, the same outputs are 5e-5 to 1e-4 of their size elsewhere, no closer to 64 bits and no further; it saves 0.3..1 %: us a
    // pass, so / with the remainder: 16 layers of 4133 tokens 120.5 / 121.7, 4 layers of 16 x 4096 tokens K8V8 119.4 / 121.2, 8 layers of 16 x 8192
    // 256.5 / 257.3.)
    const uint32_t phase = (uint32_t)bh * 40503u + (uint32_t)split * 9973u;
    const int rot = n1 > 0 ? (int)(phase % (uint32_t)n1) : 0;
    auto blk1 = [&](int i) {
        const int r = i + rot;
        return u0 + (r < n1 ? r : r - n1);
    };
    // cache block number of the i-th of phase 2's blocks (16-bit tensors), with the same rotation
    const int rot2 = n2p > 0 ? (int)(phase % (uint32_t)n2p) : 0;
    auto blk2 = [&](int i) {
        const int r = i + rot2;
        return u0 + (r < n2p ? r : r - n2p);
    };
    auto blk1c = [&](int i) { return i < n1 ? blk1(i) : u0; };    // past the range: any number, the load is an empty one
    auto after = [&](int blk) { return blk + 1 < u0 + n1 ? blk + 1 : u0; };                // the block behind blk in the sweep
    // byte offset, in the cache's exponent array, of the word this lane holds for the chunk that starts at step c0
    auto exp_offset = [&](int c0) {
        const int i = c0 + lane;
        const int r = i + rot - (i + rot >= n1 ? n1 : 0);
        return (uint32_t)((i < n1 ? u0 + r : a.n_blocks) * 4);     // beyond the range: beyond the array, reads zero
    };

    QueryRegs<GQ> Q;
    Q.nvalid = nvalid;
    Q.c = a.scale_log2e;
    Q.row = n < 2 * nvalid ? n : 2 * nvalid - 2 + (n & 1);
    Q.Aq = &aq_lds[pair][Q.row >> 1][8 * rq];
    const uint8_t *queries = reinterpret_cast<const uint8_t *>(a.q + qrow0 * kD);       // of the tile's first head

    if (key_wave) {
        // =========================================================== key wave
        // the loads are issued in the order in which their results are needed: queries, then the first blocks
        uint32_t qw[GQ];
#pragma unroll
        for (int j = 0; j < GQ; j++) {
            const uint32_t off = (uint32_t)((j < nvalid ? j : 0) * (kD * 2) + 4 * lane);
            if constexpr (kFast) {
                undefined(qw[j]);
                issue_query(qw[j], queries, off);
            } else qw[j] = *reinterpret_cast<const uint32_t *>(queries + off);
        }
        BlockStream KS = block_stream(a.lv, false, blk0, a.n_blocks, lane, NARROW);
        uint32_t kexp;                                   // exponent words of the chunk's blocks, one per lane
        CodeRegs<KB> kr[DK];
        // per-channel keys: the zero-points do not come with the blocks but for kZChunk blocks at a time, as the operand
        // of one matrix product (zero_point_terms), which saves 4 of the 12 matrix instructions of a block's scores
        // (not next to 8-bit values in a tile of 8 heads: that instantiation has no registers to spare and would spill)
        constexpr bool kZB = kFast && !KPT && !(GQ == 8 && VB == 8);
        constexpr int NLK = block_loads<KB, !kZB>();
        u32x4 zb[4];
        // byte offset, in the cache's metadata, of the 16 bytes of zero-points this lane fetches for the chunk of steps
        // that starts at z0 (beyond the range: those of some block of the range, not used)
        auto zero_point_offset = [&](int z0) {
            const int i = z0 + n;
            return (uint32_t)(blk1c(i) * (4 * meta_words(NARROW)) + (NARROW ? 256 : 512) + 16 * rq);
        };
        if constexpr (kFast) {
#pragma unroll
            for (int d = 0; d < DK; d++) undefined_regs(kr[d]);
            undefined(kexp);
            issue_exponents(kexp, KS, exp_offset(0));
            if constexpr (kZB) {
#pragma unroll
                for (int cb = 0; cb < 4; cb++) undefined(zb[cb]);
                issue_zero_points(zb, KS, n1 > 0, zero_point_offset(0));
            }
#pragma unroll
            for (int d = 0; d < DK - 1; d++) {
                end_unless(d < n1, KS);
                issue_block<KB, NARROW, !kZB>(KS, blk1c(d), kr[d]);
            }
        }
        if constexpr (kFast) await_queries<1 + (kZB ? 4 : 0) + (DK - 1) * NLK>(qw);
#pragma unroll
        for (int j = 0; j < GQ; j++) *reinterpret_cast<uint32_t *>(&aq_lds[pair][j][2 * lane]) = qw[j];
        {
            // queries divided by a power of two that brings the largest to [0.5, 1).  Per-channel keys: with the softmax
            // constant folded in, for the q * s operand.  Per-token keys: the raw fp16 queries, scaled exactly.
            constexpr bool kPerToken = KPT && KB < 16;
            float qraw[GQ][2];
            float qmax = 0.0f;
#pragma unroll
            for (int j = 0; j < GQ; j++) {
                const uint32_t w = qw[j];
                qraw[j][0] = kPerToken ? half_lo(w) : half_lo(w) * Q.c;
                qraw[j][1] = kPerToken ? half_hi(w) : half_hi(w) * Q.c;
                qmax = fmaxf(qmax, fmaxf(fabsf(qraw[j][0]), fabsf(qraw[j][1])));
            }
            // maximum over the wave: 16-lane rows by DPP, the 4 rows as unsigned integers (the values are >= 0)
            const int qrow = __builtin_bit_cast(int, row_max16(qmax));
            uint32_t qbits = (uint32_t)__builtin_amdgcn_readlane(qrow, 0);
#pragma unroll
            for (int r = 1; r < 4; r++) {
                const uint32_t o = (uint32_t)__builtin_amdgcn_readlane(qrow, 16 * r);
                qbits = o > qbits ? o : qbits;
            }
            qmax = __builtin_bit_cast(float, qbits);
            int qexp = 0;
            if (qmax > 0.0f) (void)frexpf(qmax, &qexp);      // qmax = f * 2^qexp, f in [0.5, 1)
            constexpr int kshift = CodeShift<KB < 16 ? KB : 8>::value;
            const float w0 = code_weight_inv<KB < 16 ? KB : 8>((2 * lane) & 7), w1 = code_weight_inv<KB < 16 ? KB : 8>((2 * lane + 1) & 7);
            if constexpr (kPerToken) {
                // constant A tile: row 2j = q_j * 2^(13 - qexp) / (code position weight), exact in fp16; odd rows unused
                Q.kappa = Q.c * ldexpf(1.0f, kshift + qexp - 13);
                float *qs_lds = reinterpret_cast<float *>(&L.Zk[0]);      // [head][group] sums, 4 * GQ <= 32 floats
#pragma unroll
                for (int j = 0; j < GQ; j++) {
                    *reinterpret_cast<uint32_t *>(&L.Ak[2 * j][2 * lane]) =
                        __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(ldexpf(qraw[j][0], 13 - qexp) * w0, ldexpf(qraw[j][1], 13 - qexp) * w1));
                    *reinterpret_cast<uint32_t *>(&L.Ak[2 * j + 1][2 * lane]) = 0u;
                    const float part = row_sum16(qraw[j][0] + qraw[j][1]);       // this lane row's channel group is rq
                    if (n == 0) qs_lds[4 * j + rq] = part * Q.c;
                }
                wave_lds_sync();
                if constexpr (kPairs > 1) read_operands(Q.At, &L.Ak[Q.row][8 * rq], 32);
#pragma unroll
                for (int hh = 0; hh < 2; hh++)
#pragma unroll
                    for (int g = 0; g < 4; g++) Q.qs[hh][g] = 2 * rq + hh < nvalid ? qs_lds[4 * ((2 * rq + hh) % GQ) + g] : 0.0f;
            } else {
                Q.alpha_h = ldexpf(1.0f, kshift + qexp);     // undo the code position and 2^-qexp of q
#pragma unroll
                for (int j = 0; j < GQ; j++) {
                    Q.q2[j][0] = ldexpf(qraw[j][0], -qexp) * w0;
                    Q.q2[j][1] = ldexpf(qraw[j][1], -qexp) * w1;
                    Q.q16[j] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(Q.q2[j][0], Q.q2[j][1]));
                }
            }
        }
        // fp16 rows this wave starts with: a group without packed blocks asks for them here, one with packed blocks behind
        // those (16-bit keys: a pipeline of their own)
        KeyRows rows;
        if (kEarlyRows && n1 == 0 && n2p == 0 && chunks > 0) fetch_chunk(window_chunk(a, false, bh, first_chunk), lane, rows);
        wave_lds_sync();                                // the query tile
        KeyState<GQ> W;
#pragma unroll
        for (int i = 0; i < 2; i++) { W.m[i] = -INFINITY; W.l[i] = 0.0f; }
        float s[2][2];
        if constexpr (kFast) {
            // DK register stages in rotation: stage d is consumed while the loads of the next DK - 1 units (as far as
            // there are any) are in flight.
            // The sweep goes in chunks of kChunk steps (one register of exponent words each); a chunk starts at stage 0.
            auto drain = [&]() {
                // the empty loads past the end of the range, before their registers go back to the compiler
#pragma unroll
                for (int d = 0; d < DK; d++) await_loads<0, KB>(kr[d]);
                await_exponents<0>(kexp);
                if constexpr (kZB) await_zero_points<0>(zb);
            };
            if (n1 > 0) {
                await_exponents<(DK - 1) * NLK>(kexp);                         // the first chunk's: issued ahead of the first blocks
                const PrioritySteps prio = priority_steps(n1);
                int next = blk1c(DK - 1);
                if constexpr (PAIRS == 1) __builtin_amdgcn_s_setprio(3);
                for (int c0 = 0; c0 < n1; c0 += kChunk) {
                    if (c0 > 0) {
                        issue_exponents(kexp, KS, exp_offset(c0));
                        await_exponents<0>(kexp);
                    }
                    const int cend = c0 + kChunk < n1 ? c0 + kChunk : n1;
                    for (int z0 = c0; z0 < cend; z0 += kZChunk) {
                        const int zend = z0 + kZChunk < cend ? z0 + kZChunk : cend;
                        if constexpr (kZB) {
                            // The chunk's zero-points were asked for a chunk ago (the first chunk's ahead of the first
                            // blocks): they are older than every load still allowed to be pending here.  Form the chunk's
                            // terms, then ask for the next chunk's; those four loads go out in front of the first step's
                            // block loads, so that step alone waits with four more loads allowed behind its block.
                            await_zero_points<(DK - 1) * NLK>(zb);
                            zero_point_terms<GQ>(zb, Q, L, lane);
                            wave_lds_sync();
                            issue_zero_points(zb, KS, z0 + kZChunk < n1, zero_point_offset(z0 + kZChunk));
                        }
                        bool more = true;
                        for (int i = z0; more;) {
#pragma unroll
                            for (int d = 0; d < DK; d++) {
                                if (more) {
                                    if constexpr (PAIRS == 1) priority_at_step(i, prio);
                                    end_unless(i + DK - 1 < n1, KS);
                                    issue_block<KB, NARROW, !kZB>(KS, next, kr[(d + DK - 1) % DK]);
                                    next = after(next);
                                    if constexpr (kZB) await_loads_either<(DK - 1) * NLK, 4, KB>(kr[d], i, z0);
                                    else await_block<KB, DK>(kr[d]);
                                    const uint32_t ew = (uint32_t)__builtin_amdgcn_readlane((int)kexp, i - c0);
                                    if constexpr (KPT) scores_packed_per_token<KB, GQ, NARROW>(kr[d], Q, L, lane, s);
                                    else if constexpr (kZB)
                                        scores_packed<KB, GQ, NARROW, true>(kr[d], ew, Q, L, lane, s, *reinterpret_cast<const float2 *>(&L.Zt[i - z0][rq][0]));
                                    else scores_packed<KB, GQ, NARROW>(kr[d], ew, Q, L, lane, s);
                                    softmax_publish<GQ>(s, W, L, i, lane);
                                    wg_barrier();
                                    more = ++i < zend;
                                }
                            }
                        }
                    }
                }
                if constexpr (PAIRS == 1) __builtin_amdgcn_s_setprio(0);
                drain();
                if (chunks > 0) fetch_chunk(window_chunk(a, false, bh, first_chunk), lane, rows);    // (here: on no path is `rows` held over the loop)
            } else {
                drain_unused();
                if (!kEarlyRows && chunks > 0) fetch_chunk(window_chunk(a, false, bh, first_chunk), lane, rows);
            }
        }
        if constexpr (KB == 16) {
            // 16-bit keys: a unit's rows are on their way while the one before is worked on
            const uint8_t *base = a.lv.kcode + blk0 * block_code_bytes(16);
            KeyRows next;
            if (n2p > 0) fetch_unit(base, true, blk2(0), lane, rows);
            auto step = [&](int i, const KeyRows &x, KeyRows &y) {
                fetch_unit(base, i + 1 < n2p, blk2(i + 1), lane, y);
                scores_rows<GQ>(x, 32, Q, lane, s);
                softmax_publish<GQ>(s, W, L, i, lane);
                wg_barrier();
            };
            for (int i = 0; i < n2p; i += 2) {
                step(i, rows, next);
                if (i + 1 < n2p) step(i + 1, next, rows);
            }
        } else {
            // quantized keys next to 16-bit values
            for (int i = 0; i < n2p; i++) {
                const int u = blk2(i);
                CodeRegs<KB> r;
                undefined_regs(r);
                load_block_now<KB, NARROW>(KS, u, r);
                if constexpr (KPT) scores_packed_per_token<KB, GQ, NARROW>(r, Q, L, lane, s);
                else scores_packed<KB, GQ, NARROW>(r, a.lv.bexp[blk0 + u], Q, L, lane, s);
                softmax_publish<GQ>(s, W, L, i, lane);
                wg_barrier();
            }
        }
        if (n2p > 0 && chunks > 0) fetch_chunk(window_chunk(a, false, bh, first_chunk), lane, rows);
#pragma unroll 1
        for (int i = 0; i < chunks; i++) {
            const WindowChunk w = window_chunk(a, false, bh, first_chunk + i);
            keep_new_row(w, lane);
            scores_rows<GQ>(rows, w.nt, Q, lane, s);
            if (i + 1 < chunks) fetch_chunk(window_chunk(a, false, bh, first_chunk + i + 1), lane, rows);
            softmax_publish<GQ>(s, W, L, n1 + n2p + i, lane);
            wg_barrier();
        }
        wg_barrier();                                   // the value wave consumes the last unit
        // ---- result of the key wave: reference max and sum per head
        row_sum16(W.l[0], W.l[1]);
#pragma unroll
        for (int hh = 0; hh < 2; hh++) {
            const float lsum = W.l[hh];
            const int j = 2 * rq + hh;
            if constexpr (PAIRS > 1) {
                if (n == 0) *reinterpret_cast<float2 *>(&L.Zt[j][0][0]) = make_float2(W.m[hh], lsum);
            } else if (n == 0 && j < nvalid) {
                const size_t prow = (qrow0 + j) * a.splits + split;
                store_through(a.part_ml + prow * 2, make_float2(W.m[hh], lsum));
            }
        }
    } else {
        // =========================================================== value wave (one unit behind the key wave)
        BlockStream VS = block_stream(a.lv, true, blk0, a.n_blocks, lane, NARROW);
        uint32_t vexp;
        CodeRegs<VB> vr[DV];
        if constexpr (kFast) {
#pragma unroll
            for (int d = 0; d < DV; d++) undefined_regs(vr[d]);
            undefined(vexp);
            issue_exponents(vexp, VS, exp_offset(0));
#pragma unroll
            for (int d = 0; d < DV - 1; d++) {
                end_unless(d < n1, VS);
                issue_block<VB, NARROW>(VS, blk1c(d), vr[d]);
            }
        }
        ValueRows rows;                                 // (as in the key wave)
        u32x4 fresh;
        if constexpr (VB == 16) fetch_unit(a.lv.vcode + blk0 * block_code_bytes(16), n2p > 0, n2p > 0 ? blk2(0) : 0, lane, rows);
        Q.vw0 = code_weight_inv<VB < 16 ? VB : 8>((2 * n) & 7);
        Q.vw1 = code_weight_inv<VB < 16 ? VB : 8>((2 * n + 1) & 7);
        if (kEarlyRows && n1 == 0 && n2p == 0 && chunks > 0) fetch_chunk(window_chunk(a, true, bh, first_chunk), lane, rows, fresh);
        ValueState<GQ> W;
#pragma unroll
        for (int cblk = 0; cblk < 8; cblk++) W.O[cblk] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < GQ; j++) W.accz[j] = 0.0f;
        W.ev = -100;
        wg_barrier();                                   // the key wave has produced the first unit
        if constexpr (kFast) {
            auto drain = [&]() {
#pragma unroll
                for (int d = 0; d < DV; d++) await_loads<0, VB>(vr[d]);
                await_exponents<0>(vexp);
            };
            if (n1 > 0) {
                await_exponents<(DV - 1) * block_loads<VB>()>(vexp);
                // (the first block's: nothing has to be re-based for it)
                W.ev = (int)((uint32_t)__builtin_amdgcn_readlane((int)vexp, 0) >> 16) - 32768;
                W.ev = W.ev > -100 ? W.ev : -100;
                const PrioritySteps prio = priority_steps(n1);
                int next = blk1c(DV - 1);
                if constexpr (PAIRS == 1) __builtin_amdgcn_s_setprio(3);
                for (int c0 = 0; c0 < n1; c0 += kChunk) {
                    if (c0 > 0) {
                        issue_exponents(vexp, VS, exp_offset(c0));
                        await_exponents<0>(vexp);
                    }
                    const int cend = c0 + kChunk < n1 ? c0 + kChunk : n1;
                    bool more = true;
                    for (int i = c0; more;) {
#pragma unroll
                        for (int d = 0; d < DV; d++) {
                            if (more) {
                                if constexpr (PAIRS == 1) priority_at_step(i, prio);
                                end_unless(i + DV - 1 < n1, VS);
                                issue_block<VB, NARROW>(VS, next, vr[(d + DV - 1) % DV]);
                                next = after(next);
                                await_block<VB, DV>(vr[d]);
                                const uint32_t ew = (uint32_t)__builtin_amdgcn_readlane((int)vexp, i - c0);
                                // (always true here; as a run-time test it keeps the rarely taken re-base and rescale
                                // paths out of line, without it the register count of the loop grows by half)
                                if (i < n1) {
                                    apply_rescale<GQ>(W, L, i & 1, lane);
                                    output_packed<VB, GQ, NARROW>(vr[d], ew, Q, W, L, i & 1, lane);
                                }
                                wg_barrier();
                                more = ++i < cend;
                            }
                        }
                    }
                }
                if constexpr (PAIRS == 1) __builtin_amdgcn_s_setprio(0);
                drain();
                if (chunks > 0) fetch_chunk(window_chunk(a, true, bh, first_chunk), lane, rows, fresh);
            } else {
                drain_unused();
                if (!kEarlyRows && chunks > 0) fetch_chunk(window_chunk(a, true, bh, first_chunk), lane, rows, fresh);
            }
        }
        if constexpr (VB < 16) {
            // quantized values next to 16-bit keys
            for (int i = 0; i < n2p; i++) {
                const int u = blk2(i);
                apply_rescale<GQ>(W, L, i & 1, lane);
                CodeRegs<VB> r;
                undefined_regs(r);
                load_block_now<VB, NARROW>(VS, u, r);
                output_packed<VB, GQ, NARROW>(r, a.lv.bexp[blk0 + u], Q, W, L, i & 1, lane);
                wg_barrier();
            }
        }
        // ---- un-normalised outputs of the blocks per head and channel.  The tile layout (lane = channel 16 cblk + n, rows of
        // heads 2 rq, 2 rq + 1) is turned into (lane = channels 2 lane, 2 lane + 1, all heads) through the A-tile memory, which
        // is no longer needed; they stay there while the window is taken, which needs their registers.
        static_assert(sizeof(L.Av) >= GQ * kD * sizeof(float), "output staging fits the A tiles");
        float *o_lds = reinterpret_cast<float *>(&L.Av[0].at[0][0]);
        const bool staged = VB < 16 && n1 + n2p > 0;             // (a group with nothing but the window has no such outputs)
        if constexpr (VB < 16) if (staged) {
            constexpr int vshift = CodeShift<VB>::value;
            const float wO = ldexpf(1.0f, vshift + W.ev - 14);   // high and low parts carry the same weight
            wave_lds_sync();
#pragma unroll
            for (int hh = 0; hh < 2; hh++) {
                const int j = 2 * rq + hh;
                if (j < GQ) {
#pragma unroll
                    for (int cblk = 0; cblk < 8; cblk++) o_lds[j * kD + 16 * cblk + n] = wO * (W.O[cblk][2 * hh] + W.O[cblk][2 * hh + 1]);
                }
            }
            wave_lds_sync();
            // sum_t p_t z_tg of this lane's channel group (lane >> 4), over the 16 lanes that hold its tokens
#pragma unroll
            for (int j = 0; j < GQ; j += 4) row_sum16(W.accz[j], W.accz[j + 1], W.accz[j + 2], W.accz[j + 3]);
#pragma unroll
            for (int j = 0; j < GQ; j++) {
                const float az = W.accz[j];
                float2 *t = reinterpret_cast<float2 *>(&o_lds[j * kD + 2 * lane]);
                *t = make_float2(t->x + az, t->y + az);
            }
            wave_lds_sync();
        }
        float4v R[8];                                   // contributions of fp16 rows: see output_rows, rescale_rows
        float2 shrink = make_float2(1.0f, 1.0f);
#pragma unroll
        for (int e = 0; e < 8; e++) R[e] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (VB == 16) {
            const uint8_t *base = a.lv.vcode + blk0 * block_code_bytes(16);
            ValueRows next;
            auto step = [&](int i, const ValueRows &x, ValueRows &y) {
                fetch_unit(base, i + 1 < n2p, blk2(i + 1), lane, y);
                rescale_rows<GQ>(R, shrink, L, i & 1, lane);
                output_rows<GQ>(x, R, Q, L, i & 1, lane);
                wg_barrier();
            };
            for (int i = 0; i < n2p; i += 2) {
                step(i, rows, next);
                if (i + 1 < n2p) step(i + 1, next, rows);
            }
        }
        if (n2p > 0 && chunks > 0) fetch_chunk(window_chunk(a, true, bh, first_chunk), lane, rows, fresh);
#pragma unroll 1
        for (int i = 0; i < chunks; i++) {
            const int buf = (n1 + n2p + i) & 1;
            const WindowChunk w = window_chunk(a, true, bh, first_chunk + i);
            keep_new_row(w, lane);
            settle_chunk(w, lane, rows, fresh);
            rescale_rows<GQ>(R, shrink, L, buf, lane);
            output_rows<GQ>(rows, R, Q, L, buf, lane);
            if (i + 1 < chunks) fetch_chunk(window_chunk(a, true, bh, first_chunk + i + 1), lane, rows, fresh);
            wg_barrier();
        }
        // ---- result of the value wave: un-normalised output per head and channel
        if (n2 > 0) {
            // the fp16 rows' part: channels 8 n .. + 7 of heads 2 rq and 2 rq + 1
#pragma unroll
            for (int hh = 0; hh < 2; hh++) {
                const int j = 2 * rq + hh;
                if (j >= GQ) continue;
                float r[8];
#pragma unroll
                for (int e = 0; e < 8; e++) r[e] = (1.0f / kRowLift) * join_parts(R[e][2 * hh], R[e][2 * hh + 1]);
                float4v *o = reinterpret_cast<float4v *>(&o_lds[j * kD + 8 * n]);
                float4v o0 = {r[0], r[1], r[2], r[3]}, o1 = {r[4], r[5], r[6], r[7]};
                if (staged) {
                    const float f = hh ? shrink.y : shrink.x;
                    o0 += f * o[0];
                    o1 += f * o[1];
                }
                o[0] = o0;
                o[1] = o1;
            }
            wave_lds_sync();
        }
        // Nothing of the compiler's is pending here (vmcnt(0), the other counters as they are: free).  Said for the compiler: it lays the key wave's
        // code out behind this one and takes the way there for a possible one, and would wait there, among the hand-issued loads, for loads of here.
        __builtin_amdgcn_s_waitcnt(0x0F70);
        if constexpr (PAIRS == 1) {
#pragma unroll
            for (int j = 0; j < GQ; j++)
                if (j < nvalid)
                    store_through(a.part_o + ((qrow0 + j) * a.splits + split) * kD + 2 * lane, *reinterpret_cast<const float2 *>(&o_lds[j * kD + 2 * lane]));
        }
    }
    if constexpr (PAIRS > 1) {
        for (int i = n1 + n2; i < steps; i++) wg_barrier();      // pairs with fewer units
        merge_pairs<GQ, PAIRS>(a, Ls, qrow0, nvalid, split, bh, lane, wave);
    }
}

using Args = KernelArgs<kPairs>;

struct LaunchEvents { hipEvent_t begin, end; };

template <int KB, int VB, bool NARROW, bool KPT>
hipError_t launch_gq(const Args &a, hipStream_t s, LaunchEvents ev)
{
    const int gq = a.Hq / a.Hkv;
    const int BH = a.B * a.Hkv;
    const dim3 block(128 * kPairs);
    const dim3 grid(a.splits, BH, gq <= 4 ? 1 : (gq + 7) / 8);
    if (ev.begin && ev.end) {
        // measurement: the runtime's extended launch stamps the events with the dispatch's own start and end times
        if (gq <= 4) hipExtLaunchKernelGGL((decode_mfma<KB, VB, 4, NARROW, KPT, kPairs>), grid, block, 0, s, ev.begin, ev.end, 0, a);
        else hipExtLaunchKernelGGL((decode_mfma<KB, VB, 8, NARROW, KPT, kPairs>), grid, block, 0, s, ev.begin, ev.end, 0, a);
    } else if (gq <= 4) {
        hipLaunchKernelGGL((decode_mfma<KB, VB, 4, NARROW, KPT, kPairs>), grid, block, 0, s, a);
    } else {
        hipLaunchKernelGGL((decode_mfma<KB, VB, 8, NARROW, KPT, kPairs>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

template <int KB, bool NARROW, bool KPT>
hipError_t launch_vb(const Args &a, hipStream_t s, LaunchEvents ev)
{
    switch (a.lv.vbits) {
    case 2: return launch_gq<KB, 2, NARROW, KPT>(a, s, ev);
    case 4: return launch_gq<KB, 4, NARROW, KPT>(a, s, ev);
    case 8: return launch_gq<KB, 8, NARROW, KPT>(a, s, ev);
    default: return launch_gq<KB, 16, NARROW, KPT>(a, s, ev);
    }
}

template <bool NARROW>
hipError_t launch_kb(const Args &a, hipStream_t s, LaunchEvents ev)
{
    // the key grouping only matters for quantized keys
    if (a.lv.kpt) {
        switch (a.lv.kbits) {
        case 2: return launch_vb<2, NARROW, true>(a, s, ev);
        case 4: return launch_vb<4, NARROW, true>(a, s, ev);
        case 8: return launch_vb<8, NARROW, true>(a, s, ev);
        default: break;
        }
    }
    switch (a.lv.kbits) {
    case 2: return launch_vb<2, NARROW, false>(a, s, ev);
    case 4: return launch_vb<4, NARROW, false>(a, s, ev);
    case 8: return launch_vb<8, NARROW, false>(a, s, ev);
    default: return launch_vb<16, NARROW, false>(a, s, ev);
    }
}

}  // namespace

#if KVQ_DECODE_PAIRS == 1
hipError_t launch_decode_mfma(const DecodeArgs &a, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end)
#else
hipError_t launch_decode_short(const ShortDecodeArgs &a, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end)
#endif
{
    if (a.B * a.Hkv > 65535) return hipErrorInvalidConfiguration;
    const LaunchEvents ev = {ev_begin, ev_end};
    return a.lv.narrow ? launch_kb<true>(a, s, ev) : launch_kb<false>(a, s, ev);
}

}  // namespace kvq
