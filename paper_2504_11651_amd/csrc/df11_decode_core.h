// Building blocks of the DFloat11 decoder shared by the kernels that decode
// a stream (Algorithm 1 of arXiv 2504.11651): stream loads, table lookups,
// the two decode phases, the wave prefix sum and BF16 assembly, plus the
// host-side descriptor check.  Included by the decode kernels and by the
// fused decode-and-multiply kernel.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "df11.h"
#include "df11_tables.h"

namespace df11dec {


constexpr uint32_t kScanSlots = 16;  // waves per workgroup (<= 1024 threads)
// Exponent buffer bytes past the largest block: alignment shift (< 8), codes
// decoded past a block's end, and the 4 bytes per kept lookup that a lane may
// store past a clamped start offset.
constexpr uint32_t kBufSlack = 128;

struct DecodeArgs {
    const uint8_t *exp;
    const uint8_t *sm;
    const uint32_t *gaps;      // packed Gaps read as 32-bit words
    const uint32_t *block_pos; // B + 1 entries
    const uint8_t *tables;     // LDS image (blob past its header)
    uint16_t *out;
    uint64_t total_bits;
    uint32_t n_elems;
    uint32_t num_chunks;
    uint32_t num_blocks;
    uint32_t lut_bits;
    uint32_t max_len;
    uint32_t table_lds_bytes;
    uint32_t buf_bytes;        // exponent buffer, multiple of 16
    uint32_t twin_bufs;        // T = 1024: two block buffers alternate (else one)
    uint32_t hold;             // T <= 128: a block's decode waits for the last one's stores
};

__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }

// 4 stream bytes as loaded (little endian) -> word whose bit j is stream bit j
// (the stream is most-significant-bit first within each byte).
__device__ __forceinline__ uint32_t lsb_first(uint32_t le) {
    return __builtin_bitreverse32(__builtin_bswap32(le));
}

// The kernels declare no static LDS, so the dynamically sized LDS (and the
// decode table at its start) begins at group-segment offset 0; table entries
// are read through LDS byte offsets.
__device__ __forceinline__ uint2 lds_entry(uint32_t byte_offset) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 v = *(__attribute__((address_space(3))) const u32x2 *)
        static_cast<uintptr_t>(byte_offset);
    return make_uint2(v.x, v.y);
}

// Table entry as it lies in LDS (built from the blob's entry when the tables
// are staged, so the blob keeps its format):
//   x  the (up to four) exponents, each rotated right by one bit: bits 6..0
//      are the exponent's upper seven, the ones beside the sign in a BF16's
//      high byte, and bit 7 its lowest, the one above the mantissa
//   y  bits 0..5 bits consumed, bits 8..19 eight times the number of codes,
//      bits 20..31 code start mask; 0 for an escape.
// A sum of y over a chunk's lookups is then the chunk's state in one add per
// lookup: its low byte the bit position (it starts at the chunk's first code
// and stays below 128), bits 8..19 the output position in bits (at most 64
// codes and three more).  The sum of the masks overflows out at the top.
constexpr uint32_t kMetaCount = 8, kMetaMask = 20;

__device__ __forceinline__ uint32_t rotate_exponents(uint32_t e) {  // each byte right by one bit
    return ((e >> 1) & 0x7F7F7F7Fu) | ((e << 7) & 0x80808080u);
}

__device__ __forceinline__ uint2 pack_entry(uint32_t syms, uint32_t meta) {
    // the field widths hold whatever the blob's bytes are
    return make_uint2(rotate_exponents(syms),
                      (meta & 0xFu) | ((meta & 0x700u) << 3) | ((meta & 0x0FFF0000u) << 4));
}

__device__ __forceinline__ uint32_t state_pos(uint32_t acc) { return acc & 0xFFu; }
__device__ __forceinline__ uint32_t state_out8(uint32_t acc) {
    return __builtin_amdgcn_ubfe(acc, kMetaCount, kMetaMask - kMetaCount);
}

struct Tables {
    // K-bit entries (8 bytes) at LDS offset 0
    const uint32_t *lj_last; // [33]
    const uint32_t *offset;  // [33]
    const uint8_t *sorted;   // [256]
    uint32_t addr_mask;      // (2^K - 1) << 3: entry byte offset from a shifted window
    uint32_t lut_bits;
    uint32_t max_len;
    // the same arrays over the lanes of a wave, for the common long code:
    // lane L holds lj_last[L] (all ones outside K+1 .. max_len-1) and
    // offset[L], lane i the rotated exponents sorted[4i .. 4i+3]
    uint32_t lane_lj, lane_offset, lane_sorted;
};

// The tables as a wave uses them, read from LDS: the caller's barrier after
// stage_table_blob comes first.  From memory the lanes' words are one more
// round trip before a workgroup's first block; us, from memory and from LDS:
// 16.8 M weights in 64-chunk blocks 14.97 and 14.43, 4.2 M in 256-chunk
// blocks 7.90 and 7.61 (12-bit tables 9.00 and 8.68).
__device__ __forceinline__ Tables staged_tables(const DecodeArgs &a, const uint8_t *lds) {
    Tables tb;
    const uint32_t ent_bytes = 8u << a.lut_bits;
    tb.lj_last = reinterpret_cast<const uint32_t *>(lds + ent_bytes);
    tb.offset = tb.lj_last + 33;
    tb.sorted = reinterpret_cast<const uint8_t *>(tb.offset + 33);
    tb.addr_mask = ((1u << a.lut_bits) - 1u) << 3;
    // in a vector register: an AND with a scalar operand issues at half the
    // rate (4.3 against 2.3 cycles per wave, measured)
    asm("" : "+v"(tb.addr_mask));
    tb.lut_bits = a.lut_bits;
    tb.max_len = a.max_len;
    const uint32_t lane = threadIdx.x & 63u, L = lane < 33u ? lane : 0u;
    const uint32_t lj = tb.lj_last[L];
    tb.lane_lj = lane > a.lut_bits && lane < a.max_len ? lj : 0xFFFFFFFFu;
    tb.lane_offset = tb.offset[L];
    tb.lane_sorted = rotate_exponents(reinterpret_cast<const uint32_t *>(tb.sorted)[lane]);
    return tb;
}

// Code longer than the table index: canonical length search on the
// left-justified window, then rank within the length.  For loops that only
// some lanes run.
__device__ __forceinline__ uint2 decode_long(const Tables &t, uint32_t win) {
    const uint32_t v = __builtin_bitreverse32(win);
    uint32_t L = t.lut_bits + 1;
    while (L < t.max_len && v > t.lj_last[L]) ++L;
    const uint32_t idx = ((v >> (32u - L)) + t.offset[L]) & 255u;
    const uint32_t e = t.sorted[idx];
    return make_uint2(((e >> 1) | (e << 7)) & 255u, L | (8u << kMetaCount) | (1u << kMetaMask));
}

// The same where the whole wave is active: the lanes in `todo` one after the
// other, everything about a lane's code in scalar registers.  A block of 64
// chunks has one or two such codes, nearly always in different steps, and the
// search above costs four dependent LDS reads and about 45 vector
// instructions for each; this is about 10, none of them a memory access.
__device__ __forceinline__ void decode_long_lanes(const Tables &t, uint64_t todo, uint32_t win,
                                                  uint2 &e) {
    do {
        const uint32_t l = static_cast<uint32_t>(__builtin_ctzll(todo));
        todo &= todo - 1u;
        const uint32_t v = __builtin_bitreverse32(
            static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(win), static_cast<int>(l))));
        const uint32_t L = t.lut_bits + 1u + static_cast<uint32_t>(
            __builtin_popcountll(__builtin_amdgcn_ballot_w64(v > t.lane_lj)));
        const uint32_t off = static_cast<uint32_t>(
            __builtin_amdgcn_readlane(static_cast<int>(t.lane_offset), static_cast<int>(L)));
        const uint32_t idx = ((v >> (32u - L)) + off) & 255u;
        const uint32_t four = static_cast<uint32_t>(
            __builtin_amdgcn_readlane(static_cast<int>(t.lane_sorted), static_cast<int>(idx >> 2)));
        const uint32_t sym = (four >> ((idx & 3u) << 3)) & 255u;
        const bool mine = (threadIdx.x & 63u) == l;
        e.x = mine ? sym : e.x;
        e.y = mine ? L | (8u << kMetaCount) | (1u << kMetaMask) : e.y;
    } while (todo != 0);
}

// Inclusive prefix sum over the 64 lanes of a wave: four row shifts give the
// sums within each row of 16 lanes, two row broadcasts carry row totals.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xF, 0xF, true));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xF, 0xF, true));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xF, 0xF, true));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xF, 0xF, true));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xA, 0xF, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xC, 0xF, false));
    return v;
}

// Orders this wave's LDS accesses (other lanes' writes become visible to
// later reads: LDS executes a wave's instructions in order; this keeps the
// compiler from moving accesses across).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 4 sign/mantissa bytes + 4 rotated exponents -> 4 BF16 (two words, low
// element first): the high bytes take their sign from S, the low bytes their
// top bit from E.
__device__ __forceinline__ void assemble4(uint32_t S, uint32_t E, uint32_t &o0, uint32_t &o1) {
    const uint32_t lo = (E & 0x80808080u) | (S & 0x7F7F7F7Fu);  // (e&1)<<7 | mantissa
    const uint32_t hi = (S & 0x80808080u) | (E & 0x7F7F7F7Fu);  // sign<<7 | e>>1
    o0 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
    o1 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
}

// BlockOutputPos is read-only for the whole launch and its index is uniform:
// through the constant address space these are scalar loads, which keep the
// vector memory path for the streams.
__device__ __forceinline__ const __attribute__((address_space(4))) uint32_t *
block_positions(const DecodeArgs &a) {
    return (const __attribute__((address_space(4))) uint32_t *)a.block_pos;
}

// Raw global words one lane needs for chunk c = b*T + t of block b: the
// chunk's 8 bytes, the next 4 bytes, the two 32-bit words holding Gaps[c] and
// Gaps[c+1], and the block's two BlockOutputPos entries.  T is a multiple of
// 64, so a block's first chunk and first gap start on whole words (320 bits
// of gaps per 64 chunks): every address is a uniform base plus an offset that
// depends on t alone.
struct ChunkWords {
    uint32_t x, y, z, g0, g1, bp0, bp1;
};

template <uint32_t T>
__device__ __forceinline__ ChunkWords load_chunk(const DecodeArgs &a, uint32_t b, uint32_t t) {
    static_assert(T % 64 == 0, "blocks start on whole words of Gaps");
    ChunkWords r;
    r.bp0 = block_positions(a)[b];
    r.bp1 = block_positions(a)[b + 1];
    const uint8_t *exp = a.exp + 8ull * T * b;
    const uint2 own = *reinterpret_cast<const uint2 *>(exp + 8u * t);
    r.x = own.x;
    r.y = own.y;
    r.z = *reinterpret_cast<const uint32_t *>(exp + 8u * t + 8u);
    const uint32_t *gaps = a.gaps + uint64_t{T / 64 * 10} * b;
    r.g0 = gaps[(5u * t) >> 5];
    r.g1 = gaps[((5u * t) >> 5) + 1u];
    return r;
}

// Lookups kept in registers between the count phase and the write phase;
// a chunk needing more (short codes, 4 per lookup) continues in a loop.
constexpr int kKeep = 10;
// A lookup uses up to 12 bits of its 61-bit window, so five lookups fit.
constexpr int kPerWindow = 5;
// 8-element output groups whose sign/mantissa bytes are fetched at block start.
constexpr int kPre = 4;

// One chunk's bits and code range.  s*: the chunk's bits moved up by 3 (word
// bit i+3 of s0 is stream bit i), so that a window of them masked with the
// table's index bits gives the byte offset of the entry directly; w2: the
// third word unshifted (s2 lacks its top 3 bits).
struct Chunk {
    uint32_t s0, s1, s2, w2, start, end;
};

// What the count phase leaves for the write phase, per chunk: the exponents
// of each kept lookup, and 8 times its number of codes in one byte each (0
// where the chunk had ended).
template <int N>
struct Trail {
    uint32_t sy[N], n8[(N + 3) / 4];
};

// 64 bits of the chunk's shifted words from bit p (p < 64) on: bit 3 of the
// result is stream bit p, and at least the 61 stream bits from p, or all up
// to the 92nd, are there.
__device__ __forceinline__ uint64_t window64(const Chunk &ch, uint32_t p) {
    const bool upper = p >= 32;
    const uint32_t a = upper ? ch.s1 : ch.s0;
    const uint32_t b = upper ? ch.s2 : ch.s1;
    const uint32_t c = upper ? 0u : ch.s2;
    return (static_cast<uint64_t>(__builtin_amdgcn_alignbit(c, b, p)) << 32) |
           __builtin_amdgcn_alignbit(b, a, p);
}

// 32 stream bits from bit p (p < 64) on.
__device__ __forceinline__ uint32_t window32(const Chunk &ch, uint32_t p) {
    const uint32_t w0 = __builtin_amdgcn_alignbit(ch.s1, ch.s0, 3);
    const uint32_t w1 = __builtin_amdgcn_alignbit(ch.s2, ch.s1, 3);
    return __builtin_amdgcn_alignbit(p >= 32 ? ch.w2 : w1, p >= 32 ? w1 : w0, p);
}

// Code range of chunk c from its own and the next chunk's gap.
__device__ __forceinline__ void chunk_range(const DecodeArgs &a, uint32_t c, uint32_t gap_own,
                                            uint32_t gap_next, Chunk &ch) {
    ch.start = 0;
    ch.end = 0;
    if (c < a.num_chunks) {
        ch.start = gap_own;
        const uint32_t e = (c + 1 < a.num_chunks) ? 64u + gap_next
                                                  : static_cast<uint32_t>(a.total_bits - 64ull * c);
        ch.end = min(e, 95u);
    }
}

// Chunk t of block b.  A block all of whose chunks have a successor (all but
// the stream's last block) needs no check per chunk.
template <uint32_t T>
__device__ __forceinline__ Chunk chunk_setup(const DecodeArgs &a, const ChunkWords &cw, uint32_t b,
                                             uint32_t t) {
    Chunk ch;
    const uint32_t w0 = lsb_first(cw.x), w1 = lsb_first(cw.y), w2 = lsb_first(cw.z);
    ch.s0 = w0 << 3;
    ch.s1 = __builtin_amdgcn_alignbit(w1, w0, 29);
    ch.s2 = __builtin_amdgcn_alignbit(w2, w1, 29);
    ch.w2 = w2;
    const uint64_t gv = ((static_cast<uint64_t>(__builtin_bswap32(cw.g0)) << 32) |
                         __builtin_bswap32(cw.g1))
                        << ((5u * t) & 31u);
    const uint32_t gap_own = static_cast<uint32_t>(gv >> 59);
    const uint32_t gap_next = static_cast<uint32_t>(gv >> 54) & 31u;
    if ((b + 1u) * T < a.num_chunks) {
        ch.start = gap_own;
        ch.end = 64u + gap_next;
    } else {
        chunk_range(a, b * T + t, gap_own, gap_next, ch);
    }
    return ch;
}

__device__ __forceinline__ uint2 lookup(const Tables &t, const Chunk &ch, uint32_t p) {
    uint2 e = lds_entry(static_cast<uint32_t>(window64(ch, p)) & t.addr_mask);
    if (e.y == 0u) e = decode_long(t, window32(ch, p));
    return e;
}

// ---- two chunks per lane (blocks of 128 chunks decoded by one wavefront) ----

// Raw global words for the chunk pair (c, c+1), c = b*T + t, t even: their 16
// bytes (one 128-bit load), the next 4 bytes, the two 32-bit words holding
// Gaps[c], Gaps[c+1] and Gaps[c+2], and the block's two BlockOutputPos
// entries.
struct PairWords {
    uint32_t x0, x1, x2, x3, z, g0, g1, bp0, bp1;
};

template <uint32_t T>
__device__ __forceinline__ void load_pair_streams(const DecodeArgs &a, uint32_t b, uint32_t t,
                                                  PairWords &r) {
    static_assert(T % 64 == 0, "blocks start on whole words of Gaps");
    // EncodedExponent is only 8-byte aligned (its stated alignment), and the
    // type says so; the load stays one 16-byte load
    typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));
    const uint8_t *exp = a.exp + 8ull * T * b;
    const u32x4_a8 own = *reinterpret_cast<const u32x4_a8 *>(exp + 8u * t);
    r.x0 = own.x;
    r.x1 = own.y;
    r.x2 = own.z;
    r.x3 = own.w;
    r.z = *reinterpret_cast<const uint32_t *>(exp + 8u * t + 16u);
    const uint32_t *gaps = a.gaps + uint64_t{T / 64 * 10} * b;
    r.g0 = gaps[(5u * t) >> 5];
    r.g1 = gaps[((5u * t) >> 5) + 1u];
}

template <uint32_t T>
__device__ __forceinline__ PairWords load_pair(const DecodeArgs &a, uint32_t b, uint32_t t) {
    PairWords r;
    r.bp0 = block_positions(a)[b];
    r.bp1 = block_positions(a)[b + 1];
    load_pair_streams<T>(a, b, t, r);
    return r;
}

// Decode state of chunks c (ch[0]) and c+1 (ch[1]).  The second chunk's
// window words start at the pair's third word; their low 3 shifted-in bits
// come from the first chunk's bits and only ever sit below a window's table
// index, which is masked off.
template <uint32_t T>
__device__ __forceinline__ void pair_setup(const DecodeArgs &a, const PairWords &pw, uint32_t b,
                                           uint32_t t, Chunk (&ch)[2]) {
    const uint32_t w0 = lsb_first(pw.x0), w1 = lsb_first(pw.x1), w2 = lsb_first(pw.x2),
                   w3 = lsb_first(pw.x3), w4 = lsb_first(pw.z);
    ch[0].s0 = w0 << 3;
    ch[0].s1 = __builtin_amdgcn_alignbit(w1, w0, 29);
    ch[0].s2 = ch[1].s0 = __builtin_amdgcn_alignbit(w2, w1, 29);
    ch[0].w2 = w2;
    ch[1].s1 = __builtin_amdgcn_alignbit(w3, w2, 29);
    ch[1].s2 = __builtin_amdgcn_alignbit(w4, w3, 29);
    ch[1].w2 = w4;
    const uint64_t gv = ((static_cast<uint64_t>(__builtin_bswap32(pw.g0)) << 32) |
                         __builtin_bswap32(pw.g1))
                        << ((5u * t) & 31u);
    const uint32_t gap_a = static_cast<uint32_t>(gv >> 59);
    const uint32_t gap_b = static_cast<uint32_t>(gv >> 54) & 31u;
    const uint32_t gap_c = static_cast<uint32_t>(gv >> 49) & 31u;
    if ((b + 1u) * T < a.num_chunks) {  // every chunk of the block has a successor
        ch[0].start = gap_a;
        ch[0].end = 64u + gap_b;
        ch[1].start = gap_b;
        ch[1].end = 64u + gap_c;
    } else {
        chunk_range(a, b * T + t, gap_a, gap_b, ch[0]);
        chunk_range(a, b * T + t + 1u, gap_b, gap_c, ch[1]);
    }
}

// Phase 1 for the C chunks of a lane at once: decode the codes that start in
// each chunk, keep up to N lookups per chunk, and count the codes: out8[c] =
// 8 times the count, state[c] = the state where decoding stopped.  Each step
// takes one lookup of every chunk; the lookups are independent, so their LDS
// round trips overlap.
//
// A lookup's cost is the vector instructions of its chain, so the chain is
// kept short: the window is a 64-bit register shifted down by each entry's
// length (a 64-bit shift issues like a 32-bit one, and takes the length from
// the low bits of the metadata as they are) and refilled every five lookups,
// and position and count advance in one add.  Per lookup and chunk about 30
// cycles of issue against 70 with the window selected from the chunk's words
// by position each time and position, count and last lookup kept apart.
template <int N, int C>
__device__ __forceinline__ void decode_count(const Tables &t, const Chunk (&ch)[C],
                                             Trail<N> (&tr)[C], uint32_t (&state)[C],
                                             uint32_t (&out8)[C]) {
    uint64_t win[C];
    uint32_t acc[C], last[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        acc[c] = ch[c].start;
        last[c] = 0u;
        win[c] = (static_cast<uint64_t>(__builtin_amdgcn_alignbit(ch[c].s2, ch[c].s1, ch[c].start)) << 32) |
                 __builtin_amdgcn_alignbit(ch[c].s1, ch[c].s0, ch[c].start);  // start < 32
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int q = 0; q < (N + 3) / 4; ++q) tr[c].n8[q] = 0u;
    // selector that puts byte 1 of the first operand into byte k%4 of the second
    constexpr uint32_t sel[4] = {0x03020105u, 0x03020500u, 0x03050100u, 0x05020100u};
#pragma unroll
    for (int k = 0; k < N; ++k) {
        bool act[C];
        uint64_t acting[C], any = 0;  // one bit per lane
#pragma unroll
        for (int c = 0; c < C; ++c) {
            act[c] = state_pos(acc[c]) < ch[c].end;
            acting[c] = __builtin_amdgcn_ballot_w64(act[c]);
            any |= acting[c];
            tr[c].sy[k] = 0u;
        }
        if (any == 0) continue;  // wave-uniform skip
        uint2 e[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (k % kPerWindow == 0 && k > 0) win[c] = window64(ch[c], state_pos(acc[c]));
            e[c] = lds_entry(static_cast<uint32_t>(win[c]) & t.addr_mask);
        }
        uint64_t esc[C], any_esc = 0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            esc[c] = __builtin_amdgcn_ballot_w64(e[c].y == 0u) & acting[c];
            any_esc |= esc[c];
        }
        if (__builtin_expect(any_esc != 0, 0)) {  // wave-uniform
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (esc[c] != 0) decode_long_lanes(t, esc[c], window32(ch[c], state_pos(acc[c])), e[c]);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const uint32_t m = act[c] ? e[c].y : 0u;  // done chunks keep their state
            last[c] = act[c] ? m : last[c];
            acc[c] += m;
            tr[c].n8[k / 4] = __builtin_amdgcn_perm(m, tr[c].n8[k / 4], sel[k % 4]);
            tr[c].sy[k] = e[c].x;
            win[c] >>= e[c].y & 63u;
        }
        if (__builtin_expect(any_esc != 0, 0)) {  // a long code may use up the window
#pragma unroll
            for (int c = 0; c < C; ++c) win[c] = window64(ch[c], state_pos(acc[c]));
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        state[c] = acc[c];
        uint32_t st = acc[c];
        for (uint32_t it = 0; __builtin_expect(state_pos(st) < ch[c].end, 0) && it < 96u; ++it) {
            const uint2 e = lookup(t, ch[c], state_pos(st));
            last[c] = e.y;
            st += e.y;
        }
        // codes of the last lookup that start at or past `end` belong to the next chunk
        const uint32_t last_pos = state_pos(st) - (last[c] & 0xFFu);
        out8[c] = state_out8(st) -
                  8u * __builtin_popcount((last[c] >> kMetaMask) >> min(ch[c].end - last_pos, 31u));
    }
}

// Exponent buffer: the block's exponents start kBufLead bytes into it, so that
// the word below a store's first byte is always the buffer's own.
constexpr uint32_t kBufLead = 8;

// OR 4 exponent bytes into the zeroed buffer: their first byte goes to LDS
// bit offset q8 + 8 (a multiple of 8).  The word holding the byte below takes
// the low part shifted up by 32 - s bits and the next word the rest, with
// s = 24, 16, 8 or 0 = -(q8 + 8) mod 32; shifts and alignbit use the low five
// bits of their count, so no masking is needed, and s = 0 leaves the first
// word unchanged.
__device__ __forceinline__ void or_exponents(uint32_t q8, uint32_t syms) {
    const uint32_t s = 0u - 8u - q8;
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    lds_u32 *p = reinterpret_cast<lds_u32 *>(static_cast<uintptr_t>((q8 >> 3) & ~3u));
    __hip_atomic_fetch_or(p, __builtin_amdgcn_alignbit(syms, 0u, s), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or(p + 1, syms >> (s & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Phase 2: the chunk's exponents into the block's LDS buffer, buf_bytes long
// at LDS offset buf, from exponent off8/8 of the buffer on (the kept lookups,
// then the rest of a long chunk by decoding again).  The metadata fields hold
// at most 7 codes per lookup, so with the start clamped the kept lookups stay
// inside the buffer whatever the metadata and tables hold; the rest are
// clamped one by one.
template <int N>
__device__ __forceinline__ void emit_exponents(const Tables &t, const Chunk &ch, const Trail<N> &tr,
                                               uint32_t state, uint32_t off8, uint32_t buf,
                                               uint32_t buf_bytes) {
    const uint32_t base8 = 8u * (buf + kBufLead) - 8u;
    const uint32_t first8 = base8 + umin(off8, 8u * (buf_bytes - kBufLead - 8u - 8u * N));
    uint32_t q8 = first8;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const uint32_t n8 = (tr.n8[k / 4] >> (8 * (k % 4))) & 0xFFu;
        if (n8 != 0u) {
            or_exponents(q8, tr.sy[k]);
            q8 += n8;
        }
    }
    uint32_t st = state;
    for (uint32_t it = 0; __builtin_expect(state_pos(st) < ch.end, 0) && it < 96u; ++it) {
        const uint2 e = lookup(t, ch, state_pos(st));
        or_exponents(umin(first8 + state_out8(st), base8 + 8u * (buf_bytes - kBufLead - 8u)), e.x);
        st += e.y;
    }
}

// A block's output range, clamped to the buffer and the tensor.  Outputs
// are handled in 8-element groups aligned to the tensor: group g of the
// block covers buffer bytes [8g, 8g+8), i.e. outputs g0 + 8g .. g0 + 8g + 7;
// the block owns buffer bytes [shift, lim).  Only the first and the last
// group can be partial (shared with the neighbouring block): the groups
// [full_lo, full_hi) are whole.
struct Range {
    uint32_t s, shift, lim, g0, ngroups, full_lo, full_hi;
};

__device__ __forceinline__ Range block_range(const DecodeArgs &a, uint32_t bp0, uint32_t bp1) {
    Range r;
    r.s = umin(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(bp0)), a.n_elems);
    uint32_t e = umax(umin(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(bp1)), a.n_elems), r.s);
    // at most the buffer's worth; the room above r.s is clamped so the sum
    // cannot wrap for a stream ending near 2^32 weights
    e = umin(e, r.s + umin(a.buf_bytes - kBufSlack, 0xFFFFFFFFu - r.s));
    r.shift = r.s & 7u;
    r.lim = r.shift + (e - r.s);
    r.g0 = r.s - r.shift;
    r.ngroups = (r.lim + 7u) >> 3;
    r.full_lo = r.shift ? 1u : 0u;
    r.full_hi = umax(r.lim >> 3, r.full_lo);
    return r;
}

__device__ __forceinline__ Range block_range(const DecodeArgs &a, const ChunkWords &cw) {
    return block_range(a, cw.bp0, cw.bp1);
}

__device__ __forceinline__ bool full_group(const Range &r, uint32_t g) {
    return g - r.full_lo < r.full_hi - r.full_lo;  // full_lo <= g < full_hi
}

// Byte offset, from the block's first group on, of the sign/mantissa bytes
// and exponents of group first + k*step, clamped to the block's last group
// (twice that is the offset of its outputs).
template <int P>
struct Groups {
    uint32_t at[P];
};

template <int P>
__device__ __forceinline__ Groups<P> block_groups(const Range &r, uint32_t first, uint32_t step) {
    Groups<P> gr;
    const uint32_t last8 = 8u * (umax(r.ngroups, 1u) - 1u);
#pragma unroll
    for (int k = 0; k < P; ++k) gr.at[k] = umin(8u * first + 8u * step * k, last8);
    return gr;
}

// Sign/mantissa bytes of groups first, first+step, ... (P of them).  The
// buffer is zero padded past n_elems to a multiple of 16 bytes, so a whole
// group can be read even where the block starts or ends inside it.
template <int P>
__device__ __forceinline__ void prefetch_sm(const DecodeArgs &a, const Range &r,
                                            const Groups<P> &gr, uint2 (&S)[P]) {
    const uint8_t *sm = a.sm + r.g0;
#pragma unroll
    for (int k = 0; k < P; ++k) S[k] = *reinterpret_cast<const uint2 *>(sm + gr.at[k]);
}

// Edge elements: threads 0..7 take element t of the block's first group,
// threads 8..15 element t-8 of its last group.  Buffer byte of thread t's
// element (inside [0, 8*ngroups) whenever the block has a group).
__device__ __forceinline__ uint32_t edge_byte(const Range &r, uint32_t t) {
    return (t < 8u ? 0u : (umax(r.ngroups, 1u) - 1u) << 3) + (t & 7u);
}

// The sign/mantissa byte of this thread's edge element (threads 0..15),
// fetched when the block starts like the groups' bytes.
__device__ __forceinline__ uint32_t prefetch_edge_sm(const DecodeArgs &a, const Range &r,
                                                     uint32_t t) {
    uint32_t v = 0;
    if (t < 16u) v = a.sm[r.g0 + edge_byte(r, t)];
    return v;
}

// 8 outputs from their sign/mantissa bytes and rotated exponents.
__device__ __forceinline__ uint4 assemble_group(uint2 E, uint2 S) {
    uint4 o;
    assemble4(S.x, E.x, o.x, o.y);
    assemble4(S.y, E.y, o.z, o.w);
    return o;
}

// One 16-byte non-temporal store of a whole group (the output is written
// once and not read back by this kernel); `at`: the group's byte offset among
// the sign/mantissa bytes from the block's first group on.
__device__ __forceinline__ void store_group(uint16_t *out, uint32_t at, const uint4 &o) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 ov = {o.x, o.y, o.z, o.w};
    __builtin_nontemporal_store(
        ov, reinterpret_cast<u32x4 *>(reinterpret_cast<uint8_t *>(out) + (at + at)));
}

// Assemble and store every whole group of the block: groups first + k*step.
// The first P use the bytes fetched when the block started.  Loads and
// stores share one in-order counter on this GPU, so all of those groups are
// assembled (their loads waited for) before the first store is issued;
// otherwise each wait would also wait for the stores issued before it.  They
// are assembled without a check per group (a group past the block's last
// repeats it); only the stores are guarded.
// Then the elements of the (at most two) partial groups that this block
// owns go out as one 2-byte store instruction over threads 0..15.
template <int P>
__device__ __forceinline__ void assemble_block(const DecodeArgs &a, const Range &r,
                                               const uint8_t *buf, uint32_t first, uint32_t step,
                                               const Groups<P> &gr, const uint2 (&S)[P],
                                               uint32_t edge_sm) {
    uint16_t *out = a.out + r.g0;
    uint2 E[P];
#pragma unroll
    for (int k = 0; k < P; ++k) E[k] = *reinterpret_cast<const uint2 *>(buf + gr.at[k]);
    uint4 O[P];
#pragma unroll
    for (int k = 0; k < P; ++k) O[k] = assemble_group(E[k], S[k]);
#pragma unroll
    for (int k = 0; k < P; ++k)  // assembled here, not inside the guarded stores
        asm volatile("" : "+v"(O[k].x), "+v"(O[k].y), "+v"(O[k].z), "+v"(O[k].w));
#pragma unroll
    for (int k = 0; k < P; ++k) {
        // full_lo is 0 or 1, so only the first of a thread's groups can lie below it
        const uint32_t hi = r.full_hi - umin(r.full_hi, step * k);
        if (first < hi && (k > 0 || first >= r.full_lo)) store_group(out, gr.at[k], O[k]);
    }
    for (uint32_t g = first + P * step; g < r.full_hi; g += step)
        store_group(out, g << 3,
                    assemble_group(reinterpret_cast<const uint2 *>(buf)[g],
                                   *reinterpret_cast<const uint2 *>(a.sm + r.g0 + (g << 3))));
    if (first < 16u) {
        const uint32_t t = first;
        const uint32_t el = edge_byte(r, t);
        const uint32_t g = el >> 3;
        // the last group is taken by threads 8..15 only when it is not also the first
        const bool mine = r.ngroups != 0u && !full_group(r, g) && (t < 8u || g != 0u) &&
                          el >= r.shift && el < r.lim;
        if (mine) {
            const uint32_t e = buf[el];  // rotated: lowest bit at the top
            out[el] = static_cast<uint16_t>(((edge_sm & 0x80u) << 8) | ((e & 0x7Fu) << 8) |
                                            (e & 0x80u) | (edge_sm & 0x7Fu));
        }
    }
}

// Workgroups are dispatched to the 8 XCDs round robin and each XCD has its
// own L2.  Within every run of 32 workgroups this numbering gives the 4 that
// share an XCD neighbouring indices, so neighbouring blocks, which share the
// cache lines at their boundaries, are mostly decoded under one L2, while
// the blocks in flight still form one contiguous window of the stream.  A
// bijection of [0, n): a trailing partial run keeps its own numbers.
__device__ __forceinline__ uint32_t xcd_grouped_index(uint32_t g, uint32_t n) {
    constexpr uint32_t kXcds = 8u, kPer = 4u, kRun = kXcds * kPer;
    const uint32_t base = g - g % kRun;
    if (base + kRun > n) return g;
    return base + (g % kXcds) * kPer + (g % kRun) / kXcds;
}

// The blob into LDS: entries repacked, the long-code arrays as they are.
__device__ __forceinline__ void stage_table_blob(const DecodeArgs &a, uint8_t *lds, uint32_t tid,
                                                 uint32_t nthreads) {
    const uint4 *src = reinterpret_cast<const uint4 *>(a.tables);
    uint4 *dst = reinterpret_cast<uint4 *>(lds);
    const uint32_t entries = 1u << (a.lut_bits - 1u);  // 16-byte pieces: two entries each
    for (uint32_t i = tid; i < (a.table_lds_bytes >> 4); i += nthreads) {
        uint4 v = src[i];
        if (i < entries) {
            const uint2 e0 = pack_entry(v.x, v.y), e1 = pack_entry(v.z, v.w);
            v = make_uint4(e0.x, e0.y, e1.x, e1.y);
        }
        dst[i] = v;
    }
}

// ---- host side ------------------------------------------------------------

inline bool layout_supported(uint32_t T) {
    return T == 64 || T == 128 || T == 256 || T == 512 || T == 1024;
}

// Workgroups of `lds` bytes that a CU's LDS holds at once.  gfx950 hands LDS
// out in pieces of 1280 bytes; the occupancy query counts plain bytes, and a
// persistent grid one workgroup per CU too large runs in two unequal turns.
inline uint32_t lds_fit(uint32_t cu_lds, uint32_t lds) {
    constexpr uint32_t kPiece = 1280;
    return lds ? cu_lds / ((lds + kPiece - 1) / kPiece * kPiece) : ~0u >> 1;
}

inline uint32_t buf_bytes_for(uint32_t max_elems) {
    return (max_elems + kBufSlack + 15u) & ~15u;
}

inline int check_stream(const df11_stream *s) {
    if (!s) return DF11_E_INVALID_ARG;
    const df11_sizes &z = s->sizes;
    if (s->layout.bytes_per_thread != 8) return DF11_E_UNSUPPORTED;
    if (!layout_supported(s->layout.threads_per_block)) return DF11_E_UNSUPPORTED;
    if (s->layout.lut_bits < 8 || s->layout.lut_bits > 12) return DF11_E_INVALID_ARG;
    if (z.n_elems == 0) return DF11_OK;
    if (!s->exp || !s->sm || !s->gaps || !s->block_pos || !s->tables) return DF11_E_INVALID_ARG;
    if (z.n_elems > 0xFFFFFFFFull || z.num_blocks > 0xFFFFFFFFull / 1024) return DF11_E_INVALID_ARG;
    if (z.max_code_len > 32 || z.table_bytes != df11tab::blob_bytes(s->layout.lut_bits))
        return DF11_E_INVALID_ARG;
    const uint64_t T = s->layout.threads_per_block;
    if (z.exp_bytes < z.num_blocks * 8 * T + 16) return DF11_E_INVALID_ARG;
    if (z.gap_bytes < 4 * ((5 * (z.num_blocks * T + 1) + 31) / 32 + 2)) return DF11_E_INVALID_ARG;
    if (z.num_chunks > z.num_blocks * T) return DF11_E_INVALID_ARG;
    if (z.max_elems_per_block > 64u * T) return DF11_E_INVALID_ARG;
    if (z.sm_bytes < ((z.n_elems + 15) & ~uint64_t{15}) + 16) return DF11_E_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(s->sm) & 15u) || (reinterpret_cast<uintptr_t>(s->exp) & 7u) ||
        (reinterpret_cast<uintptr_t>(s->gaps) & 3u) || (reinterpret_cast<uintptr_t>(s->tables) & 15u) ||
        (reinterpret_cast<uintptr_t>(s->block_pos) & 3u))
        return DF11_E_INVALID_ARG;
    return DF11_OK;
}

}  // namespace df11dec
