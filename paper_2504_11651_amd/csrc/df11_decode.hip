// DFloat11 decompression on gfx950 (Algorithm 1 of arXiv 2504.11651,
// re-designed for CDNA4).
//
// A block of T chunks (the paper's "thread block") is decoded by one
// wavefront when T = 64 (a chunk per lane) or T = 128 (two adjacent chunks
// per lane, decoded as two interleaved lookup chains) -- the block's prefix
// sum is then a wave-level DPP scan and no workgroup barrier is needed, so
// the waves of a CU drift into different phases and decode overlaps memory
// streaming -- or, when T >= 256, by one workgroup: T threads with a chunk
// each (T = 256, 512), or T/2 threads whose waves take 128 of the chunks as
// lane pairs (T = 1024).  The grid is persistent:
// decode tables are staged into LDS once per workgroup and shared by all of
// its waves.
//
// Per block:
//   1. every lane loads its 8-byte chunk of EncodedExponent plus the next
//      4 bytes (or its two chunks' 16 bytes plus the next 4), and the 5-bit
//      Gaps of its chunks and of the next chunk;
//   2. phase 1 (count): starting at the gap, decode with the multi-symbol
//      table until the code start reaches the next chunk's first code;
//   3. exclusive scan of the counts (wave DPP scan, plus LDS across waves
//      for T >= 256) gives each lane its output position (Sec. 2.3.2);
//   4. phase 2 (emit): replay the lookups phase 1 kept in registers (a
//      chunk that needed more decodes its remaining codes again) and OR the
//      exponent bytes into an LDS buffer at their output positions.  The
//      waves of a CU run this phase at a higher priority than decoding, and
//      step 5 higher still.  A lookup may run past the lane's
//      last code; the extra codes are the next lanes' first codes, decoded
//      from the same bits, so they land on their own positions with their
//      own values and need no masking;
//   5. assemble BF16 = sign<<15 | exponent<<7 | mantissa (Algorithm 1) for
//      8 consecutive outputs per lane and step: one 8-byte PackedSignMantissa
//      load (issued when the block starts), one 8-byte LDS read, one 16-byte
//      store; consecutive lanes take consecutive groups, so a wave stores
//      1 KiB contiguous per instruction.  The block's first and last group
//      may be shared with its neighbours; their elements go out as one
//      2-byte store over 16 lanes.  No per-element gather (the paper
//      gathers sign/mantissa per element).
// Integer work only; no MFMA.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <vector>

#include "df11.h"
#include "df11_decode_core.h"
#include "df11_tables.h"

namespace {

using namespace df11dec;

// T = 64: every wave owns whole blocks; W waves per workgroup share the tables.
template <uint32_t W>
__global__ __launch_bounds__(64 * W) void df11_decode_wave_kernel(DecodeArgs a) {
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // block indices stay scalar
    const uint32_t first_block = xcd_grouped_index(blockIdx.x, gridDim.x) * W + wave;
    const uint32_t stride = gridDim.x * W;
    // the first block's words are requested before the tables are staged,
    // so the two memory round trips overlap
    ChunkWords cw{};
    if (first_block < a.num_blocks) cw = load_chunk<64>(a, first_block, lane);
    stage_table_blob(a, lds, tid, 64 * W);
    const uint32_t buf_off = a.table_lds_bytes + wave * a.buf_bytes;
    uint8_t *buf = lds + buf_off + kBufLead;
    __syncthreads();
    if (first_block >= a.num_blocks) return;
    const Tables tb = staged_tables(a, lds);
    Chunk ch[1] = {chunk_setup<64>(a, cw, first_block, lane)};
    Range r = block_range(a, cw);

    for (uint32_t b = first_block; b < a.num_blocks; b += stride) {
        // loads for this block's assembly and the next block's decode
        const uint32_t bn = b + stride;
        ChunkWords nxt = cw;
        if (bn < a.num_blocks) nxt = load_chunk<64>(a, bn, lane);
        const Groups<kPre> gr = block_groups<kPre>(r, lane, 64u);
        uint2 S[kPre];
        prefetch_sm(a, r, gr, S);
        const uint32_t edge_sm = prefetch_edge_sm(a, r, lane);

        if (a.hold) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");  // as below, 5 issued
        wave_lds_sync();  // this wave's reads of the previous block are issued
        for (uint32_t i = lane; i < (a.buf_bytes >> 4); i += 64u)
            reinterpret_cast<uint4 *>(lds + buf_off)[i] = make_uint4(0u, 0u, 0u, 0u);

        Trail<kKeep> tr[1];
        uint32_t state[1], out8[1];
        decode_count(tb, ch, tr, state, out8);
        const uint32_t excl8 = wave_inclusive_scan(out8[0]) - out8[0];
        // Waves near their memory phase issue first: the CU's decoding waves
        // (priority 0) fill the gaps, and the loads and stores of the waves
        // that have finished decoding reach the memory system sooner.
        __builtin_amdgcn_s_setprio(1);
        wave_lds_sync();
        emit_exponents(tb, ch[0], tr[0], state[0], 8u * r.shift + excl8, buf_off, a.buf_bytes);
        wave_lds_sync();

        __builtin_amdgcn_s_setprio(2);
        assemble_block(a, r, buf, lane, 64u, gr, S, edge_sm);
        __builtin_amdgcn_s_setprio(0);
        cw = nxt;
        ch[0] = chunk_setup<64>(a, cw, bn, lane);
        r = block_range(a, cw);
    }
}

// Sign/mantissa groups fetched at block start when a lane owns two chunks (a
// 128-chunk block holds about twice the outputs of a 64-chunk one).
constexpr int kPrePair = 7;

// T = 128: one wave per block as well, lane l owning chunks 2l and 2l+1 of
// it.  Its 16 bytes come in one 128-bit load, the two chunks decode
// interleaved (independent table lookups in flight together), and the
// block's count scan, buffer, edges and positions are shared by twice the
// outputs.
template <uint32_t W>
__global__ __launch_bounds__(64 * W) void df11_decode_pair_kernel(DecodeArgs a) {
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t first_block = xcd_grouped_index(blockIdx.x, gridDim.x) * W + wave;
    const uint32_t stride = gridDim.x * W;
    PairWords pw{};
    if (first_block < a.num_blocks) pw = load_pair<128>(a, first_block, 2u * lane);
    stage_table_blob(a, lds, tid, 64 * W);
    const uint32_t buf_off = a.table_lds_bytes + wave * a.buf_bytes;
    uint8_t *buf = lds + buf_off + kBufLead;
    __syncthreads();
    if (first_block >= a.num_blocks) return;
    const Tables tb = staged_tables(a, lds);
    Chunk ch[2];
    pair_setup<128>(a, pw, first_block, 2u * lane, ch);
    Range r = block_range(a, pw.bp0, pw.bp1);

    for (uint32_t b = first_block; b < a.num_blocks; b += stride) {
        const uint32_t bn = b + stride;
        PairWords nxt = pw;
        if (bn < a.num_blocks) nxt = load_pair<128>(a, bn, 2u * lane);
        const Groups<kPrePair> gr = block_groups<kPrePair>(r, lane, 64u);
        uint2 S[kPrePair];
        prefetch_sm(a, r, gr, S);
        const uint32_t edge_sm = prefetch_edge_sm(a, r, lane);
        // Vector memory operations complete in order: with the 8 just issued
        // still out, the wave's stores before them are done.  It holds back
        // nothing the block needs yet; it bounds what the wave has in flight.
        if (a.hold) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");

        wave_lds_sync();
        for (uint32_t i = lane; i < (a.buf_bytes >> 4); i += 64u)
            reinterpret_cast<uint4 *>(lds + buf_off)[i] = make_uint4(0u, 0u, 0u, 0u);

        Trail<kKeep> tr[2];
        uint32_t state[2], out8[2];
        decode_count(tb, ch, tr, state, out8);
        const uint32_t both8 = out8[0] + out8[1];
        const uint32_t off8 = 8u * r.shift + wave_inclusive_scan(both8) - both8;
        __builtin_amdgcn_s_setprio(1);
        wave_lds_sync();
        emit_exponents(tb, ch[0], tr[0], state[0], off8, buf_off, a.buf_bytes);
        emit_exponents(tb, ch[1], tr[1], state[1], off8 + out8[0], buf_off, a.buf_bytes);
        wave_lds_sync();

        __builtin_amdgcn_s_setprio(2);
        assemble_block(a, r, buf, lane, 64u, gr, S, edge_sm);
        __builtin_amdgcn_s_setprio(0);
        pw = nxt;
        pair_setup<128>(a, pw, bn, 2u * lane, ch);
        r = block_range(a, pw.bp0, pw.bp1);
    }
}

// T = 1024: one workgroup of T/2 threads per block, each wave decoding 128
// chunks as lane pairs like the kernel above.  The waves' counts meet in
// LDS, every wave ORs its exponents into one block buffer, and the workgroup
// assembles the block together.  Where LDS holds two block buffers they
// alternate between blocks: a buffer is cleared while the other is still
// being assembled, so a block needs two barriers (counts, then exponents).
// With one buffer, a third barrier waits for the previous block's assembly.
template <uint32_t T>
__global__ __launch_bounds__(T / 2) void df11_decode_block_pair_kernel(DecodeArgs a) {
    constexpr uint32_t NT = T / 2;
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    PairWords pw{};
    if (blockIdx.x < a.num_blocks) pw = load_pair<T>(a, blockIdx.x, 2u * tid);
    stage_table_blob(a, lds, tid, NT);
    uint32_t *wave_sums = reinterpret_cast<uint32_t *>(lds + a.table_lds_bytes);
    const uint32_t buf0 = a.table_lds_bytes + 4 * kScanSlots;
    __syncthreads();
    if (blockIdx.x >= a.num_blocks) return;
    const Tables tb = staged_tables(a, lds);
    Chunk ch[2];
    pair_setup<T>(a, pw, blockIdx.x, 2u * tid, ch);
    Range r = block_range(a, pw.bp0, pw.bp1);

    uint32_t parity = 0;
    for (uint32_t b = blockIdx.x; b < a.num_blocks; b += gridDim.x) {
        const uint32_t bn = b + gridDim.x;
        PairWords nxt = pw;
        if (bn < a.num_blocks) nxt = load_pair<T>(a, bn, 2u * tid);
        const Groups<kPrePair> gr = block_groups<kPrePair>(r, tid, NT);
        uint2 S[kPrePair];
        prefetch_sm(a, r, gr, S);
        const uint32_t edge_sm = prefetch_edge_sm(a, r, tid);

        // with two buffers this one was last read two blocks ago, before the
        // previous block's barriers
        if (!a.twin_bufs) __syncthreads();  // the previous block is assembled
        const uint32_t buf_off = buf0 + (a.twin_bufs ? parity : 0u) * a.buf_bytes;
        uint8_t *buf = lds + buf_off + kBufLead;
        for (uint32_t i = tid; i < (a.buf_bytes >> 4); i += NT)
            reinterpret_cast<uint4 *>(lds + buf_off)[i] = make_uint4(0u, 0u, 0u, 0u);

        Trail<kKeep> tr[2];
        uint32_t state[2], out8[2];
        decode_count(tb, ch, tr, state, out8);
        const uint32_t both8 = out8[0] + out8[1];
        const uint32_t incl = wave_inclusive_scan(both8);
        if (lane == 63u) wave_sums[wave] = incl;
        __syncthreads();  // every wave's count is in, the buffer is cleared
        uint32_t before = 0;
        for (uint32_t w = 0; w < wave; ++w) before += wave_sums[w];
        const uint32_t off8 = 8u * r.shift + before + incl - both8;
        emit_exponents(tb, ch[0], tr[0], state[0], off8, buf_off, a.buf_bytes);
        emit_exponents(tb, ch[1], tr[1], state[1], off8 + out8[0], buf_off, a.buf_bytes);
        __syncthreads();  // the block's exponents are all in the buffer

        assemble_block(a, r, buf, tid, NT, gr, S, edge_sm);
        parity ^= 1u;
        pw = nxt;
        pair_setup<T>(a, pw, bn, 2u * tid, ch);
        r = block_range(a, pw.bp0, pw.bp1);
    }
}

// T = 256, 512: one workgroup of T threads per block, a chunk per thread.
// (Two chunks per lane would halve the waves of a workgroup, and the tables
// staged per workgroup would then cap the waves per CU.)
template <uint32_t T>
__global__ __launch_bounds__(T) void df11_decode_block_kernel(DecodeArgs a) {
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = tid >> 6;
    stage_table_blob(a, lds, tid, T);
    uint32_t *wave_sums = reinterpret_cast<uint32_t *>(lds + a.table_lds_bytes);
    const uint32_t buf_off = a.table_lds_bytes + 4 * kScanSlots;
    uint8_t *buf = lds + buf_off + kBufLead;

    if (blockIdx.x >= a.num_blocks) return;
    ChunkWords cw = load_chunk<T>(a, blockIdx.x, tid);
    __syncthreads();
    const Tables tb = staged_tables(a, lds);
    Chunk ch[1] = {chunk_setup<T>(a, cw, blockIdx.x, tid)};
    Range r = block_range(a, cw);

    for (uint32_t b = blockIdx.x; b < a.num_blocks; b += gridDim.x) {
        const uint32_t bn = b + gridDim.x;
        ChunkWords nxt = cw;
        if (bn < a.num_blocks) nxt = load_chunk<T>(a, bn, tid);
        const Groups<kPre> gr = block_groups<kPre>(r, tid, T);
        uint2 S[kPre];
        prefetch_sm(a, r, gr, S);
        const uint32_t edge_sm = prefetch_edge_sm(a, r, tid);

        __syncthreads();  // the previous block's buffer is consumed
        for (uint32_t i = tid; i < (a.buf_bytes >> 4); i += T)
            reinterpret_cast<uint4 *>(lds + buf_off)[i] = make_uint4(0u, 0u, 0u, 0u);

        Trail<kKeep> tr[1];
        uint32_t state[1], out8[1];
        decode_count(tb, ch, tr, state, out8);

        const uint32_t incl = wave_inclusive_scan(out8[0]);
        if (lane == 63u) wave_sums[wave] = incl;
        __syncthreads();
        uint32_t before = 0;
        for (uint32_t w = 0; w < wave; ++w) before += wave_sums[w];
        emit_exponents(tb, ch[0], tr[0], state[0], 8u * r.shift + before + incl - out8[0], buf_off,
                       a.buf_bytes);
        __syncthreads();

        assemble_block(a, r, buf, tid, T, gr, S, edge_sm);
        cw = nxt;
        ch[0] = chunk_setup<T>(a, cw, bn, tid);
        r = block_range(a, cw);
    }
}

using KernelFn = void (*)(DecodeArgs);

struct LaunchShape {
    uint32_t threads, lut_bits, buf, most, large;  // key
    KernelFn fn;
    uint32_t block, lds, per_cu, waves_per_group, twin_bufs;
};

struct DeviceInfo {
    int cus = 0;
    int max_lds = 0;                 // bytes of LDS one workgroup may use
    uint32_t lds_granted[11] = {};   // dynamic LDS limit set per kernel instance (slot)
    std::vector<LaunchShape> shapes; // launch shapes already worked out
};

std::mutex g_mu;
std::vector<DeviceInfo> g_dev;

constexpr uint32_t kWaveChoices[4] = {4, 8, 12, 16};

// Waves per SIMD.  A stream's reads and writes are spread over every wave's
// block, and the more blocks are in flight at once the less of the memory's
// rate their mix reaches; fewer waves than the registers and LDS allow are
// faster as soon as they still cover the decode's latency.  Times in us on
// an MI355X, streams rotating so that none is cached; "before" is the same
// rule's line when every wave decoded longer and 4 to 6 per SIMD were best.
//   weights, T, mean code  before   2 waves   3 waves  3, hold   4 waves  4, hold   5 waves
//   855.6 M  128  2.69      562       519       565      542       595
//   300.0 M  128  2.59      192.2     176.0     194.1    185.5     204.7
//   218.1 M  128  2.59      140.1     130.2     142.1    134.3     149.2
//   218.1 M  128  2.64      140.3     135.4     142.3    134.6     149.8
//    91.7 M  128  2.64       59.3      60.6      58.7     57.4      61.6
//   218.1 M  128  2.85      140.7     138.6     142.5    135.1     150.7
//    80.0 M  128  2.59       52.7      51.2      53.8     51.5      54.4
//    67.0 M  128  2.59       44.9      46.9      46.2               44.6
//    16.0 M  128  2.59       14.6      15.7      13.4               13.2
//   190.0 M   64  2.59      121.5     150         118.5             126.9    118.3     134.3
//   100.0 M   64  2.85       66.2                  62.3             68.6     63.9      71.7
//    50.0 M   64  2.85       30.6                  31.3             32.5     29.4      32.7
//    50.0 M   64  2.59       31.0                  29.2             31.7               32.9
//    24.0 M   64  2.59       16.8                  16.9             17.2     16.8      17.5
//    20.0 M   64  2.85       15.7                  16.1             14.9               15.2
//    16.8 M   64  2.59       13.1      17.0        13.7             13.0     13.2      12.7
//   329.3 M  256  2.59      222.6                 206.1            226.3
//   120.0 M  256  2.59       83.5     102          77.8             83.1               84.4
//   218.1 M  256  2.64      150.5                                  149.9
//   120.0 M  256  2.85       84.7     114          84.8             83.1               87.2
//   120.0 M  512  2.59       86.3     108                           78.6               78.7
// "hold": a wave waits for its stores before it starts the next block.  With
// longer codes the lookups per weight grow and two waves no longer cover them;
// a third one that holds does, without as many blocks in flight.
// A stream of few blocks per wave takes more waves instead: its last round
// and the latency of each round dominate.
struct WaveRule {
    uint32_t per_simd;   // 0: every wave that fits
    bool hold;
    bool large = false;  // T <= 128: among equal counts the largest workgroups
};

// Chunks per CU up to which a T = 64 stream takes 5 waves (2.65 rounds of
// blocks), then 4 with hold (until 4.6 rounds of them, with long codes until
// a stream is long), and from which a stream is long (12 rounds of two waves
// on 128 chunks) or very long.
constexpr uint64_t kFiveWaves = 3400, kFourWaves = 4725, kLongChunks = 12288,
                   kVeryLongChunks = 65536;

WaveRule wave_rule(const df11_stream *s, uint64_t cus) {
    const df11_sizes &z = s->sizes;
    const uint32_t T = s->layout.threads_per_block;
    const bool long_codes = z.total_bits > z.n_elems * 11 / 4;  // mean above 2.75 bits
    if (T == 64) {
        // 33 KB of tables per workgroup: a short stream takes few, large ones
        // (us, before, 4-wave and 12-wave workgroups: 4.2 M weights 7.4, 8.2,
        // 6.5; 16.8 M 15.9, 16.5, 15.1; 24 M 19.2, 20.4, 17.8)
        if (s->layout.lut_bits == 12 && z.num_chunks <= kFourWaves * cus) return {0u, false, true};
        if (z.num_chunks <= kFiveWaves * cus) return {5u, false};
        if (z.num_chunks <= (long_codes ? kLongChunks : kFourWaves) * cus) return {4u, true};
        return {3u, false};
    }
    if (z.num_chunks < kLongChunks * cus) return {0u, false};
    const bool mixed = z.total_bits * 50 > z.n_elems * 131;  // mean above 2.62 bits
    if (T == 128) {
        const bool three = long_codes || (mixed && z.num_chunks < kVeryLongChunks * cus);
        return {three ? 3u : 2u, three};
    }
    if (T == 256 && !mixed) return {3u, false};
    return {4u, false};
}

constexpr size_t kMaxShapes = 64;  // cached launch shapes per device

KernelFn wave_kernel(uint32_t W) {
    switch (W) {
        case 4: return df11_decode_wave_kernel<4>;
        case 8: return df11_decode_wave_kernel<8>;
        case 12: return df11_decode_wave_kernel<12>;
        case 16: return df11_decode_wave_kernel<16>;
        default: return nullptr;
    }
}

KernelFn pair_kernel(uint32_t W) {
    switch (W) {
        case 4: return df11_decode_pair_kernel<4>;
        case 8: return df11_decode_pair_kernel<8>;
        case 12: return df11_decode_pair_kernel<12>;
        case 16: return df11_decode_pair_kernel<16>;
        default: return nullptr;
    }
}

// Slots of lds_granted: 0-3 wave kernels, 4-7 pair kernels, 8-10 below.
KernelFn block_kernel(uint32_t T, int *slot) {
    switch (T) {
        case 256: *slot = 8; return df11_decode_block_kernel<256>;
        case 512: *slot = 9; return df11_decode_block_kernel<512>;
        case 1024: *slot = 10; return df11_decode_block_pair_kernel<1024>;
        default: return nullptr;
    }
}

// Lets a kernel use `lds` bytes of dynamic LDS and returns how many of its
// workgroups fit on one CU (0 when none does).
int fit(DeviceInfo &di, int slot, KernelFn fn, uint32_t threads, uint32_t lds, int *per_cu) {
    *per_cu = 0;
    if (lds > static_cast<uint32_t>(di.max_lds)) return DF11_OK;
    if (lds > 65536u && di.lds_granted[slot] < lds) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(lds)) != hipSuccess)
            return DF11_E_HIP;
        di.lds_granted[slot] = lds;
    }
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, reinterpret_cast<const void *>(fn),
                                                     static_cast<int>(threads), lds) != hipSuccess)
        return DF11_E_HIP;
    *per_cu = std::min(*per_cu, static_cast<int>(lds_fit(static_cast<uint32_t>(di.max_lds), lds)));
    return DF11_OK;
}

int shape_for(const df11_stream *s, KernelFn *fn, uint32_t *grid, uint32_t *block, uint32_t *lds,
              uint32_t *twin_bufs, uint32_t *hold) {
    const uint32_t T = s->layout.threads_per_block;
    const uint32_t K = s->layout.lut_bits;
    const uint32_t tab = static_cast<uint32_t>(df11tab::lds_bytes(K));
    const uint32_t buf = buf_bytes_for(s->sizes.max_elems_per_block);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return DF11_E_HIP;
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_dev.size() <= static_cast<size_t>(dev)) g_dev.resize(dev + 1);
    DeviceInfo &di = g_dev[dev];
    if (!di.cus) {
        if (hipDeviceGetAttribute(&di.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipDeviceGetAttribute(&di.max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
                hipSuccess)
            return DF11_E_HIP;
    }
    const WaveRule rule = wave_rule(s, static_cast<uint64_t>(di.cus));
    const uint32_t most = 4u * (rule.per_simd ? rule.per_simd : 16u);  // waves per CU; 4 SIMDs
    const LaunchShape *found = nullptr;
    for (const LaunchShape &ls : di.shapes)
        if (ls.threads == T && ls.lut_bits == K && ls.buf == buf && ls.most == most &&
            ls.large == rule.large)
            found = &ls;
    if (!found) {
        LaunchShape ls{T, K, buf, most, rule.large, nullptr, 0, 0, 0, 1, 0};
        if (T == 64 || T == 128) {
            // one wave per block: the workgroup size that comes nearest to the
            // rule's waves per CU from below; on a tie as the rule says
            int best_waves = 0;
            for (int i = 0; i < 4; ++i) {
                const uint32_t W = kWaveChoices[i];
                const KernelFn fn = T == 64 ? wave_kernel(W) : pair_kernel(W);
                int pc = 0;
                int rc = fit(di, T == 64 ? i : 4 + i, fn, 64 * W, tab + W * buf, &pc);
                if (rc) return rc;
                pc = std::min(pc, static_cast<int>(most / W));
                const int waves = pc * static_cast<int>(W);
                if (waves > best_waves || (rule.large && waves > 0 && waves == best_waves)) {
                    best_waves = waves;
                    ls.fn = fn;
                    ls.block = 64 * W;
                    ls.lds = tab + W * buf;
                    ls.per_cu = static_cast<uint32_t>(pc);
                    ls.waves_per_group = W;
                }
            }
            if (!best_waves) return DF11_E_UNSUPPORTED;
        } else if (T == 1024) {
            int slot = 0, pc = 0;
            ls.fn = block_kernel(T, &slot);
            ls.block = T / 2;
            ls.twin_bufs = 1;
            ls.lds = tab + 4 * kScanSlots + 2 * buf;  // two block buffers
            int rc = fit(di, slot, ls.fn, T / 2, ls.lds, &pc);
            if (rc) return rc;
            if (pc < 1) {  // one buffer (very compressible streams: large blocks)
                ls.twin_bufs = 0;
                ls.lds = tab + 4 * kScanSlots + buf;
                rc = fit(di, slot, ls.fn, T / 2, ls.lds, &pc);
                if (rc) return rc;
            }
            if (pc < 1) return DF11_E_UNSUPPORTED;
            ls.per_cu = static_cast<uint32_t>(pc);
        } else {
            int slot = 0, pc = 0;
            ls.fn = block_kernel(T, &slot);
            ls.block = T;
            ls.lds = tab + 4 * kScanSlots + buf;
            int rc = fit(di, slot, ls.fn, T, ls.lds, &pc);
            if (rc) return rc;
            if (pc < 1) return DF11_E_UNSUPPORTED;
            ls.per_cu = static_cast<uint32_t>(pc);
        }
        // (a workgroup of T >= 256 is a block: at least one, whatever the rule)
        ls.per_cu = std::min(ls.per_cu, std::max(most * 64u / ls.block, 1u));
        if (di.shapes.size() >= kMaxShapes) di.shapes.erase(di.shapes.begin());  // oldest goes
        di.shapes.push_back(ls);
        found = &di.shapes.back();
    }
    *fn = found->fn;
    *block = found->block;
    *lds = found->lds;
    *twin_bufs = found->twin_bufs;
    const uint64_t W = found->waves_per_group;
    const uint64_t nb = s->sizes.num_blocks;
    const uint64_t blocks_needed = (nb + W - 1) / W;
    *hold = rule.hold;
    uint64_t g = static_cast<uint64_t>(di.cus) * found->per_cu;
    if (g > blocks_needed) g = blocks_needed;
    *grid = static_cast<uint32_t>(g ? g : 1);
    return DF11_OK;
}

}  // namespace

extern "C" {

int df11_decode_launch_shape(const df11_stream *s, uint32_t *grid, uint32_t *block,
                             uint32_t *lds_bytes) {
    int rc = check_stream(s);
    if (rc) return rc;
    if (!grid || !block || !lds_bytes) return DF11_E_INVALID_ARG;
    KernelFn fn;
    uint32_t twin, hold;
    return shape_for(s, &fn, grid, block, lds_bytes, &twin, &hold);
}

int df11_decode_block(const df11_stream *s, uint16_t *out, hipStream_t stream) {
    int rc = check_stream(s);
    if (rc) return rc;
    if (s->sizes.n_elems == 0) return DF11_OK;
    if (!out || (reinterpret_cast<uintptr_t>(out) & 15u)) return DF11_E_INVALID_ARG;
    KernelFn fn;
    uint32_t grid, block, lds, twin, hold;
    rc = shape_for(s, &fn, &grid, &block, &lds, &twin, &hold);
    if (rc) return rc;
    DecodeArgs a;
    a.exp = s->exp;
    a.sm = s->sm;
    a.gaps = reinterpret_cast<const uint32_t *>(s->gaps);
    a.block_pos = s->block_pos;
    a.tables = s->tables + df11tab::kHeaderBytes;
    a.out = out;
    a.total_bits = s->sizes.total_bits;
    a.n_elems = static_cast<uint32_t>(s->sizes.n_elems);
    a.num_chunks = static_cast<uint32_t>(s->sizes.num_chunks);
    a.num_blocks = static_cast<uint32_t>(s->sizes.num_blocks);
    a.lut_bits = s->layout.lut_bits;
    a.max_len = s->sizes.max_code_len;
    a.table_lds_bytes = static_cast<uint32_t>(df11tab::lds_bytes(s->layout.lut_bits));
    a.buf_bytes = buf_bytes_for(s->sizes.max_elems_per_block);
    a.twin_bufs = twin;
    a.hold = hold;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), lds, stream, a);
    return hipGetLastError() == hipSuccess ? DF11_OK : DF11_E_HIP;
}

}  // extern "C"
