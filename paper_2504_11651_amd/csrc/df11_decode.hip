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

        if (a.hold) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");  // as below, 5 loads
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
        // Vector memory operations complete in order: with the 8 loads of
        // sign/mantissa bytes just issued still out, the wave's stores are done,
        // and so are the loads of the next block's words that were issued before
        // those 8.  The wait for the latter is part of what "hold" measured.
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
// faster as long as they still cover the decode's latency.  How many that takes
// follows from the lookups per weight, that is from the mean code length against
// the table's index width K.  A stream of few blocks per wave takes more waves:
// its last round and the latency of each round dominate.
struct WaveRule {
    uint32_t per_simd;   // 0: every wave that fits
    bool hold;           // a wave waits for its stores, and its next block's words, before a block
    bool large = false;  // the largest workgroups of which two fit a CU, among equal counts
};

// Times in us on an MI355X by graph replay, streams rotating ("all": every
// wave that fits, 4 to 8; "h": with hold; "before": 4 to 6 per SIMD, when every
// wave decoded longer).  Codes / K is the mean code length over the index width.
//   weights   T   K  codes  codes/K  before   2      3      3h     4      4h     5      all
//   218.1 M  128 11  2.59    0.24     141.4  133.9  141.9  134.9  148.9  147.4
//   600.0 M  128 11  2.67    0.24     390.9  357.2  392.4  374.1  414.8  403.6
//   120.0 M  128 11  2.67    0.24      77.5   75.2   80.2   77.0
//   120.0 M  128 11  2.59    0.24      77.7   75.6   79.0   75.3
//   218.1 M  128 12  2.67    0.22     142.7  131.4  144.1  136.8  153.4  150.1
//   218.0 M  128 11  2.17    0.20     136.7  132.6  137.1  134.6  147.5  142.1
//   218.0 M  128 11  1.63    0.15     140.5  171.0  136.7  141.0  140.6  139.3
//   218.1 M  128 11  2.85    0.26     140.2  138.8  142.3  135.6  151.0  146.4
//    80.0 M  128 11  2.85    0.26      55.4   55.7   55.5   53.1   57.4   57.2
//   218.1 M  128 10  2.59    0.26     141.8  145.8  141.4  134.6  149.0  146.0
//   218.0 M  128 11  3.24    0.29     143.1  149.0  143.6  135.6  155.2  146.0
//   218.0 M  128 11  3.53    0.32     147.0  161.1  141.4  140.2  157.5  145.9
//   100.0 M  128 11  3.53    0.32      67.3   75.5   64.9   67.8   70.5   64.6
//   218.1 M  128  9  2.67    0.30     151.6  202.3  156.3  166.4  152.0  148.6
//   218.1 M  128  8  2.59    0.32     165.1  205.0  156.0  166.1  151.4  149.0
//   218.0 M  128 11  4.53    0.41     184.4  225.8  172.7  192.3  160.4  168.7
//   218.0 M  128 11  8.00    0.73     242.5  326.1  242.1  263.6  211.1  226.1
//   130.0 M  128 11  1.63    0.15      88.1  105.1   85.1   89.6   85.4   85.7
//    20.0 M   64 11  2.59    0.24      17.8          17.1          16.9   17.5   16.6   17.0
//    28.0 M   64 11  2.85    0.26      22.6          21.6          21.6   22.2   21.4   22.1
//    32.0 M   64 11  2.59    0.24      24.4          24.0          24.1   24.6   23.5   24.1
//    36.0 M   64 11  2.67    0.24      26.7          25.7          26.0   26.4   26.2   26.7
//    36.0 M   64 11  2.85    0.26      27.5          25.2          26.7   26.1   26.9   28.2
//    60.0 M   64 11  2.85    0.26      41.4          39.3          42.1   39.4   43.4   44.1
//   190.0 M   64 11  2.59    0.24     122.4  138.0  120.0  122.1  128.6  118.9  135.5  137.6
//   190.0 M   64 11  2.85    0.26     124.3  147.8  116.4  128.6  129.6  117.9  137.0  139.8
//   190.0 M   64  9  2.59    0.29     129.5  164.2  124.7  141.4  129.8  122.7  133.9  139.4
//    28.0 M   64  9  2.67    0.30      23.2          23.6          21.8   23.2   21.5   21.5
//    32.0 M   64  9  2.67    0.30      25.0          29.4          26.0   27.6   26.0   24.7
//    36.0 M   64  9  2.67    0.30      28.3          28.1          26.0   28.2   26.8   26.5
//    28.0 M   64 12  2.59    0.22      21.6          22.5          21.5   23.3          21.8
//    36.0 M   64 12  2.59    0.22      26.9          26.9          27.4   27.3          28.1
//    60.0 M   64 12  2.59    0.22      42.5          40.8          41.9   40.5          45.4
//   100.0 M   64 11  3.24    0.29      71.3   84.2   67.3   79.0   68.9   66.9   71.9   74.2
//   100.0 M   64 11  3.53    0.32      75.5   90.2   68.9   83.3   68.5   69.5   71.8   74.8
//   190.0 M   64  9  2.67    0.30     138.0  195.2  145.1  163.5  132.3  139.5  135.6  142.4
//   190.0 M   64  8  2.59    0.32     145.2  201.3  150.1  167.5  133.2  140.3  136.1  141.1
//   100.0 M   64 11  4.53    0.41      94.1  126.1   95.2  109.3   81.1   92.0   78.0   82.3
//   100.0 M   64 11  8.00    0.73     120.3  192.7  137.6  153.4  113.9  125.8  101.6   97.9
//   100.0 M   64 11  1.00    0.09      64.5   98.2   76.8   79.8   67.5   69.2          62.4
//   100.0 M   64 11  1.63    0.15      57.0   66.4   54.2   57.6   55.9   54.9   56.7   57.8
//   218.1 M  256 11  2.59    0.24     150.5  182.6  139.5         149.4         153.9  153.0
//   218.1 M  256 11  2.85    0.26     151.8  194.5  145.5         150.4         155.4  153.4
//   120.0 M  256 11  3.24    0.29      88.6  119.6   89.5          82.9          86.7   86.7
//   218.1 M  256  9  2.59    0.29     161.7  220.9  165.7         148.5         156.0  154.8
//   218.1 M  256  9  2.85    0.32     167.0  256.2  189.0         163.3         158.8  161.4
//   120.0 M  256 11  8.00    0.73     156.4  263.1  190.0         156.9         141.0  130.5
//   218.1 M  512 11  2.59    0.24     155.0  195.6                138.9                148.5
//   120.0 M  512 11  3.53    0.32      98.5  136.5                 90.1                 89.0
//   218.1 M  512  9  2.85    0.32     176.8  273.3                177.7                160.2
//   120.0 M  512 11  8.00    0.73     163.8  278.6                168.3                145.0
//   218.1 M 1024 11  2.59    0.24     152.8  170.4                                     147.9

// With 12-bit tables every workgroup copies 33 KB of them: short streams take
// few, large workgroups (us, before, 4-wave and 12-wave workgroups: 4.2 M
// weights 7.4, 8.2, 6.5; 16.8 M 15.9, 16.5, 15.1; 24 M of 2.85 bits, 4- and
// 8-wave ones 20.5, 19.7).

// Chunks per CU up to which a T = 64 stream is short (4.4 rounds of five waves'
// blocks), with 12-bit tables very short, and from which one of larger blocks
// is long (12 rounds of two waves on 128 chunks) or very long (40).
constexpr uint64_t kShortChunks = 5632, kVeryShortChunks = 3400, kLongChunks = 12288,
                   kVeryLongChunks = 40960;

WaveRule wave_rule(const df11_stream *s, uint64_t cus) {
    const df11_sizes &z = s->sizes;
    const uint64_t bits = z.total_bits, n = z.n_elems, K = s->layout.lut_bits;
    const uint32_t T = s->layout.threads_per_block;
    const bool is_long = z.num_chunks >= kLongChunks * cus;
    // lookups per weight: codes / K above a number of thousandths; an index of
    // 8 or 9 bits also meets more codes that are longer than it
    const auto above = [&](uint64_t thousandths) { return bits * 1000 > n * K * thousandths; };
    const bool more = above(K < 10 ? 290 : 330), many = above(400);
    if (T == 64) {
        const bool one = bits * 2 < n * 3;  // nearly one symbol: blocks of up to 4096 weights
        if (one || many) return {0u, false};
        const bool is_short = z.num_chunks <= kShortChunks * cus;
        if (K == 12 && is_short) return {z.num_chunks <= kVeryShortChunks * cus ? 0u : 4u, false, true};
        if (more) return {is_short ? 0u : 4u, false};
        return {is_short ? 5u : 3u, false};
    }
    if (!is_long || many) return {0u, false};
    if (T == 128) {
        if (more) return {4u, true};
        if (bits < n * 2) return {0u, false};
        // two waves cover the lookups of codes of 2.4 to 2.75 bits; shorter
        // codes make larger blocks, longer ones more lookups.  Above 2.62 bits
        // (several standard deviations in one block) only from 40 thousand chunks
        // per CU on: a decode that finds nothing of its stream and its output in
        // the caches waits for them with two waves.  2 waves and 3 with hold, us,
        // streams rotating and after 1 GiB of other reads: 218 M weights of 2.59
        // bits 131.4, 135.2 and 136.5, 135.1; of 2.64 136.0, 136.6 and 143.6,
        // 138.2; 260 M of 2.67 154.5, 159.6 and 160.1, 159.0.
        const bool mixed = bits * 50 > n * 131;
        const bool two = K > 10 && bits * 5 > n * 12 && bits * 4 < n * 11 &&
                         (!mixed || z.num_chunks >= kVeryLongChunks * cus);
        return two ? WaveRule{2u, false} : WaveRule{3u, true};
    }
    if (T == 256) return {above(275) ? 4u : 3u, false};
    if (T == 512) return {more ? 0u : 4u, false};
    return {0u, false};  // T = 1024: 4 per SIMD at most
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
                if (waves > best_waves || (rule.large && pc > 1 && waves == best_waves)) {
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
