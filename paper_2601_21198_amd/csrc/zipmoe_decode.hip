// Device side of libzipmoe: zm_decode_experts and its gfx950 kernels.
//
// One launch decodes every tensor of the experts a MoE layer's gate selected
// (ZipMoE, arXiv 2601.21198, Sec. 3.1 "Real-time Inference"): each wavefront
// takes one stream of one E-chunk, entropy-decodes its exponent bytes and merges
// them with the raw sign-mantissa bytes into bf16 words (the tensor recovery
// step of Sec. 3.3) without the exponents ever leaving registers.
//
// Work decomposition
//   grid    x: workgroups of kWaves consecutive streams, y: tensor (or x through all tensors)
//   wave    one stream: stream_values consecutive values, tiles of 512 (or eight tiles of several short streams, decode_bundle)
//   lane j  owns values 8j..8j+7 of every tile: one 64-bit load of
//           sign-mantissa bytes and one 128-bit store of bf16 words per tile,
//           both contiguous across the wave (512 B and 1 KiB per instruction)
//
// Per wave
//   1. one read of the chunk's table entry locates the stream, and the decode table is requested meanwhile; the stream's bytes (64
//      lane-length bytes, then the 64 lane bitstreams back to back) are requested with 128-bit loads (a4), because
//      decoding can not start without them, and go to LDS;
//   2. the sign-mantissa bytes of the stream's first tiles are requested behind them, the others as tiles are finished;
//   3. the decode table goes to LDS (a3) as 16-bit entries, code length in the low bits and symbol where a bf16 word has it:
//      256 entries for codes of at most eight bits; longer codes take 16 more for each beginning that they share;
//   4. a wavefront prefix sum over the 64 lane-length bytes gives every lane the first and the last bit of
//      its own bitstream (a6): what varies from lane to lane is where its input lies, its output positions
//      are fixed;
//   5. lock-step decode (a5): a lane's bitstream holds the first half of its symbols from its first bit upwards
//      and the second half, last symbol first, from its last bit downwards, so every lane runs two independent
//      decode chains at once (the lookups of one overlap the latency of the other).  Per chain it keeps two
//      words of the bitstream, a bit position and the index of its next word; per round it extracts a 32-bit
//      window with one funnel shift (one chain reads reversed bits) and decodes four symbols by table lookup, or
//      two where longer codes do not fit; the next word is requested at the start of the round, so that a chain that crosses a word
//      boundary finds it there;
//   6. the eight decoded entries are merged with the sign-mantissa bytes
//      by byte-parallel bit operations and stored (a8).
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "zipmoe.h"
#include "zipmoe_extent.h"
#include "zipmoe_kinds.h"

namespace {

using namespace zipmoe;

constexpr int kMaxTensorsPerCall = 256;
constexpr int kMaxTasks = 48;     // tensors per launch; 84 B each keeps the kernel arguments under 4 KiB
constexpr int kFewTasks = 6;      // tensors of a launch with small arguments: two experts of three matrices
constexpr int kRawBuffer = 0x00027000;   // last word of a descriptor of untyped memory

// One tensor to decode.  Its parts may live in separate allocations (a cache may keep only some of them
// resident), so each has a pointer of its own.
struct Task {
    const uint8_t *lut;       // decode table: 2^max_len entries of 16 bits
    const uint8_t *sm;        // sign-mantissa section
    const uint8_t *echunks;   // E-chunk region (what the blob holds from e_offset on)
    const uint64_t *table;    // chunk table (entries of 8 + 4*(streams_per_chunk+1) bytes, rounded up to 8); offsets count from the start of the blob
    uint16_t *out;
    uint64_t e_offset;        // blob offset of the E-chunk region
    uint64_t e_size;          // bytes in the E-chunk region
    uint32_t stream_values;
    uint32_t streams_per_chunk;
    uint32_t per_chunk;       // reciprocal of streams_per_chunk, see chunk_of
    uint32_t n_streams;
    uint32_t last_values;     // values of the last stream
    uint32_t code;            // longest code length | shift of the reciprocal << 4 | lane quantum << 9
};
__host__ __device__ constexpr uint32_t max_len_of(uint32_t code) { return code & 15u; }
__host__ __device__ constexpr uint32_t quantum_of(uint32_t code) { return code >> 9; }

// The chunk that stream g lies in, g / streams_per_chunk: with 2^k the next power of two from the divisor on, r = ceil(2^(31+k) / divisor)
// is below 2^32 and exact for every g < 2^31.  (The compiler's division by a value it does not know goes through the
// floating-point reciprocal, 30 instructions in front of a wave's first read.)
__device__ __forceinline__ uint32_t chunk_of(uint32_t g, uint32_t per_chunk, uint32_t code)
{
    return __umulhi(2u * g, per_chunk) >> (code >> 4 & 31u);
}

// Kernel arguments of a launch of up to N tensors.  The runtime copies all of them, used or not, into the device's
// memory for every launch, so a launch of few tensors takes a smaller kind: one matrix of 256 x 512 called again and again
// 7.2 us with 4 KB, 6.9 with 0.5, waited for every time 21.6 and 16.5; three of 2048 x 1408 8.7 and 8.5.  (Those that are whole blobs
// cut alike a smaller one still, Few.)
// grid: x = workgroup inside the tensor, y = tensor.  kFlat, for tensors of very different lengths: x counts through
// the workgroups of all tensors, first_block[k] being the first one of tensor k.  (A kind of its own: a flag among the
// arguments would be one more read that every wave waits for.)
template <int N, bool kFlat>
struct Launch {
    uint32_t n_tasks;
    uint32_t stream_cap_words;   // LDS words reserved per wave for its stream
    uint32_t long_slots;         // long codes: shared eight-bit beginnings that the LDS table has room for
    uint32_t pad;
    Task task[N];
    uint32_t first_block[kFlat ? N : 1];
};
static_assert(sizeof(Launch<kMaxTasks, true>) <= 4096, "kernel arguments must stay under 4 KiB");
static_assert(kMaxTasks <= 64, "a wave finds its tensor with one value per lane");

// What the tensors of one shape share, and what is left of a tensor: 16 bytes, so that a launch takes five times as many.
struct Shape {
    uint64_t sm_offset, e_offset;
    uint32_t lut_offset, table_offset;
    uint32_t stream_values, streams_per_chunk, per_chunk, n_streams, last_values, code;
};
struct Packed {
    uint32_t blob;       // bits 4..35 of the blob's address
    uint32_t high;       // bits 36..47 of the blob's address, 8 bits of shape number, bits 36..47 of the output's address
    uint32_t out;        // bits 4..35 of the output's address
    uint32_t e_units;    // bytes in the E-chunk region / 256
};
constexpr int kMaxPacked = 240, kMaxShapes = 4;
// Values per tensor, on average, from which on a call's tensors travel that way.  It would pay below as well: 100 tensors of
// 50000 values 14.0 us in launches of 48, 7.1 in one; 192 of 8192 19.3 and 9.5.  The line keeps the number of launches that
// zm_decode_launch_shapes tells of for smaller tensors.
constexpr uint64_t kPackedValues = 1u << 16;
struct PackedLaunch {
    uint32_t n_tasks;
    uint32_t stream_cap_words;
    uint32_t long_slots;
    uint32_t pad;
    Packed task[kMaxPacked];
    Shape shape[kMaxShapes];
};
static_assert(sizeof(PackedLaunch) <= 4096, "kernel arguments must stay under 4 KiB");

// Up to six blobs cut alike, in 112 bytes, because the host takes longer for a launch with more: 2.75 us up to 112 B, 3.45 from 116 B on,
// 4.2 with 4 KB (a kernel that does nothing).  Prepared calls from Python, in turn in one process: one tensor 3.8 -> 3.55 us, three 4.1 ->
// 3.65, six 4.2 -> 3.75 against a Launch<6>.  Unpacking them costs a wave a few scalar instructions: one matrix of 256 x 512 3.88 -> 3.92 us
// on the GPU.  (With the first 56 bytes preloaded into scalar registers, so that a wave's first read is the chunk table's, launches
// of many short waves were slower than with reads: 4096 streams of 512 values 3.65 -> 3.75 us.)
struct Few {
    // [0] stream_values / 512 | longest code length << 7 | log2 of streams_per_chunk << 11 | lane quantum << 16 | long_slots << 24
    // [1] n_streams  [2] last_values | lut_offset << 16  [3] table_offset  [4] sm_offset / 256  [5] e_offset / 256
    uint32_t lead[6];
    const uint8_t *low;            // the lowest blob
    uint32_t to[kFewTasks];        // from there to tensor k's, / 256
    uint16_t *out;                 // the lowest output
    uint32_t to_out[kFewTasks];    // from there to tensor k's, / 16
    uint32_t e_units[kFewTasks];   // bytes in the E-chunk region / 256
};
static_assert(sizeof(Few) == 112 && offsetof(Few, out) == 56);

// The tensor that a workgroup works on and the workgroup's number inside the tensor.
template <int N, bool kFlat>
__device__ __forceinline__ Task task_of(const Launch<N, kFlat> &P, uint32_t lane, uint32_t &block)
{
    uint32_t k = blockIdx.y;
    block = blockIdx.x;
    if constexpr (kFlat) {
        // every lane looks at one tensor's first workgroup; those that start at or before this one are the first k + 1
        const uint32_t first = lane < P.n_tasks ? P.first_block[lane] : ~0u;
        k = static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(first <= blockIdx.x))) - 1u;
        block = blockIdx.x - static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(first), static_cast<int>(k)));
    }
    return P.task[k];            // one batch of scalar loads
}

__device__ __forceinline__ Task task_of(const PackedLaunch &P, uint32_t, uint32_t &block)
{
    block = blockIdx.x;
    const Packed p = P.task[blockIdx.y];
    const Shape s = P.shape[(p.high >> 12) & (kMaxShapes - 1u)];
    const uint8_t *blob = reinterpret_cast<const uint8_t *>(static_cast<uint64_t>(p.blob) << 4 | static_cast<uint64_t>(p.high & 0xfffu) << 36);
    uint16_t *out = reinterpret_cast<uint16_t *>(static_cast<uint64_t>(p.out) << 4 | static_cast<uint64_t>(p.high >> 20) << 36);
    return Task{blob + s.lut_offset, blob + s.sm_offset, blob + s.e_offset, reinterpret_cast<const uint64_t *>(blob + s.table_offset), out,
                s.e_offset, static_cast<uint64_t>(p.e_units) * 256u, s.stream_values, s.streams_per_chunk, s.per_chunk, s.n_streams, s.last_values, s.code};
}

// LDS words of a table of long codes with `slots` shared beginnings (LongTable), a multiple of four
__host__ __device__ constexpr uint32_t long_table_words(uint32_t slots)
{
    return (256u + ((1u << (ZM_MAX_CODE_LEN - 8)) - 1u) * slots + 7u) / 8u * 4u;
}

// LDS words a wave reserves for one stream of the launch's longest kind: the length bytes, the code bits
// of a lane bounded by the longest code, the rounding of every lane to the quantum, the padding to 16 bytes,
// and two words a lane may read past its last one.
template <class Words>
__host__ __device__ constexpr Words stream_cap_words(Words stream_values, uint32_t max_len_bound, uint32_t quantum)
{
    return (kLaneBytes + 8u * (stream_values / 64u * max_len_bound + quantum) + 16u + 8u + 15u) / 16u * 4u;
}

// Exclusive prefix sum of x over the 64 lanes of the wave (a6), by data-parallel primitives: an inclusive
// scan inside each row of 16 lanes (shifts by 1, 2, 4, 8), then lane 15 of row 0 and 2 is added to the next
// row, then lane 31 to rows 2 and 3.  Lanes with no source keep the `old` operand, zero.
__device__ __forceinline__ uint32_t wave_exclusive_sum(uint32_t x)
{
    uint32_t v = x;
    v += __builtin_amdgcn_update_dpp(0u, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0u, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0u, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0u, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return v - x;
}

// Sec. 3.3 recovery of four values at once: e4 and sm4 hold four exponent bytes
// and four sign-mantissa bytes; the results are the four bf16 words, two per register.
__device__ __forceinline__ void recover4(uint32_t e4, uint32_t sm4, uint32_t &w01, uint32_t &w23)
{
    const uint32_t hi4 = (sm4 & 0x80808080u) | ((e4 >> 1) & 0x7F7F7F7Fu);   // s eeeeeee
    const uint32_t lo4 = ((e4 << 7) & 0x80808080u) | (sm4 & 0x7F7F7F7Fu);   // e mmmmmmm
    w01 = __builtin_amdgcn_perm(hi4, lo4, 0x05010400u);
    w23 = __builtin_amdgcn_perm(hi4, lo4, 0x07030602u);
}

// Where they go: the first n_values of stream_base, lane j's eight words of tile k at k * kTile + 8 * j.  Buffer stores,
// because 128-bit device-scope stores exist as these only; the descriptor covers the wave's words and nothing else.
template <Stores kStores>
struct Sink {
    __amdgpu_buffer_rsrc_t words;
    uint32_t lane_offset;
    // stream_base and n_values are the same for all lanes
    __device__ __forceinline__ Sink(uint16_t *stream_base, uint32_t n_values, uint32_t lane)
        : words(__builtin_amdgcn_make_buffer_rsrc(stream_base, 0, static_cast<int>(2u * n_values), kRawBuffer)),
          lane_offset(lane * 16u) {}

    __device__ __forceinline__ void store(uint32_t tile, uint4 w) const
    {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        constexpr int kFlags = kStores == kStreaming ? 2 : kStores == kThrough ? 16 : 0;      // the instruction's nt and sc1 bits
        __builtin_amdgcn_raw_buffer_store_b128((u32x4){w.x, w.y, w.z, w.w}, words, static_cast<int>(lane_offset + tile * (2u * kTile)), 0, kFlags);
    }

    // for a lane that owns fewer than eight values of the tile: one word at a time, and those past the end of the
    // stream are past the end of the descriptor too, which drops them
    __device__ __forceinline__ void store_partial(uint32_t tile, uint4 w) const
    {
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q)
            __builtin_amdgcn_raw_buffer_store_b16(static_cast<uint16_t>(ws[q >> 1] >> (16 * (q & 1))), words,
                                                  static_cast<int>(lane_offset + tile * (2u * kTile) + 2u * q), 0, 0);
    }
};

__device__ __forceinline__ uint4 recover8(uint2 e, uint2 sm)
{
    uint4 w;
    recover4(e.x, sm.x, w.x, w.y);
    recover4(e.y, sm.y, w.z, w.w);
    return w;
}

constexpr uint32_t kTableEntries = 256;   // the LDS table of codes of at most eight bits resolves them all at once

// The LDS table of a tensor whose codes have up to L = 9..12 bits.  Take the next L bits of a stream as a number v, first
// bit highest.  The canonical code orders them by length: beginnings of eight bits that longer codes share come last.
// With T beginnings that decide the code by themselves, the table holds one entry for each of these and then the
// 2^(L-8) entries of every other beginning, and the entry of v is max(v >> (L-8), v - skip): up to T the first term is the
// larger one, from there on the second, and they meet in T.  So a code of any length takes one LDS read and no branch.
// (Before, the table held the 256 beginnings, and a wave in which one lane met a long code, one step in two, branched to
// a second look-up; and a window was refilled after every two symbols.  One / two / four / eight experts of 1024 x 2048 x 3
// with codes of up to 12 bits, streaming stores, inputs in the last-level cache: 9.5 / 13.2 / 19.8 / 31.8 us then,
// 7.0 / 9.8 / 15.6 / 27.8 us now.)
// At most half as many beginnings are shared as there are symbols: each by two codes or more.  The table has room for that
// many; where a description counts fewer symbols than the blob's table has, codes are looked up in that one.
struct LongTable {
    uint32_t shift;      // 32 - L
    int32_t skip;        // (T << (L-8)) - T

    // bits: what is left of a 32-bit window, first bit highest; zeros behind its last bit
    __device__ __forceinline__ uint32_t index(uint32_t bits) const
    {
        const int32_t whole = static_cast<int32_t>(bits >> 24), late = static_cast<int32_t>(bits >> shift) - skip;
        return static_cast<uint32_t>(whole > late ? whole : late);
    }
};

// A shift reads five bits of its amount, so an entry is one as it stands.  Written out: the compiler would put the `and` that the
// language asks for back in front of the next look-up, and a field extract behind it.
__device__ __forceinline__ uint32_t shifted_down(uint32_t x, uint32_t by) { uint32_t r; asm("v_lshrrev_b32_e32 %0, %1, %2" : "=v"(r) : "v"(by), "v"(x)); return r; }
__device__ __forceinline__ uint32_t shifted_up(uint32_t x, uint32_t by) { uint32_t r; asm("v_lshlrev_b32_e32 %0, %1, %2" : "=v"(r) : "v"(by), "v"(x)); return r; }
// All ones where bit kBit of x is set, else zero (likewise: as a condition it takes a comparison more).
template <int kBit>
__device__ __forceinline__ uint32_t spread(uint32_t x) { uint32_t r; asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(r) : "v"(x), "n"(kBit)); return r; }

// Bits of `mask` from a, the others from b: one instruction.
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

// An entry of the LDS table: the code's length in its low bits, the symbol in bits 7..14, where a bf16 word has its exponent.  So the
// entry is the shift to the next code as it stands (shifts read five bits), a sum of four has the bits used in its low seven, and two
// entries side by side take the sign-mantissa bytes in place of all other bits (merge2).  Made from two entries of a blob, symbol in the low
// byte and length in the high one; bit 15 holds anything.
constexpr uint32_t kExponentBits = 0x7f807f80u;
__device__ __forceinline__ uint32_t entry_pair(uint32_t v) { return pick(kExponentBits, v << 7, v >> 8); }

// Two bf16 words from two entries and their two sign-mantissa bytes, twice each: s eeeeeee e mmmmmmm.
__device__ __forceinline__ uint32_t merge2(uint32_t entries, uint32_t sm_twice) { return pick(kExponentBits, entries, sm_twice); }

// Lock-step decoder state of one lane (a5): two chains, one reading the lane's bitstream upwards from its
// first bit (the first half of the lane's symbols, in order), one reading it downwards from its last bit (the
// second half, last symbol first).
// kLong = false: every code has at most eight bits, four symbols per 32-bit window.  kLong = true: codes of up to
// ZM_MAX_CODE_LEN bits.  Two symbols per window are safe; four nearly always fit as well, since long codes are the rare
// ones by construction: quad tries four, and its caller falls back to safe_quad where a lane's four have more than 32
// bits between them.
// kFromBlob: the table in LDS does not hold all of the tensor's codes, and tab is the blob's own.
template <bool kLong, bool kFromBlob = false>
struct Decoder {
    const uint32_t *words;        // the stream as staged in LDS (length bytes included)
    uint32_t last_word;           // highest index a read may use
    LongTable table;              // kLong only
    // Upward chain: words q and q+1 of the bitstream, bits of lo already used (< 32 at the start of a round), index of word q+2.
    // Downward chain, short codes: the same of the bitstream from its end, every word reversed, so that it reads upwards as well.
    // Long codes: dhi is the word that holds the bits just below the read position, of which its low dpos bits (0..31) are still
    // unread, dlo the word below it, dnext the index of the word below that.
    uint32_t lo = 0, hi = 0, pos = 0, next = 0;
    uint32_t dlo = 0, dhi = 0, dpos = 0, dnext = 0;

    // first_bit, end_bit: where this lane's bitstream starts and ends, counted from the first payload bit
    __device__ __forceinline__ void start(uint32_t first_bit, uint32_t end_bit)
    {
        const uint32_t q = kLaneBytes / 4 + (first_bit >> 5);
        pos = first_bit & 31u;
        lo = words[min(q, last_word)];
        hi = words[min(q + 1u, last_word)];
        next = q + 2u;
        const uint32_t end = kLong ? end_bit : end_bit - 1u;                    // a bitstream has at least eight bits
        const uint32_t w = min(kLaneBytes / 4 + (end >> 5), last_word);         // >= 16, so the indices below stay >= 14
        const uint32_t top = words[w], below = words[w - 1u];
        dnext = w - 2u;
        if constexpr (kLong) {
            dpos = end & 31u;
            dhi = top;
            dlo = below;
        } else {
            dpos = ~end & 31u;
            dlo = __builtin_bitreverse32(top);
            dhi = __builtin_bitreverse32(below);
        }
    }

    // The entry of the code at the beginning of a window: its lowest bits (short codes) or its highest (long codes).
    __device__ __forceinline__ uint32_t look(const uint16_t *tab, uint32_t win) const
    {
        if constexpr (kFromBlob) return entry_pair(tab[__builtin_bitreverse32(win >> table.shift) >> table.shift]);
        else if constexpr (kLong) return tab[table.index(win)];
        else return tab[win & 0xffu];
    }

    // One round: R symbols of each chain.  up / down receive the R entries in the order read; the result is the larger
    // of the two chains' bits used, of which no more than 32 are real.
    // A chain's step is a look-up, a shift of the window by the entry, and the next address: two instructions between one read
    // and the next, the rest is off the chain.  Where a launch is bound by its waves' chains, us: one matrix of 256 x 512 4.00 -> 3.86, one
    // expert of 2048 x 1408 x 3, cached, 6.23 -> 5.98, two in streams of 16384 values 13.1 -> 12.5, of 32768 18.1 -> 17.2, against bits
    // used that were summed up and codes extracted from an unmoved window (three instructions; a round with its merging and stores 56
    // vector instructions instead of 44).
    template <int R>
    __device__ __forceinline__ uint32_t round(const uint16_t *tab, uint32_t (&up)[R], uint32_t (&down)[R])
    {
        // the words the chains take if the round crosses a word boundary: asked for now, used after the round
        const uint32_t fresh = words[min(next, last_word)];
        uint32_t dfresh = words[min(dnext, last_word)];
        uint32_t win = __builtin_amdgcn_alignbit(hi, lo, pos), dwin = __builtin_amdgcn_alignbit(dhi, dlo, dpos);
        if constexpr (kLong) win = __builtin_bitreverse32(win);
        uint32_t used = 0, dused = 0;                 // in the low seven bits; those above hold sums of symbols
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const uint32_t v = look(tab, win), dv = look(tab, dwin);
            up[k] = v;
            down[k] = dv;
            if (k + 1 < R) {
                win = kLong ? shifted_up(win, v) : shifted_down(win, v);
                dwin = kLong ? shifted_up(dwin, dv) : shifted_down(dwin, dv);
            }
            used += v;
            dused += dv;
        }
        // written without branches so that a whole tile pair is one basic block: the masks are all ones where the chain has used
        // up its first word
        pos += used;
        const uint32_t take = spread<5>(pos);
        pos &= 31u;
        lo = pick(take, hi, lo);
        hi = pick(take, fresh, hi);
        next -= take;
        if constexpr (kLong) {
            dpos -= dused;                            // -48..31 in the low seven bits
            const uint32_t dtake = spread<6>(dpos);
            dpos &= 31u;
            dhi = pick(dtake, dlo, dhi);
            dlo = pick(dtake, dfresh, dlo);
            dnext += dtake;
        } else {
            dpos += dused;
            const uint32_t dtake = spread<5>(dpos);
            dpos &= 31u;
            dlo = pick(dtake, dhi, dlo);
            dhi = pick(dtake, __builtin_bitreverse32(dfresh), dhi);
            dnext += dtake;
        }
        return kLong ? max(used & 127u, dused & 127u) : 0u;
    }

    // Four symbols of each chain, as entries, two per register in value order: half a tile's of this lane each.  most: the
    // largest number of bits that a round has used (long codes only).
    struct Quad { uint2 up, down; };
    __device__ __forceinline__ Quad quad(const uint16_t *tab, uint32_t &most)
    {
        uint32_t up[4], down[4];
        most = max(most, round(tab, up, down));
        return Quad{make_uint2(pack(up[0], up[1]), pack(up[2], up[3])), make_uint2(pack(down[3], down[2]), pack(down[1], down[0]))};
    }

    __device__ __forceinline__ Quad safe_quad(const uint16_t *tab)
    {
        if constexpr (kLong) {
            uint32_t ua[2], da[2], ub[2], db[2];
            round(tab, ua, da);
            round(tab, ub, db);
            return Quad{make_uint2(pack(ua[0], ua[1]), pack(ub[0], ub[1])), make_uint2(pack(db[1], db[0]), pack(da[1], da[0]))};
        } else {
            uint32_t most = 0;
            return quad(tab, most);
        }
    }

    static __device__ __forceinline__ uint32_t pack(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
};

// One lane's eight bf16 words of a tile from its entries, values 0..3 and 4..7, and its sign-mantissa bytes.
__device__ __forceinline__ uint4 merge8(uint2 e03, uint2 e47, uint2 sm)
{
    return make_uint4(merge2(e03.x, __builtin_amdgcn_perm(sm.x, sm.x, 0x01010000u)), merge2(e03.y, __builtin_amdgcn_perm(sm.x, sm.x, 0x03030202u)),
                      merge2(e47.x, __builtin_amdgcn_perm(sm.y, sm.y, 0x01010000u)), merge2(e47.y, __builtin_amdgcn_perm(sm.y, sm.y, 0x03030202u)));
}

// One byte per value of a stream (sign-mantissa bytes, or a raw chunk's exponent bytes), read as 64 bits per lane and
// tile.  The descriptor covers the stream's bytes, rounded up to whole groups of eight (the section is padded): a lane
// or a tile past them reads zeros and touches no memory.
struct ByteSource {
    __amdgpu_buffer_rsrc_t bytes;
    uint32_t lane_offset;
    __device__ __forceinline__ ByteSource(const uint8_t *stream_base, uint32_t n_values, uint32_t lane)
        : bytes(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(stream_base), 0, static_cast<int>((n_values + 7u) & ~7u), kRawBuffer)),
          lane_offset(lane * 8u) {}
    __device__ __forceinline__ uint2 load(uint32_t tile) const
    {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(bytes, static_cast<int>(lane_offset + tile * kTile), 0, 0);
        return make_uint2(v.x, v.y);
    }
};

// Stores one lane's eight values of a tile, or those that it has.
template <Stores kStores>
__device__ __forceinline__ void finish_tile(const Sink<kStores> &out, uint32_t tile, uint4 w, int32_t mine)
{
    const int32_t left = mine - static_cast<int32_t>(tile * kTile);
    if (left >= 8) out.store(tile, w);
    else if (left > 0) out.store_partial(tile, w);
}

// Decodes a coded stream from both ends: pair p is tile p (upward chain) and tile tiles - 1 - p (downward chain), and
// up[p % kPairs] / down[p % kPairs] receive their sign-mantissa bytes.  The first kAhead pairs' have been asked for by
// the caller, the others of the first kPairs pairs are asked for when pair p - kAhead is done.

// Pairs first .. first + kPairs - 1.  Returns how many are done: with long codes, a pair in which a lane's four symbols had more
// bits than a window is left alone, with the decoder as it was in front of it.
template <bool kLong, int kAhead, Stores kStores>
__device__ __forceinline__ uint32_t decode_group(Decoder<kLong> &dec, const uint16_t *tab, const Sink<kStores> &out, const ByteSource &sm,
                                                 uint32_t first, uint32_t tiles, uint2 (&up)[kPairs], uint2 (&down)[kPairs])
{
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
        const uint32_t lo = first + i, hi = tiles - 1u - lo;
        const Decoder<kLong> before = dec;
        uint32_t most = 0;
        // a tile's eight symbols come in two quads: the upward chain gives values 0..3 first, the
        // downward chain values 4..7 first
        const auto a = dec.quad(tab, most), b = dec.quad(tab, most);
        if constexpr (kLong) {
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(most > 32u) != 0, 0)) {
                dec = before;
                return static_cast<uint32_t>(i);
            }
        }
        out.store(lo, merge8(a.up, b.up, up[i]));
        out.store(hi, merge8(b.down, a.down, down[i]));
        if (i + kAhead < kPairs) {
            up[i + kAhead] = sm.load(lo + kAhead);
            down[i + kAhead] = sm.load(hi - kAhead);
        }
    }
    return kPairs;
}

// Streams of whole tiles, a multiple of eight of them: returns the pairs that are done.  The next group's bytes are asked for when a
// group is begun, into registers of their own: they come while it is decoded, and as they are asked for in front of its stores, the
// wait for them is not a wait for these.  The last group asks for tiles that read as zero and touch no memory, and groups take turns
// with the registers, so that the same requests follow a group's bytes on every way to their use: where the compiler can not
// count them, or has to move the bytes, it waits for more than is needed.
template <bool kLong, Stores kStores>
__device__ __forceinline__ uint32_t decode_groups(Decoder<kLong> &dec, const uint16_t *tab, const Sink<kStores> &out, const ByteSource &sm,
                                                  uint32_t tiles, uint2 (&up)[kPairs], uint2 (&down)[kPairs])
{
    constexpr uint32_t kOutside = 1u << 20;        // tiles; no stream has as many
    uint2 other_up[kPairs], other_down[kPairs];
    uint32_t done = 0;
    // the next group, with the one after it asked for; false: nothing is left to do here
    auto group = [&](uint2 (&u)[kPairs], uint2 (&d)[kPairs], uint2 (&next_u)[kPairs], uint2 (&next_d)[kPairs]) {
        const uint32_t next = done + kPairs, skip = 2u * next >= tiles ? kOutside : 0u;
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            next_u[i] = sm.load(next + i + skip);
            next_d[i] = sm.load(tiles - 1u - next - i + skip);
        }
        const uint32_t more = decode_group<kLong, kPairs>(dec, tab, out, sm, done, tiles, u, d);
        done += more;
        return more == kPairs && 2u * done < tiles;
    };
    if (group(up, down, other_up, other_down))
        while (group(other_up, other_down, up, down) && group(up, down, other_up, other_down)) {}
    return done;
}

// Any stream, from pair `first` on: short ones, last ones, ones dense in long codes.  With an odd number of tiles the last
// pair is the middle tile alone, whose low half comes from the upward and whose high half from the downward chain.  The
// caller has asked for two pairs (up[0], up[1]).  Only the last tile of a stream can be cut off, and that is one of pair 0.
// kTurns pairs take turns with as many registers, in a loop body of as many pairs: rolled to one pair, with the next one's bytes moved into its
// registers, every pair waited for these bytes and for its own stores, 0.8 us.  us before / now: 24 tensors of 2.1 M values down to 1/300 of it
// 8.17 / 7.06, 3000 streams of 2048 values 5.24 / 4.75 (long codes 6.69 / 6.22), four experts of 1024 x 2048 x 3 in streams of 6144 19.97 / 18.95.  Four turns
// where a wave has the registers; in the last of these launches they cost two waves per SIMD: 20.76.
template <bool kLong, Kind kKind>
constexpr int kSlots = kLong || kKind == kShortStreams || kKind == kFitting || kKind == kMixed ? 2 : kPairs;

template <bool kLong, bool kFromBlob, int kTurns, Stores kStores>
__device__ __forceinline__ void decode_any_stream(Decoder<kLong, kFromBlob> &dec, const uint16_t *tab, const Sink<kStores> &out, const ByteSource &sm,
                                                  uint32_t first, uint32_t tiles, int32_t mine, uint2 (&up)[kPairs], uint2 (&down)[kPairs])
{
#pragma unroll
    for (int i = 2; i < kTurns; ++i) {
        up[i] = sm.load(first + i);
        down[i] = sm.load(tiles - 1u - first - i);
    }
    // true: that was the last one
    auto pair = [&](auto slot) {
        constexpr int i = slot.value;
        const uint32_t lo = first + i, hi = tiles - 1u - lo;
        const auto a = dec.safe_quad(tab);
        if (lo == hi) {
            const uint4 w = merge8(a.up, a.down, up[i]);
            if (i == 0) finish_tile(out, lo, w, mine);
            else out.store(lo, w);
            return true;
        }
        const auto b = dec.safe_quad(tab);
        out.store(lo, merge8(a.up, b.up, up[i]));
        if (i == 0) finish_tile(out, hi, merge8(b.down, a.down, down[i]), mine);
        else out.store(hi, merge8(b.down, a.down, down[i]));
        if (lo + 1u >= hi) return true;
        up[i] = sm.load(lo + kTurns);
        down[i] = sm.load(hi - kTurns);
        return false;
    };
#pragma unroll 1
    for (;; first += kTurns) {
        if (pair(std::integral_constant<int, 0>())) return;
        if constexpr (kTurns > 1)
            if (pair(std::integral_constant<int, 1>())) return;
        if constexpr (kTurns == 4)
            if (pair(std::integral_constant<int, 2>()) || pair(std::integral_constant<int, 3>())) return;
    }
}

// A chunk that is stored raw: its exponent bytes lie in memory as they are.  Four tiles are asked for before the first
// is merged.
template <Stores kStores>
__device__ __forceinline__ void merge_raw_stream(const Sink<kStores> &out, const ByteSource &raw, const ByteSource &sm,
                                                 uint32_t tiles, int32_t mine)
{
    for (uint32_t first = 0; first < tiles; first += kPairs) {
        uint2 e[kPairs], s[kPairs];
#pragma unroll
        for (int k = 0; k < kPairs; ++k) { e[k] = raw.load(first + k); s[k] = sm.load(first + k); }
#pragma unroll
        for (int k = 0; k < kPairs; ++k) finish_tile(out, first + k, recover8(e[k], s[k]), mine);
    }
}

// What no kernel writes, read through the scalar cache where the address is the same for all lanes.
template <class T>
using Constant = __attribute__((address_space(4))) T;

// LDS written by some lanes of this wave is read by others: order the LDS accesses only
__device__ __forceinline__ void order_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// a3: a tensor's decode table -> LDS, in entries of the decoder's form.  Every wave of the workgroup writes the
// same bytes (LDS word writes are atomic), so a wave may read as soon as its own writes are done: no workgroup barrier.
template <bool kLong>
struct TableStage {
    const uint16_t *lut;             // the blob's table
    uint32_t max_len;
    uint2 lut4;                      // entries 4 * lane .. + 3, of codes shorter than eight bits replicated over the index bits above
    uint32_t lut_tail = 0;           // long codes: see put

    __device__ __forceinline__ void ask(const Task &t, uint32_t lane)
    {
        lut = reinterpret_cast<const uint16_t *>(t.lut);
        max_len = max_len_of(t.code);
        if constexpr (kLong) {
            lut4 = reinterpret_cast<const uint2 *>(lut)[lane];
        } else {
            const uint32_t mask = (1u << max_len) - 1u;
            lut4 = make_uint2(*reinterpret_cast<const uint32_t *>(lut + (4u * lane & mask)), *reinterpret_cast<const uint32_t *>(lut + (4u * lane + 2u & mask)));
        }
    }

    __device__ __forceinline__ void ask_tail(uint32_t lane)
    {
        if constexpr (kLong) lut_tail = lut[__builtin_bitreverse32((1u << max_len) - 64u + lane) >> (32u - max_len)];
    }

    // narrow: the table has no room for all shared beginnings
    __device__ __forceinline__ void put(uint16_t *tab, uint32_t lane, uint32_t long_slots, LongTable &table, bool &narrow) const
    {
        const uint32_t i = 4u * lane;
        const uint2 e = lut4;
        if constexpr (!kLong) {
            reinterpret_cast<uint2 *>(tab)[lane] = make_uint2(entry_pair(e.x), entry_pair(e.y));
        } else {
            // The blob's table is indexed with a code's first bit lowest, so the number v of LongTable has to be reversed;
            // its first 256 entries are those of the eight-bit beginnings, with a length above eight at shared ones.
            // The last 64 values of v belong to long codes if any are (lut_tail); they are asked for before it is known how many
            // more there are, which on Gaussian weights is none.
            const uint32_t more = max_len - 8u;
            uint32_t n_shared = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t v = (k & 2 ? e.y : e.x) >> (16 * (k & 1)) & 0xffffu;
                n_shared += static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64((v >> 8) > 8u)));
            }
            narrow = n_shared > long_slots;
            n_shared = min(n_shared, long_slots);
            const uint32_t whole_codes = kTableEntries - n_shared, late = n_shared << more;
            table.shift = 32u - max_len;
            table.skip = static_cast<int32_t>((whole_codes << more) - whole_codes);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t v = (k & 2 ? e.y : e.x) >> (16 * (k & 1)) & 0xffffu;
                const uint32_t at = __builtin_bitreverse32(i + k) >> 24;
                if (at < whole_codes) tab[at] = static_cast<uint16_t>(entry_pair(v));
            }
            if (lane + late >= 64u) tab[whole_codes + late - 64u + lane] = static_cast<uint16_t>(entry_pair(lut_tail));
            for (uint32_t k = lane; k + 64u < late; k += 64u) {
                const uint32_t v = lut[__builtin_bitreverse32((whole_codes << more) + k) >> (32u - max_len)];
                tab[whole_codes + k] = static_cast<uint16_t>(entry_pair(v));
            }
        }
    }
};

// Stream g of a tensor, by one wave.  kLong: codes of more than eight bits; kStores: how the output is written; tab: LDS for the decode
// table; words: LDS for the stream, cap_words of it; long_slots: as in Launch; kOneTile: many of the streams are of one tile
template <bool kLong, Stores kStores, Kind kKind, bool kOneTile>
__device__ __forceinline__ void decode_stream(const Task &t, uint32_t g, uint16_t *tab, uint32_t *words, uint32_t cap_words, uint32_t long_slots)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t W = t.stream_values;
    const uint32_t quantum = quantum_of(t.code);
    const uint32_t stride = (8u + 4u * (t.streams_per_chunk + 1u) + 7u) & ~7u;     // bytes of a chunk-table entry
    const uint64_t v0 = static_cast<uint64_t>(g) * W;              // first value of the stream in the tensor
    const uint32_t sn = g + 1u < t.n_streams ? W : t.last_values, tiles = (sn + kTile - 1) / kTile;
    const int32_t mine = static_cast<int32_t>(sn) - static_cast<int32_t>(lane * 8u);   // values left from this lane's first one

    // one read of the chunk's table entry gives the chunk's place and mode and this stream's extent
    const uint32_t c = chunk_of(g, t.per_chunk, t.code), s = g - c * t.streams_per_chunk;
    const Constant<uint8_t> *entry = (const Constant<uint8_t> *)(reinterpret_cast<const uint8_t *>(t.table) + static_cast<uint64_t>(c) * stride);
    const uint64_t ent = *(const Constant<uint64_t> *)entry;
    const uint32_t o0 = ((const Constant<uint32_t> *)(entry + 8))[s], o1 = ((const Constant<uint32_t> *)(entry + 8))[s + 1u];

    // The decode table is asked for meanwhile: behind the sign-mantissa bytes it would be served behind them, and decoding
    // waits for it.
    TableStage<kLong> stage_table;
    stage_table.ask(t, lane);
    asm volatile("" :: "s"(ent), "s"(o0), "s"(o1));        // with one wait: the compiler would read o0 and o1 where they are used

    bool active = true;
    const uint8_t *raw = nullptr;
    // The stream's first vectors, lane + 64 k, wait in registers until the other requests are out: 2 KiB, more than a typical
    // stream of 4096 values, 4, or 12, as much as one of 32768.  (What is copied in the loop below waits for every vector anew: streams
    // of 32768 values, two / eight experts of 1024 x 2048 x 3, 20.7 / 45.5 us with 2 KiB, 17.8 / 37.8 with 12 and the next group of
    // tiles asked for early, of 16384 values 13.2 / 32.8 and 12.1 / 32.1.)  What lies past 4 KiB is left out in one step: one tensor of 32760
    // values in streams of 8192 8.33 -> 7.93 us, four experts of three tensors of 70001 6.14 -> 5.78.
    constexpr uint32_t kHeld = kKind == kDeep ? 12 : kKind == kMixed ? 4 : 2, kFirst = kHeld < 4 ? kHeld : 4;
    u32x4 held[kHeld];
    uint32_t n_held = 0;
    bool dense = false;          // long codes: four symbols of a lane are likely to have more bits than a window
    const uint64_t chunk = ent & ~15ull, at = chunk - t.e_offset;            // offsets inside the blob and the E-chunk region
    const uint32_t mode = static_cast<uint32_t>(ent & 15ull);
    if (mode == ZM_MODE_CODED) {
        // a4: the stream's bytes, 128 bits per lane per load.  They are requested before the (larger)
        // sign-mantissa bytes because decoding can not start without them.  What is not held is copied here.
        active = stream_inside(chunk, o0, o1, t.e_offset, t.e_size);
        if (active) {
            const uint32_t nvec = min((o1 - o0) >> 4, cap_words >> 2);
            if constexpr (kLong) dense = 2u * (o1 - o0) > sn;          // more than four bits a value
            const u32x4 *src = reinterpret_cast<const u32x4 *>(t.echunks + at + o0);
            u32x4 *dst = reinterpret_cast<u32x4 *>(words);
            n_held = min(nvec, 64u * kHeld);
#pragma unroll
            for (uint32_t k = 0; k < kFirst; ++k)
                if (lane + 64u * k < n_held) held[k] = src[lane + 64u * k];
            if (kFirst < kHeld && n_held > 64u * kFirst) {
#pragma unroll
                for (uint32_t k = kFirst; k < kHeld; ++k)
                    if (lane + 64u * k < n_held) held[k] = src[lane + 64u * k];
            }
            for (uint32_t i = 64u * kHeld + lane; i < nvec; i += 64) dst[i] = src[i];
        }
    } else {
        raw = t.echunks + at + static_cast<uint64_t>(s) * W;
        active = mode == ZM_MODE_RAW && raw_stream_inside(chunk, static_cast<uint64_t>(s) * W, (sn + 15u) & ~15u, t.e_offset, t.e_size);
    }
    stage_table.ask_tail(lane);
    // Next in the request order: the sign-mantissa bytes of the first tiles.  They stay in flight while the
    // stream is staged and decoding starts.  up[i] / down[i] hold those of a pair of tiles, one from either end.
    constexpr int kAhead = pairs_ahead(kKind, kLong, kStores);
    constexpr bool kGroups = kKind == kDeep || kKind == kMixed;          // there may be streams of several groups
    const bool coded = mode == ZM_MODE_CODED;
    const bool straight = kKind != kShortStreams && (kGroups ? sn % kGroupValues == 0 : sn == kGroupValues) && !dense;     // whole groups of tiles, decoded without a look at their ends
    const bool groups = kGroups && straight && (kKind == kDeep || tiles > kGroup);                     // all of them are asked for group by group
    uint2 up[kPairs], down[kPairs];
    const ByteSource sm(t.sm + v0, sn, lane), first_sm(t.sm + v0, coded && active ? sn : 0u, lane);
    auto ask = [&](int i) {        // tiles that the stream does not have read as zero and touch no memory
        up[i] = first_sm.load(i);
        down[i] = first_sm.load(tiles - 1u - i);
    };
    LongTable table{0u, 0};
    bool narrow = false;         // long codes: the table has no room for all shared beginnings
    auto stage = [&] {
        stage_table.put(tab, lane, long_slots, table, narrow);
        u32x4 *dst = reinterpret_cast<u32x4 *>(words);
#pragma unroll
        for (uint32_t k = 0; k < kFirst; ++k)
            if (lane + 64u * k < n_held) dst[lane + 64u * k] = held[k];
        if (kFirst < kHeld && n_held > 64u * kFirst) {
#pragma unroll
            for (uint32_t k = kFirst; k < kHeld; ++k)
                if (lane + 64u * k < n_held) dst[lane + 64u * k] = held[k];
        }
    };
    // The requests that follow a stream's are known to be so many when it is copied: no branch lies in between.  Where the
    // compiler can not count them it waits for all of them, and decoding does not start before the sign-mantissa bytes have come.
    // (One expert of 1024 x 2048 x 3, streaming stores 5.40 -> 5.18 us, eight 26.8 -> 26.55, one matrix of 256 x 512 3.92 -> 3.80.)
    ask(0);
    if (groups) {
#pragma unroll
        for (int i = 1; i < kPairs; ++i) ask(i);
        stage();
    } else if (kAhead == 2 || !straight) {
        ask(1);
        stage();
    } else {
#pragma unroll
        for (int i = 1; i < kAhead; ++i) ask(i);
        stage();
    }
    order_lds();
    if (!active) return;

    const Sink<kStores> out(t.out + v0, sn, lane);

    if (!coded) {
        merge_raw_stream(out, ByteSource(raw, sn, lane), sm, tiles, mine);
        return;
    }
    // a6: this lane's bitstream has 8 * tiles + quantum * (its length byte) bits and starts where
    // the bitstreams of the lanes below it end
    const uint32_t units = reinterpret_cast<const uint8_t *>(words)[lane];
    const uint32_t bits = 8u * tiles + quantum * units;
    const uint32_t first = wave_exclusive_sum(bits);
    if constexpr (kLong) {
        if (__builtin_expect(narrow, 0)) {
            Decoder<true, true> dec;
            dec.words = words; dec.last_word = cap_words - 1u;
            dec.table = table;
            dec.start(first, first + bits);
            // one turn: with two, for tables that only a damaged blob has, streams shorter than a group took 65 registers, seven waves per SIMD
            decode_any_stream<true, true, 1>(dec, stage_table.lut, out, sm, 0u, tiles, mine, up, down);
            return;
        }
    }
    // A stream of one tile has no turns to take, and in their loop it waited for all that its turns would have asked for.  us: 2000 / 8000 streams of 512 values,
    // cached 2.96 / 4.88 -> 2.86 / 4.68, long codes 3.41 / 5.87 -> 3.33 / 5.61.
    if (kOneTile && tiles == 1u) {
        Decoder<kLong> dec;
        dec.words = words; dec.last_word = cap_words - 1u;
        dec.table = table;
        dec.start(first, first + bits);
        const auto e = dec.safe_quad(tab);
        finish_tile(out, 0u, merge8(e.up, e.down, up[0]), mine);
        return;
    }
    Decoder<kLong> dec;
    dec.words = words; dec.last_word = cap_words - 1u;
    dec.table = table;
    dec.start(first, first + bits);
    uint32_t done = 0;
    if (straight) {
        if (groups) done = decode_groups(dec, tab, out, sm, tiles, up, down);
        else done = decode_group<kLong, kAhead>(dec, tab, out, sm, 0u, tiles, up, down);
        if (!kLong || 2u * done >= tiles) return;
        up[0] = sm.load(done); down[0] = sm.load(tiles - 1u - done);
        up[1] = sm.load(done + 1u); down[1] = sm.load(tiles - 2u - done);
    }
    decode_any_stream<kLong, false, kSlots<kLong, kKind>>(dec, tab, out, sm, done, tiles, mine, up, down);
}

// kBundle consecutive streams of a tensor, eight tiles together, by one wave: where streams are short, a wave's life is mostly the chain of
// dependent reads in front of a few look-ups, and this puts eight tiles behind one chain and interleaves the look-ups of two streams.  Lane k
// reads the chunk-table entry of stream k; the streams follow one another in memory, coded and raw ones, and are fetched as one piece.  Raw ones are
// merged from it, coded ones beside raw ones decoded one at a time.  A round of long codes that had more bits than a window is done again in two halves;
// where the decoders as they were would cost a wave per SIMD (110 registers instead of 95), the stream is.  One wave that went through its
// streams one after another, each with its own reads, held up a whole launch (us for 24000 streams of
// 512 values, a wave per stream / such waves / now: codes of up to 12 bits, rows scaled by exp(N(0,1)), 12.3 / 17.3 / 8.6; one piece of 4096 values in a thousand raw
// 10.2 / 13.3 / 8.5).  That is left for what a damaged table has.  The rest of a tensor that is no whole bundle is decoded by a wave per stream.
template <bool kLong, Stores kStores, Kind kKind, int kBundle>
__device__ __forceinline__ void decode_bundle(const Task &t, uint32_t wave_of_tensor, uint16_t *tab, uint32_t *words, uint32_t cap_words, uint32_t long_slots)
{
    constexpr uint32_t kTilesEach = kGroup / kBundle, kValues = kTilesEach * kTile;
    constexpr bool kAgain = kLong && (kTilesEach <= 2 || kKind == kMany);      // rounds are done again, not streams
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t bundles = whole_bundles(t.n_streams, t.last_values, kBundle);
    const uint32_t alone = wave_of_tensor - min(wave_of_tensor, bundles), g0 = (wave_of_tensor - alone) * kBundle + alone;
    if (g0 >= t.n_streams) return;
    uint32_t one_by_one = 1u;        // streams to be decoded by themselves, bit k is stream g0 + k
    if (wave_of_tensor < bundles) {
        const uint32_t stride = (8u + 4u * (t.streams_per_chunk + 1u) + 7u) & ~7u;
        const uint64_t v0 = static_cast<uint64_t>(g0) * kValues;
        const uint32_t quantum = quantum_of(t.code);

        const uint32_t k_of = lane & (kBundle - 1u), g = g0 + k_of;
        const uint32_t c = chunk_of(g, t.per_chunk, t.code), s = g - c * t.streams_per_chunk;
        const uint8_t *entry = reinterpret_cast<const uint8_t *>(t.table) + static_cast<uint64_t>(c) * stride;
        const uint64_t ent = *reinterpret_cast<const uint64_t *>(entry);
        const uint32_t o0 = reinterpret_cast<const uint32_t *>(entry + 8)[s], o1 = reinterpret_cast<const uint32_t *>(entry + 8)[s + 1u];
        TableStage<kLong> stage_table;
        stage_table.ask(t, lane);

        constexpr uint32_t kHeld = 4;        // KiB that wait in registers
        const uint32_t room = 4u * kBundle * cap_words;
        const uint64_t chunk = ent & ~15ull;
        uint64_t from0;
        uint32_t rel, total, raws = 0;       // this lane's stream and the end of the last one, from from0; bit k of raws: stream g0 + k is raw
        // whether all lanes' streams, `bytes` at `at` in the region, are one piece that finds room
        auto one_piece = [&](bool inside, uint64_t at, uint32_t bytes) {
            const uint64_t from = reinterpret_cast<uint64_t>(t.echunks) + (chunk - t.e_offset) + at;
            from0 = static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(from >> 32), 0))) << 32 |
                    static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(from), 0));
            rel = static_cast<uint32_t>(from - from0);
            const uint32_t end = rel + bytes, before = __builtin_amdgcn_update_dpp(0u, end, 0x111, 0xf, 0xf, false);       // row_shr:1
            total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(end), kBundle - 1));
            const bool simple = inside && !((from | bytes) & 15u) && from - from0 <= room && (k_of == 0 || rel == before) && bytes <= room && end <= room;
            return __builtin_amdgcn_ballot_w64(simple) == ~0ull;
        };
        const bool coded = (ent & 15ull) == ZM_MODE_CODED && stream_inside(chunk, o0, o1, t.e_offset, t.e_size);
        bool piece_found = one_piece(coded, o0, o1 - o0);
        if (__builtin_expect(!piece_found, 0)) {
            const uint64_t raw_at = static_cast<uint64_t>(s) * kValues;
            const bool raw = (ent & 15ull) == ZM_MODE_RAW;
            raws = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(raw)) & ((1u << kBundle) - 1u);
            piece_found = one_piece(raw ? raw_stream_inside(chunk, raw_at, kValues, t.e_offset, t.e_size) : coded, raw ? raw_at : o0, raw ? kValues : o1 - o0);
        }
        one_by_one = (1u << kBundle) - 1u;
        if (piece_found) {
            const u32x4 *const piece_at = reinterpret_cast<const u32x4 *>(from0);
            if (__builtin_expect(total > 1024u * kHeld, 0))
                for (uint32_t i = 64u * kHeld + lane; i < total / 16u; i += 64u) reinterpret_cast<u32x4 *>(words)[i] = piece_at[i];
            u32x4 held[kHeld];
            const __amdgpu_buffer_rsrc_t piece = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(from0), 0, static_cast<int>(total), kRawBuffer);
#pragma unroll
            for (uint32_t k = 0; k < kHeld; ++k) held[k] = __builtin_amdgcn_raw_buffer_load_b128(piece, static_cast<int>(16u * lane + 1024u * k), 0, 0);
            stage_table.ask_tail(lane);
            // sign-mantissa bytes, in the order of use: two streams take turns, each from both ends
            const ByteSource sm(t.sm + v0, kGroupValues, lane);
            auto tile_of = [](uint32_t i) {
                if (kTilesEach == 1) return i;
                const uint32_t pair = i / (2u * kTilesEach), p = i % (2u * kTilesEach) / 4u, which = i & 3u;
                return (2u * pair + which / 2u) * kTilesEach + (which & 1u ? kTilesEach - 1u - p : p);
            };
            constexpr uint32_t kAhead = bundle_ahead(kKind, kStores);
            uint2 byte8[kGroup];
#pragma unroll
            for (uint32_t i = 0; i < kAhead; ++i) byte8[i] = sm.load(tile_of(i));
            LongTable table{0u, 0};
            bool narrow = false;
            stage_table.put(tab, lane, long_slots, table, narrow);
#pragma unroll
            for (uint32_t k = 0; k < kHeld; ++k)
                if (16u * lane + 1024u * k < total) reinterpret_cast<u32x4 *>(words)[lane + 64u * k] = held[k];
            order_lds();
            if (!narrow) {
                const Sink<kStores> out(t.out + v0, kGroupValues, lane);
                one_by_one = 0;
                uint32_t rest = 0;           // bit k: stream g0 + k is left for the loop below
                auto place_of = [&](uint32_t k) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(rel), static_cast<int>(k))) / 4u; };      // words
                if (__builtin_expect(raws != 0, 0)) {
                    rest = raws ^ ((1u << kBundle) - 1u);
#pragma unroll
                    for (uint32_t i = kAhead; i < kGroup; ++i) byte8[i] = sm.load(tile_of(i));
#pragma unroll
                    for (uint32_t i = 0; i < kGroup; ++i) {
                        const uint32_t k = tile_of(i) / kTilesEach;
                        if (raws >> k & 1u)
                            out.store(tile_of(i), recover8(reinterpret_cast<const uint2 *>(words + place_of(k))[tile_of(i) % kTilesEach * 64u + lane], byte8[i]));
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < kBundle; k += 2) {
                        const uint32_t at0 = place_of(k), at1 = place_of(k + 1);
                        const uint32_t *const w0 = words + at0, *const w1 = words + at1;
                        // two streams' prefix sums in one: 64 lanes of at most 8 * 4 + 2 * 255 bits
                        const uint32_t bits0 = 8u * kTilesEach + quantum * reinterpret_cast<const uint8_t *>(w0)[lane], bits1 = 8u * kTilesEach + quantum * reinterpret_cast<const uint8_t *>(w1)[lane];
                        const uint32_t first = wave_exclusive_sum(bits0 | bits1 << 16);
                        Decoder<kLong> d0, d1;
                        d0.words = w0; d1.words = w1;
                        d0.last_word = kBundle * cap_words - 1u - at0;
                        d1.last_word = kBundle * cap_words - 1u - at1;
                        d0.table = d1.table = table;
                        d0.start(first & 0xffffu, (first & 0xffffu) + bits0);
                        d1.start(first >> 16, (first >> 16) + bits1);
                        const uint32_t done = k * kTilesEach;          // tiles
                        auto more = [&](uint32_t i) { if (i + kAhead < kGroup) byte8[i + kAhead] = sm.load(tile_of(i + kAhead)); };
                        uint32_t most0 = 0, most1 = 0;
                        auto again = [&] { return kAgain && __builtin_expect(__builtin_amdgcn_ballot_w64(max(most0, most1) > 32u) != 0, 0); };
                        if constexpr (kTilesEach == 1) {
                            const Decoder<kLong> before0 = d0, before1 = d1;
                            auto a0 = d0.quad(tab, most0), a1 = d1.quad(tab, most1);
                            if (again()) {
                                d0 = before0; d1 = before1;
                                a0 = d0.safe_quad(tab); a1 = d1.safe_quad(tab);
                            }
                            out.store(done, merge8(a0.up, a0.down, byte8[done]));
                            out.store(done + 1u, merge8(a1.up, a1.down, byte8[done + 1u]));
                            more(done); more(done + 1u);
                        } else {
#pragma unroll
                            for (uint32_t p = 0; p < kTilesEach / 2u; ++p) {
                                const Decoder<kLong> before0 = d0, before1 = d1;
                                if (kAgain) most0 = most1 = 0;
                                auto a0 = d0.quad(tab, most0), a1 = d1.quad(tab, most1), b0 = d0.quad(tab, most0), b1 = d1.quad(tab, most1);
                                if (again()) {
                                    d0 = before0; d1 = before1;
                                    a0 = d0.safe_quad(tab); a1 = d1.safe_quad(tab);
                                    b0 = d0.safe_quad(tab); b1 = d1.safe_quad(tab);
                                }
                                const uint32_t i = done + 4u * p;
                                out.store(tile_of(i), merge8(a0.up, b0.up, byte8[i]));
                                out.store(tile_of(i + 1u), merge8(b0.down, a0.down, byte8[i + 1u]));
                                out.store(tile_of(i + 2u), merge8(a1.up, b1.up, byte8[i + 2u]));
                                out.store(tile_of(i + 3u), merge8(b1.down, a1.down, byte8[i + 3u]));
                                more(i); more(i + 1u); more(i + 2u); more(i + 3u);
                            }
                            if constexpr (kLong && !kAgain)
                                rest |= (__builtin_amdgcn_ballot_w64(most0 > 32u) ? 1u << k : 0u) | (__builtin_amdgcn_ballot_w64(most1 > 32u) ? 2u << k : 0u);
                        }
                    }
                }
                while (__builtin_expect(rest != 0, 0)) {
                    const uint32_t k = static_cast<uint32_t>(__builtin_ctz(rest)), at = place_of(k);
                    rest &= rest - 1u;
                    const ByteSource its_sm(t.sm + v0 + k * kValues, kValues, lane);
                    uint2 up[kPairs], down[kPairs];
#pragma unroll
                    for (uint32_t i = 0; i < 2; ++i) {
                        up[i] = its_sm.load(i);
                        down[i] = its_sm.load(kTilesEach - 1u - i);
                    }
                    const uint32_t bits = 8u * kTilesEach + quantum * reinterpret_cast<const uint8_t *>(words + at)[lane], first = wave_exclusive_sum(bits);
                    Decoder<kLong> dec;
                    dec.words = words + at;
                    dec.last_word = kBundle * cap_words - 1u - at;
                    dec.table = table;
                    dec.start(first, first + bits);
                    decode_any_stream<kLong, false, 2>(dec, tab, Sink<kStores>(t.out + v0 + k * kValues, kValues, lane), its_sm, 0u, kTilesEach,
                                                       static_cast<int32_t>(kValues) - static_cast<int32_t>(lane * 8u), up, down);
                }
            }
        }
    }
    while (one_by_one) {
        const uint32_t k = static_cast<uint32_t>(__builtin_ctz(one_by_one));
        one_by_one &= one_by_one - 1u;
        decode_stream<kLong, kStores, kShortStreams, false>(t, g0 + k, tab, words, cap_words, long_slots);
    }
}

// What a wave decodes: a stream, or kBundle of them.  kWaves: waves per workgroup; cap_words: LDS words reserved for a stream
template <bool kLong, int kWaves, Stores kStores, Kind kKind, int kBundle>
__device__ __forceinline__ void decode_block(const Task &t, uint32_t block, uint32_t cap_words, uint32_t long_slots)
{
    // The decode table of the workgroup's tensor, at a fixed LDS address: one 16-bit read gives a code's length and its
    // symbol.  (Two byte tables, one read each, were 2-4 % slower: twice the LDS instructions, whose random accesses
    // collide on banks.)  That of long codes lies in front of the streams, as long as the launch's widest tensor needs.
    __shared__ __align__(16) uint16_t short_tab[kLong ? 8 : kTableEntries];
    extern __shared__ __align__(16) uint32_t dynamic_lds[];
    uint16_t *const tab = kLong ? reinterpret_cast<uint16_t *>(dynamic_lds) : short_tab;

    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t g = block * kWaves + wave;
    uint32_t *words = dynamic_lds + (kLong ? long_table_words(long_slots) : 0u) + wave * cap_words * kBundle;
    if constexpr (kBundle > 1) decode_bundle<kLong, kStores, kKind, kBundle>(t, g, tab, words, cap_words, long_slots);
    else if (g < t.n_streams) decode_stream<kLong, kStores, kKind, kKind == kShortStreams>(t, g, tab, words, cap_words, long_slots);
}

template <bool kLong, int kWaves, Stores kStores, Kind kKind, int kBundle, class Args>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(1, kBundle > 1 ? bundle_waves(kKind, kLong) : most_waves(kKind, kLong)))) zm_decode_kernel(const Args P)
{
    uint32_t block;
    const Task t = task_of(P, threadIdx.x & 63u, block);
    const uint32_t cap_words = P.stream_cap_words, long_slots = kLong ? P.long_slots : 0u;
    // All of the arguments with one wait: the compiler would read each where it is first used, one wait after another.  One
    // expert of 2048 x 1408 x 3 6.28 -> 6.09 us, one matrix of 1024 x 2048 in streams of 512 values 3.66 -> 3.45 (with the
    // chunk-table entry read at once, the look-up table asked for before the stream, and no division).
    asm volatile("" :: "s"(t.lut), "s"(t.sm), "s"(t.echunks), "s"(t.table), "s"(t.out), "s"(t.e_offset), "s"(t.e_size), "s"(t.stream_values),
                       "s"(t.streams_per_chunk), "s"(t.per_chunk), "s"(t.n_streams), "s"(t.last_values), "s"(t.code), "s"(cap_words), "s"(long_slots));
    decode_block<kLong, kWaves, kStores, kKind, kBundle>(t, block, cap_words, long_slots);
}

template <bool kLong, int kWaves, Stores kStores, Kind kKind, int kBundle>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(1, kBundle > 1 ? bundle_waves(kKind, kLong) : most_waves(kKind, kLong)))) zm_decode_few_kernel(const Few P)
{
    const uint32_t k = blockIdx.y;
    const uint32_t code = P.lead[0], n_streams = P.lead[1], last_lut = P.lead[2], table_offset = P.lead[3], sm_units = P.lead[4], e_at = P.lead[5];
    const uint8_t *low = P.low;
    const uint32_t to = P.to[k], to_out = P.to_out[k], e_units = P.e_units[k];
    uint16_t *out = P.out;
    asm volatile("" :: "s"(code), "s"(n_streams), "s"(last_lut), "s"(table_offset), "s"(sm_units), "s"(e_at), "s"(low), "s"(to), "s"(to_out), "s"(e_units), "s"(out));
    const uint8_t *blob = low + static_cast<uint64_t>(to) * 256u;
    const uint32_t W = (code & 127u) * kTile, max_len = code >> 7 & 15u, shift = code >> 11 & 31u, quantum = code >> 16 & 255u, long_slots = code >> 24;
    const uint64_t e_offset = static_cast<uint64_t>(e_at) * 256u;
    const Task t{blob + (last_lut >> 16), blob + static_cast<uint64_t>(sm_units) * 256u, blob + e_offset, reinterpret_cast<const uint64_t *>(blob + table_offset),
                 out + static_cast<uint64_t>(to_out) * 8u, e_offset, static_cast<uint64_t>(e_units) * 256u, W, 1u << shift, 1u << 31, n_streams,
                 last_lut & 0xffffu, max_len | shift << 4 | quantum << 9};
    decode_block<kLong, kWaves, kStores, kKind, kBundle>(t, blockIdx.x, stream_cap_words(W, kLong ? ZM_MAX_CODE_LEN : 8u, quantum), long_slots);
}

// Stand-alone tensor recovery (Sec. 3.3): lane j merges values 8j..8j+7 of its wave's tiles -- per tile a 64-bit load from each
// input and one 128-bit store, all contiguous across the wave.  Bound by the memory.  A wave asks for all of its tiles before it merges
// the first; one, two, four and eight of them, us with buffers that are not cached: 58.7 M values (non-temporal stores, one wave per workgroup,
// four per SIMD) 42.0 (four waves per workgroup) / 39.5 / 39.6 / 40.7, 37.7 M 26.2 / 25.5 / 24.8 / 25.1.  Four waves per workgroup take 39.7 with
// four tiles; six or eight per SIMD 39.8.  With device-scope stores and four waves per workgroup, not cached 25 M 20.9 / 20.0 / 20.1 / -, 6.3 M 6.85 /
// 6.6 / 6.55 / -, three sets that stay cached 6.3 M 5.0 / 4.3 / 4.1 / -, 4.2 M 2.6 / 2.7 / 2.8 / -, 1 M 1.66 / 1.69 / 1.76 / -: small tensors
// need the waves.
template <Stores kStores, int kTiles, int kWaves>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(1, kStores == kStreaming ? 4 : 8)))
zm_recover_kernel(const uint8_t *__restrict__ e, const uint8_t *__restrict__ sm, uint16_t *__restrict__ out, uint64_t n)
{
    constexpr uint32_t kWaveValues = kTiles * kTile;
    const uint32_t lane = threadIdx.x & 63u;
    // the first workgroup takes the tensor's end, whose last wave takes longer than the others
    const uint64_t block = blockIdx.x ? blockIdx.x - 1u : (n - 1u) / (kWaves * kWaveValues);
    const uint64_t first = (block * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kWaveValues;
    if (first >= n) return;
    const uint32_t have = n - first < kWaveValues ? static_cast<uint32_t>(n - first) : kWaveValues;
    const Sink<kStores> sink(out + first, have, lane);
    if (have == kWaveValues) {
        const ByteSource es(e + first, have, lane), ss(sm + first, have, lane);
        uint2 ev[kTiles], sv[kTiles];
#pragma unroll
        for (int k = 0; k < kTiles; ++k) { ev[k] = es.load(k); sv[k] = ss.load(k); }
#pragma unroll
        for (int k = 0; k < kTiles; ++k) sink.store(static_cast<uint32_t>(k), recover8(ev[k], sv[k]));
        return;
    }
    // The tensor's last wave: whole groups of eight are read as above, past them nothing; the one lane that owns a part of a group reads
    // it byte by byte.  All at once: tile by tile this wave alone took a microsecond (7.0 M values, cached, 4.6 us).
    const ByteSource es(e + first, have & ~7u, lane), ss(sm + first, have & ~7u, lane);
    uint2 ev[kTiles], sv[kTiles];
#pragma unroll
    for (int k = 0; k < kTiles; ++k) { ev[k] = es.load(k); sv[k] = ss.load(k); }
    if ((have & 7u) && lane == (have >> 3 & 63u)) {
        const uint32_t group = have & ~7u, left = have & 7u;
        uint32_t eb[2] = {0u, 0u}, sb[2] = {0u, 0u};
#pragma unroll
        for (uint32_t q = 0; q < 7; ++q) {
            const uint64_t i = first + group + (q < left ? q : 0u);       // past the end: the group's first byte again
            eb[q >> 2] |= static_cast<uint32_t>(e[i]) << (8 * (q & 3));
            sb[q >> 2] |= static_cast<uint32_t>(sm[i]) << (8 * (q & 3));
        }
        sink.store_partial(have / kTile, recover8(make_uint2(eb[0], eb[1]), make_uint2(sb[0], sb[1])));
    }
#pragma unroll
    for (int k = 0; k < kTiles; ++k)
        if (k * kTile + lane * 8u + 8u <= have) sink.store(static_cast<uint32_t>(k), recover8(ev[k], sv[k]));
}

// Streams share a workgroup's LDS up to this size; one that is longer by itself is refused.  A table of long codes
// (0.5 to 4.3 KB) comes on top, so that the line does not depend on the tensor's symbols.
constexpr size_t kLdsLimit = 64 * 1024;
template <bool kLong>
constexpr size_t kBesideStreams = kLong ? 1056 : 2 * kTableEntries;
template <bool kLong>
constexpr size_t kStaticLds = kLong ? 16 : 2 * kTableEntries;
constexpr uint64_t kLastLevelCacheBytes = 256ull << 20;   // MI355X Infinity Cache
// What a launch leaves dirty in the L2 caches (eight of 4 MiB) is written back when it ends; device-scope stores spread that
// over the launch.  Experts of 1024 x 2048 x 3 (12 MiB each), us per call with ordinary / device-scope stores, short codes unless it says long:
//   out, MiB                              48            72            96            96, long      192           288
//   one set, all cached                   13.6 / 11.9   21.4 / 20.1   27.4 / 25.8   29.0 / 27.1   60.7 / 57.9   88.3 / 84.8
//   inputs from HBM, one output set       15.3 / 15.2   23.0 / 21.4   28.9 / 26.9   30.8 / 29.5   59.6 / 58.3   86.5 / 84.7
//   neither cached                        18.0 / 17.5   25.7 / 24.9   32.5 / 31.4   34.7 / 34.1   59.5 / 58.1   86.4 / 84.4
//   the same and a kernel that reads      26.1 / 25.2   36.9 / 35.5   46.9 / 45.6   49.1 / 47.8   92.3 / 90.9   143.9 / 141.3
// Device-scope stores are ahead in every row, and from streams of 512 to 16384 values, but for one place: launches of short codes that find
// places for all of their waves (up to 56 MiB) and take turns with two or three sets that stay cached.  There, from 38 MiB on (two
// sets in turn, MiB: 36 11.2 / 11.2, 38 11.4 / 12.4, 48 13.6 / 14.5, 52 15.3 / 15.6, 54 15.8 / 16.0), fewer waves help neither (three / four /
// five / six at 48 MiB: 14.0 / 14.4 / 14.7 / 14.5), and these keep ordinary stores.
constexpr uint64_t kThroughBytes = 36ull << 20;

// From seven eighths of the last-level cache on non-temporal stores are ahead whatever the caller does: outputs so large leave the cache before they are read or
// written again, and push out what is read meanwhile.  Below, the decode by itself is, but a product that reads the output next finds nothing of it in the
// cache.  us device-scope / non-temporal, experts of 1024 x 2048 x 3 (long codes), one output set; read: with a product over all of it:
//   out, MiB                              168                          192                          216                          228                          252
//   one set                               46.7 / 43.6  (56.6 / 44.7)   54.8 / 49.6  (62.7 / 50.5)   62.7 / 55.6  (69.0 / 57.0)   67.0 / 58.6  (73.4 / 59.9)   73.9 / 64.6  (80.1 / 65.6)
//   the same, read                        70.8 / 74.8  (74.8 / 76.6)   83.1 / 85.4  (86.6 / 88.8)   98.2 / 98.6  (102.0 / 103.5) 108.8 / 104.1 (113.9 / 112.8) 128.8 / 117.8 (132.6 / 125.5)
//   inputs from HBM                       45.8 / 48.9  (49.9 / 54.6)   57.4 / 55.4  (62.0 / 60.9)   64.0 / 62.2  (69.2 / 69.1)   66.9 / 65.4  (73.4 / 72.6)   73.8 / 71.9  (79.9 / 79.5)
//   the same, read                        71.6 / 80.4  (75.0 / 85.7)   82.5 / 90.9  (86.0 / 96.0)   99.0 / 101.3 (103.3 / 107.9) 109.7 / 106.6 (113.9 / 113.4) 127.4 / 117.1 (131.6 / 124.6)
//   neither cached, read                  78.1 / 80.7  (81.6 / 85.9)   92.4 / 90.6  (95.8 / 96.3)   107.5 / 101.2 (111.9 / 108.0) 113.8 / 106.3 (118.3 / 113.8) 128.0 / 116.8 (132.0 / 124.3)
// Experts of 512 x 1024 x 3, inputs from HBM, read: 192 84.1 / 91.9, 216 99.6 / 102.1, 228 109.8 / 107.2.
constexpr uint64_t kStreamingBytes = kLastLevelCacheBytes / 8 * 7;

// How a launch writes, for the caller's policy.
Stores stores_of(int policy, const Streams &s)
{
    return policy == ZM_STORES_STREAMING || (policy == ZM_STORES_AUTO && s.out_bytes() >= kStreamingBytes) ? kStreaming : kThrough;
}

// Where the shapes of a call's launches go when they are asked for instead of launched.
struct Recorder {
    zm_launch_shape *out;
    int cap;
    int n = 0;
};

// What a launch needs to know beside its kernel arguments.
struct Plan {
    Bundle bundle;
    dim3 grid;
    uint32_t n_tasks;
    size_t lds;              // dynamic part: the streams
    Streams streams;
    int stores;
    hipStream_t stream;
    Recorder *rec;
};

// args: an Args, or something that begins like one
template <bool kLong, int kWaves, Stores kStores, Kind kKind, int kBundle, class Args>
int launch_kernel(void *args, const Plan &p)
{
    void *argv[] = {args};
    const void *fn;
    if constexpr (std::is_same<Args, Few>::value) fn = reinterpret_cast<const void *>(&zm_decode_few_kernel<kLong, kWaves, kStores, kKind, kBundle>);
    else fn = reinterpret_cast<const void *>(&zm_decode_kernel<kLong, kWaves, kStores, kKind, kBundle, Args>);
    // the launch's own status: an error left behind by an earlier, unrelated call is not this call's
    return hipLaunchKernel(fn, p.grid, dim3(64 * kWaves), argv, p.lds, p.stream) == hipSuccess ? ZM_OK : ZM_E_HIP;
}

template <bool kLong, int kWaves, Kind kKind, class Args, int kBundle = 1>
int launch_stores(void *args, const Plan &p, Stores kind)
{
    if constexpr (kKind == kFitting && !kLong && kBundle == 1)
        if (kind == kThrough && p.streams.out_bytes() > kThroughBytes && p.streams.one_group == p.streams.n && p.streams.n <= kManyStreams)
            return launch_kernel<kLong, kWaves, kOrdinary, kKind, 1, Args>(args, p);
    if constexpr (kKind != kSparse)
        if (kind == kStreaming) return launch_kernel<kLong, kWaves, kStreaming, kKind, kBundle, Args>(args, p);
    return launch_kernel<kLong, kWaves, kThrough, kKind, kBundle, Args>(args, p);
}

// What bundle_of answers.
template <bool kLong, class Args>
int launch_bundles(void *args, const Plan &p, Stores kind)
{
    const bool many = p.bundle.kind == kMany;
    if (p.bundle.streams == 8u) return launch_stores<kLong, 2, kLong ? kMany : kFitting, Args, 8>(args, p, kind);
    if (p.bundle.streams == 4u) {
        if constexpr (kLong)
            if (many) return launch_stores<kLong, 2, kMany, Args, 4>(args, p, kind);
        return launch_stores<kLong, 2, kFitting, Args, 4>(args, p, kind);
    }
    if constexpr (kLong)
        if (many) return launch_stores<kLong, 2, kMany, Args, 2>(args, p, kind);
    return launch_stores<kLong, 2, kFitting, Args, 2>(args, p, kind);
}

template <bool kLong, int kWaves, class Args>
int launch_args(void *args, const Plan &p)
{
    const Stores kind = stores_of(p.stores, p.streams);
    if (p.rec) {
        if (p.rec->n < p.rec->cap)
            p.rec->out[p.rec->n] = zm_launch_shape{kLong ? 2u : 4u, static_cast<uint32_t>(kWaves), kind == kStreaming ? 1u : 0u, p.grid.x,
                                                   p.n_tasks, static_cast<uint32_t>(p.lds + kStaticLds<kLong>)};
        ++p.rec->n;
        return ZM_OK;
    }
    if constexpr (kWaves == 2) {
        if (p.bundle.streams > 1) return launch_bundles<kLong, Args>(args, p, kind);
        switch (kind_of(kLong, p.streams, kind)) {
        case kShortStreams: return launch_stores<kLong, kWaves, kShortStreams, Args>(args, p, kind);
        case kSparse: return launch_stores<kLong, kWaves, kSparse, Args>(args, p, kind);
        case kFitting: return launch_stores<kLong, kWaves, kFitting, Args>(args, p, kind);
        case kMany: return launch_stores<kLong, kWaves, kMany, Args>(args, p, kind);
        case kMixed:
            if constexpr (!kLong) return launch_stores<kLong, kWaves, kMixed, Args>(args, p, kind);
            break;
        case kDeep: break;
        }
    }
    return launch_stores<kLong, kWaves, kDeep, Args>(args, p, kind);
}

// Whether a launch numbers its workgroups through all tensors instead of giving every tensor as many as the largest has.
// Workgroups that exit at once still have to be started; finding the tensor by its first workgroup costs every wave one
// more read.  Calls of tensors whose lengths fall off, with everything marshalled beforehand (from Python a call of 24 tensors
// is bound by its marshalling), us with a workgroup row per tensor / numbered through:
//   24 tensors of 2.1 M values down to 1/3: 17.6 / 17.7, to 1/30: 10.0 / 9.0, to 1/300: 9.5 / 7.5
//   48 tensors of 0.5 M values to 1/3: 9.4 / 9.4, to 1/30: 9.1 / 6.8;  of 0.13 M values to 1/300: 5.9 / 5.9
bool number_through(uint64_t useful, uint64_t started)
{
    const uint64_t idle = started - useful;
    return idle > 2048 || (idle > 1024 && idle > useful);
}

template <bool kLong, int kWaves, int N>
int launch_tasks(Launch<N, true> &L, size_t cap, int stores, hipStream_t stream, Recorder *rec)
{
    const size_t streams = 4 * kWaves * cap, table = kLong ? 4 * long_table_words(L.long_slots) : 0;
    if (streams + kBesideStreams<kLong> > kLdsLimit) {
        if constexpr (kWaves > 1) return launch_tasks<kLong, kWaves / 2>(L, cap, stores, stream, rec);
        else return ZM_E_ARG;                   // stream too long to stage in LDS
    }
    Streams streams_of;
    for (uint32_t k = 0; k < L.n_tasks; ++k) streams_of.add(L.task[k].stream_values, L.task[k].n_streams, L.task[k].last_values, L.task[k].e_size);
    const Bundle bundle = kWaves == 2 ? bundle_of(kLong, streams_of, stores_of(stores, streams_of)) : Bundle{1u, kShortStreams};
    const size_t lds = streams * bundle.streams + table;       // dynamic part
    uint32_t blocks = 0;            // of the largest tensor
    uint64_t total = 0;
    for (uint32_t k = 0; k < L.n_tasks; ++k) {
        const uint32_t b = (waves_of(L.task[k].n_streams, L.task[k].last_values, bundle.streams) + kWaves - 1) / kWaves;
        L.first_block[k] = static_cast<uint32_t>(total);
        blocks = b > blocks ? b : blocks;
        total += b;
    }
    if (!blocks) return ZM_OK;
    // without the workgroup numbers the arguments are the same up to the end of the tasks
    using Rows = Launch<N, false>;
    using Through = Launch<N, true>;
    static_assert(offsetof(Through, task) == offsetof(Rows, task) && sizeof(Rows) <= sizeof(Through));
    // a launch admits 2^32 - 1 threads in x
    if (total <= UINT32_MAX / (64u * kWaves) && number_through(total, static_cast<uint64_t>(blocks) * L.n_tasks))
        return launch_args<kLong, kWaves, Through>(&L, Plan{bundle, dim3(static_cast<uint32_t>(total)), L.n_tasks, lds, streams_of, stores, stream, rec});
    return launch_args<kLong, kWaves, Rows>(&L, Plan{bundle, dim3(blocks, L.n_tasks), L.n_tasks, lds, streams_of, stores, stream, rec});
}

// Collects the tensors of one round length and launches them.
template <bool kLong>
struct Group {
    static constexpr uint32_t kLenBound = kLong ? ZM_MAX_CODE_LEN : 8;
    int n = 0;                        // tensors to come, all launches together
    bool may_share = false;           // they are many and large enough for packed launches; if so:
    uint64_t blocks = 0;              // workgroups of two streams that they need
    uint32_t most_blocks = 0;         // of the largest one
    bool packable = true;             // every one has the layout of a blob and an address that fits a Packed
    uint32_t n_shapes = 0;
    Shape shape[kMaxShapes];
    Packed packed[kMaxTensorsPerCall];

    static bool same(const Shape &a, const Shape &b)
    {
        return a.last_values == b.last_values && a.per_chunk == b.per_chunk && a.sm_offset == b.sm_offset && a.e_offset == b.e_offset && a.lut_offset == b.lut_offset &&
               a.table_offset == b.table_offset && a.stream_values == b.stream_values && a.streams_per_chunk == b.streams_per_chunk &&
               a.n_streams == b.n_streams && a.code == b.code;
    }

    // LDS words per wave that tensors of these streams need
    struct Cap {
        uint32_t max_stream = 0, max_quantum = 1, long_slots = 0;
        void see(const Task &t, const zm_tensor_info &ti)
        {
            const uint32_t slots = (ti.n_present < kTableEntries ? ti.n_present : kTableEntries) / 2;
            long_slots = long_slots > slots ? long_slots : slots;
            max_stream = max_stream > t.stream_values ? max_stream : t.stream_values;
            max_quantum = max_quantum > quantum_of(t.code) ? max_quantum : quantum_of(t.code);
        }
        size_t words() const { return stream_cap_words<size_t>(max_stream, kLenBound, max_quantum); }
    };
    Cap cap_of_all;

    // First pass: what the launches will have to hold.
    void count(const Task &t, const zm_tensor_info &ti)
    {
        ++n;
        if (!may_share) return;
        const uint32_t b = (t.n_streams + 1u) / 2u;
        blocks += b;
        most_blocks = most_blocks > b ? most_blocks : b;
        cap_of_all.see(t, ti);
        packable = packable && (packed[n - 1] = pack(t, ti)).high != kUnpackable;
    }

    static constexpr uint32_t kUnpackable = ~0u;      // no device address has all of bits 36..47 set

    // Whether the tensor's parts lie as in a blob at address b.
    static bool whole_blob(const Task &t, const zm_tensor_info &ti, uint64_t b)
    {
        return reinterpret_cast<uint64_t>(t.sm) == b + ti.sm_offset && reinterpret_cast<uint64_t>(t.echunks) == b + ti.e_offset &&
               reinterpret_cast<uint64_t>(t.table) == b + ti.table_offset && !(t.e_size & 255) && t.e_size >> 8 <= UINT32_MAX;
    }

    Packed pack(const Task &t, const zm_tensor_info &ti)
    {
        const Packed no{0, kUnpackable, 0, 0};
        const uint64_t b = reinterpret_cast<uint64_t>(t.lut) - ti.lut_offset, o = reinterpret_cast<uint64_t>(t.out);
        if (ti.lut_offset > UINT32_MAX || ti.table_offset > UINT32_MAX || !whole_blob(t, ti, b) || (b & 15) || b >> 48 || o >> 48) return no;
        const Shape s{ti.sm_offset, ti.e_offset, static_cast<uint32_t>(ti.lut_offset), static_cast<uint32_t>(ti.table_offset),
                      t.stream_values, t.streams_per_chunk, t.per_chunk, t.n_streams, t.last_values, t.code};
        uint32_t k;
        for (k = 0; k < n_shapes; ++k) if (same(shape[k], s)) break;
        if (k == n_shapes) {
            if (n_shapes == kMaxShapes) return no;
            shape[n_shapes++] = s;
        }
        return Packed{static_cast<uint32_t>(b >> 4), static_cast<uint32_t>(b >> 36) | k << 12 | static_cast<uint32_t>(o >> 36) << 20,
                      static_cast<uint32_t>(o >> 4), static_cast<uint32_t>(t.e_size >> 8)};
    }

    // Second pass: next(t) yields the group's tensors in order, with their descriptions.  Two streams per workgroup: on one MoE layer call of
    // 118 MB one, two and four waves per workgroup are within 1 % of each other, eight are 5 % slower.
    template <typename Next>
    int launch(Next next, int stores, hipStream_t stream, Recorder *rec)
    {
        if (n <= kFewTasks) {
            int rc;
            return launch_few(next, stores, stream, rec, rc) ? rc : launch_wide<kFewTasks>(next, stores, stream, rec);
        }
        if (may_share && packable && rows_pay() && 8 * cap_of_all.words() + kBesideStreams<kLong> <= kLdsLimit) return launch_packed(stores, stream, rec);
        return launch_wide<kMaxTasks>(next, stores, stream, rec);
    }

    // Where the tensors fit a Few: launches them, and sets rc.
    template <typename Next>
    bool launch_few(Next next, int stores, hipStream_t stream, Recorder *rec, int &rc)
    {
        Task t[kFewTasks];
        uint64_t blob[kFewTasks], low = UINT64_MAX, low_out = UINT64_MAX;
        const zm_tensor_info *ti = nullptr;
        Cap cap;
        for (int k = 0; k < n; ++k) {
            const zm_tensor_info &tk = next(t[k]);
            cap.see(t[k], tk);
            blob[k] = reinterpret_cast<uint64_t>(t[k].lut) - tk.lut_offset;
            const uint64_t out = reinterpret_cast<uint64_t>(t[k].out);
            if (blob[k] & 255 || !whole_blob(t[k], tk, blob[k])) return false;
            if (k && !(t[k].last_values == t[0].last_values && t[k].n_streams == t[0].n_streams && t[k].stream_values == t[0].stream_values &&
                       t[k].streams_per_chunk == t[0].streams_per_chunk && t[k].code == t[0].code && tk.lut_offset == ti->lut_offset &&
                       tk.table_offset == ti->table_offset && tk.sm_offset == ti->sm_offset && tk.e_offset == ti->e_offset)) return false;
            ti = &tk;
            low = low < blob[k] ? low : blob[k];
            low_out = low_out < out ? low_out : out;
        }
        const uint32_t shift = t[0].code >> 4 & 31u, quantum = quantum_of(t[0].code), W = t[0].stream_values;
        if (t[0].streams_per_chunk != 1u << shift || quantum > 255 || W / kTile > 127 || ti->lut_offset > 0xffff || ti->table_offset > UINT32_MAX ||
            (ti->sm_offset | ti->e_offset) & 255 || ti->e_offset >> 8 > UINT32_MAX) return false;
        Few F;
        const uint32_t lead[6] = {W / kTile | max_len_of(t[0].code) << 7 | shift << 11 | quantum << 16 | (kLong ? cap.long_slots : 0u) << 24, t[0].n_streams,
                                  t[0].last_values | static_cast<uint32_t>(ti->lut_offset) << 16, static_cast<uint32_t>(ti->table_offset),
                                  static_cast<uint32_t>(ti->sm_offset >> 8), static_cast<uint32_t>(ti->e_offset >> 8)};
        for (int i = 0; i < 6; ++i) F.lead[i] = lead[i];
        F.low = reinterpret_cast<const uint8_t *>(low);
        F.out = reinterpret_cast<uint16_t *>(low_out);
        for (int k = 0; k < kFewTasks; ++k) {
            const int j = k < n ? k : 0;
            const uint64_t to = (blob[j] - low) >> 8, to_out = (reinterpret_cast<uint64_t>(t[j].out) - low_out) >> 4;
            if (to > UINT32_MAX || to_out > UINT32_MAX) return false;
            F.to[k] = static_cast<uint32_t>(to);
            F.to_out[k] = static_cast<uint32_t>(to_out);
            F.e_units[k] = static_cast<uint32_t>(t[j].e_size >> 8);
        }
        const size_t words = cap.words(), table = kLong ? 4 * long_table_words(cap.long_slots) : 0;
        Streams streams_of;
        for (int k = 0; k < n; ++k) streams_of.add(W, t[k].n_streams, t[k].last_values, t[k].e_size);
        auto plan = [&](uint32_t waves) {
            const Bundle bundle = waves == 2 ? bundle_of(kLong, streams_of, stores_of(stores, streams_of)) : Bundle{1u, kShortStreams};
            return Plan{bundle, dim3((waves_of(t[0].n_streams, t[0].last_values, bundle.streams) + waves - 1) / waves, static_cast<uint32_t>(n)), static_cast<uint32_t>(n), 4 * waves * bundle.streams * words + table, streams_of, stores, stream, rec};
        };
        if (8 * words + kBesideStreams<kLong> <= kLdsLimit) rc = launch_args<kLong, 2, Few>(&F, plan(2));
        else if (4 * words + kBesideStreams<kLong> <= kLdsLimit) rc = launch_args<kLong, 1, Few>(&F, plan(1));
        else rc = ZM_E_ARG;                     // stream too long to stage in LDS
        return true;
    }

    template <int N, typename Next>
    int launch_wide(Next next, int stores, hipStream_t stream, Recorder *rec)
    {
        Launch<N, true> L;
        for (int left = n; left > 0; left -= static_cast<int>(L.n_tasks)) {
            L.n_tasks = static_cast<uint32_t>(left < N ? left : N);
            Cap cap;
            for (uint32_t k = 0; k < L.n_tasks; ++k) {
                const zm_tensor_info &ti = next(L.task[k]);
                cap.see(L.task[k], ti);
            }
            L.long_slots = cap.long_slots;
            L.stream_cap_words = static_cast<uint32_t>(cap.words());
            const int rc = launch_tasks<kLong, 2>(L, cap.words(), stores, stream, rec);
            if (rc != ZM_OK) return rc;
        }
        return ZM_OK;
    }

    // The same tensors in one launch where wide arguments would need one per 48 of them: a launch after another waits
    // for it to drain, and its first waves for their first bytes.  51 / 96 / 192 tensors of 512 x 1024: 21.3 / 37.7 /
    // 77.0 us in launches of 48, 19.1 / 35.2 / 65.4 us in one.
    // Packed launches have a row of workgroups per tensor, as many as the largest needs.  Workgroups that exit at once take
    // 0.2 ns each to start and a launch saved is worth 1.3 to 3.4 us, so lengths that fall off too far take the launches of
    // 48, which are numbered through; beside four times fewer that work, the idle ones start unnoticed.  us packed / in
    // launches of 48: one tensor of 14.7 M values and 191 of 0.13 M (113 K idle per launch saved, 70 for one that works)
    // 91.5 / 28.9; one of 2.9 M and 60 of 65536 (21 K, 25) 12.4 / 9.2; one of 2.1 M and 100 of 0.5 M (10 K, 3) 30.1 / 33.1.
    static constexpr uint64_t kIdlePerLaunch = 16384;
    bool rows_pay() const
    {
        const uint64_t idle = static_cast<uint64_t>(most_blocks) * static_cast<uint64_t>(n) - blocks;
        return idle <= kIdlePerLaunch * static_cast<uint64_t>(launches_of(kMaxTasks) - launches_of(kMaxPacked)) || idle <= 4 * blocks;
    }
    int launches_of(int tensors) const { return (n + tensors - 1) / tensors; }

    int launch_packed(int stores, hipStream_t stream, Recorder *rec)
    {
        const size_t cap = cap_of_all.words();
        PackedLaunch L;
        L.stream_cap_words = static_cast<uint32_t>(cap);
        L.long_slots = cap_of_all.long_slots;
        uint64_t n_values[kMaxShapes];
        for (uint32_t k = 0; k < n_shapes; ++k) {
            L.shape[k] = shape[k];
            n_values[k] = Streams::values_of(shape[k].stream_values, shape[k].n_streams, shape[k].last_values);
        }
        const int launches = launches_of(kMaxPacked), each = (n + launches - 1) / launches;
        for (int at = 0; at < n; at += static_cast<int>(L.n_tasks)) {
            L.n_tasks = static_cast<uint32_t>(n - at < each ? n - at : each);
            uint32_t blocks = 0, count[kMaxShapes] = {}, raw[kMaxShapes] = {};
            uint64_t e_bytes[kMaxShapes] = {};
            for (uint32_t k = 0; k < L.n_tasks; ++k) {
                L.task[k] = packed[at + static_cast<int>(k)];
                const uint32_t of = L.task[k].high >> 12 & (kMaxShapes - 1u);
                const uint64_t e_size = static_cast<uint64_t>(L.task[k].e_units) * 256u;
                ++count[of];
                raw[of] += Streams::is_raw(e_size, n_values[of]);
                e_bytes[of] += e_size;
            }
            Streams streams_of;
            for (uint32_t k = 0; k < n_shapes; ++k)
                if (count[k]) streams_of.add(shape[k].stream_values, shape[k].n_streams, n_values[k], count[k], raw[k], e_bytes[k]);
            const Bundle bundle = bundle_of(kLong, streams_of, stores_of(stores, streams_of));
            for (uint32_t k = 0; k < n_shapes; ++k) {
                const uint32_t b = (waves_of(shape[k].n_streams, shape[k].last_values, bundle.streams) + 1u) / 2u;
                if (count[k]) blocks = b > blocks ? b : blocks;
            }
            const int rc = launch_args<kLong, 2, PackedLaunch>(&L, Plan{bundle, dim3(blocks, L.n_tasks), L.n_tasks, 8 * bundle.streams * cap + (kLong ? 4 * long_table_words(L.long_slots) : 0), streams_of, stores, stream, rec});
            if (rc != ZM_OK) return rc;
        }
        return ZM_OK;
    }
};

// Checks one tensor's description and fills its task.  skip: the tensor is empty.
int make_task(const zm_tensor_parts &pt, const zm_tensor_info &ti, void *out, Task &t, bool &skip)
{
    skip = ti.n_values == 0;
    if (skip) return ZM_OK;
    if (!pt.table || !pt.chunk_offsets || !pt.sm || !pt.echunks || !out) return ZM_E_ARG;
    if ((reinterpret_cast<uintptr_t>(pt.table) & 15) || (reinterpret_cast<uintptr_t>(pt.chunk_offsets) & 7) ||
        (reinterpret_cast<uintptr_t>(pt.sm) & 15) || (reinterpret_cast<uintptr_t>(pt.echunks) & 15) ||
        (reinterpret_cast<uintptr_t>(out) & 15)) return ZM_E_ARG;
    if (ti.stream_values == 0 || ti.stream_values % kTile || ti.chunk_values == 0 || ti.chunk_values % ti.stream_values) return ZM_E_ARG;
    if (ti.max_len < 1 || ti.max_len > ZM_MAX_CODE_LEN) return ZM_E_ARG;
    const uint32_t span = (ti.max_len - 1) * (ti.stream_values / 64);
    if (ti.lane_quantum != (span + 254) / 255 + (span == 0)) return ZM_E_ARG;
    // no sum here may wrap past 2^64
    const uint64_t n_streams = (ti.n_values - 1) / ti.stream_values + 1;
    if (n_streams > 0x7FFFFFFFull) return ZM_E_ARG;
    if (ti.e_offset > ti.blob_size || ti.sm_offset > ti.e_offset || ((ti.n_values + 255) & ~255ull) > ti.e_offset - ti.sm_offset) return ZM_E_ARG;
    if (ti.table_stride != ((8u + 4u * (ti.chunk_values / ti.stream_values + 1u) + 7u) & ~7u)) return ZM_E_ARG;
    t.lut = static_cast<const uint8_t *>(pt.table);
    t.sm = static_cast<const uint8_t *>(pt.sm);
    t.echunks = static_cast<const uint8_t *>(pt.echunks);
    t.table = static_cast<const uint64_t *>(pt.chunk_offsets);
    t.out = static_cast<uint16_t *>(out);
    t.e_offset = ti.e_offset;
    t.e_size = ti.blob_size - ti.e_offset;
    t.stream_values = ti.stream_values;
    t.streams_per_chunk = ti.chunk_values / ti.stream_values;
    t.n_streams = static_cast<uint32_t>(n_streams);
    t.last_values = static_cast<uint32_t>(ti.n_values - (n_streams - 1) * ti.stream_values);
    // a power of two, the usual case, takes no division: this runs twice per tensor of a call
    const uint32_t shift = t.streams_per_chunk > 1 ? 32u - static_cast<uint32_t>(__builtin_clz(t.streams_per_chunk - 1)) : 0u;
    t.per_chunk = t.streams_per_chunk == 1u << shift ? 1u << 31
                                                     : static_cast<uint32_t>(((1ull << (31 + shift)) + t.streams_per_chunk - 1) / t.streams_per_chunk);
    t.code = ti.max_len | shift << 4 | ti.lane_quantum << 9;
    return ZM_OK;
}

// describe(i, t, skip, ti) fills tensor i's task and names its description, info(i) only names it; implemented by the entry
// points.
template <typename Describe, typename Info>
int decode_call(int n_tensors, Describe describe, Info info, int stores, hipStream_t stream, Recorder *rec = nullptr)
{
    if (stores != ZM_STORES_AUTO && stores != ZM_STORES_CACHED && stores != ZM_STORES_STREAMING) return ZM_E_ARG;
    Group<false> short_codes;
    Group<true> long_codes;
    if (n_tensors > kMaxTasks) {
        // Only what packed launches may take is looked over for them.  (With all tensors looked over, calls that the host
        // bounds took longer: 60 tensors of 8192 values 8.8 -> 9.3 us, 256 of 2048 26.6 -> 27.7.)
        uint64_t n_all = 0, n_short = 0, values_all = 0, values_short = 0;
        for (int i = 0; i < n_tensors; ++i) {
            const zm_tensor_info &ti = info(i);
            const uint64_t values = ti.n_values, is_short = ti.max_len <= 8;
            n_all += values != 0;
            values_all += values;
            n_short += (values != 0) & is_short;
            values_short += is_short ? values : 0;
        }
        auto share = [](uint64_t n, uint64_t values) { return n > kMaxTasks && values / kPackedValues >= n; };
        short_codes.may_share = share(n_short, values_short);
        long_codes.may_share = share(n_all - n_short, values_all - values_short);
    }
    // first pass: every tensor is checked before anything is launched
    for (int i = 0; i < n_tensors; ++i) {
        Task t; bool skip; const zm_tensor_info *ti;
        const int rc = describe(i, t, skip, ti);
        if (rc != ZM_OK) return rc;
        if (skip) continue;
        if (max_len_of(t.code) <= 8) short_codes.count(t, *ti);
        else long_codes.count(t, *ti);
    }
    // the tensors of one group, in the call's order
    auto members = [&](bool want_short) {
        return [&, want_short, i = 0](Task &t) mutable -> const zm_tensor_info & {
            for (;;) {
                bool skip; const zm_tensor_info *ti;
                describe(i++, t, skip, ti);
                if (!skip && (max_len_of(t.code) <= 8) == want_short) return *ti;
            }
        };
    };
    if (short_codes.n) {
        const int rc = short_codes.launch(members(true), stores, stream, rec);
        if (rc != ZM_OK) return rc;
    }
    return long_codes.n ? long_codes.launch(members(false), stores, stream, rec) : ZM_OK;
}

}  // namespace

extern "C" int zm_decode_tensors(const zm_tensor_parts *parts, const zm_tensor_info *infos, int n_tensors,
                                 void *const *out_bf16, void *stream)
{
    if (n_tensors == 0) return ZM_OK;
    if (!parts || !infos || !out_bf16 || n_tensors < 0 || n_tensors > kMaxTensorsPerCall) return ZM_E_ARG;
    auto describe = [&](int i, Task &t, bool &skip, const zm_tensor_info *&ti) {
        ti = infos + i;
        return make_task(parts[i], *ti, out_bf16[i], t, skip);
    };
    return decode_call(n_tensors, describe, [&](int i) -> const zm_tensor_info & { return infos[i]; }, ZM_STORES_AUTO, static_cast<hipStream_t>(stream));
}

extern "C" int zm_decode_launch_shapes(const zm_tensor_info *infos, int n_tensors, int stores,
                                       zm_launch_shape *shapes_out, int shapes_cap, int *n_shapes)
{
    if (!infos || n_tensors < 0 || n_tensors > kMaxTensorsPerCall || shapes_cap < 0 || (shapes_cap && !shapes_out) || !n_shapes) return ZM_E_ARG;
    // the same path as a decode call, with placeholder addresses and a recorder in place of the launches; the parts lie as
    // in a blob, where that keeps them aligned
    uint8_t *const somewhere = reinterpret_cast<uint8_t *>(uintptr_t{4096});
    Recorder rec{shapes_out, shapes_cap};
    auto describe = [&](int i, Task &t, bool &skip, const zm_tensor_info *&described) {
        const zm_tensor_info &ti = *(described = infos + i);
        const bool aligned = !((ti.lut_offset | ti.sm_offset | ti.e_offset) & 15) && !(ti.table_offset & 7);
        const zm_tensor_parts pt = aligned ? zm_tensor_parts{somewhere + ti.lut_offset, somewhere + ti.table_offset, somewhere + ti.sm_offset, somewhere + ti.e_offset}
                                           : zm_tensor_parts{somewhere, somewhere, somewhere, somewhere};
        return make_task(pt, ti, somewhere, t, skip);
    };
    const int rc = decode_call(n_tensors, describe, [&](int i) -> const zm_tensor_info & { return infos[i]; }, stores, nullptr, &rec);
    *n_shapes = rec.n;
    return rc;
}

extern "C" int zm_decode_experts_stores(const void *const *blobs, const uint64_t *const *chunk_offsets,
                                        const zm_tensor_info *infos, int n_experts, int tensors_per_expert,
                                        const int32_t *expert_ids, int n_selected,
                                        void *const *out_bf16, int stores, void *stream)
{
    if (n_selected == 0) return ZM_OK;
    if (!blobs || !chunk_offsets || !infos || !expert_ids || !out_bf16) return ZM_E_ARG;
    if (n_experts <= 0 || tensors_per_expert <= 0 || n_selected < 0) return ZM_E_ARG;
    if (static_cast<long>(n_selected) * tensors_per_expert > kMaxTensorsPerCall) return ZM_E_ARG;
    for (int j = 0; j < n_selected; ++j)
        if (expert_ids[j] < 0 || expert_ids[j] >= n_experts) return ZM_E_ARG;
    auto index = [&](int i) { return static_cast<size_t>(expert_ids[i / tensors_per_expert]) * tensors_per_expert + i % tensors_per_expert; };
    auto describe = [&](int i, Task &t, bool &skip, const zm_tensor_info *&described) {
        const size_t src = index(i);
        const zm_tensor_info &ti = *(described = infos + src);
        skip = ti.n_values == 0;
        if (skip) return ZM_OK;
        if (!blobs[src]) return ZM_E_ARG;
        const uint8_t *blob = static_cast<const uint8_t *>(blobs[src]);
        const zm_tensor_parts pt{blob + ti.lut_offset, chunk_offsets[src], blob + ti.sm_offset, blob + ti.e_offset};
        return make_task(pt, ti, out_bf16[i], t, skip);
    };
    return decode_call(n_selected * tensors_per_expert, describe, [&](int i) -> const zm_tensor_info & { return infos[index(i)]; }, stores, static_cast<hipStream_t>(stream));
}

extern "C" int zm_decode_experts(const void *const *blobs, const uint64_t *const *chunk_offsets,
                                 const zm_tensor_info *infos, int n_experts, int tensors_per_expert,
                                 const int32_t *expert_ids, int n_selected,
                                 void *const *out_bf16, void *stream)
{
    return zm_decode_experts_stores(blobs, chunk_offsets, infos, n_experts, tensors_per_expert, expert_ids, n_selected,
                                    out_bf16, ZM_STORES_AUTO, stream);
}

extern "C" int zm_recover(const void *exponents, const void *sign_mantissa, size_t n_values, void *out_bf16, void *stream)
{
    if (n_values == 0) return ZM_OK;
    if (!exponents || !sign_mantissa || !out_bf16) return ZM_E_ARG;
    if ((reinterpret_cast<uintptr_t>(exponents) & 7) || (reinterpret_cast<uintptr_t>(sign_mantissa) & 7) ||
        (reinterpret_cast<uintptr_t>(out_bf16) & 15)) return ZM_E_ARG;
    constexpr uint64_t kSmallTensor = 5ull << 20;
    constexpr int kRecoverTiles = 4;
    const uint8_t *e = static_cast<const uint8_t *>(exponents), *sm = static_cast<const uint8_t *>(sign_mantissa);
    uint16_t *out = static_cast<uint16_t *>(out_bf16);
    uint64_t n = n_values;
    // A launch that moves more than half of the last-level cache (four bytes per value) writes with non-temporal
    // stores: measured on 58.7 M-value tensors 40.5 against 42.0 us with one tile per wave.  Smaller ones write with device-scope
    // stores.  us, ordinary / device-scope (one tile):
    //   values                                                    1.0 M        1.6 M        2.1 M        2.9 M        4.2 M        5.0 M
    //   exponents just copied from the host, nothing else cached   3.63 / 3.58  4.01 / 3.91  4.48 / 4.16  4.93 / 4.63  5.80 / 5.57  7.08 / 6.69
    //   values                                                    1.0 M        1.6 M        2.4 M        3.0 M        4.2 M        4.6 M
    //   three sets in turn                                         2.04 / 1.96  2.18 / 2.19  2.47 / 2.31  2.79 / 2.51  3.36 / 2.76  4.26 / 3.22
    //   nothing cached, graph replay                               2.47 / 2.59  3.21 / 3.45  3.84 / 3.95  4.26 / 4.42  4.86 / 4.98  5.84 / 5.94
    // The first row, taken from the profiler's trace, is what recovery is for: exponent bytes that the host has decompressed arrive by a copy, which
    // leaves them in the last-level cache.  The last is the one in which ordinary stores are ahead.  One tile against four: 4.6 M three sets
    // 3.22 / 3.22, one set 2.86 / 3.15, not cached 5.94 / 6.09, 5.2 M 3.15 / 3.28 (one set), 6.40 / 6.35; 6.0 M three sets 4.43 / 4.20.
    const bool streaming = 4 * n > kLastLevelCacheBytes / 2, small = n <= kSmallTensor;
    const uint64_t per_block = small ? 4 * kTile : streaming ? kRecoverTiles * kTile : 4 * kRecoverTiles * kTile;
    const uint64_t blocks = (n + per_block - 1) / per_block;
    if (blocks > 0x7FFFFFFFull) return ZM_E_ARG;
    void *args[] = {&e, &sm, &out, &n};
    const void *fn = streaming ? reinterpret_cast<const void *>(&zm_recover_kernel<kStreaming, kRecoverTiles, 1>)
                     : small   ? reinterpret_cast<const void *>(&zm_recover_kernel<kThrough, 1, 4>)
                               : reinterpret_cast<const void *>(&zm_recover_kernel<kThrough, kRecoverTiles, 4>);
    return hipLaunchKernel(fn, dim3(static_cast<uint32_t>(blocks)), dim3(streaming ? 64 : 256),
                           args, 0, static_cast<hipStream_t>(stream)) == hipSuccess ? ZM_OK : ZM_E_HIP;
}
