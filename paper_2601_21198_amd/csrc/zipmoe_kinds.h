// Which kernel decodes a launch: what its streams are, how many waves of it a SIMD holds at most and how early a wave asks for its
// sign-mantissa bytes.  Plain C++: the rule is host code, its answers are template arguments of the kernels.
//
// A launch that finds places for all of its waves is the faster the more it has; one that does not is bound by the memory, which serves fewer
// waves, with fewer places open at a time, faster -- if they decode straight through.  Streams that do not (shorter than a group of tiles, no
// whole groups, raw) wait for each tile and need the waves.  Figures are us, GPU time by graph replay, of experts of 1024 x 2048 x 3
// with inputs and outputs that are not cached unless they say otherwise; nt: non-temporal stores, dev: device-scope stores.
#pragma once
#include <cstdint>

namespace zipmoe {

constexpr uint32_t kTile = 512;
constexpr int kGroup = 8;                 // tiles of a stream that are decoded straight through; tile i and tile 7 - i are a pair
constexpr int kPairs = kGroup / 2;
constexpr uint32_t kGroupValues = kGroup * kTile;
constexpr uint64_t kSimds = 1024;         // 256 CUs of four
constexpr uint64_t kManyStreams = 7 * kSimds;      // that many are at work at a time with seven waves per SIMD

// How a wave writes its bf16 words.
//   kOrdinary   the lines stay dirty in the L2 caches; what is left of them is written back when the kernel ends
//   kThrough    device-scope stores: the L2 caches keep the line and pass it on to the last-level cache at once
//   kStreaming  non-temporal: the output fills most of the last-level cache, or the caller said that its buffers are
//               not cache-resident
enum Stores { kOrdinary, kThrough, kStreaming };

//   kShortStreams  streams shorter than a group: bound by their waves' latencies, so as many as go
//   kSparse        of one group, so few that a wave has its SIMD (nearly) to itself, dev
//   kFitting       of one group, in launches that find places for all of their waves, or nearly; streams of no whole groups and raw ones whatever their number
//   kMany          of one group, in launches of more
//   kMixed         of one group and of other lengths in one launch; long ones of no whole groups
//   kDeep          of several whole groups
enum Kind { kShortStreams, kSparse, kFitting, kMany, kMixed, kDeep };

// What a launch decodes.
struct Streams {
    uint64_t n = 0;
    uint64_t one_group = 0, in_groups = 0;       // of tensors whose streams are one whole group of tiles, and several
    uint64_t values = 0, raw_values = 0;         // values, and those of tensors that are stored raw
    uint64_t e_bytes = 0;                        // in the E-chunk regions
    uint32_t longest = 0, shortest = ~0u;        // values of the longest and the shortest kind of stream
    // tensors cut alike, `raw` of them stored raw
    void add(uint32_t stream_values, uint32_t n_streams, uint64_t n_values, uint32_t tensors, uint32_t raw, uint64_t e_size)
    {
        const uint64_t streams = static_cast<uint64_t>(tensors) * n_streams;
        n += streams;
        one_group += stream_values == kGroupValues ? streams : 0u;
        in_groups += stream_values > kGroupValues && stream_values % kGroupValues == 0 ? streams : 0u;
        values += tensors * n_values;
        raw_values += raw * n_values;
        e_bytes += e_size;
        longest = longest > stream_values ? longest : stream_values;
        shortest = shortest < stream_values ? shortest : stream_values;
    }
    void add(uint32_t stream_values, uint32_t n_streams, uint32_t last_values, uint64_t e_size)
    {
        const uint64_t n_values = values_of(stream_values, n_streams, last_values);
        add(stream_values, n_streams, n_values, 1u, is_raw(e_size, n_values), e_size);
    }
    static constexpr uint64_t values_of(uint32_t stream_values, uint32_t n_streams, uint32_t last_values)
    {
        return static_cast<uint64_t>(n_streams - 1u) * stream_values + last_values;
    }
    static constexpr bool is_raw(uint64_t e_size, uint64_t n_values) { return e_size >= n_values; }        // a coded chunk is smaller than a raw one
    uint64_t out_bytes() const { return 2 * values; }
};

// stores: kThrough or kStreaming.
//   kDeep / kMixed, longer streams.  A launch of nothing but whole groups: three waves (most_waves).  With 23 tensors in streams of 4096 values, one
//     of 8192 ran dev 35.2 with three waves and all pairs ahead, 31.8 as kMixed (nt 29.9 / 28.9); with 23 of 1024 values 53.1 / 39.2.  nt keeps kDeep
//     from half the streams on: of eight tensors of 8192 and four of 4096, 17.4 against 19.1 (dev 21.9 / 21.5).  Whole groups need it, the
//     others are held by LDS at four waves or less: of 10240 values 16 experts nt 70.0 as kDeep, 65.5 as kMixed, dev 73.4 / 68.7.  Long codes have
//     no kMixed: as kDeep they are ahead there (10240 values, eight experts dev 44.6, 47.1 as kFitting).
//   no whole groups, longer than one: 6144 values, four experts nt 20.9 with three waves, 18.3 with seven, dev 23.9 / 20.2; long codes, 4608 values,
//     eight experts dev 43.6 with three, 38.6 with five.
//   kShortStreams: 3072 values, eight experts nt 33.8 with eight waves, 33.2 with seven.  Long codes: 2048 values, eight experts nt
//     38.9 with eight, 36.2 with five, but two (6144 streams, which find places) 9.1 / 9.9, all cached; 1024 values, eight dev 39.3 / 41.6.
//   kMixed, streams of one group and others: 23 tensors of 4096 values and one of 1024 nt 32.4 with three waves, 32.6 with seven, 30.6 as kMixed, dev 34.6 /
//     33.6 / 32.5.  Where the others are more it is kFitting: one of 4096 and 23 of 1024 nt 33.5 as kMixed, 31.8 as kFitting, dev 36.1 / 33.6.
//   kSparse: see pairs_ahead.
//   raw: every chunk of a tensor's, eight experts nt 37.0 with three waves, 34.8 with seven, dev 40.1 / 37.2.  (Dense codes are not raw: eight experts with
//     codes of seven bits dev 37.3 with three, 39.3 with seven.)
inline Kind kind_of(bool long_codes, const Streams &s, Stores stores)
{
    const bool streaming = stores == kStreaming;
    if (s.in_groups || s.longest > 2 * kGroupValues)
        return long_codes || s.in_groups == s.n || (streaming && 2 * s.in_groups >= s.n) ? kDeep : kMixed;
    if (s.longest <= 1024u || (s.longest < kGroupValues && (long_codes ? s.n <= 8 * kSimds : s.longest <= 2048u))) return kShortStreams;
    if (s.one_group < s.n) return !long_codes && 2 * s.one_group >= s.n ? kMixed : kFitting;
    if (!streaming && s.n <= (long_codes ? kSimds : 3 * kSimds)) return kSparse;
    return s.n > (long_codes && !streaming ? 5 * kSimds : kManyStreams) && 2 * s.raw_values <= s.values ? kMany : kFitting;
}

// Waves that a SIMD holds at most (the registers would admit six to eight; the compiler is told, and reserves what keeps the others out.
// Keeping them out by LDS instead is not as good: four experts with long codes nt 20.0 against 19.2).
//   kShortStreams  eight experts in streams of 512 values at seven / eight waves: 31.6 / 30.3, long codes at five / eight 48.1 / 38.7
//   kFitting       four experts (6144 streams), all cached, at three / five / seven waves: 14.9 / 14.4 / 13.5.  Long codes at four / five: three experts
//                  (4608) dev, three sets cached 12.9 / 11.6, four (6144) nt 19.9 / 19.3, dev 20.0 / 20.7
//   kMany          three; at three / four / six: one layer of 4096 x 4096 x 3 nt 29.7 / 30.2 / 30.8, two 55.4 / 56.1 / 57.1, two of
//                  14336 x 4096 x 3 185.4 / 189.1 / 190.7, dev one of 4096 x 4096 x 3 31.1 / 31.0 / 31.5, two 57.3 / 58.2 / 59.1, 48 of 512 x 1024 x 3
//                  44.8 / 45.1 / 45.8 (five).  Long codes four: eight experts nt at four / five / eight 31.8 / 32.8 / 34.6, dev 34.4 / 34.6 / 35.5
//   kMixed         six, of what LDS admits: 11 tensors of 4096 values and one of 1024 dev 18.9 at four, 18.6 at six, one of 8192 and 11 of 1024 23.1 / 21.3
//   kDeep          three.  8192 values, four / eight / 16 experts at three 15.1 / 26.9 / 61.8, at four 16.2 / 26.9 / 62.1, uncapped 16.2 / 28.4 /
//                  63.6; of longer ones LDS holds fewer
constexpr int most_waves(Kind kind, bool long_codes)
{
    return kind == kShortStreams ? 8 : kind == kSparse || kind == kFitting ? (long_codes ? 5 : 7) : kind == kMany ? (long_codes ? 4 : 3) : kind == kMixed ? 6 : 3;
}

// Pairs of tiles of a group whose sign-mantissa bytes a wave asks for before it decodes the first; pair i + that many is asked for when pair i is
// done.  All up front, the thousands of waves that start together queue behind each other's late tiles; few, a wave waits for a load
// behind its own stores.
//   short codes    two: four experts of 2048 x 1408 x 3 nt with four / three / two ahead 18.98 / 18.91 / 18.86, 16 experts 57.9 / 56.0 / 55.6 (one 59.2).
//                  kFitting dev one: two experts of 2048 x 1408 x 3 (4224 streams), three sets cached, two / one 11.1 / 10.2, three 11.2 / 10.9; up to
//                  three waves per SIMD two: one expert 7.0 / 7.7; with ordinary stores no difference (four experts 18.1 / 18.0): two.  kMixed nt
//                  four: 23 tensors of 4096 values and one of 1024 two / four 32.2 / 30.6
//   long codes     nt four: one / four: two experts 10.8 / 10.3, eight 34.3 / 31.8, four of 2048 x 1408 x 3 25.0 / 24.4, 16 60.1 / 60.7, two of
//                  14336 x 4096 x 3 193.7 / 198.3.  dev one: one / four: two experts 11.8 / 13.9, eight 34.4 / 35.2; up to one wave per SIMD four: 12
//                  tensors of 300001 values (888 streams) 7.7 / 6.8, one expert (1536) 8.8 / 9.0
constexpr int pairs_ahead(Kind kind, bool long_codes, Stores stores)
{
    if (kind == kShortStreams) return 2;         // never straight through
    if (kind == kDeep) return kPairs;
    if (stores == kStreaming) return long_codes || kind == kMixed ? kPairs : 2;
    return kind == kSparse ? (long_codes ? kPairs : 2) : long_codes || (kind == kFitting && stores == kThrough) ? 1 : 2;
}

// Streams of 512, 1024 and 2048 values, all of a launch cut alike: whether a wave takes eight tiles of them, and the kind of kernel that does it
// (kFitting or kMany; streams == 1: it does not).
struct Bundle {
    uint32_t streams;
    Kind kind;
};

// us, three tensors of Gaussian weights, a wave per stream / bundles as kFitting / as kMany (one figure where there is only one); cached: three sets in
// turn, device-scope stores; else nothing cached.
//   short codes, streams        cached                 dev                    nt
//     512:   9000              5.2 /  5.4             6.9 /  6.9             6.6 /  6.6
//           24000              9.9 /  8.5            12.8 / 10.5            12.5 /  9.8
//    1024:  12000              8.5 /  8.2            10.5 / 10.1            10.6 /  9.2
//           24000             14.3 / 15.2            17.7 / 18.7            17.0 / 18.0
//    2048:   6500              9.0 /  8.7 / 10.3     11.9 / 10.8 / 12.3     10.4 /  9.4
//            8000             10.3 /  9.9 / 11.2     14.2 / 12.8 / 13.9     11.9 / 10.7
//           12000             14.2 / 14.9 / 14.0     18.6 / 18.1 / 17.6     17.4 / 17.7
//           24000             31.9 / 32.0 / 30.9     32.0 / 32.0 / 31.0     30.3 / 31.2
//           24576, 24 tensors 32.1 /      / 33.2     32.0 /      / 33.1     31.0
//   long codes
//     512:   8000              5.5 /  6.2             7.3 /  7.2             7.0 /  7.1
//            9500              6.3 /  6.3             8.2 /  7.8             7.8 /  7.4
//           24000             11.9 /  8.5            14.6 / 10.8            13.9 / 10.7
//    1024:   6000              6.1 /  6.5 /  6.4      7.9 /  7.8 /  7.7      7.5 /  7.4 /  7.6
//            8000              7.2 /  6.8 /  6.7     10.1 /  8.8 /  8.9      9.4 /  7.8 /  8.8
//           16000             11.7 / 10.2 / 11.9     15.3 / 14.7 / 14.5     13.3 / 11.9 / 13.1
//           24000             15.8 / 15.7 / 14.6     19.9 / 19.5 / 19.0     19.1 / 19.1 / 18.3
//    2048:   3000              6.2 /  6.7 /  6.3      8.5 /  7.9 /  7.7      7.3 /  7.5 /  7.6
//            4500              7.4 /  8.0 /  7.7     10.7 /  9.8 /  9.5      9.5 /  9.2 /  9.4
//            6500              9.2 /  9.0 / 10.7     13.5 / 11.5 / 12.6     11.9 / 11.1 / 12.0
//            8000             10.6 /  9.9 / 11.8     15.7 / 14.1 / 14.1     12.9 / 12.0 / 13.0
//           12000             14.5 / 15.3 / 14.5     20.4 / 19.0 / 18.5     18.4 / 18.8 / 17.6
//           24000             35.3 / 33.7 / 32.2     35.8 / 33.8 / 32.2     32.5 / 32.4 / 31.3
//   denser long codes, a wave per stream / bundles; e: bytes a stream
//     512:   9500, e 296          6.5 /  6.5             8.2 /  7.9             7.9 /  7.6
//            9500, e 347          6.7 /  6.9             8.2 /  9.2             8.0 /  8.4
//           12000, e 347          7.6 /  7.1             9.6 /  9.6             9.2 /  9.0
//           24000, e 347         12.3 / 10.1            14.6 / 12.7            14.2 / 12.0
//    1024:   8000, e 521          7.3 /  7.6             9.9 /  9.0             9.7 /  8.7
//           12000, e 521          9.7 /  9.5            11.9 / 11.0            11.9 / 11.4
//            8000, e 623          7.6 /  8.2            10.2 /  9.4             9.9 /  9.2
//           24000, e 623         19.1 / 19.5            20.4 / 20.0            19.6 / 19.1
//    2048:   8000, e 976         11.5 / 11.8            16.1 / 14.8            13.5 / 13.4
//           12000, e 976         18.7 / 18.4            22.2 / 19.5            20.0 / 18.6
// So waves of one stream stay where all of them find places, and for short codes in large launches where they are bound by the memory
// already (2048 values as kMany gain with three large tensors, but lose with the many of a usual call); device-scope stores of few streams that stay cached decide where the lines lie, though cold ones would gain earlier.  Raw tensors are not
// bundled, nor streams of more than a kilobyte, nor what has no room for its streams at all.  Raw chunks among coded ones make no difference.  What is left: 4096 long
// codes of rare symbols in a row, 2048 values a stream, where most rounds are done again: one such piece in a hundred, 6500 streams, 10.7 / 12.2, 14.7 / 15.2, 12.5 / 13.7.
inline Bundle bundle_of(bool long_codes, const Streams &s, Stores stores)
{
    const Bundle none{1u, kShortStreams};
    if (s.shortest != s.longest || 2 * s.raw_values > s.values || s.e_bytes > 1024 * s.n || s.e_bytes < 80 * s.n) return none;
    const bool streaming = stores == kStreaming;
    // long codes: more bytes a stream than these, of which 64 are lengths
    auto denser = [&](uint64_t bytes) { return long_codes && s.e_bytes > bytes * s.n; };
    switch (s.longest) {
    case 512u: return s.n > (denser(320) ? 12 : 9) * kSimds ? Bundle{8u, long_codes ? kMany : kFitting} : none;
    case 1024u:
        if (!streaming && denser(576)) return none;
        if (s.n <= (streaming ? (long_codes ? 7 : 8) : denser(464) ? 12 : long_codes ? 7 : 10) * kSimds) return none;
        return s.n <= 16 * kSimds ? Bundle{4u, kFitting} : long_codes ? Bundle{4u, kMany} : none;
    case 2048u:
        if (s.n <= (streaming ? (long_codes ? 4 : 5) : denser(864) ? 9 : 6) * kSimds) return none;
        return s.n <= 9 * kSimds ? Bundle{2u, kFitting} : long_codes ? Bundle{2u, kMany} : none;
    default: return none;
    }
}

constexpr int bundle_waves(Kind kind, bool long_codes) { return kind == kMany ? 3 : long_codes ? 5 : 6; }
// Tiles whose sign-mantissa bytes are asked for before the first is decoded.  Bundles of short codes as kFitting, nt, with eight / four: 12000 streams of 1024
// values 9.1 / 10.0 us; dev 10.5 / 10.1.
constexpr uint32_t bundle_ahead(Kind kind, Stores stores) { return kind == kFitting && stores == kStreaming ? 8u : 4u; }

// Whole bundles of a tensor: none holds a stream that is cut off.
constexpr uint32_t whole_bundles(uint32_t n_streams, uint32_t last_values, uint32_t bundle)
{
    return (n_streams - (last_values % (kGroupValues / bundle) ? 1u : 0u)) / bundle;
}
// Waves that a tensor takes: one for every whole bundle, and for every stream behind them.
constexpr uint32_t waves_of(uint32_t n_streams, uint32_t last_values, uint32_t bundle)
{
    return bundle == 1u ? n_streams : n_streams - whole_bundles(n_streams, last_values, bundle) * (bundle - 1u);
}
}  // namespace zipmoe
