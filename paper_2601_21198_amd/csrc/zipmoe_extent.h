// Whether what a chunk-table entry points at lies in its blob's E-chunk region.  The kernels read nothing else of a blob at a place
// that the blob itself names, so these are what stands between a damaged table and a read out of range: written without a sum
// that could wrap.  (constexpr: for host and device.)
#pragma once
#include <cstdint>

#include "zipmoe.h"

namespace zipmoe {

constexpr uint32_t kLaneBytes = 64;   // a stream opens with one length byte per lane

// The coded stream at bytes o0..o1 of the chunk at blob offset `chunk`, with the region at e_offset, e_size bytes long; e_offset + e_size is
// the blob's size, so a chunk in front of the region comes out behind its end.
constexpr bool stream_inside(uint64_t chunk, uint32_t o0, uint32_t o1, uint64_t e_offset, uint64_t e_size)
{
    const uint64_t at = chunk - e_offset;
    return at <= e_size && o1 <= e_size - at && o1 >= o0 && o1 - o0 >= kLaneBytes;
}

// The raw stream of `bytes` bytes that starts `first` bytes into the chunk.
constexpr bool raw_stream_inside(uint64_t chunk, uint64_t first, uint32_t bytes, uint64_t e_offset, uint64_t e_size)
{
    const uint64_t at = chunk - e_offset;
    return at <= e_size && first <= e_size - at && bytes <= e_size - at - first;
}

}  // namespace zipmoe
