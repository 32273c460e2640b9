// zipmoe_cache.hip built as host code, with a runtime that knows which memory a kernel could reach.  Each scenario
// creates a cache of two experts, one tensor each, fetches both and prints what moved and whether a launch would have
// left mapped memory:  "<bytes that differ> <parts by kernel> <parts by copy> <unmapped reads> <misaligned parts>"
// With a third argument that names how a fetch ends it prints how many copies and launches nothing has waited for when the
// cache is gone.
#include "zipmoe_cache.hip"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string_view>

thread_local dim3 blockIdx, threadIdx;

static std::map<const uint8_t *, size_t> allocations;      // mapped host memory: start, bytes
static long by_kernel, by_copy, unmapped, misaligned;
static hipError_t last_error = hipSuccess;

static std::map<const uint8_t *, size_t>::iterator allocation_of(const void *p)
{
    const uint8_t *q = static_cast<const uint8_t *>(p);
    auto it = allocations.upper_bound(q);
    if (it == allocations.begin()) return allocations.end();
    --it;
    return q < it->first + it->second ? it : allocations.end();
}

hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    *a = hipPointerAttribute_t{};
    if (allocation_of(p) != allocations.end()) { a->type = hipMemoryTypeHost; a->devicePointer = a->hostPointer = const_cast<void *>(p); }
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p)
{
    const auto it = allocation_of(p);
    if (it == allocations.end()) return last_error = hipErrorNotFound;
    *base = const_cast<uint8_t *>(it->first); *size = it->second;
    return hipSuccess;
}

// What is under way: work is numbered per stream; an event, and a stream, know up to which number each stream's is over once they are passed.
using Passed = std::map<hipStream_t, long>;
static std::map<hipStream_t, long> issued;
static std::map<hipStream_t, Passed> behind;
static std::map<hipEvent_t, Passed> recorded;
static std::map<hipEvent_t, bool> in_capture;              // recorded in a capture: nothing outside of it can wait for that
static Passed over;                                        // what the host has waited for
static bool capturing;                                     // the caller's stream
static uintptr_t handles;
static void pass(Passed &to, const Passed &from) { for (const auto &[s, n] : from) to[s] = std::max(to[s], n); }
static void issue(hipStream_t s) { if (!capturing) ++issued[s]; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(++handles); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = reinterpret_cast<hipEvent_t>(++handles); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    in_capture[e] = capturing;
    recorded[e].clear();
    if (!capturing) { recorded[e] = behind[s]; recorded[e][s] = issued[s]; }
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    if (in_capture[e] && !capturing) return last_error = hipErrorCapturedEvent;
    pass(behind[s], recorded[e]);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { pass(over, behind[s]); over[s] = issued[s]; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *status)
{
    *status = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
static long under_way() { long n = 0; for (const auto &[s, k] : issued) n += k - over[s]; return n; }

hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind kind, hipStream_t stream)
{
    issue(stream);
    std::memcpy(dst, src, bytes);
    by_copy += kind == hipMemcpyHostToDevice;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t, hipStream_t stream)
{
    issue(stream);
    if (kernel != reinterpret_cast<const void *>(&zm_cache_fetch_kernel)) std::abort();
    const Parts P = *static_cast<const Parts *>(args[0]);
    by_kernel += P.n_parts;
    for (uint32_t k = 0; k < P.n_parts; ++k) {
        misaligned += ((reinterpret_cast<uintptr_t>(P.part[k].src) | reinterpret_cast<uintptr_t>(P.part[k].dst)) & 15) != 0;
        for (uint64_t i = 0; i < P.part[k].n; ++i) unmapped += allocation_of(P.part[k].src + i) == allocations.end();
    }
    if (misaligned) return hipSuccess;
    for (blockIdx.x = 0; blockIdx.x < grid.x; ++blockIdx.x)
        for (threadIdx.x = 0; threadIdx.x < block.x; ++threadIdx.x) zm_cache_fetch_kernel(P);
    return hipSuccess;
}

// compares the parts that the cache hands to the decoder with the host's bytes
static std::vector<std::vector<uint8_t>> want_sm, want_e;
static long differing;
static int decoded;
static bool refuse;                                        // as the decoder does with streams that do not fit its LDS
extern "C" int zm_decode_tensors(const zm_tensor_parts *parts, const zm_tensor_info *, int n, void *const *, void *)
{
    if (refuse && n) return ZM_E_ARG;
    for (int i = 0; i < n; ++i, ++decoded) {
        const auto &sm = want_sm[decoded % 2], &e = want_e[decoded % 2];
        for (size_t k = 0; k < sm.size(); ++k) differing += static_cast<const uint8_t *>(parts[i].sm)[k] != sm[k];
        for (size_t k = 0; k < e.size(); ++k) differing += static_cast<const uint8_t *>(parts[i].echunks)[k] != e[k];
    }
    return ZM_OK;
}

int main(int argc, char **argv)
{
    if (argc < 2) return 2;
    const std::string_view what = argv[1];
    const bool packed = argc > 2 && std::string_view(argv[2]) == "packed";
    zm_tensor_info t{};
    t.n_values = 12000; t.lut_offset = 384; t.table_offset = 896; t.sm_offset = 1024; t.e_offset = 1024 + 12032; t.blob_size = t.e_offset + 2048;
    t.table_stride = 16; t.n_chunks = 3;
    if (what == "odd-end") t.blob_size -= 250;
    if (what == "odd-sections") { t.sm_offset += 8; t.e_offset += 24; }
    zm_tensor_info infos[2] = {t, t};
    zm_cache_config config{2, 1, {0, 0, 0, 0}, 0, 2};
    // host memory whose every page a caller may map or not; 4 KiB pages
    const size_t room = 1 << 16;
    std::vector<uint8_t *> blob(2), image(2);
    std::vector<const void *> blob_p(2), image_p(2);
    for (int e = 0; e < 2; ++e) {
        blob[e] = static_cast<uint8_t *>(std::aligned_alloc(4096, room));
        image[e] = static_cast<uint8_t *>(std::aligned_alloc(4096, room));
        for (size_t i = 0; i < room; ++i) blob[e][i] = static_cast<uint8_t>(1 + (i * 131 + e * 7) % 251);
        blob_p[e] = blob[e]; image_p[e] = image[e];
        want_sm.emplace_back(blob[e] + t.sm_offset, blob[e] + t.e_offset);
        want_e.emplace_back(blob[e] + t.e_offset, blob[e] + t.blob_size);
        if (packed && zm_cache_pack_expert(&config, infos, blob_p.data(), e, image[e], room) != ZM_OK) return 3;
        uint8_t *source = packed ? image[e] : blob[e];
        if (what == "hole") allocations[source] = allocations[source + 3 * 4096] = 4096;      // the last byte is in page 3
        else if (what != "pageable") allocations[source] = room;
    }
    size_t bytes = 0;
    if (zm_cache_arena_bytes(&config, infos, &bytes) != ZM_OK) return 4;
    uint8_t *arena = static_cast<uint8_t *>(std::aligned_alloc(256, up256(bytes)));
    std::memset(arena, 0, bytes);
    zm_cache *cache = nullptr;
    last_error = hipErrorInvalidValue;                  // of some earlier call of the program's
    if (zm_cache_create(&config, blob_p.data(), packed ? image_p.data() : nullptr, infos, arena, bytes, &cache) != ZM_OK) return 5;
    by_copy = 0;                                        // the tables
    if (what == "unmapped-later") allocations.clear();  // still valid memory, as the contract asks
    const int32_t ids[2] = {0, 1};
    void *out[2];
    if (argc > 3) {
        const std::string_view ends = argv[3];
        over = issued;                                  // the tables: creation has waited for them
        if (ends == "captured") {
            if (zm_cache_fetch(cache, ids, 2, out, nullptr, nullptr) != ZM_OK) return 6;
            capturing = true;
        }
        refuse = ends == "refused";
        if (zm_cache_fetch(cache, ids, 2, out, nullptr, nullptr) != (refuse ? ZM_E_ARG : ZM_OK)) return 6;
        capturing = false;
        const bool any = under_way() > 0;
        zm_cache_destroy(cache);
        std::printf("%d %ld %ld\n", any, under_way(), differing);
        return 0;
    }
    if (zm_cache_fetch(cache, ids, 2, out, nullptr, nullptr) != ZM_OK) return 6;
    zm_cache_destroy(cache);
    if (last_error != hipErrorInvalidValue) return 7;   // not the cache's to clear
    std::printf("%ld %ld %ld %ld %ld\n", differing, by_kernel, by_copy, unmapped, misaligned);
    return 0;
}
