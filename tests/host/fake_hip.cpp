// A HIP runtime without a device, for tests of the library's host side: memory is host memory, streams are
// names, kernels do not run.  A launch is recorded, and what its work list says is copied out of the library's memory at
// that moment; the copy of a list that a kernel leaves in device memory for later launches is made here.
// Loaded with global symbols before libpbkv.so, whose calls then come here.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "pbkv_internal.h"

namespace {

struct Launch {
    std::string name;
    dim3 grid, block;
    hipStream_t stream;
    pbkv::AttnParams attn;
    pbkv::DecodeParams decode;
    std::vector<pbkv::TileDesc> tiles;
    std::vector<pbkv::RangeDesc> ranges;
    std::vector<pbkv::MergeDesc> merges;
    std::vector<uint32_t> units;
};

std::mutex mu;
std::map<const void *, std::string> kernels;
std::map<void *, size_t> device_memory;
std::vector<Launch> launches;
std::map<std::string, int64_t> counts;
int64_t live = 0, limit = INT64_MAX;
int capturing = 0;
hipError_t last_error = hipSuccess;
thread_local dim3 cfg_grid, cfg_block;
thread_local size_t cfg_shmem;
thread_local hipStream_t cfg_stream;

bool has(const std::string &s, const char *part) { return s.find(part) != std::string::npos; }

}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    kernels[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shmem, hipStream_t s) {
    cfg_grid = g; cfg_block = b; cfg_shmem = shmem; cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shmem, hipStream_t *s) {
    *g = cfg_grid; *b = cfg_block; *shmem = cfg_shmem; *s = cfg_stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t s) {
    std::lock_guard<std::mutex> lock(mu);
    Launch l{};
    l.name = kernels.count(f) ? kernels[f] : "?";
    l.grid = grid; l.block = block; l.stream = s;
    if ((uint64_t)grid.x * block.x >= ((uint64_t)1 << 32)) return last_error = hipErrorInvalidConfiguration;
    const bool merge = has(l.name, "merge_kernel");
    if (has(l.name, "attn_")) {
        const pbkv::AttnParams p = *(const pbkv::AttnParams *)args[0];
        l.attn = p;
        if (merge) {
            l.merges.assign(p.merges, p.merges + p.n_merges);
            if (p.mirror_merges) memcpy(p.mirror_merges, p.merges, p.n_merges * sizeof *p.merges);
        } else {
            l.tiles.assign(p.tiles, p.tiles + p.n_tiles);
            if (p.mirror) memcpy(p.mirror, p.tiles, p.n_tiles * sizeof *p.tiles);
            if (p.units) l.units.assign(p.units, p.units + p.n_units);
            if (p.mirror_units) memcpy(p.mirror_units, p.units, p.n_units * sizeof *p.units);
            if (p.ranges) {
                l.ranges.assign(p.ranges, p.ranges + p.n_tiles);
                if (p.mirror_ranges) memcpy(p.mirror_ranges, p.ranges, p.n_tiles * sizeof *p.ranges);
            }
        }
    } else if (has(l.name, "decode_")) {
        l.decode = *(const pbkv::DecodeParams *)args[0];
        if (!merge && l.decode.mirror_reqs)
            memcpy(l.decode.mirror_reqs, l.decode.reqs, l.decode.n_reqs * sizeof *l.decode.reqs);
    }
    launches.push_back(std::move(l));
    return hipSuccess;
}

hipError_t hipMalloc(void **out, size_t n) {
    std::lock_guard<std::mutex> lock(mu);
    counts["hipMalloc"]++;
    if (live + (int64_t)n > limit) return last_error = hipErrorOutOfMemory;
    *out = aligned_alloc(256, (n + 255) & ~(size_t)255);      // (pages that nothing writes take no memory)
    device_memory[*out] = n;
    live += (int64_t)n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::mutex> lock(mu);
    if (!device_memory.count(p)) return last_error = hipErrorInvalidValue;
    live -= (int64_t)device_memory[p];
    device_memory.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **out, size_t n, unsigned) { *out = aligned_alloc(256, (n + 255) & ~(size_t)255); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **out, void *p, unsigned) { *out = p; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **out, const void *) { static void *m = aligned_alloc(256, 16u << 20); *out = m; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { hipError_t e = last_error; last_error = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipDeviceSynchronize() { counts["hipDeviceSynchronize"]++; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { counts["hipStreamSynchronize"]++; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { static intptr_t n; *e = (hipEvent_t)(++n); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { counts["hipEventRecord"]++; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
    memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}

// ---- what the tests ask for ----
void fake_limit_device_memory(int64_t bytes_more) { limit = bytes_more < 0 ? INT64_MAX : live + bytes_more; }
int64_t fake_live() { return live; }
int64_t fake_count(const char *what) { return counts[what]; }
int fake_launches() { return (int)launches.size(); }
void fake_forget() { launches.clear(); counts.clear(); }
const char *fake_name(int i) { return launches[i].name.c_str(); }
// grid, threads, stream, tiles, merges, waves, scratch, counters, list
void fake_launch(int i, int64_t *o) {
    const Launch &l = launches[i];
    const bool dec = has(l.name, "decode_");
    o[0] = l.grid.x; o[1] = l.block.x; o[2] = (int64_t)l.stream;
    o[3] = (int64_t)l.tiles.size(); o[4] = l.attn.n_merges; o[5] = l.attn.waves;
    o[6] = (int64_t)(dec ? l.decode.scratch : l.attn.partial);
    o[7] = (int64_t)l.decode.counters;
    o[8] = (int64_t)(dec ? (const void *)l.decode.reqs : (const void *)l.attn.tiles);
}
// req, tok0, prefix, new, row0, part, kt0, kt1
void fake_tiles(int i, int64_t *o) {
    const Launch &l = launches[i];
    for (size_t k = 0; k < l.tiles.size(); k++, o += 8) {
        const pbkv::TileDesc &t = l.tiles[k];
        const pbkv::RangeDesc r = l.ranges.empty() ? pbkv::RangeDesc{-1, 0, INT32_MAX, 0} : l.ranges[k];
        o[0] = t.req; o[1] = t.tok0; o[2] = t.prefix_len; o[3] = t.new_len; o[4] = t.row0;
        o[5] = r.part; o[6] = r.kt0; o[7] = r.kt1;
    }
}
// the work-groups per KV head that the list names (none: all of every tile)
int fake_unit_count(int i) { return (int)launches[i].units.size(); }
void fake_units(int i, int64_t *o) {
    for (uint32_t u : launches[i].units) { *o++ = u >> 2; *o++ = u & 3; }
}
// where the partial results of tiles and of merged blocks (first slot, slots of a part) stand
void fake_slots(int i, int64_t *o) {
    for (const pbkv::RangeDesc &r : launches[i].ranges) *o++ = r.slot;
}
void fake_places(int i, int64_t *o) {
    for (const pbkv::MergeDesc &m : launches[i].merges) { *o++ = m.slot0; *o++ = m.splits; }
}
// tok0, new, part0, parts, row0
void fake_merges(int i, int64_t *o) {
    for (const pbkv::MergeDesc &m : launches[i].merges) {
        o[0] = m.tok0; o[1] = m.new_len; o[2] = m.part0; o[3] = m.n_parts; o[4] = m.row0;
        o += 5;
    }
}

}  // extern "C"
