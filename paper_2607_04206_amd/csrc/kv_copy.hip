// Paged-KV export / import kernels for gfx950 and their C ABI entry points.
//
// One work-group per (listed page, 256 / (2 D) heads, tensor): grid.x walks
// the plan's page records, the head groups of a page next to each other, grid.y
// picks K (0) or V (1). A page's chunk of one KV head is 16 slots x D
// contiguous in the pool; in the packed buffers slot s of that head is row
// row0 + s, Hkv x D elements apart. A thread moves one 16-byte piece, so the
// pool side reads or writes whole 4 KiB (2 KiB at D = 64, two heads) chunks and
// the packed side whole 256-byte (128-byte) rows. Both directions move bytes
// only and are bound by HBM. Many short work-groups keep more bytes in flight
// than one per page that walked the heads four at a time, and the rows of one
// slot are written close together in time. Measured, export + import: 32
// requests of the 32/32 model (304 MB packed) 252 -> 209 us, with the stores
// below; 8 requests (91 MB) 68 -> 62; 48 requests of the 28/4 model (91 MB)
// 62.6 -> 61.2; two or four heads per work-group in between.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "../../include/sangam_kv.h"
#include "kv_format.h"

namespace sangam {
void set_error(const std::string& msg);
void clear_error();
const KvPlanHeader* check_kv_plan(const void* plan);
}  // namespace sangam

using namespace sangam;

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct KvCopyArgs {
    const KvPageRec* recs;
    const uint16_t* src[2];  // K, V (pool for export, packed for import)
    uint16_t* dst[2];
    int32_t hkv;
    uint32_t groups;  // head groups of a page
};

// Work-groups of one launch: the grid's threads are counted in 32 bits.
constexpr int64_t kMaxBlocks = (int64_t(1) << 32) / 256 - 1;

// Packed bytes (K and V) from which the stores are nontemporal: with as many
// bytes read, the copy no longer fits the 256 MiB Infinity Cache. Measured,
// export + import with plain -> with nontemporal stores: 91 MB 62.0 -> 64.8 us
// (the import reads what the export left in the cache), 147 MB 102 -> 99,
// 176 MB 137 -> 127, 247 MB 191 -> 181, 304 MB 219 -> 209, 785 MB 591 -> 570.
constexpr int64_t kStreamBytes = int64_t(128) << 20;

template <int D, bool EXPORT, bool STREAM>
__global__ __launch_bounds__(256) void kv_copy_kernel(KvCopyArgs a) {
    constexpr int NC = D / 8;             // 16-byte pieces of a row
    constexpr int HPG = 256 / (16 * NC);  // heads of a work-group
    const uint32_t page = blockIdx.x / a.groups;
    const KvPageRec r = a.recs[page];
    const int t = blockIdx.y;
    const int tid = threadIdx.x;
    const int pos = tid % NC;
    const int s = (tid / NC) % 16;
    const int h = int(blockIdx.x - page * a.groups) * HPG + tid / (16 * NC);
    if (s >= r.nslots || h >= a.hkv) return;  // no position in this slot (last page of an item), no head
    const size_t pool = (((size_t)r.page * a.hkv + h) * 16 + s) * D + pos * 8;
    const size_t pack = ((size_t)(r.row0 + s) * a.hkv + h) * D + pos * 8;
    const u32x4 v = *(const u32x4*)(a.src[t] + (EXPORT ? pool : pack));
    u32x4* const dst = (u32x4*)(a.dst[t] + (EXPORT ? pack : pool));
    if (STREAM) __builtin_nontemporal_store(v, dst);
    else *dst = v;
}

template <int D>
const void* copy_fn(bool is_export, bool stream) {
    if (is_export)
        return stream ? reinterpret_cast<const void*>(&kv_copy_kernel<D, true, true>)
                      : reinterpret_cast<const void*>(&kv_copy_kernel<D, true, false>);
    return stream ? reinterpret_cast<const void*>(&kv_copy_kernel<D, false, true>)
                  : reinterpret_cast<const void*>(&kv_copy_kernel<D, false, false>);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

sangam_status run_copy(bool is_export, const void* plan_host, const void* plan_dev, const void* src_k,
                       const void* src_v, void* dst_k, void* dst_v, void* stream) {
    clear_error();
    const KvPlanHeader* h = check_kv_plan(plan_host);
    if (!h) {
        set_error("plan_host is not a KV transfer plan of this library version");
        return SANGAM_ERR_PLAN;
    }
    if (!plan_dev || !src_k || !src_v || !dst_k || !dst_v) {
        set_error("plan_dev and the K / V source and destination pointers must not be NULL");
        return SANGAM_ERR_INVALID_ARG;
    }
    if (!aligned16(plan_dev) || !aligned16(src_k) || !aligned16(src_v) || !aligned16(dst_k) || !aligned16(dst_v)) {
        set_error("plan_dev and the K / V buffers must be 16-byte aligned");
        return SANGAM_ERR_ALIGN;
    }
    KvCopyArgs args;
    const KvPageRec* recs = reinterpret_cast<const KvPageRec*>(static_cast<const uint8_t*>(plan_dev) + h->off_pages);
    args.src[0] = static_cast<const uint16_t*>(src_k);
    args.src[1] = static_cast<const uint16_t*>(src_v);
    args.dst[0] = static_cast<uint16_t*>(dst_k);
    args.dst[1] = static_cast<uint16_t*>(dst_v);
    args.hkv = h->hkv;
    const int heads = 256 / (2 * h->d);  // of a work-group
    args.groups = uint32_t((h->hkv + heads - 1) / heads);
    const bool nt = h->total_rows * h->hkv * h->d * 4 > kStreamBytes;
    const void* fn = h->d == 128 ? copy_fn<128>(is_export, nt) : copy_fn<64>(is_export, nt);
    void* kargs[] = {&args};
    const int64_t step = std::max<int64_t>(kMaxBlocks / args.groups, 1);  // pages of a launch
    for (int64_t first = 0; first < h->total_pages; first += step) {
        args.recs = recs + first;
        const int64_t pages = std::min<int64_t>(step, h->total_pages - first);
        const hipError_t e = hipLaunchKernel(fn, dim3(unsigned(pages * args.groups), 2), dim3(256), kargs, 0,
                                             static_cast<hipStream_t>(stream));
        if (e != hipSuccess) {
            set_error(std::string(is_export ? "kv export" : "kv import") + " launch: " + hipGetErrorString(e));
            return SANGAM_ERR_HIP;
        }
    }
    return SANGAM_OK;
}

}  // namespace

extern "C" sangam_status sangam_kv_export(const void* plan_host, const void* plan_dev, const void* k_cache,
                                          const void* v_cache, void* k_packed, void* v_packed, void* stream) {
    return run_copy(true, plan_host, plan_dev, k_cache, v_cache, k_packed, v_packed, stream);
}

extern "C" sangam_status sangam_kv_import(const void* plan_host, const void* plan_dev, const void* k_packed,
                                          const void* v_packed, void* k_cache, void* v_cache, void* stream) {
    return run_copy(false, plan_host, plan_dev, k_packed, v_packed, k_cache, v_cache, stream);
}
