// Appending a decode step's rows for gfx950: one launch for all the arrays a
// step writes (keys and values of every layer into the cache, its queries
// into their buffers).
//
// One thread per 16-byte chunk.  The copies are a few hundred KB at most, so
// what counts is the number of launches: a step that wrote its arrays one
// torch copy each made three launches of 3.3 us and their host work.  A
// driver cycle of 128 steps over 4 layers (32 query and 8 kv-heads each) went
// from 2.32 to 1.40 ms, of which the host's calls are nearly all.
#include "device_common.h"
#include "internal.h"

namespace bkv {
namespace {

constexpr int kThreads = 256;

struct AppendArgs {
    bkv_rows a[BKV_APPEND_MAX];
    int first[BKV_APPEND_MAX + 1];  // first chunk of each array; the last entry is the total
    int cpr;                        // chunks per row
};

__global__ __launch_bounds__(kThreads) void append_kernel(AppendArgs p) {
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= p.first[BKV_APPEND_MAX]) return;
    int k = 0;
#pragma unroll
    for (int j = 1; j < BKV_APPEND_MAX; ++j) k += i >= p.first[j];
    bkv_rows r = p.a[0];  // selected by comparison: an index into the arguments would go through scratch
    int f = p.first[0];
#pragma unroll
    for (int j = 1; j < BKV_APPEND_MAX; ++j)
        if (k == j) {
            r = p.a[j];
            f = p.first[j];
        }
    const int h = ((int)i - f) / p.cpr, c = ((int)i - f) % p.cpr;
    *reinterpret_cast<dev::u32x4*>(static_cast<char*>(r.dst) + h * r.dst_stride + c * 16) =
        *reinterpret_cast<const dev::u32x4*>(static_cast<const char*>(r.src) + h * r.src_stride + c * 16);
}

}  // namespace
}  // namespace bkv

extern "C" bkv_status bkv_append_rows(const bkv_rows* arrays, int32_t n, int32_t row_bytes, hipStream_t stream) {
    using namespace bkv;
    if (n < 0 || n > BKV_APPEND_MAX || row_bytes <= 0 || row_bytes % 16 != 0) return BKV_ERR_SHAPE;
    if (n > 0 && !arrays) return BKV_ERR_INVALID;
    AppendArgs p{};
    p.cpr = row_bytes / 16;
    long long total = 0;
    for (int k = 0; k < n; ++k) {
        const bkv_rows& r = arrays[k];
        if (r.heads < 0 || r.heads > 0x7fffffffLL) return BKV_ERR_SHAPE;
        if (r.heads > 0 && (!r.src || !r.dst)) return BKV_ERR_INVALID;
        if (((reinterpret_cast<uintptr_t>(r.src) | reinterpret_cast<uintptr_t>(r.dst) | (uintptr_t)r.src_stride |
              (uintptr_t)r.dst_stride) & 15u) != 0)
            return BKV_ERR_INVALID;
        p.a[k] = r;
        p.first[k] = (int)total;
        total += r.heads * p.cpr;
        if (total > 0x7fffffffLL) return BKV_ERR_SHAPE;
    }
    if (total == 0) return BKV_OK;
    for (int k = n; k <= BKV_APPEND_MAX; ++k) p.first[k] = (int)total;
    hipLaunchKernelGGL(append_kernel, dim3((unsigned)((total + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream, p);
    return hipGetLastError() == hipSuccess ? BKV_OK : BKV_ERR_HIP;
}
