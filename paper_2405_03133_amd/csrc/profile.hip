// Optional per-kernel-class timing with HIP events on the caller's stream.
// Off by default; when on, every launch of the hot path is bracketed by a pair
// of events and tagged with the algorithmic FLOPs and bytes of that launch, so
// a benchmark can report achieved TFLOP/s and GB/s per kernel class without an
// external profiler.
#include "lory_internal.h"

#include <string.h>

#include <vector>

namespace lory {
namespace prof {

namespace {

struct Record {
    int cls;
    hipEvent_t start, stop;
    double flops, bytes;
    hipEvent_t counted;   // NULL, or follows the count of the segments that have merged values of their own
    int segments;
    double seg_bytes;
};

bool g_on = false;
std::vector<Record> g_records;
std::vector<hipEvent_t> g_pool;
int32_t *g_counts = nullptr;   // per record, in host memory that the GPU writes; kept to the end of the process

const char *const kNames[kNumClasses] = {"route",     "merge",     "gemm_gate_up", "swiglu_fwd", "gemm_down",
                                         "gemm_dA",   "swiglu_bwd", "gemm_dX",   "gemm_dW_gate_up",
                                         "gemm_dW_down", "scatter_dots", "dw_reduce", "route_bwd", "dense_skinny",
                                         "fused_gate_up", "fused_down", "fused_dA", "fused_dX", "fused_dW_dots"};

// Events are created when timing is switched on (and by lory_profile_read, which returns
// them to the pool), never inside a launch: a launch only takes events from the pool and
// goes untimed when the pool is empty.
constexpr size_t kMaxRecords = 2048;   // timed launches between two reads
constexpr size_t kPoolEvents = 3 * kMaxRecords;

hipEvent_t get_event()
{
    if (g_pool.empty()) return nullptr;
    hipEvent_t e = g_pool.back();
    g_pool.pop_back();
    return e;
}

void fill_pool()
{
    g_pool.reserve(kPoolEvents);
    g_records.reserve(kMaxRecords);
    if (!g_counts && hipHostMalloc((void **)&g_counts, kMaxRecords * sizeof(int32_t), hipHostMallocDefault) != hipSuccess)
        g_counts = nullptr;
    while (g_pool.size() < kPoolEvents) {
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) break;
        g_pool.push_back(e);
    }
}

__global__ __launch_bounds__(256) void count_segments_kernel(const int32_t *map, int S, int32_t *out)
{
    __shared__ int part[4];
    int n = 0;
    for (int s = threadIdx.x; s - (int)threadIdx.x < S; s += 256) n += __popcll(__ballot(s < S && map[s] == s));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) *out = part[0] + part[1] + part[2] + part[3];
}

}  // namespace

bool enabled() { return g_on; }

Range::Range(hipStream_t st, int cls, double flops, double bytes) : st_(st), idx_(-1)
{
    if (!g_on) return;
    Record r = {};
    r.cls = cls;
    r.flops = flops;
    r.bytes = bytes;
    if (g_pool.size() < 2 || g_records.size() == g_records.capacity()) return;  // untimed launch
    r.start = get_event();
    r.stop = get_event();
    hipEventRecord(r.start, st);
    g_records.push_back(r);
    idx_ = (int)g_records.size() - 1;
}

Range::~Range()
{
    if (idx_ >= 0) hipEventRecord(g_records[idx_].stop, st_);
}

void shared_segments(hipStream_t st, int idx, const int32_t *map, int S, double seg_bytes)
{
    if (idx < 0 || !map || !g_counts || g_pool.empty()) return;
    Record &r = g_records[idx];
    r.segments = S;
    r.seg_bytes = seg_bytes;
    hipLaunchKernelGGL(count_segments_kernel, dim3(1), dim3(256), 0, st, map, S, g_counts + idx);
    r.counted = get_event();
    hipEventRecord(r.counted, st);
}

int set_enabled(int on)
{
    g_on = on != 0;
    if (g_on) fill_pool();
    return LORY_OK;
}

int read(lory_kernel_stat *out, int max_out, int *n_out)
{
    lory_kernel_stat acc[kNumClasses];
    memset(acc, 0, sizeof(acc));
    for (int c = 0; c < kNumClasses; ++c) strncpy(acc[c].name, kNames[c], sizeof(acc[c].name) - 1);
    int rc = LORY_OK;
    for (size_t i = 0; i < g_records.size(); ++i) {
        const Record &r = g_records[i];
        float ms = 0.f;
        if (hipEventSynchronize(r.stop) != hipSuccess || (r.counted && hipEventSynchronize(r.counted) != hipSuccess) ||
            hipEventElapsedTime(&ms, r.start, r.stop) != hipSuccess) {
            rc = LORY_ERR_DEVICE;
        } else {
            acc[r.cls].launches += 1;
            acc[r.cls].ms += ms;
            acc[r.cls].flops += r.flops;
            acc[r.cls].bytes += r.bytes - (r.counted ? r.seg_bytes * (r.segments - g_counts[i]) : 0.0);
        }
        if (r.counted) g_pool.push_back(r.counted);
        g_pool.push_back(r.start);
        g_pool.push_back(r.stop);
    }
    g_records.clear();
    int n = 0;
    for (int c = 0; c < kNumClasses && n < max_out; ++c)
        if (acc[c].launches > 0) out[n++] = acc[c];
    *n_out = n;
    return rc;
}

}  // namespace prof
}  // namespace lory
