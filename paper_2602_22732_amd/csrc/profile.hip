// Optional per-kernel timing with HIP events on the stream the kernels run on.
// Off by default; when switched on, every kernel launch of the library is
// bracketed by two events.  Used by the benchmark to attribute time to kernels.
#include <vector>

#include "common.h"

namespace {
struct Record { hipEvent_t start, stop; int cls; double flops, bytes; int slot; int64_t rows; };  // slot: row count of the launch (-1: as counted)
bool g_on = false;
std::vector<Record> g_records;       // events in flight since the last read
std::vector<Record> g_pool;          // recycled event pairs
const size_t kMaxRecords = 1 << 16;
// Row counts that only the device knows: copied here on the stream, read with the events.  Pinned, allocated at the first such count, kept.
const int kMaxSlots = 1 << 14;
int32_t *g_slots = nullptr;
int g_slots_used = 0;
// the slot in force and the rows the launches are counted with (a thread's own: decodes of several threads do not touch one another's)
thread_local int t_slot = -1;
thread_local int64_t t_rows = 0;
const char *kNames[KC_COUNT] = {"gemm_bf16_tile", "gemm_simple", "cross_attn_flash_bf16",
                                "cross_attn_simple", "self_attn_step", "trunk_self_attn", "rmsnorm", "fuse_gate", "select_rows",
                                "select_request", "gather_rows", "broadcast_rows", "v_transpose", "gemm_bf16_ring", "masked_softmax_rows",
                                "gemm_fp8_ring", "quantize_rows", "context_attn_flash_bf16", "distinct_rows"};
}  // namespace

ProfScope::ProfScope(int cls, hipStream_t st, double flops, double bytes) : idx_(-1), st_(st) {
    if (!g_on || g_records.size() >= kMaxRecords) return;
    Record r;
    if (!g_pool.empty()) {
        r = g_pool.back();
        g_pool.pop_back();
    } else {
        if (hipEventCreate(&r.start) != hipSuccess) return;
        if (hipEventCreate(&r.stop) != hipSuccess) {
            (void)hipEventDestroy(r.start);
            return;
        }
    }
    r.cls = cls;
    r.flops = flops;
    r.bytes = bytes;
    r.slot = t_slot;
    r.rows = t_rows;
    (void)hipEventRecord(r.start, st);
    g_records.push_back(r);
    idx_ = (int)g_records.size() - 1;
}

ProfScope::~ProfScope() {
    if (idx_ >= 0) (void)hipEventRecord(g_records[idx_].stop, st_);
}

void prof_rows(const int32_t *count_dev, int64_t rows, hipStream_t st) {
    t_slot = -1;
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (!count_dev || !g_on || g_slots_used >= kMaxSlots || hipStreamIsCapturing(st, &capturing) != hipSuccess || capturing != hipStreamCaptureStatusNone) return;
    if (!g_slots && hipHostMalloc((void **)&g_slots, kMaxSlots * sizeof(int32_t)) != hipSuccess) {
        g_slots = nullptr;
        return;
    }
    if (hipMemcpyAsync(g_slots + g_slots_used, count_dev, sizeof(int32_t), hipMemcpyDeviceToHost, st) != hipSuccess) return;
    t_slot = g_slots_used++;
    t_rows = rows;
}

extern "C" {

int gr4ad_profile_enable(int on) {
    g_on = on != 0;
    return GR4AD_OK;
}

int gr4ad_profile_kernel_count(void) { return KC_COUNT; }

const char *gr4ad_profile_kernel_name(int cls) { return (cls >= 0 && cls < KC_COUNT) ? kNames[cls] : ""; }

int gr4ad_profile_read(double *ms, double *flops, double *bytes, int64_t *launches, int reset) {
    if (!ms || !flops || !bytes || !launches) return GR4AD_EINVAL;
    for (int i = 0; i < KC_COUNT; i++) { ms[i] = 0; flops[i] = 0; bytes[i] = 0; launches[i] = 0; }
    for (const Record &r : g_records) {
        if (hipEventSynchronize(r.stop) != hipSuccess) return GR4AD_EHIP;
        float t = 0;
        if (hipEventElapsedTime(&t, r.start, r.stop) != hipSuccess) return GR4AD_EHIP;
        ms[r.cls] += t;
        const double f = r.slot < 0 ? 1.0 : (double)g_slots[r.slot] / (double)r.rows;
        flops[r.cls] += r.flops * f;
        bytes[r.cls] += r.bytes * f;
        launches[r.cls] += 1;
    }
    if (reset) {
        for (const Record &r : g_records) g_pool.push_back(r);
        g_records.clear();
        g_slots_used = 0;
    }
    return GR4AD_OK;
}

}  // extern "C"
