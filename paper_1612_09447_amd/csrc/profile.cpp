// Per-kernel-class timing with HIP events. Classes of one kernel take the
// start/stop events of the launch itself (hipExtLaunchKernelGGL: the
// kernel's own execution, as a kernel trace reports it); the V-cycle class
// brackets its launches with events recorded on the stream. A launch that does
// the work of two classes (a folded operator) counts, with its whole time, in
// both.
#include "eqs_internal.h"

namespace eqs {

static hipEvent_t next_event(eqs_ctx* c) {
    if (c->prof_next == c->prof_pool.size()) {
        hipEvent_t e;
        EQS_HIP(hipEventCreate(&e));
        c->prof_pool.push_back(e);
    }
    return c->prof_pool[c->prof_next++];
}

// slot of the class's next launch
static std::pair<hipEvent_t, hipEvent_t>& slot(eqs_ctx* c, int cls) {
    auto& v = c->prof_ev[cls];
    if (v.size() <= (size_t)c->prof_used[cls]) v.resize((size_t)c->prof_used[cls] + 1);
    return v[(size_t)c->prof_used[cls]];
}

void prof_begin(eqs_ctx* c, int cls, hipStream_t s) {
    if (!(c->prof_mask & (1u << cls))) return;
    auto& p = slot(c, cls);
    p = {next_event(c), next_event(c)};
    EQS_HIP(hipEventRecord(p.first, s));
}

bool prof_pair(eqs_ctx* c, int cls, hipEvent_t* e0, hipEvent_t* e1, int cls2) {
    auto on = [&](int k) { return k >= 0 && (c->prof_mask & (1u << k)); };  // negative: never timed
    if (!on(cls) && !on(cls2)) return false;
    *e0 = next_event(c);
    *e1 = next_event(c);
    for (int k : {cls, cls2})
        if (on(k)) {
            slot(c, k) = {*e0, *e1};
            c->prof_used[k]++;
        }
    return true;
}

// The class's last launch did the work of two of its launches: the second is
// counted with no time of its own.
void prof_again(eqs_ctx* c, int cls) {
    if (!(c->prof_mask & (1u << cls)) || c->prof_used[cls] == 0) return;
    const hipEvent_t e = c->prof_ev[cls][(size_t)c->prof_used[cls] - 1].second;
    slot(c, cls) = {e, e};
    c->prof_used[cls]++;
}

void prof_end(eqs_ctx* c, int cls, hipStream_t s) {
    if (!(c->prof_mask & (1u << cls))) return;
    EQS_HIP(hipEventRecord(c->prof_ev[cls][(size_t)c->prof_used[cls]].second, s));
    c->prof_used[cls]++;
}

void prof_release(eqs_ctx* c) {
    for (hipEvent_t e : c->prof_pool) (void)hipEventDestroy(e);
    c->prof_pool.clear();
    c->prof_next = 0;
    for (auto& v : c->prof_ev) v.clear();
    for (auto& u : c->prof_used) u = 0;
    c->prof_mask = 0;
}

}  // namespace eqs

extern "C" int eqs_profile_enable_impl(eqs_ctx* c, uint32_t mask) {
    for (auto& u : c->prof_used) u = 0;
    c->prof_next = 0;
    c->prof_mask = mask & ((1u << EQS_KCLASS_COUNT) - 1);
    return EQS_OK;
}

extern "C" int eqs_profile_read_impl(eqs_ctx* c, int32_t cls, int64_t* launches, double* total_ms) {
    EQS_HIP(hipStreamSynchronize(c->stream));
    double ms = 0.0;
    for (int64_t i = 0; i < c->prof_used[cls]; ++i) {
        float t = 0.0f;
        EQS_HIP(hipEventElapsedTime(&t, c->prof_ev[cls][(size_t)i].first, c->prof_ev[cls][(size_t)i].second));
        ms += t;
    }
    *launches = c->prof_used[cls];
    *total_ms = ms;
    return EQS_OK;
}
