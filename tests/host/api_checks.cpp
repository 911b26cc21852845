// What a handle does when memory or a launch fails, and what it touches while
// earlier runs are still on their way: rqa_api.cpp against a HIP runtime and an
// engine made here (host memory; streams whose destruction is noted; an engine
// that writes a run's records when the stream is waited for, as the kernels do).
// Built with AddressSanitizer: writing to a block that the handle has freed, or
// reading through a null pointer, ends the program.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <set>
#include <vector>

#include "rqa_internal.h"

using namespace rqa;

#define CHECK(c) \
    do { if (!(c)) { std::fprintf(stderr, "line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

// ---- the runtime ----
struct FakeStream {
    bool capturing = false;
    std::vector<std::function<void()>> work;   // done when the stream is waited for
};
static std::set<FakeStream *> streams;
static bool fail_host_malloc = false, fail_malloc = false;
static int host_mallocs = 0;
static FakeStream *fs(hipStream_t s) {
    CHECK(streams.count(reinterpret_cast<FakeStream *>(s)));   // not one that was destroyed
    return reinterpret_cast<FakeStream *>(s);
}
static hipStream_t make_stream() {
    FakeStream *f = new FakeStream;
    streams.insert(f);
    return reinterpret_cast<hipStream_t>(f);
}
static bool any_capture() {
    for (FakeStream *f : streams) if (f->capturing) return true;
    return false;
}

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) {
    for (FakeStream *f : streams) {
        CHECK(!f->capturing);
        for (auto &w : f->work) w();
        f->work.clear();
    }
    return hipSuccess;
}
hipError_t hipDeviceTotalMem(size_t *b, hipDevice_t) { *b = size_t(288) << 30; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
    CHECK(!any_capture());
    if (fail_malloc) return hipErrorOutOfMemory;
    *p = std::calloc(n, 1);
    return hipSuccess;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    CHECK(!any_capture());
    ++host_mallocs;
    if (fail_host_malloc) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = make_stream(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) {
    delete fs(s);
    streams.erase(reinterpret_cast<FakeStream *>(s));
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    CHECK(!fs(s)->capturing);
    for (auto &f : fs(s)->work) f();
    fs(s)->work.clear();
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
    *c = fs(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    fs(st)->work.push_back([=] { std::memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 1.f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    return hipErrorNotSupported;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
}

// ---- the engine: every line of a job of n vectors has length 1, n of them ----
static enum { kWorks, kRefuses, kFailsLate, kNeverRuns } engine = kWorks;
namespace rqa {
KParams make_kparams(const rqa_params &p) { KParams k{}; k.m = p.m; return k; }
size_t engine_launch_scratch_bytes(size_t n) { return 1024 * n; }
size_t engine_job_scratch_bytes(const Job &) { return 4096; }
int engine_band_strips(const Job &, size_t) { return 0; }
JobPlan engine_job_plan(const Job &) { return JobPlan{}; }
void engine_batch_segs(std::vector<Job> &) {}
int engine_default_waves(int64_t) { return 4; }
int64_t engine_plot_tail_floats(const KParams &) { return 64; }
int64_t engine_plot_scratch_floats(const KParams &, int64_t n, int64_t nb, bool cross) {
    return 64 + nb + (cross ? n : 0);
}
static bool plot_boxes;
int engine_plot(const KParams &, const float *, int64_t, const float *, int64_t, uint64_t *, int64_t,
                float *, bool boxes, hipStream_t) { plot_boxes = boxes; return RQA_OK; }
int engine_launch(const std::vector<Job> &jobs, void *, void *, hipEvent_t, int, hipStream_t st,
                  const PhaseEvents *, AuxStreams *) {
    if (engine == kRefuses) return RQA_EINVAL;
    if (engine == kNeverRuns) return RQA_OK;
    for (const Job &j : jobs)
        fs(st)->work.push_back([=] {
            JobStats s{};
            const uint64_t n = static_cast<uint64_t>(j.n_vec);
            for (int k = 0; k < 3; ++k) {
                s.cnt_all[k] = s.mass_all[k] = n;
                s.longest[k] = 1;
                uint64_t *h = j.hist + k * j.hist_len();
                std::memset(h, 0, sizeof(uint64_t) * j.hist_len());
                h[1] = n;
                if (j.host_hist)
                    std::memcpy(static_cast<uint64_t *>(j.host_hist) + k * j.hist_len(), h,
                                sizeof(uint64_t) * j.hist_len());
            }
            std::memset(j.flag, 0, 8);
            std::memcpy(reinterpret_cast<char *>(j.flag) + 8, &s, sizeof s);
            if (!j.host_info) return;
            std::memcpy(static_cast<char *>(j.host_info) + 8, &s, sizeof s);
            const uint32_t head[2] = {0u, j.run};
            std::memcpy(j.host_info, head, sizeof head);
        });
    return engine == kFailsLate ? RQA_EDEVICE : RQA_OK;
}
void measures_from_stats(const JobStats &st, int64_t n, int64_t, const rqa_params &, rqa_measures *out) {
    std::memset(out, 0, sizeof *out);
    out->n_rec = st.cnt_all[0];
    out->n_vec = n;
}
void measures_from_hist(const uint64_t *, const uint64_t *, const uint64_t *, int64_t, const rqa_params &,
                        rqa_measures *) {}
}  // namespace rqa

// ---- the checks ----
static const float *const kSeries = reinterpret_cast<const float *>(4096);

static rqa_handle *handle() {
    rqa_handle *h = nullptr;
    CHECK(rqa_create(&h, 1, 1, 0.5f, 3, 2, 2, 2, 1) == RQA_OK);
    CHECK(rqa_set_tiling(h, 4, 0) == RQA_OK);   // no trials
    return h;
}
// The last run was one of n points, and its results are its own.
static void expect(rqa_handle *h, int64_t n) {
    rqa_measures m;
    std::vector<uint64_t> d(n + 1, 7), v(n + 1, 7), w(n + 1, 7);
    CHECK(rqa_result(h, &m, d.data(), v.data(), w.data(), n + 1) == RQA_OK);
    CHECK(m.n_vec == n && m.n_rec == static_cast<uint64_t>(n));
    for (auto *x : {&d, &v, &w})
        for (int64_t k = 0; k <= n; ++k) CHECK((*x)[k] == (k == 1 ? static_cast<uint64_t>(n) : 0u));
}
static int batch(rqa_handle *h, int count, hipStream_t st) {
    std::vector<int64_t> off(count, 0), len(count);
    for (int k = 0; k < count; ++k) len[k] = 10 + k;
    return rqa_run_batch(h, kSeries, 10 + count, off.data(), len.data(), count, st);
}
static void expect_batch(rqa_handle *h, int count) {
    std::vector<rqa_measures> m(count);
    CHECK(rqa_result_batch_all(h, m.data(), nullptr, count) == RQA_OK);
    for (int k = 0; k < count; ++k) CHECK(m[k].n_vec == 10 + k && m[k].n_rec == static_cast<uint64_t>(10 + k));
}

constexpr int64_t kShort = 100, kLonger = 16383, kLong = 40000;   // kLonger: the last that is published

int main() {
    // No run.
    rqa_handle *h = handle();
    CHECK(rqa_result(h, nullptr, nullptr, nullptr, nullptr, 0) == RQA_ESTATE);
    rqa_destroy(h);

    // Runs of growing size, each on a stream that is gone when the next begins.
    h = handle();
    for (int64_t n : {kShort, kLonger, kLong, kShort}) {
        hipStream_t st = make_stream();
        CHECK(rqa_run(h, kSeries, n, st) == RQA_OK);
        expect(h, n);
        CHECK(batch(h, 300, st) == RQA_OK);
        expect_batch(h, 300);
        if (n != kLong) CHECK(hipStreamDestroy(st) == hipSuccess);
    }
    hipStream_t one = make_stream(), two = make_stream();
    CHECK(rqa_run(h, kSeries, kShort, one) == RQA_OK);
    expect(h, kShort);
    rqa_destroy(h);

    // A larger run begins while an earlier one still has its records to write.
    h = handle();
    CHECK(rqa_run(h, kSeries, kLong, one) == RQA_OK);   // (the workspace of both)
    expect(h, kLong);
    CHECK(rqa_run(h, kSeries, kShort, one) == RQA_OK);
    CHECK(rqa_run(h, kSeries, kLonger, two) == RQA_OK);
    expect(h, kLonger);
    CHECK(hipStreamSynchronize(one) == hipSuccess);
    expect(h, kLonger);
    rqa_destroy(h);

    // No pinned memory: the results are copied, and the next run is as before.
    for (int64_t n : {kShort, kLonger, kLong}) {
        h = handle();
        CHECK(batch(h, 20, one) == RQA_OK);   // (staging for what follows)
        expect_batch(h, 20);
        fail_host_malloc = true;
        CHECK(rqa_run(h, kSeries, n, one) == RQA_OK);
        rqa_measures m;
        CHECK(rqa_result(h, &m, nullptr, nullptr, nullptr, 0) == RQA_OK && m.n_vec == n);
        std::vector<uint64_t> d(n + 1);
        const int rc = rqa_result(h, &m, d.data(), nullptr, nullptr, n + 1);
        CHECK(rc == (8 * 3 * (n + 1) + 256 <= 20 * 256 ? RQA_OK : RQA_ENOMEM));
        fail_host_malloc = false;
        expect(h, n);
        CHECK(rqa_run(h, kSeries, n, one) == RQA_OK);
        expect(h, n);
        rqa_destroy(h);
    }

    // A launch that fails leaves the run before it, fetched or not.
    for (int fetched = 0; fetched < 2; ++fetched) {
        for (int64_t n : {kShort, kLonger}) {
            h = handle();
            CHECK(rqa_run(h, kSeries, n, one) == RQA_OK);
            if (fetched) expect(h, n);
            engine = kRefuses;
            CHECK(rqa_run(h, kSeries, n, one) == RQA_EINVAL);
            CHECK(batch(h, 200, one) == RQA_EINVAL);      // (larger: records of its own)
            CHECK(rqa_run(h, kSeries, kLong, two) == RQA_EINVAL);
            engine = kWorks;
            fail_malloc = true;
            CHECK(rqa_run(h, kSeries, int64_t(1) << 22, two) == RQA_ENOMEM);
            fail_malloc = false;
            expect(h, n);
            CHECK(rqa_run(h, kSeries, kLong, two) == RQA_OK);
            expect(h, kLong);
            rqa_destroy(h);
        }
        h = handle();
        CHECK(batch(h, 200, one) == RQA_OK);
        if (fetched) expect_batch(h, 200);
        engine = kRefuses;
        CHECK(rqa_run(h, kSeries, kLonger, one) == RQA_EINVAL);
        engine = kWorks;
        expect_batch(h, 200);
        // Histograms that were in a workspace which has gone are an error.
        fail_malloc = true;
        CHECK(rqa_run(h, kSeries, int64_t(1) << 22, two) == RQA_ENOMEM);
        fail_malloc = false;
        std::vector<uint64_t> d(300);
        CHECK(rqa_result_batch(h, 3, nullptr, d.data(), nullptr, nullptr, 300) == RQA_EDEVICE);
        rqa_destroy(h);
    }

    // A launch that fails after kernels of it were enqueued, and one whose kernels
    // did not run, have no result: not their own, and not an earlier run's.
    for (int late = 0; late < 2; ++late) {
        h = handle();
        CHECK(rqa_run(h, kSeries, kLonger, one) == RQA_OK);
        engine = late ? kFailsLate : kNeverRuns;
        CHECK(rqa_run(h, kSeries, kShort, one) == (late ? RQA_EDEVICE : RQA_OK));
        engine = kWorks;
        rqa_measures m;
        CHECK(rqa_result(h, &m, nullptr, nullptr, nullptr, 0) == RQA_EDEVICE);
        CHECK(rqa_run(h, kSeries, kShort, one) == RQA_OK);
        expect(h, kShort);
        rqa_destroy(h);
    }

    // A captured run allocates nothing and waits for nothing.
    h = handle();
    CHECK(rqa_run(h, kSeries, kLong, one) == RQA_OK);
    expect(h, kLong);
    const int before = host_mallocs;
    fs(two)->capturing = true;
    CHECK(rqa_run(h, kSeries, kShort, two) == RQA_OK);
    fs(two)->capturing = false;
    CHECK(host_mallocs == before);
    expect(h, kShort);
    rqa_destroy(h);

    // Nor does a captured plot with more boxes than one before it: it has none.
    h = handle();
    uint64_t *bits = reinterpret_cast<uint64_t *>(4096);
    CHECK(rqa_plot(h, kSeries, 640, bits, 10, one) == RQA_OK && plot_boxes);
    fs(two)->capturing = true;
    CHECK(rqa_plot_cross(h, kSeries, 5000, kSeries, 640, bits, 10, two) == RQA_OK && !plot_boxes);
    CHECK(rqa_plot(h, kSeries, 600, bits, 10, two) == RQA_OK && plot_boxes);
    fs(two)->capturing = false;
    CHECK(rqa_plot_cross(h, kSeries, 5000, kSeries, 640, bits, 10, two) == RQA_OK && plot_boxes);
    rqa_destroy(h);

    // Trials: the neighbour of four waves is eight, but two for short strips, whose
    // launch has no use for more.
    struct { int64_t n; int count, other; } shapes[] = {
        {2000, 1, 2}, {2000, 300, 2}, {3000, 1, 2}, {3000, 31, 2}, {3000, 32, 8}, {3000, 300, 8}, {5000, 1, 8}};
    for (const auto &s : shapes) {
        CHECK(rqa_create(&h, 1, 1, 0.5f, 3, 2, 2, 2, 1) == RQA_OK);
        std::vector<int64_t> off(s.count, 0), len(s.count, s.n);
        for (int k = 0; k < 3; ++k) {
            CHECK(rqa_run_batch(h, kSeries, s.n, off.data(), len.data(), s.count, one) == RQA_OK);
            int32_t waves = 0, graph = 0;
            CHECK(rqa_last_launch(h, &waves, &graph) == RQA_OK);
            CHECK(waves == (k == 1 ? s.other : 4));
            CHECK(rqa_result_batch_all(h, std::vector<rqa_measures>(s.count).data(), nullptr, s.count) == RQA_OK);
        }
        rqa_destroy(h);
    }

    CHECK(hipStreamDestroy(one) == hipSuccess && hipStreamDestroy(two) == hipSuccess);
    return 0;
}
