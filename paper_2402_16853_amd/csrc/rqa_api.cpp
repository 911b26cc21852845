// C ABI of librqa: parameter validation, device workspace, enqueue of the hot
// path on the caller's stream, and result retrieval (Sect. 7: Settings ->
// RQAComputation.create -> run -> RQAResult; missing devices and invalid input
// are reported as errors, never aborts).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <limits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "rqa_internal.h"

namespace rqa {

int validate_params(const rqa_params &p) {
    if (p.m < 1 || p.tau < 1) return RQA_EINVAL;
    if (!(p.eps >= 0.0f) || std::isinf(p.eps)) return RQA_EINVAL;
    if (p.norm < RQA_NORM_L1 || p.norm > RQA_NORM_LINF) return RQA_EINVAL;
    if (p.lmin < 1 || p.vmin < 1 || p.wmin < 1 || p.theiler < 0) return RQA_EINVAL;
    // (m-1)*tau must fit comfortably in 32 bits for device index arithmetic.
    if (static_cast<int64_t>(p.m - 1) * p.tau > (int64_t(1) << 30)) return RQA_EINVAL;
    return RQA_OK;
}

Workspace::~Workspace() {
    if (base) {
        int cur = -1;
        hipGetDevice(&cur);
        if (device >= 0 && cur != device) hipSetDevice(device);
        hipFree(base);
        if (device >= 0 && cur != device && cur >= 0) hipSetDevice(cur);
    }
}

int Workspace::reserve(size_t need) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return RQA_EDEVICE;
    need = (need + 255) & ~size_t(255);
    if (base && device == dev && bytes >= need) return RQA_OK;
    if (base) {
        if (device != dev) {
            hipSetDevice(device);
            hipDeviceSynchronize();
            hipFree(base);
            hipSetDevice(dev);
        } else {
            hipDeviceSynchronize();
            hipFree(base);
        }
        base = nullptr;
        bytes = 0;
    }
    void *p = nullptr;
    if (hipMalloc(&p, need) != hipSuccess) {
        (void)hipGetLastError();
        return RQA_ENOMEM;
    }
    base = p;
    bytes = need;
    device = dev;
    return RQA_OK;
}

}  // namespace rqa

using namespace rqa;

// ---------------------------------------------------------------------------
// Workgroup-shape autotuner.  For a launch signature (norm, m, size class,
// number of jobs) it times each candidate shape on real runs (tiles, stitch and
// statistics, measured with hipEvents when the run's result is fetched) and then keeps the
// fastest.  Results never depend on the shape, so trial runs are ordinary runs.
// The table is process-wide; with RQA_AUTOTUNE_CACHE=<file> decisions persist
// across processes as "key waves" lines.
// ---------------------------------------------------------------------------
namespace {

constexpr int kNumCandidates = 3;

struct TuneEntry {
    int cand[kNumCandidates] = {};   // trials: the default shape, its neighbour, the default again
    int ncand = 0;
    int next = 0;          // next candidate to try
    int best = 0;          // best waves so far
    double best_ms = 1e300;
    bool done = false;
};

// Three trials: the default shape, its neighbour, and the default again, because a
// signature's first run is a cold one: with one run per shape the 65,521-point Lorenz
// series settled on 4 waves (640 us) instead of 8 (500 us).  The neighbour is 4 of 8
// waves, and 8 of 4, or 2 where the strips are short: below 2,048 delay vectors, and
// in a launch of few jobs below 4,096.  Runs with 2 / 4 / 8 waves, us: uniform points,
// 2,000: 92 / 103 / 131, 3,000: 122 / 122 / 149, 4,100: 121 / 115 / 124, 30,000: 860 /
// 563 / 495; 1,000 windows of 1,200 1,423 / 1,495 / 1,599, of 3,958 (m = 5) 6,276 / 4,128 /
// 3,677; 300 of 3,000 Lorenz points 626 / 496 / 488; Lorenz and sine runs as uniform ones.
void tune_init(TuneEntry &e, int dflt, int64_t nmax, int32_t count) {
    const bool low = nmax < 2048 || (nmax < 4096 && count < 32);
    const int other = dflt > 4 ? 4 : low ? 2 : 8;
    e.ncand = 3;
    e.cand[0] = e.cand[2] = dflt;
    e.cand[1] = other;
}

std::mutex g_tune_mu;
std::map<std::string, TuneEntry> g_tune;
bool g_tune_loaded = false;

void tune_load_locked() {
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char *path = std::getenv("RQA_AUTOTUNE_CACHE");
    if (!path) return;
    std::ifstream f(path);
    std::string key;
    int waves;
    while (f >> key >> waves) {
        if (waves < 1 || waves > 8) continue;
        TuneEntry &e = g_tune[key];
        e.best = waves;
        e.done = true;
    }
}

void tune_store_locked(const std::string &key, int waves) {
    const char *path = std::getenv("RQA_AUTOTUNE_CACHE");
    if (!path) return;
    std::ofstream f(path, std::ios::app);
    f << key << " " << waves << "\n";
}

int ilog2(int64_t v) {
    int l = 0;
    while (v > 1) { v >>= 1; ++l; }
    return l;
}

std::string tune_key(const rqa_params &p, int64_t nmax, int32_t count) {
    char buf[96];
    std::snprintf(buf, sizeof buf, "norm%d_m%d_n2^%d_jobs2^%d_w%d", p.norm, p.m <= 6 ? p.m : 0,
                  ilog2(nmax), ilog2(count), p.theiler > 64 ? 65 : p.theiler);
    return buf;
}

uint64_t fnv(uint64_t h, const void *data, size_t bytes) {
    const unsigned char *c = static_cast<const unsigned char *>(data);
    for (size_t k = 0; k < bytes; ++k) h = (h ^ c[k]) * 1099511628211ull;
    return h;
}

}  // namespace

struct rqa_handle {
    rqa_params p{};
    Workspace ws;
    void *staging = nullptr;        // pinned host buffer for launch descriptors
    size_t staging_bytes = 0;
    hipEvent_t staging_free = nullptr;   // recorded when a launch has read `staging`
    bool profiling = false;
    bool prof_valid = false;
    PhaseEvents prof{};
    int waves = 0;                  // 0 = autotuned
    int groups = 0;                 // 0 = fill the device
    int64_t ws_limit = 0;           // line-summary bytes of a one-series run (0 = default)
    JobPlan plan{};                 // how the last run's first job was cut
    bool has_run = false;
    bool batched = false;
    hipStream_t stream = nullptr;
    std::vector<int64_t> nvec;      // per job: rows (delay vectors)
    std::vector<int64_t> ncols;     // per job: columns
    std::vector<int64_t> hlen;      // per job: histogram entries
    std::vector<size_t> job_off;    // per job: byte offset of its histograms in ws.base
    size_t info_block_off = 0;      // info records (flag + statistics) of all jobs
    size_t hist_block_off = 0;      // histograms of all jobs, contiguous
    size_t hist_block_bytes = 0;
    bool on_device = false;         // ... of the last run are still in the workspace
    // Pinned memory that a launch writes its info records to, and behind them (one
    // short job) its histograms.  A block stays until the handle goes, also when a
    // larger one has taken its place: an earlier run, or a graph that the caller
    // captured, may still write to it.  Each is at least twice as large as the one
    // before, so all of them are less than two of the last.
    char *pub = nullptr;
    size_t pub_bytes = 0;
    char *pub_old[48] = {};
    int pub_olds = 0;
    char *rec = nullptr;            // the last run's records there (nullptr: none, they are copied)
    bool rec_hist = false;          // and its histograms
    uint32_t run = 0;               // number of the last run, which its records carry
    uint32_t run_next = 1;
    char *info_copy = nullptr;      // records copied from the device (rec == nullptr)
    size_t info_copy_bytes = 0;
    uint64_t *host_cache = nullptr;
    size_t host_cache_bytes = 0;
    bool info_valid = false;
    bool cache_valid = false;
    bool last_from_graph = false;   // the last run was a graph replay
    // autotuning trial in flight
    bool trial = false;
    int trial_waves = 0;
    std::string trial_key;
    // graph replay of repeated identical launches
    uint64_t last_sig = 0;
    uint64_t graph_sig = 0;
    uint32_t graph_run = 0;         // number of the run that was captured
    hipGraphExec_t graph = nullptr;
    void *graph_staging = nullptr;
    hipStream_t capture_stream = nullptr;
    // recurrence plot output: tail scratch, and the event after the last plot
    float *plot_tail = nullptr;
    size_t plot_tail_bytes = 0;
    hipEvent_t plot_done = nullptr;
};

namespace {

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

void drop_graph(rqa_handle *h) {
    if (h->graph) hipGraphExecDestroy(h->graph);
    if (h->graph_staging) hipHostFree(h->graph_staging);
    h->graph = nullptr;
    h->graph_staging = nullptr;
    h->graph_sig = 0;
}

int ensure_events(rqa_handle *h) {
    if (!h->prof.ev[0]) {
        for (hipEvent_t &e : h->prof.ev)
            if (hipEventCreate(&e) != hipSuccess) return RQA_EDEVICE;
    }
    return RQA_OK;
}

// Pinned memory of at least `need` bytes for a launch on `st` to write its results
// to, or nullptr: none to be had, or `st` is being captured, where no memory may
// be allocated.  The results are then copied from the device when they are
// fetched.
char *result_block(rqa_handle *h, size_t need, hipStream_t st) {
    if (h->pub_bytes >= need) return h->pub;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (cap != hipStreamCaptureStatusNone || h->pub_olds == 48) return nullptr;
    const size_t size = std::max(need, 2 * h->pub_bytes);
    void *p = nullptr;
    if (hipHostMalloc(&p, size, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::memset(p, 0, size);   // no run is number 0: records that none has written
    if (h->pub) h->pub_old[h->pub_olds++] = h->pub;
    h->pub = static_cast<char *>(p);
    h->pub_bytes = size;
    return h->pub;
}

// Capture the launch of `jobs` into a graph (own staging buffer, own capture
// stream) and instantiate it.
int capture_graph(rqa_handle *h, const std::vector<Job> &jobs, char *base, uint64_t sig) {
    drop_graph(h);
    if (!h->capture_stream &&
        hipStreamCreateWithFlags(&h->capture_stream, hipStreamNonBlocking) != hipSuccess)
        return RQA_EDEVICE;
    if (hipHostMalloc(&h->graph_staging, align256(engine_launch_scratch_bytes(jobs.size())),
                      hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        h->graph_staging = nullptr;
        return RQA_ENOMEM;
    }
    if (hipStreamBeginCapture(h->capture_stream, hipStreamCaptureModeRelaxed) != hipSuccess)
        return RQA_EDEVICE;
    int rc = engine_launch(jobs, base, h->graph_staging, nullptr, h->groups, h->capture_stream,
                           nullptr);
    hipGraph_t g = nullptr;
    const hipError_t ec = hipStreamEndCapture(h->capture_stream, &g);
    if (rc != RQA_OK || ec != hipSuccess || !g) {
        if (g) hipGraphDestroy(g);
        (void)hipGetLastError();
        drop_graph(h);
        return rc != RQA_OK ? rc : RQA_EDEVICE;
    }
    const hipError_t ei = hipGraphInstantiate(&h->graph, g, nullptr, nullptr, 0);
    hipGraphDestroy(g);
    if (ei != hipSuccess) {
        (void)hipGetLastError();
        h->graph = nullptr;
        drop_graph(h);
        return RQA_EDEVICE;
    }
    h->graph_sig = sig;
    h->graph_run = jobs[0].run;
    return RQA_OK;
}

// Lay out the workspace for `jobs` and enqueue them: [launch scratch][info
// records of every job][histograms of every job][job scratch].  The launch also
// writes the records, and the histograms of one short job, to pinned memory; a
// batch's histograms are copied, when asked for, in one go.  `sig` identifies the
// launch apart from the workspace; an identical repeat replays a captured graph.
// The handle goes on describing the run before until the launch has succeeded.
int launch(rqa_handle *h, std::vector<Job> &jobs, int waves, bool trial, const std::string &key,
           uint64_t sig, void *stream, bool batched) {
    const int32_t count = static_cast<int32_t>(jobs.size());
    std::vector<int64_t> nvec(count), ncols(count), hlen(count);
    std::vector<size_t> off(count);
    size_t total = align256(engine_launch_scratch_bytes(count));
    const size_t info_block_off = total;
    total += align256(kInfoBytes * static_cast<size_t>(count));
    const size_t hist_block_off = total;
    for (int32_t w = 0; w < count; ++w) {
        jobs[w].waves = waves;
        jobs[w].fine = count == 1;
    }
    if (count > 1) engine_batch_segs(jobs);
    // A job run alone (a series, a cross pair or a given matrix) is cut into
    // row bands when its line summaries would exceed the workspace limit.
    if (count == 1) {
        size_t limit = static_cast<size_t>(h->ws_limit);
        if (limit == 0) {
            int dev = 0;
            size_t total_mem = 0;
            if (hipGetDevice(&dev) != hipSuccess || hipDeviceTotalMem(&total_mem, dev) != hipSuccess)
                return RQA_EDEVICE;
            limit = total_mem / 4;
        }
        jobs[0].band_strips = engine_band_strips(jobs[0], limit);
        sig = fnv(sig, &jobs[0].band_strips, sizeof jobs[0].band_strips);
    }
    Job first = jobs[0];
    const JobPlan plan = engine_job_plan(first);
    for (int32_t w = 0; w < count; ++w) {
        nvec[w] = jobs[w].n_vec;
        ncols[w] = jobs[w].mode == kModeAuto ? jobs[w].n_vec : jobs[w].n_cols;
        hlen[w] = jobs[w].hist_len();
        off[w] = total;
        total += align256(sizeof(uint64_t) * 3 * static_cast<size_t>(hlen[w]));
    }
    const size_t hist_block_bytes = total - hist_block_off;
    std::vector<size_t> soff(count);
    for (int32_t w = 0; w < count; ++w) {
        soff[w] = total;
        total += align256(engine_job_scratch_bytes(jobs[w]));
    }
    const void *old_base = h->ws.base;
    const size_t old_bytes = h->ws.bytes;
    int rc = h->ws.reserve(total);
    if (h->ws.base != old_base || h->ws.bytes != old_bytes) {   // (also where the reserve has failed)
        h->on_device = false;
        drop_graph(h);
    }
    if (rc != RQA_OK) return rc;
    const size_t stage = align256(engine_launch_scratch_bytes(count));
    if (!h->staging_free &&
        hipEventCreateWithFlags(&h->staging_free, hipEventDisableTiming) != hipSuccess)
        return RQA_EDEVICE;
    if (h->staging_bytes < stage) {
        if (h->has_run) hipEventSynchronize(h->staging_free);
        if (h->staging) hipHostFree(h->staging);
        h->staging = nullptr;
        h->staging_bytes = 0;
        if (hipHostMalloc(&h->staging, stage, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return RQA_ENOMEM;
        }
        h->staging_bytes = stage;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t rec_bytes = kInfoBytes * static_cast<size_t>(count);
    bool rec_hist = count == 1 && hlen[0] <= kPublishEntries;
    char *rec = result_block(
        h, rec_bytes + (rec_hist ? sizeof(uint64_t) * 3 * static_cast<size_t>(hlen[0]) : 0), st);
    if (!rec && rec_hist) {
        rec_hist = false;
        rec = result_block(h, rec_bytes, st);
    }
    uint32_t run = h->run_next++;
    if (run == 0) run = h->run_next++;
    char *base = static_cast<char *>(h->ws.base);
    for (int32_t w = 0; w < count; ++w) {
        Job &jb = jobs[w];
        jb.host_info = rec ? rec + kInfoBytes * static_cast<size_t>(w) : nullptr;
        jb.host_hist = rec_hist ? rec + rec_bytes : nullptr;
        jb.run = run;
        jb.hist = reinterpret_cast<uint64_t *>(base + off[w]);
        jb.flag = reinterpret_cast<int *>(base + info_block_off + kInfoBytes * w);
        jb.scratch = base + soff[w];
    }

    sig = fnv(sig, &h->p, sizeof h->p);
    sig = fnv(sig, &waves, sizeof waves);
    sig = fnv(sig, &h->groups, sizeof h->groups);
    sig = fnv(sig, &base, sizeof base);
    sig = fnv(sig, &rec, sizeof rec);
    sig = fnv(sig, &rec_hist, sizeof rec_hist);
    const bool plain = !h->profiling && !trial;

    h->last_from_graph = false;
    if (plain && h->graph && h->graph_sig == sig) {
        if (hipGraphLaunch(h->graph, st) != hipSuccess) return RQA_EDEVICE;
        h->prof_valid = false;
        h->last_from_graph = true;
        run = h->graph_run;
    } else if (plain && h->last_sig == sig && capture_graph(h, jobs, base, sig) == RQA_OK) {
        if (hipGraphLaunch(h->graph, st) != hipSuccess) return RQA_EDEVICE;
        h->prof_valid = false;
        h->last_from_graph = true;
        run = h->graph_run;
    } else {
        const bool timed = h->profiling || trial;
        if (timed && (rc = ensure_events(h)) != RQA_OK) return rc;
        rc = engine_launch(jobs, base, h->staging, h->staging_free, h->groups, st,
                           timed ? &h->prof : nullptr);
        h->prof_valid = timed && rc == RQA_OK;
        if (rc == RQA_EDEVICE) h->on_device = false;   // some of its kernels may have been enqueued
        if (rc != RQA_OK) return rc;
    }
    h->last_sig = sig;
    h->plan = plan;
    h->trial = trial;
    h->trial_waves = waves;
    h->trial_key = key;
    h->nvec = std::move(nvec);
    h->ncols = std::move(ncols);
    h->hlen = std::move(hlen);
    h->job_off = std::move(off);
    h->info_block_off = info_block_off;
    h->hist_block_off = hist_block_off;
    h->hist_block_bytes = hist_block_bytes;
    h->info_valid = false;
    h->cache_valid = false;
    h->on_device = true;
    h->rec = rec;
    h->rec_hist = rec_hist;
    h->run = run;
    h->stream = st;
    h->has_run = true;
    h->batched = batched;
    return RQA_OK;
}

int enqueue(rqa_handle *h, const float *d_series, int64_t n_points, const int64_t *offsets,
            const int64_t *lengths, int32_t count, void *stream, bool batched) {
    if (!h || !d_series) return RQA_EINVAL;
    std::vector<Job> jobs(count);
    const KParams kp = make_kparams(h->p);
    int64_t nmax = 0;
    for (int32_t w = 0; w < count; ++w) {
        const int64_t o = offsets ? offsets[w] : 0;
        const int64_t len = lengths ? lengths[w] : n_points;
        if (o < 0 || len < 0 || o > n_points || len > n_points - o) return RQA_EINVAL;
        const int64_t nv = len - static_cast<int64_t>(h->p.m - 1) * h->p.tau;
        if (nv < 1) return RQA_ETOOSHORT;
        if (nv > (int64_t(1) << 31) - 2) return RQA_EINVAL;
        Job &jb = jobs[w];
        jb.series = d_series + o;
        jb.n_points = len;
        jb.n_vec = nv;
        jb.n_cols = nv;
        jb.kp = kp;
        nmax = std::max(nmax, nv);
    }

    // Workgroup shape: fixed by rqa_set_tiling, else tuned per signature.
    bool trial = false;
    int waves = h->waves;
    std::string key;
    if (waves == 0) {
        key = tune_key(h->p, nmax, count);
        std::lock_guard<std::mutex> lk(g_tune_mu);
        tune_load_locked();
        TuneEntry &e = g_tune[key];
        if (!e.done && e.ncand == 0) tune_init(e, engine_default_waves(nmax), nmax, count);
        if (e.done) {
            waves = e.best;
        } else {
            waves = e.cand[e.next];
            trial = true;
        }
    }
    uint64_t sig = 1469598103934665603ull;
    const int32_t mode = kModeAuto;
    sig = fnv(sig, &mode, sizeof mode);
    sig = fnv(sig, &d_series, sizeof d_series);
    sig = fnv(sig, &n_points, sizeof n_points);
    sig = fnv(sig, &count, sizeof count);
    if (offsets) sig = fnv(sig, offsets, sizeof(int64_t) * count);
    if (lengths) sig = fnv(sig, lengths, sizeof(int64_t) * count);
    return launch(h, jobs, waves, trial, key, sig, stream, batched);
}

// Waves per workgroup of a full matrix.  The default shape's rule is one for the rows;
// many cells behind few rows (from 2^27, and 2,048 rows: four strips of eight waves)
// take eight waves too, 24 instead of 16 on a CU.  Cross recurrence with four and with
// eight, us: uniform points (m = 5) 8,000 x 200,000 1,152 and 1,060, 3,388 x 94,121 350 and
// 341; Lorenz 222 and 211 there, logistic 2,560 x 60,000 298 and 317.  Fewer rows lose
// more (1,800 x 80,000: logistic 257 and 314, uniform 244 and 250, sine 177 and 164).  A given
// matrix, which has no predicate, takes four up to 24,576 rows: half-full ones of 20,000^2
// 694 us with four, 764 with eight (a tenth full 387, 370), of 30,000^2 1,342 and 1,278.
int full_waves(const Job &jb) {
    if (jb.mode == kModeMatrix && jb.n_vec < 24576) return 4;
    const bool wide = jb.n_vec >= 2048 && jb.n_vec * jb.n_cols >= int64_t(1) << 27;
    return engine_default_waves(wide ? std::max(jb.n_vec, jb.n_cols) : jb.n_vec);
}

// One job over a full (not symmetric) matrix: the cross recurrence matrix of
// (a, b), or a given bit matrix.
int enqueue_full(rqa_handle *h, Job jb, void *stream) {
    if (jb.n_vec > (int64_t(1) << 31) - 2 || jb.n_cols > (int64_t(1) << 31) - 2)
        return RQA_EINVAL;
    jb.kp = make_kparams(h->p);
    const int waves = h->waves > 0 ? h->waves : full_waves(jb);
    std::vector<Job> jobs(1, jb);
    uint64_t sig = 1469598103934665603ull;
    sig = fnv(sig, &jb.mode, sizeof jb.mode);
    sig = fnv(sig, &jb.series, sizeof jb.series);
    sig = fnv(sig, &jb.n_points, sizeof jb.n_points);
    sig = fnv(sig, &jb.series_b, sizeof jb.series_b);
    sig = fnv(sig, &jb.n_points_b, sizeof jb.n_points_b);
    sig = fnv(sig, &jb.bits, sizeof jb.bits);
    sig = fnv(sig, &jb.n_vec, sizeof jb.n_vec);
    sig = fnv(sig, &jb.n_cols, sizeof jb.n_cols);
    sig = fnv(sig, &jb.words, sizeof jb.words);
    return launch(h, jobs, waves, false, std::string(), sig, stream, false);
}

// Record the time of a finished autotuning trial: tiles, stitch and statistics
// (fewer waves per workgroup mean more strips to stitch: 65,521 Lorenz points take
// 0.39 + 0.10 ms with 8 waves, 0.45 + 0.16 with 4).
void finish_trial(rqa_handle *h) {
    if (!h->trial) return;
    h->trial = false;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, h->prof.ev[1], h->prof.ev[3]) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    std::lock_guard<std::mutex> lk(g_tune_mu);
    TuneEntry &e = g_tune[h->trial_key];
    const int w = h->trial_waves;
    if (e.done || e.ncand == 0 || e.cand[e.next] != w) return;
    if (ms < e.best_ms) {
        e.best_ms = ms;
        e.best = w;
    }
    if (++e.next >= e.ncand) {
        e.done = true;
        tune_store_locked(h->trial_key, e.best);
    }
}

int fetch(rqa_handle *h, int32_t index, rqa_measures *out, uint64_t *diag, uint64_t *vert,
          uint64_t *white, int64_t hist_len) {
    if (!h) return RQA_EINVAL;
    if (!h->has_run) return RQA_ESTATE;
    if (index < 0 || index >= static_cast<int32_t>(h->nvec.size())) return RQA_EINVAL;
    const int64_t n = h->nvec[index];
    const int64_t hl = h->hlen[index];
    if ((diag || vert || white) && hist_len < hl) return RQA_ESIZE;
    // Grow a pinned host buffer.
    auto grow = [](void **buf, size_t *have, size_t need) -> int {
        if (*have >= need) return RQA_OK;
        if (*buf) hipHostFree(*buf);
        *buf = nullptr;
        *have = 0;
        if (hipHostMalloc(buf, need, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return RQA_ENOMEM;
        }
        *have = need;
        return RQA_OK;
    };
    if (!h->info_valid) {
        // Every job's flag and statistics are in host memory once the launch
        // has passed, or are copied there.
        if (!h->rec) {
            const size_t need = kInfoBytes * h->nvec.size();
            if (h->info_copy_bytes < need) {
                std::free(h->info_copy);
                h->info_copy = static_cast<char *>(std::malloc(need));
                h->info_copy_bytes = h->info_copy ? need : 0;
                if (!h->info_copy) return RQA_ENOMEM;
            }
            if (!h->on_device ||
                hipMemcpyAsync(h->info_copy, static_cast<const char *>(h->ws.base) + h->info_block_off,
                               need, hipMemcpyDeviceToHost, h->stream) != hipSuccess)
                return RQA_EDEVICE;
        }
        if (hipStreamSynchronize(h->stream) != hipSuccess) return RQA_EDEVICE;
        finish_trial(h);
        h->info_valid = true;
    }
    const char *info = (h->rec ? h->rec : h->info_copy) + kInfoBytes * static_cast<size_t>(index);
    if (h->rec) {
        // Another number: this run's kernels did not run, or those of a later
        // launch that failed have written over its record.
        uint32_t run = 0;
        std::memcpy(&run, info + 4, sizeof run);
        if (run != h->run) return RQA_EDEVICE;
    }
    int flag = 0;
    std::memcpy(&flag, info, sizeof(int));
    if (flag & 1) return RQA_ENONFINITE;
    if (flag) return RQA_EDEVICE;   // internal consistency check failed on the device
    if (diag || vert || white) {
        // Entries above a histogram's longest line are zero (the device
        // statistics hold the longest lines), so only the prefixes cross PCIe
        // and the tails are cleared on the host.  A launch of one job copies
        // its three prefixes; a batch copies the block of all its jobs once.
        JobStats st;
        std::memcpy(&st, info + 8, sizeof st);
        int64_t used[3];
        for (int k = 0; k < 3; ++k)
            used[k] = std::min<int64_t>(hl, static_cast<int64_t>(st.longest[k]) + 1);
        const bool single = h->nvec.size() == 1;
        if (!h->cache_valid && !h->rec_hist) {
            if (!h->on_device) return RQA_EDEVICE;
            int rc = grow(reinterpret_cast<void **>(&h->host_cache), &h->host_cache_bytes,
                          h->hist_block_bytes);
            if (rc != RQA_OK) return rc;
            const char *dev = static_cast<const char *>(h->ws.base) + h->hist_block_off;
            bool ok = true;
            if (single) {
                for (int k = 0; k < 3 && ok; ++k)
                    ok = hipMemcpyAsync(reinterpret_cast<char *>(h->host_cache) +
                                            sizeof(uint64_t) * k * hl,
                                        dev + sizeof(uint64_t) * k * hl, sizeof(uint64_t) * used[k],
                                        hipMemcpyDeviceToHost, h->stream) == hipSuccess;
            } else {
                ok = hipMemcpyAsync(h->host_cache, dev, h->hist_block_bytes, hipMemcpyDeviceToHost,
                                    h->stream) == hipSuccess;
            }
            if (!ok || hipStreamSynchronize(h->stream) != hipSuccess) return RQA_EDEVICE;
            h->cache_valid = true;
        }
        const uint64_t *hd = reinterpret_cast<const uint64_t *>(
            h->rec_hist ? h->rec + kInfoBytes
                        : reinterpret_cast<const char *>(h->host_cache) +
                              (h->job_off[index] - h->hist_block_off));
        uint64_t *dst[3] = {diag, vert, white};
        for (int k = 0; k < 3; ++k) {
            if (!dst[k]) continue;
            std::memcpy(dst[k], hd + k * hl, sizeof(uint64_t) * used[k]);
            std::memset(dst[k] + used[k], 0, sizeof(uint64_t) * (hl - used[k]));
        }
    }
    if (out) {
        JobStats st;
        std::memcpy(&st, info + 8, sizeof st);
        measures_from_stats(st, n, h->ncols[index], h->p, out);
    }
    return RQA_OK;
}

}  // namespace

extern "C" {

int rqa_create(rqa_handle **out, int32_t m, int32_t tau, float eps, int32_t norm, int32_t lmin,
               int32_t vmin, int32_t wmin, int32_t theiler) {
    if (!out) return RQA_EINVAL;
    rqa_params p{m, tau, eps, norm, lmin, vmin, wmin, theiler};
    const int rc = validate_params(p);
    if (rc != RQA_OK) return rc;
    rqa_handle *h = new (std::nothrow) rqa_handle;
    if (!h) return RQA_ENOMEM;
    h->p = p;
    *out = h;
    return RQA_OK;
}

int rqa_hist_len(const rqa_handle *h, int64_t n_points, int64_t *len) {
    if (!h || !len) return RQA_EINVAL;
    const int64_t nv = n_points - static_cast<int64_t>(h->p.m - 1) * h->p.tau;
    if (nv < 1) return RQA_ETOOSHORT;
    *len = nv + 1;
    return RQA_OK;
}

int rqa_run(rqa_handle *h, const float *d_series, int64_t n_points, void *hip_stream) {
    if (!h) return RQA_EINVAL;
    if (n_points < 0) return RQA_EINVAL;
    return enqueue(h, d_series, n_points, nullptr, nullptr, 1, hip_stream, false);
}

int rqa_cross_hist_len(const rqa_handle *h, int64_t na_points, int64_t nb_points, int64_t *len) {
    if (!h || !len) return RQA_EINVAL;
    const int64_t d = static_cast<int64_t>(h->p.m - 1) * h->p.tau;
    const int64_t na = na_points - d, nb = nb_points - d;
    if (na < 1 || nb < 1) return RQA_ETOOSHORT;
    *len = std::max(na, nb) + 1;
    return RQA_OK;
}

int rqa_run_cross(rqa_handle *h, const float *d_a, int64_t na_points, const float *d_b,
                  int64_t nb_points, void *hip_stream) {
    if (!h || !d_a || !d_b || na_points < 0 || nb_points < 0) return RQA_EINVAL;
    const int64_t d = static_cast<int64_t>(h->p.m - 1) * h->p.tau;
    Job jb;
    jb.mode = kModeCross;
    jb.series = d_a;
    jb.n_points = na_points;
    jb.n_vec = na_points - d;
    jb.series_b = d_b;
    jb.n_points_b = nb_points;
    jb.n_cols = nb_points - d;
    if (jb.n_vec < 1 || jb.n_cols < 1) return RQA_ETOOSHORT;
    return enqueue_full(h, jb, hip_stream);
}

int rqa_run_matrix(rqa_handle *h, const uint64_t *d_bits, int64_t n_rows, int64_t n_cols,
                   int64_t words_per_row, void *hip_stream) {
    if (!h || !d_bits || n_rows < 1 || n_cols < 1 || words_per_row < (n_cols + 63) / 64)
        return RQA_EINVAL;
    Job jb;
    jb.mode = kModeMatrix;
    jb.n_vec = n_rows;
    jb.n_cols = n_cols;
    jb.bits = d_bits;
    jb.words = words_per_row;
    return enqueue_full(h, jb, hip_stream);
}

namespace {

// Enqueue a recurrence plot; the tail scratch is reused, so a plot waits (on the
// device) for the previous one of this handle.
int plot(rqa_handle *h, const float *a, int64_t na_points, const float *b, int64_t nb_points,
         uint64_t *d_bits, int64_t words, void *hip_stream) {
    const KParams kp = make_kparams(h->p);
    const int64_t d = static_cast<int64_t>(h->p.m - 1) * h->p.tau;
    const int64_t na = na_points - d, nb = b ? nb_points - d : na;
    if (na < 1 || nb < 1) return RQA_ETOOSHORT;
    if (na > (int64_t(1) << 31) - 2 || nb > (int64_t(1) << 31) - 2) return RQA_EINVAL;
    if (words < (nb + 63) / 64) return RQA_ESIZE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const size_t need = sizeof(float) * static_cast<size_t>(engine_plot_scratch_floats(kp, na, nb, b != nullptr));
    if (!h->plot_done && hipEventCreateWithFlags(&h->plot_done, hipEventDisableTiming) != hipSuccess)
        return RQA_EDEVICE;
    bool boxes = true;
    if (h->plot_tail_bytes < need && h->plot_tail_bytes >= sizeof(float) * engine_plot_tail_floats(kp)) {
        // A plot that is being captured allocates nothing: without room for its
        // boxes it evaluates every pair.
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        boxes = hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone;
        if (!boxes) (void)hipGetLastError();
    }
    if (boxes && h->plot_tail_bytes < need) {
        if (h->plot_tail) {
            hipEventSynchronize(h->plot_done);
            hipFree(h->plot_tail);
        }
        h->plot_tail = nullptr;
        h->plot_tail_bytes = 0;
        if (hipMalloc(&h->plot_tail, need) != hipSuccess) {
            (void)hipGetLastError();
            return RQA_ENOMEM;
        }
        h->plot_tail_bytes = need;
    } else if (hipStreamWaitEvent(st, h->plot_done, 0) != hipSuccess) {
        return RQA_EDEVICE;
    }
    const int rc = engine_plot(kp, a, na_points, b, nb_points, d_bits, words, h->plot_tail, boxes, st);
    if (rc != RQA_OK) return rc;
    return hipEventRecord(h->plot_done, st) == hipSuccess ? RQA_OK : RQA_EDEVICE;
}

}  // namespace

int rqa_plot(rqa_handle *h, const float *d_series, int64_t n_points, uint64_t *d_bits,
             int64_t words_per_row, void *hip_stream) {
    if (!h || !d_series || !d_bits || n_points < 0 || words_per_row < 1) return RQA_EINVAL;
    return plot(h, d_series, n_points, nullptr, 0, d_bits, words_per_row, hip_stream);
}

int rqa_plot_cross(rqa_handle *h, const float *d_a, int64_t na_points, const float *d_b,
                   int64_t nb_points, uint64_t *d_bits, int64_t words_per_row, void *hip_stream) {
    if (!h || !d_a || !d_b || !d_bits || na_points < 0 || nb_points < 0 || words_per_row < 1)
        return RQA_EINVAL;
    return plot(h, d_a, na_points, d_b, nb_points, d_bits, words_per_row, hip_stream);
}

int rqa_result(rqa_handle *h, rqa_measures *out, uint64_t *diag, uint64_t *vert, uint64_t *white,
               int64_t hist_len) {
    if (h && h->has_run && h->batched) return RQA_ESTATE;
    return fetch(h, 0, out, diag, vert, white, hist_len);
}

int rqa_run_batch(rqa_handle *h, const float *d_series, int64_t n_points, const int64_t *offsets,
                  const int64_t *lengths, int32_t count, void *hip_stream) {
    if (!h || !offsets || !lengths || count < 1 || n_points < 0) return RQA_EINVAL;
    return enqueue(h, d_series, n_points, offsets, lengths, count, hip_stream, true);
}

int rqa_result_batch(rqa_handle *h, int32_t index, rqa_measures *out, uint64_t *diag,
                     uint64_t *vert, uint64_t *white, int64_t hist_len) {
    return fetch(h, index, out, diag, vert, white, hist_len);
}

int rqa_result_batch_all(rqa_handle *h, rqa_measures *out, int32_t *status, int32_t count) {
    if (!h || !out || count < 1) return RQA_EINVAL;
    if (!h->has_run) return RQA_ESTATE;
    if (count != static_cast<int32_t>(h->nvec.size())) return RQA_ESIZE;
    int first = RQA_OK;
    for (int32_t k = 0; k < count; ++k) {
        const int rc = fetch(h, k, &out[k], nullptr, nullptr, nullptr, 0);
        if (rc != RQA_OK) {
            // No result for this window: NaN measures, nothing recurrent.
            const double nan = std::numeric_limits<double>::quiet_NaN();
            out[k] = rqa_measures{nan, nan, nan, nan, nan, nan, nan, nan, nan, nan, nan, nan, nan,
                                  0u, h->nvec[k]};
            if (first == RQA_OK) first = rc;
        }
        if (status) status[k] = rc;
    }
    return first;
}

int rqa_measures_from_hist(const uint64_t *diag, const uint64_t *vert, const uint64_t *white,
                           int64_t n, const rqa_params *p, rqa_measures *out) {
    if (!diag || !vert || !white || !p || !out || n < 1) return RQA_EINVAL;
    const int rc = validate_params(*p);
    if (rc != RQA_OK) return rc;
    measures_from_hist(diag, vert, white, n, *p, out);
    return RQA_OK;
}

int rqa_set_tiling(rqa_handle *h, int32_t waves_per_group, int32_t groups) {
    if (!h || waves_per_group < 0 || waves_per_group > 8 || groups < 0) return RQA_EINVAL;
    h->waves = waves_per_group;
    h->groups = groups;
    return RQA_OK;
}

int rqa_set_profiling(rqa_handle *h, int32_t enable) {
    if (!h) return RQA_EINVAL;
    h->profiling = enable != 0;
    h->prof_valid = false;
    return RQA_OK;
}

int rqa_get_timings(rqa_handle *h, double *prepare_ms, double *tiles_ms, double *stitch_ms) {
    if (!h) return RQA_EINVAL;
    if (!h->prof_valid) return RQA_ESTATE;
    if (hipEventSynchronize(h->prof.ev[3]) != hipSuccess) return RQA_EDEVICE;
    float a = 0.f, b = 0.f, c = 0.f;
    if (hipEventElapsedTime(&a, h->prof.ev[0], h->prof.ev[1]) != hipSuccess ||
        hipEventElapsedTime(&b, h->prof.ev[1], h->prof.ev[2]) != hipSuccess ||
        hipEventElapsedTime(&c, h->prof.ev[2], h->prof.ev[3]) != hipSuccess)
        return RQA_EDEVICE;
    if (prepare_ms) *prepare_ms = a;
    if (tiles_ms) *tiles_ms = b;
    if (stitch_ms) *stitch_ms = c;
    return RQA_OK;
}

int rqa_last_launch(const rqa_handle *h, int32_t *waves, int32_t *graph_replay) {
    if (!h) return RQA_EINVAL;
    if (!h->has_run) return RQA_ESTATE;
    if (waves) *waves = h->trial_waves;
    if (graph_replay) *graph_replay = h->last_from_graph ? 1 : 0;
    return RQA_OK;
}

int rqa_workspace_plan(const rqa_params *p, int64_t n_points, int32_t waves, int64_t limit_bytes,
                       int32_t *bands, int32_t *band_strips, int32_t *segs,
                       int64_t *workspace_bytes) {
    if (!p || waves < 0 || waves > 8 || limit_bytes < 0) return RQA_EINVAL;
    int rc = validate_params(*p);
    if (rc != RQA_OK) return rc;
    const int64_t nv = n_points - static_cast<int64_t>(p->m - 1) * p->tau;
    if (nv < 1) return RQA_ETOOSHORT;
    if (nv > (int64_t(1) << 31) - 2) return RQA_EINVAL;
    Job jb;
    jb.n_points = n_points;
    jb.n_vec = nv;
    jb.n_cols = nv;
    jb.kp = make_kparams(*p);
    jb.waves = waves > 0 ? waves : engine_default_waves(nv);
    jb.fine = true;
    jb.band_strips = engine_band_strips(jb, static_cast<size_t>(limit_bytes));
    const JobPlan plan = engine_job_plan(jb);
    if (bands) *bands = plan.bands;
    if (band_strips) *band_strips = plan.band_strips;
    if (segs) *segs = plan.segs;
    if (workspace_bytes) *workspace_bytes = static_cast<int64_t>(plan.scratch_bytes);
    return RQA_OK;
}

int rqa_set_workspace_limit(rqa_handle *h, int64_t bytes) {
    if (!h || bytes < 0) return RQA_EINVAL;
    h->ws_limit = bytes;
    return RQA_OK;
}

int rqa_last_plan(const rqa_handle *h, int32_t *bands, int32_t *band_strips, int32_t *segs,
                  int32_t *strip_rows, int64_t *workspace_bytes) {
    if (!h) return RQA_EINVAL;
    if (!h->has_run) return RQA_ESTATE;
    if (bands) *bands = h->plan.bands;
    if (band_strips) *band_strips = h->plan.band_strips;
    if (segs) *segs = h->plan.segs;
    if (strip_rows) *strip_rows = h->plan.strip_rows;
    if (workspace_bytes) *workspace_bytes = static_cast<int64_t>(h->plan.scratch_bytes);
    return RQA_OK;
}

void rqa_destroy(rqa_handle *h) {
    if (!h) return;
    if (h->has_run) hipStreamSynchronize(h->stream);
    if (h->staging) hipHostFree(h->staging);
    if (h->staging_free) hipEventDestroy(h->staging_free);
    for (hipEvent_t e : h->prof.ev)
        if (e) hipEventDestroy(e);
    drop_graph(h);
    if (h->capture_stream) hipStreamDestroy(h->capture_stream);
    if (h->host_cache) hipHostFree(h->host_cache);
    if (h->pub) hipHostFree(h->pub);
    for (int k = 0; k < h->pub_olds; ++k) hipHostFree(h->pub_old[k]);
    std::free(h->info_copy);
    if (h->plot_done) {
        hipEventSynchronize(h->plot_done);
        hipEventDestroy(h->plot_done);
    }
    if (h->plot_tail) hipFree(h->plot_tail);
    delete h;
}

const char *rqa_strerror(int code) {
    switch (code) {
        case RQA_OK: return "ok";
        case RQA_EINVAL: return "invalid argument";
        case RQA_ETOOSHORT: return "series too short for the embedding (fewer than one delay vector)";
        case RQA_ENOMEM: return "out of memory";
        case RQA_EDEVICE: return "HIP device error";
        case RQA_ENONFINITE: return "series contains NaN or infinity";
        case RQA_ESIZE: return "output buffer too small";
        case RQA_ESTATE: return "invalid call order";
        case RQA_EBUDGET: return "job exceeds the memory budget (server pool or static scratch)";
        case RQA_EAGAIN: return "job not finished";
        case RQA_ENOTFOUND: return "unknown ticket";
        default: return "unknown error";
    }
}

}  // extern "C"
