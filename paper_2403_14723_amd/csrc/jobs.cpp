// gpolylla_mesh_jobs: meshes a list of host-resident triangulations with the
// host<->device copies of one group of jobs overlapped with the copies and
// the work of the next.
//
// One host thread and three streams: an upload stream, the context's stream
// (builds and meshing runs, in job order) and a download stream.  Per group
// of jobs (consecutive jobs up to a triangle budget, meshed as one batch):
//   1. queue the uploads of the next group's inputs;
//   2. wait for the previous group's meshing run to finish and queue its
//      downloads, so they run while this group builds and the next uploads;
//   3. build this group's half-edge structures (after its uploads; one host
//      wait for the whole group) and queue its meshing run;
//   4. give back the memory of groups whose downloads have completed (at
//      most two meshed groups hold memory at once).
// Memory goes back to the context's pool only after the host has seen the
// downloads that read it complete, so the pool's reuse stays ordered.
#include <semaphore.h>

#include <algorithm>
#include <chrono>
#include <cstring>
#include <deque>
#include <exception>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "runtime_internal.h"

using namespace gprt;

namespace {

struct Group {
    int j0 = 0, j1 = 0;                // jobs [j0, j1)
    std::vector<void *> dxy, dtri;     // uploaded inputs (until the builds)
    hipEvent_t uploaded = nullptr;     // the uploads have finished
    int up_rc = GP_OK;
    std::vector<int> job;              // job of each meshed entry
    std::vector<gp_mesh *> meshes;
    std::vector<gp_result *> res;
    hipEvent_t copied = nullptr;       // the group's downloads have finished
    bool queued = false;               // downloads queued
};

void group_free(Group &g) {
    for (gp_result *r : g.res) gpolylla_result_free(r);
    for (gp_mesh *m : g.meshes) gpolylla_mesh_free(m);
    g.res.clear();
    g.meshes.clear();
    if (g.copied) (void)hipEventDestroy(g.copied);
    g.copied = nullptr;
    if (g.uploaded) (void)hipEventDestroy(g.uploaded);
    g.uploaded = nullptr;
}

// Waits for the group's meshing run and queues the downloads of every job's
// outputs on the copy stream.
void group_download(gp_job *jobs, Group &g, hipStream_t cs) {
    for (size_t k = 0; k < g.res.size(); k++) {
        gp_job &jb = jobs[g.job[k]];
        gp_result_info info;
        int rc = gpolylla_result_info(g.res[k], &info);   // waits for the run
        gp_result_dev dv{};
        if (rc == GP_OK) rc = gpolylla_result_device(g.res[k], &dv);
        if (rc == GP_OK) {
            jb.npoly = info.npoly;
            jb.nloop_he = info.nloop_he;
            const size_t nh = (size_t)info.nh, P = (size_t)info.npoly, F = (size_t)info.nloop_he;
            hipError_t e = hipSuccess;
            if (jb.next && nh) e = hipMemcpyAsync(jb.next, dv.next, 4 * nh, hipMemcpyDeviceToHost, cs);
            if (e == hipSuccess && jb.prev && nh)
                e = hipMemcpyAsync(jb.prev, dv.prev, 4 * nh, hipMemcpyDeviceToHost, cs);
            if (e == hipSuccess && P) e = hipMemcpyAsync(jb.seeds, dv.seeds, 4 * P, hipMemcpyDeviceToHost, cs);
            if (e == hipSuccess)
                e = hipMemcpyAsync(jb.loop_off, dv.loop_off, 4 * (P + 1), hipMemcpyDeviceToHost, cs);
            if (e == hipSuccess && F) e = hipMemcpyAsync(jb.loop_he, dv.loop_he, 4 * F, hipMemcpyDeviceToHost, cs);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                rc = GP_EHIP;
            }
        }
        jb.status = rc;
    }
    if (hipEventCreateWithFlags(&g.copied, hipEventDisableTiming) != hipSuccess ||
        hipEventRecord(g.copied, cs) != hipSuccess) {
        (void)hipGetLastError();
        if (g.copied) (void)hipEventDestroy(g.copied);
        g.copied = nullptr;
        (void)hipStreamSynchronize(cs);   // without the event: wait here
    }
    g.queued = true;
}

// Waits for the group's downloads, then frees its device memory.
void group_finish(Group &g, hipStream_t cs) {
    if (!g.copied || hipEventSynchronize(g.copied) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(cs);
    }
    group_free(g);
}

// ---- small jobs: packed copies, one build-and-mesh launch per group -------
//
// A list whose jobs all fit one workgroup (gp::kJobSmallTri triangles,
// gp::kJobSmallV vertices) is not worth a build and a batched run per group:
// the dozen runtime calls per job that those take would bound it.  Each
// group's inputs are packed into one pinned staging block and uploaded with
// one copy; one launch builds and meshes every job (k_small_jobs); one copy
// brings every output back, and the host hands each job its part.  Groups
// overlap (small_jobs_run).

bool small_jobs_fit(const gp_ctx *c, const gp_job *jobs, int n) {
    int max_nt = 0;
    for (int i = 0; i < n; i++) {
        if (jobs[i].nt > gp::kJobSmallTri || jobs[i].nv > gp::kJobSmallV) return false;
        max_nt = std::max(max_nt, jobs[i].nt);
    }
    return c->cfg.small_max >= max_nt && gp::small_job_lds_bytes(max_nt) <= (size_t)c->cfg.lds_max;
}

// Byte offsets of one job's parts: inputs (xy, tri) in the upload block,
// outputs in the device block after them: every job's counts, seeds, loop_off
// and loop_he, then every job's next and prev (copied back when a job of the
// group asks for them).
struct SmallLayout {
    size_t xy, tri, counts, next, prev, seeds, loop_off, loop_he;
};

// One packed group in flight: its layout, staging blocks and device block.
struct SmallGroup {
    int j0 = 0, j1 = 0;
    std::vector<SmallLayout> lay;
    char *up = nullptr, *down = nullptr;
    size_t up_bytes = 0, out_bytes = 0;
    void *dev = nullptr;
    hipEvent_t done = nullptr;
    hipStream_t stream = nullptr;
    int rc = GP_OK;
    bool unpacked = false;
};

// Packs jobs [j0, j1) and queues their upload, the launch and the download.
void small_group_start(gp_ctx *c, gp_job *jobs, SmallGroup &g, hipStream_t s) {
    g.stream = s;
    const int n = g.j1 - g.j0;
    try {
        g.lay.assign(n, SmallLayout{});
    } catch (const std::bad_alloc &) {
        g.rc = GP_ENOMEM;
        return;
    }
    size_t in_bytes = 0, out_bytes = 0;
    bool links = false;   // a job asks for next and prev
    int max_nt = 0;
    for (int k = 0; k < n; k++) {
        const gp_job &jb = jobs[g.j0 + k];
        const size_t nh = 3 * (size_t)jb.nt;
        SmallLayout &L = g.lay[k];
        L.xy = in_bytes;
        in_bytes += align_up(8 * (size_t)jb.nv, 16);
        L.tri = in_bytes;
        in_bytes += align_up(12 * (size_t)jb.nt, 16);
        L.counts = out_bytes;
        out_bytes += align_up(4 * (size_t)gp::kJobCounts, 16);
        L.seeds = out_bytes;
        out_bytes += align_up(4 * (size_t)jb.nt + 4, 16);
        L.loop_off = out_bytes;
        out_bytes += align_up(4 * (size_t)jb.nt + 8, 16);
        L.loop_he = out_bytes;
        out_bytes += align_up(4 * nh + 4, 16);
        max_nt = std::max(max_nt, jb.nt);
        links |= jb.next != nullptr;
    }
    g.out_bytes = out_bytes;   // what is copied back
    for (int k = 0; k < n; k++) {
        const size_t nh = 3 * (size_t)jobs[g.j0 + k].nt;
        g.lay[k].next = out_bytes;
        out_bytes += align_up(4 * nh + 4, 16);
        g.lay[k].prev = out_bytes;
        out_bytes += align_up(4 * nh + 4, 16);
    }
    if (links) g.out_bytes = out_bytes;
    const size_t desc_off = align_up(in_bytes, 256);
    g.up_bytes = desc_off + sizeof(gp::SmallJob) * (size_t)n;   // inputs, then descriptors
    const size_t out_off = align_up(g.up_bytes, 256);
    g.rc = c->pool.alloc(out_off + out_bytes, &g.dev);
    if (g.rc != GP_OK) return;
    g.up = static_cast<char *>(pinned_take(c, g.up_bytes));
    g.down = static_cast<char *>(pinned_take(c, g.out_bytes));
    if (!g.up || !g.down || hipEventCreateWithFlags(&g.done, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        g.rc = GP_ENOMEM;
        return;
    }
    char *d = static_cast<char *>(g.dev);
    gp::SmallJob *descs = reinterpret_cast<gp::SmallJob *>(g.up + desc_off);
    for (int k = 0; k < n; k++) {
        const gp_job &jb = jobs[g.j0 + k];
        const SmallLayout &L = g.lay[k];
        if (jb.nv) std::memcpy(g.up + L.xy, jb.xy, 8 * (size_t)jb.nv);
        if (jb.nt) std::memcpy(g.up + L.tri, jb.tri, 12 * (size_t)jb.nt);
        gp::SmallJob &sj = descs[k];
        sj.xy = reinterpret_cast<const int2 *>(d + L.xy);
        sj.tri = reinterpret_cast<const int32_t *>(d + L.tri);
        sj.nv = jb.nv;
        sj.nt = jb.nt;
        sj.org = sj.twin = nullptr;   // (stay in LDS)
        sj.counts = reinterpret_cast<int32_t *>(d + out_off + L.counts);
        sj.next_o = reinterpret_cast<int32_t *>(d + out_off + L.next);
        sj.prev_o = reinterpret_cast<int32_t *>(d + out_off + L.prev);
        sj.seeds = reinterpret_cast<int32_t *>(d + out_off + L.seeds);
        sj.loop_off = reinterpret_cast<int32_t *>(d + out_off + L.loop_off);
        sj.loop_he = reinterpret_cast<int32_t *>(d + out_off + L.loop_he);
        sj.xy_out = nullptr;
        sj.build_only = 0;
        sj.pad = 0;
    }
    if (hipMemcpyAsync(d, g.up, g.up_bytes, hipMemcpyHostToDevice, s) != hipSuccess ||
        gp::launch_small_jobs(reinterpret_cast<const gp::SmallJob *>(d + desc_off), n, max_nt, s) !=
            hipSuccess ||
        hipMemcpyAsync(g.down, d + out_off, g.out_bytes, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipEventRecord(g.done, s) != hipSuccess) {
        (void)hipGetLastError();
        g.rc = GP_EHIP;
    }
}

// Waits for a started group and hands each job its outputs and status.  May
// run on another thread than the one that starts groups: it touches the
// group's own blocks and jobs only.
void small_group_unpack(gp_job *jobs, SmallGroup &g) {
    if (g.rc == GP_OK && hipEventSynchronize(g.done) != hipSuccess) {
        (void)hipGetLastError();
        g.rc = GP_EHIP;
    }
    if (g.rc != GP_OK) (void)hipStreamSynchronize(g.stream);   // nothing may still read or write the blocks
    for (int k = 0; k < g.j1 - g.j0 && g.rc == GP_OK; k++) {
        gp_job &jb = jobs[g.j0 + k];
        const SmallLayout &L = g.lay[k];
        const int32_t *cnt = reinterpret_cast<const int32_t *>(g.down + L.counts);
        const uint64_t key = (uint64_t)(uint32_t)cnt[8] | ((uint64_t)(uint32_t)cnt[9] << 32);
        gp::MeshCounters mc;
        std::memcpy(&mc, cnt, sizeof mc);
        if (key != ~0ull) {
            jb.status = -(int)(key & 0xff);
            continue;
        }
        if (mc.err || mc.npoly < 0 || mc.npoly > jb.nt || mc.nloop < 0 || mc.nloop > 3 * jb.nt) {
            jb.status = GP_ECORRUPT;
            continue;
        }
        const size_t nh = 3 * (size_t)jb.nt;
        jb.npoly = mc.npoly;
        jb.nloop_he = mc.nloop;
        if (jb.next && nh) std::memcpy(jb.next, g.down + L.next, 4 * nh);
        if (jb.prev && nh) std::memcpy(jb.prev, g.down + L.prev, 4 * nh);
        if (mc.npoly) std::memcpy(jb.seeds, g.down + L.seeds, 4 * (size_t)mc.npoly);
        std::memcpy(jb.loop_off, g.down + L.loop_off, 4 * ((size_t)mc.npoly + 1));
        if (mc.nloop) std::memcpy(jb.loop_he, g.down + L.loop_he, 4 * (size_t)mc.nloop);
        jb.status = GP_OK;
    }
    if (g.rc != GP_OK)
        for (int k = g.j0; k < g.j1; k++) jobs[k].status = g.rc;
}

// Gives an unpacked group's memory back (on the calling thread: the pool and
// the pinned blocks belong to the context).
void small_group_free(gp_ctx *c, SmallGroup &g) {
    if (g.up) pinned_give(c, g.up, g.up_bytes);
    if (g.down) pinned_give(c, g.down, g.out_bytes);
    if (g.dev) c->pool.release(g.dev);
    if (g.done) (void)hipEventDestroy(g.done);
    g = SmallGroup{};
}

// Groups in flight at once, the threads that unpack besides the caller's, and
// the triangles of a group when the caller names no size.  A list in one group
// is packed, copied in, meshed, copied out and unpacked one after the other:
// 3,050 us for 512 jobs of 2,048 triangles (17 MB in, 35 MB out).  In groups the
// device works on some while the host packs the next and the helpers unpack the
// last: 1,750 us with one stream and one helper, 1,600 us with two streams (a
// group's inputs go up while another's outputs come down), 1,450 us with two
// helpers, 1,360 us with threads and stream kept between calls.  Half the triangles to a group is as fast, twice as many is slower
// (1,900 us: too few groups to overlap).
constexpr int kGroupsInFlight = 5, kHelpers = 2;
constexpr int64_t kPackedTriangles = 128 << 10, kLargeGroup = 8 << 20;

}  // namespace

// What the packed lists of a context keep between calls: the helper threads
// (asleep meanwhile), the second stream, and the groups of the list that runs.
// Made by the first list of more than one group, given back with the context.
// A helper that the system has not scheduled yet holds nothing up: the
// caller's thread takes the groups that no helper has.  (Threads and a stream
// made by each call cost it 250 us, and up to 2 ms when the joins had to wait
// for threads that had not run.)  Nor does the caller's thread sleep while helpers
// work: after work that had kept every CPU busy, others of which still spin (a
// parallel loop's workers), a thread that slept waits 3 to 4 ms for its turn.  So
// it took 4 to 5 ms for every other such list that it waited for on a condition
// variable (whose notification, too, may wait for a thread that was notified
// before and has not run), all groups unpacked within 1.4; a semaphore polled
// for a while takes 1.5 to 2.4 (3.5 with one thread and one group).
struct gprt::JobCrew {
    int device = 0;
    hipStream_t second = nullptr;
    hipEvent_t before = nullptr;
    std::vector<std::thread> helpers;
    std::mutex mu;
    // posted for each group started, to the helpers in turn: the same groups of a
    // list that is run again then go to the cores that had them (a list of 100
    // jobs in two groups: 450 us, and 535 in half of the processes when any helper
    // woke), and for each group that a helper has unpacked
    sem_t work[kHelpers], finished;
    bool quit = false;
    bool alone = false;   // the caller's thread unpacks every group, in order
    gp_job *jobs = nullptr;
    std::deque<SmallGroup> live;   // started groups, oldest first (its elements stay where they are)
    size_t started = 0, taken = 0, done = 0, freed = 0;   // groups so far, in order

    static void wait(sem_t &s) {
        while (sem_wait(&s) != 0) {
        }   // (a signal)
    }
    // Unpacks the oldest group that no thread has taken.
    void unpack_one(std::unique_lock<std::mutex> &lk) {
        SmallGroup &g = live[taken++ - freed];
        lk.unlock();
        small_group_unpack(jobs, g);
        lk.lock();
        g.unpacked = true;
        while (done < started && live[done - freed].unpacked) done++;
    }
    void help(int me) {
        (void)hipSetDevice(device);
        while (true) {
            wait(work[me]);
            std::unique_lock<std::mutex> lk(mu);
            if (quit) return;
            if (taken == started || alone) continue;
            unpack_one(lk);
            lk.unlock();
            sem_post(&finished);
        }
    }
    // Until a helper has unpacked a group, now or since the caller last waited.
    // The caller's thread stays awake for as long as that takes with helpers
    // that run (as it does in the runtime's own waits).
    void wait_finished(std::unique_lock<std::mutex> &lk) {
        lk.unlock();
        const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(5);
        bool got = false;
        do got = sem_trywait(&finished) == 0;
        while (!got && std::chrono::steady_clock::now() < until);
        if (!got) wait(finished);
        lk.lock();
    }
    void free_done(gp_ctx *c) {
        for (; freed < done; freed++) {
            small_group_free(c, live.front());
            live.pop_front();
        }
    }
    // Until every started group has been unpacked and its memory given back.
    void drain(gp_ctx *c) {
        std::unique_lock<std::mutex> lk(mu);
        while (taken < started) unpack_one(lk);
        while (done < started) wait_finished(lk);
        free_done(c);
    }
    explicit JobCrew(int dev) : device(dev) {
        if (hipStreamCreateWithFlags(&second, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&before, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            if (second) (void)hipStreamDestroy(second);
            second = nullptr;
        }
        for (sem_t &w : work) sem_init(&w, 0, 0);
        sem_init(&finished, 0, 0);
        try {
            helpers.reserve(kHelpers);
            for (int k = 0; k < kHelpers; k++) helpers.emplace_back([this, k]() { help(k); });
        } catch (const std::exception &) {
        }   // (no thread to be had, or no memory for it: the caller's does all)
    }
    ~JobCrew() {
        {
            std::lock_guard<std::mutex> lk(mu);
            quit = true;
        }
        for (sem_t &w : work) sem_post(&w);
        for (std::thread &t : helpers) t.join();
        for (sem_t &w : work) sem_destroy(&w);
        sem_destroy(&finished);
        if (before) (void)hipEventDestroy(before);
        if (second) (void)hipStreamDestroy(second);
    }
};

void gprt::job_crew_free(gp_ctx *c) {
    delete c->crew;
    c->crew = nullptr;
}

namespace {

// Arrays that jobs of a list share, by what each job may read or write.
enum class Shared {
    nothing,
    outputs,   // an output array of one and an output array of another, of whatever kind
    inputs     // an output array of one and an input array of another
};

Shared shared_arrays(const gp_job *jobs, int n) {
    struct Range {
        uintptr_t at, end;
        bool operator<(const Range &o) const { return at < o.at; }
    };
    constexpr int kKinds = 5;
    std::vector<Range> kind[kKinds];
    Range span[kKinds] = {};   // of all ranges of a kind
    for (int q = 0; q < kKinds; q++) {
        std::vector<Range> &r = kind[q];
        r.reserve(n);
        for (int k = 0; k < n; k++) {
            const gp_job &j = jobs[k];
            const int32_t *const at[kKinds] = {j.next, j.prev, j.loop_he, j.seeds, j.loop_off};
            const size_t nt = (size_t)j.nt, ints = q < 3 ? 3 * nt : q == 3 ? nt : nt + 1;
            if (at[q] && ints) r.push_back({(uintptr_t)at[q], (uintptr_t)(at[q] + ints)});
        }
        if (!std::is_sorted(r.begin(), r.end())) std::sort(r.begin(), r.end());
        for (const Range &x : r) span[q] = span[q].end ? Range{span[q].at, std::max(span[q].end, x.end)} : x;
    }
    const auto meet = [](const Range &a, const Range &b) { return a.at < b.end && b.at < a.end; };
    const auto overlap = [](const std::vector<Range> &r) {
        for (size_t k = 1; k < r.size(); k++)
            if (r[k - 1].end > r[k].at) return true;
        return false;
    };
    // every kind by itself; all together only if their spans meet (arrays of the
    // kinds are often apart, or one array per kind cut up for the jobs)
    bool outputs = false, mixed = false;
    for (int q = 0; q < kKinds; q++) {
        outputs |= overlap(kind[q]);
        for (int p = 0; p < q; p++) mixed |= meet(span[p], span[q]);
    }
    const auto in_a_span = [&](const Range &x) {
        return std::any_of(span, span + kKinds, [&](const Range &s) { return meet(s, x); });
    };
    std::vector<Range> all;
    const auto merge = [&]() {
        for (const std::vector<Range> &r : kind) {
            const size_t m = all.size();
            all.insert(all.end(), r.begin(), r.end());
            std::inplace_merge(all.begin(), all.begin() + m, all.end());
        }
    };
    if (!outputs && mixed) {
        merge();
        outputs = overlap(all);
    }
    for (int k = 0; k < n; k++) {
        const gp_job &j = jobs[k];
        for (const Range &x : {Range{(uintptr_t)j.xy, (uintptr_t)(j.xy + 2 * (size_t)j.nv)},
                               Range{(uintptr_t)j.tri, (uintptr_t)(j.tri + 3 * (size_t)j.nt)}}) {
            if (x.at == x.end || !in_a_span(x)) continue;
            if (outputs) return Shared::inputs;   // (as far as is known)
            if (all.empty()) merge();
            auto after = std::upper_bound(all.begin(), all.end(), x);
            if ((after != all.end() && meet(*after, x)) || (after != all.begin() && meet(after[-1], x)))
                return Shared::inputs;
        }
    }
    return outputs ? Shared::outputs : Shared::nothing;
}

// Runs a list of small jobs as one group, if it has at most `triangles` triangles
// (0: kPackedTriangles), or in groups of as many, but at most kPackedTriangles.
// (Five groups of the size that a caller gives take 2.5 times the memory that two
// took, and a context's first list pays for it: 2,048 jobs of 2,048 triangles in
// groups of 512K 37 ms, 23 with two groups in flight, now 18; repeated lists 4.7
// ms, 8.1 and 4.6.)  Jobs that share output arrays (a caller may want only the
// last one's) are unpacked in order, by one thread.  Where one job's outputs lie
// over another's inputs, groups are as large as given (0: kLargeGroup) and two at
// most are in flight, so that a job's inputs are read before the outputs of the
// others of its group and of the group before are written.
void small_jobs_run(gp_ctx *c, gp_job *jobs, int n, int64_t triangles) {
    int64_t budget = triangles > 0 ? triangles : kPackedTriangles, total = 0;
    for (int k = 0; k < n && total <= budget; k++) total += jobs[k].nt;
    Shared shared = Shared::nothing;
    if (total > budget || n >= 65536) {   // more than one group
        budget = std::min(budget, kPackedTriangles);
        try {
            shared = shared_arrays(jobs, n);
        } catch (const std::bad_alloc &) {
            shared = Shared::inputs;   // (not known)
        }
    }
    if (shared == Shared::inputs) budget = triangles > 0 ? triangles : kLargeGroup;
    const size_t in_flight = shared == Shared::inputs ? 2 : kGroupsInFlight;
    JobCrew *crew = c->crew;
    // Every second group goes to a stream of its own, so that one group's inputs
    // go up while another's outputs come down.  Its blocks may still be in use
    // by earlier work on the context's stream, so it starts after that.
    hipStream_t streams[2] = {c->stream, c->stream};
    int j0 = 0;
    for (int k = 0; j0 < n; k++) {
        SmallGroup g;
        int64_t tri = 0;
        g.j0 = g.j1 = j0;
        while (g.j1 < n && g.j1 - g.j0 < 65535 && (g.j1 == g.j0 || tri + jobs[g.j1].nt <= budget))
            tri += jobs[g.j1++].nt;
        j0 = g.j1;
        if (k == 0 && j0 < n) {
            if (!crew) crew = c->crew = new (std::nothrow) JobCrew(c->device);
            if (crew) {
                std::lock_guard<std::mutex> lk(crew->mu);
                crew->alone = shared != Shared::nothing;
            }
            if (crew && crew->second) {
                if (hipEventRecord(crew->before, c->stream) == hipSuccess &&
                    hipStreamWaitEvent(crew->second, crew->before, 0) == hipSuccess)
                    streams[1] = crew->second;
                else
                    (void)hipGetLastError();
            }
        }
        small_group_start(c, jobs, g, streams[k % 2]);
        if (g.rc == GP_ENOMEM && crew && k > 0) {   // no room beside the groups in flight: alone, then
            const int first = g.j0, end = g.j1;
            small_group_free(c, g);
            crew->drain(c);
            g.j0 = first;
            g.j1 = end;
            small_group_start(c, jobs, g, streams[k % 2]);
        }
        if (!crew || (k == 0 && j0 == n)) {   // a list of one group, or no memory for the crew
            small_group_unpack(jobs, g);
            small_group_free(c, g);
            continue;
        }
        std::unique_lock<std::mutex> lk(crew->mu);
        crew->jobs = jobs;
        try {
            crew->live.push_back(std::move(g));
        } catch (const std::bad_alloc &) {   // (g is as it was) in its turn, by this thread
            lk.unlock();
            crew->drain(c);
            small_group_unpack(jobs, g);
            small_group_free(c, g);
            continue;
        }
        crew->started++;
        if (!crew->alone) sem_post(&crew->work[k % kHelpers]);
        while (crew->started - crew->done >= in_flight) {
            if (crew->taken < crew->started &&
                (crew->alone || crew->helpers.empty() || crew->started - crew->taken >= in_flight - 1))
                crew->unpack_one(lk);
            else
                crew->wait_finished(lk);
        }
        crew->free_done(c);
    }
    if (crew) crew->drain(c);
}

}  // namespace

extern "C" {

int gpolylla_mesh_jobs(gp_ctx *c, gp_job *jobs, int32_t n, int64_t group_triangles, uint32_t flags) {
    if (!c || n < 0 || (n > 0 && !jobs)) return GP_EINVAL;
    if (flags & ~(uint32_t)GP_GRAPH) return GP_EINVAL;
    for (int i = 0; i < n; i++) {
        const gp_job &j = jobs[i];
        if (j.nv < 0 || j.nt < 0 || (j.nv > 0 && !j.xy) || (j.nt > 0 && !j.tri) || !j.seeds || !j.loop_off ||
            !j.loop_he || ((j.next == nullptr) != (j.prev == nullptr)))
            return GP_EINVAL;
        if (3ll * j.nt >= (1ll << 31)) return GP_ERANGE;
    }
    for (int i = 0; i < n; i++) {
        jobs[i].npoly = jobs[i].nloop_he = 0;
        jobs[i].status = GP_OK;
    }
    if (n == 0) return GP_OK;
    const int64_t budget = group_triangles > 0 ? group_triangles : kLargeGroup;
    DeviceGuard dg(c->device);
    if (small_jobs_fit(c, jobs, n)) {   // every job builds and meshes in one workgroup
        small_jobs_run(c, jobs, n, group_triangles);
        int rc_all = GP_OK;
        for (int i = 0; i < n; i++)
            if (jobs[i].status != GP_OK && rc_all == GP_OK) rc_all = jobs[i].status;
        return rc_all;
    }
    hipStream_t us = nullptr, cs = nullptr;   // uploads, downloads
    if (hipStreamCreateWithFlags(&us, hipStreamNonBlocking) != hipSuccess ||
        hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        if (us) (void)hipStreamDestroy(us);
        return GP_EHIP;
    }
    hipStream_t s = c->stream;
    const uint32_t mesh_flags = GP_ASYNC | (flags & GP_GRAPH);
    std::deque<Group> live;   // groups holding device memory, oldest first
    int next_job = 0;

    // Forms the next group and queues the uploads of its inputs on the
    // upload stream.
    auto prepare = [&](Group &g) {
        g.j0 = next_job;
        int64_t tri = 0;
        while (next_job < n && (next_job == g.j0 || tri + jobs[next_job].nt <= budget)) tri += jobs[next_job++].nt;
        g.j1 = next_job;
        const int gn = g.j1 - g.j0;
        g.dxy.assign(gn, nullptr);
        g.dtri.assign(gn, nullptr);
        g.up_rc = GP_OK;
        for (int k = 0; k < gn && g.up_rc == GP_OK; k++) {
            const gp_job &jb = jobs[g.j0 + k];
            g.up_rc = c->pool.alloc(8 * (size_t)std::max(jb.nv, 1), &g.dxy[k]);
            if (g.up_rc == GP_OK) g.up_rc = c->pool.alloc(12 * (size_t)std::max(jb.nt, 1), &g.dtri[k]);
            if (g.up_rc == GP_OK && jb.nv &&
                hipMemcpyAsync(g.dxy[k], jb.xy, 8 * (size_t)jb.nv, hipMemcpyHostToDevice, us) != hipSuccess)
                g.up_rc = GP_EHIP;
            if (g.up_rc == GP_OK && jb.nt &&
                hipMemcpyAsync(g.dtri[k], jb.tri, 12 * (size_t)jb.nt, hipMemcpyHostToDevice, us) != hipSuccess)
                g.up_rc = GP_EHIP;
        }
        if (g.up_rc == GP_OK && (hipEventCreateWithFlags(&g.uploaded, hipEventDisableTiming) != hipSuccess ||
                                 hipEventRecord(g.uploaded, us) != hipSuccess))
            g.up_rc = GP_EHIP;
        if (g.up_rc != GP_OK) (void)hipGetLastError();
    };

    Group cur;
    prepare(cur);
    while (true) {
        // 1. the next group's uploads, while this group builds
        Group nxt;
        const bool more = next_job < n;
        if (more) prepare(nxt);
        // 2. the previous group's downloads, overlapping both
        if (!live.empty() && !live.back().queued) group_download(jobs, live.back(), cs);
        // 3. this group's builds (after its uploads) and one meshing run
        const int gn = cur.j1 - cur.j0;
        if (cur.up_rc == GP_OK && hipStreamWaitEvent(s, cur.uploaded, 0) != hipSuccess) {
            (void)hipGetLastError();
            cur.up_rc = GP_EHIP;
        }
        if (cur.up_rc != GP_OK) {
            (void)hipStreamSynchronize(us);   // its uploads may still read the inputs
            for (int k = 0; k < gn; k++) jobs[cur.j0 + k].status = cur.up_rc;
        } else {
            std::vector<const int32_t *> pxy(gn), ptri(gn);
            std::vector<int32_t> nv(gn), nt(gn);
            std::vector<gp_mesh *> ms(gn, nullptr);
            std::vector<int> st(gn, GP_OK);
            for (int k = 0; k < gn; k++) {
                pxy[k] = static_cast<const int32_t *>(cur.dxy[k]);
                ptri[k] = static_cast<const int32_t *>(cur.dtri[k]);
                nv[k] = jobs[cur.j0 + k].nv;
                nt[k] = jobs[cur.j0 + k].nt;
            }
            const int b = gprt::build_many(c, gn, pxy.data(), nv.data(), ptri.data(), nt.data(), GP_IN_DEVICE,
                                           ms.data(), st.data());
            for (int k = 0; k < gn; k++) {
                const int r = b != GP_OK ? b : st[k];
                jobs[cur.j0 + k].status = r;
                if (r == GP_OK) {
                    cur.meshes.push_back(ms[k]);
                    cur.job.push_back(cur.j0 + k);
                }
            }
        }
        // the builds have drained the stream: the uploaded inputs are free
        for (void *p : cur.dxy) c->pool.release(p);
        for (void *p : cur.dtri) c->pool.release(p);
        cur.dxy.clear();
        cur.dtri.clear();
        if (!cur.meshes.empty()) {
            cur.res.assign(cur.meshes.size(), nullptr);
            const int mr =
                gpolylla_mesh_batch(c, cur.meshes.data(), (int32_t)cur.meshes.size(), mesh_flags, cur.res.data());
            if (mr != GP_OK) {
                for (int idx : cur.job) jobs[idx].status = mr;
                cur.res.clear();
                for (gp_mesh *m : cur.meshes) gpolylla_mesh_free(m);
                cur.meshes.clear();
                cur.job.clear();
            }
        }
        live.push_back(std::move(cur));
        // 4. at most two meshed groups hold memory: the one being downloaded
        //    and the one just queued
        while (live.size() > 2) {
            if (!live.front().queued) group_download(jobs, live.front(), cs);
            group_finish(live.front(), cs);
            live.pop_front();
        }
        if (!more) break;
        cur = std::move(nxt);
    }
    while (!live.empty()) {
        if (!live.front().queued) group_download(jobs, live.front(), cs);
        group_finish(live.front(), cs);
        live.pop_front();
    }
    (void)hipStreamDestroy(cs);
    (void)hipStreamDestroy(us);
    int rc_all = GP_OK;
    for (int i = 0; i < n; i++)
        if (jobs[i].status != GP_OK && rc_all == GP_OK) rc_all = jobs[i].status;
    return rc_all;
}

}  // extern "C"
