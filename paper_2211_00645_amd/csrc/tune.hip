// tune.hip -- launch-shape tuning: the on-disk cache of tuned shapes shared
// by the batch and single-stack tuners, and the single-stack tuner.
//
// The vector kernel's plane pacing has a cliff: paced a little below the
// rate the memory system sustains, every wavefront keeps to the schedule;
// paced above it, the wavefronts fall behind, stop sleeping and drift apart,
// and the launch runs at the unpaced speed, 10-25% slower.  Where the cliff
// lies depends on the frame (how many waves a row needs, the read/write
// mix) and differs by a few percent between devices, so a fixed pace either
// leaves speed unused or sits past the cliff.  The tuner measures it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "common.hpp"
#include "tune.hpp"
#include "deskew.h"

namespace dsk {

namespace {
std::mutex g_file_mu;
}

std::string arch_name() {
    int dev = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&p, dev) != hipSuccess)
        return "unknown";
    std::string a(p.gcnArchName);
    const size_t c = a.find(':');
    return c == std::string::npos ? a : a.substr(0, c);
}

bool tune_cache_lookup(const std::string &key, dsk_tune *t, double *ms, int *mode) {
    const char *path = std::getenv("DSK_TUNE_CACHE");
    if (!path || !*path) return false;
    std::lock_guard<std::mutex> lk(g_file_mu);
    std::FILE *f = std::fopen(path, "r");
    if (!f) return false;
    char line[512];
    bool found = false;
    while (std::fgets(line, sizeof line, f)) {
        char k[256];
        dsk_tune c{};
        double m = 0.0;
        int md = 0;
        const int got = std::sscanf(
            line,
            " \"%255[^\"]\": {\"block\": %d, \"per_thread\": %d, \"nt_store\": %d, "
            "\"unroll\": %d, \"wg_per_cu\": %d, \"pace_gbs\": %d, \"ms\": %lf, \"mode\": %d}",
            k, &c.block, &c.per_thread, &c.nt_store, &c.unroll, &c.wg_per_cu, &c.pace_gbs, &m,
            &md);
        if (got >= 8 && key == k && tune_ok(c) && md >= 0 && md <= 2) {
            *t = c;
            *ms = m;
            if (mode) *mode = got == 9 ? md : 0;
            found = true;
        }
    }
    std::fclose(f);
    return found;
}

void tune_cache_store(const std::string &key, const dsk_tune &t, double ms, int mode) {
    const char *path = std::getenv("DSK_TUNE_CACHE");
    if (!path || !*path) return;
    std::lock_guard<std::mutex> lk(g_file_mu);
    // Keep every other entry, replace this key, rewrite the file.
    std::vector<std::string> keep;
    if (std::FILE *f = std::fopen(path, "r")) {
        char line[512];
        while (std::fgets(line, sizeof line, f)) {
            char k[256];
            if (std::sscanf(line, " \"%255[^\"]\":", k) == 1 && key != k) {
                std::string s(line);
                while (!s.empty() && (s.back() == '\n' || s.back() == ',')) s.pop_back();
                keep.push_back(s);
            }
        }
        std::fclose(f);
    }
    char ent[512];
    std::snprintf(ent, sizeof ent,
                  "  \"%s\": {\"block\": %d, \"per_thread\": %d, \"nt_store\": %d, "
                  "\"unroll\": %d, \"wg_per_cu\": %d, \"pace_gbs\": %d, \"ms\": %.6f, "
                  "\"mode\": %d}",
                  key.c_str(), t.block, t.per_thread, t.nt_store, t.unroll, t.wg_per_cu,
                  t.pace_gbs, ms, mode);
    keep.push_back(ent);
    const std::string tmp = std::string(path) + ".tmp";
    std::FILE *f = std::fopen(tmp.c_str(), "w");
    if (!f) return;
    std::fputs("{\n", f);
    for (size_t i = 0; i < keep.size(); ++i)
        std::fprintf(f, "%s%s\n", keep[i].c_str(), i + 1 < keep.size() ? "," : "");
    std::fputs("}\n", f);
    std::fclose(f);
    std::rename(tmp.c_str(), path);
}

}  // namespace dsk

using namespace dsk;

namespace {

// Shapes the single-stack tuner times.  With a volume: one 4-column group
// per lane with a 2- or 4-plane pipeline, and two groups per lane, each
// unpaced and paced over the range where the cliff lies on the frames
// measured (5000-6000 GB/s; one group per lane, 2-plane pipeline, in
// 100 GB/s steps); the default shape is always a candidate.
// Without a volume nothing is paced: groups and pipeline depth only.
std::vector<dsk_tune> fwd_candidates(bool paced) {
    if (!paced) {
        // without a volume: the default (paced at 9000), its shape unpaced
        // and at 12000, a 2-plane pipeline unpaced and at 9000, two groups
        // per lane unpaced
        std::vector<dsk_tune> c{kDefaultProjTune, dsk_tune{64, 4, 1, 4, 0, 0},
                                dsk_tune{64, 4, 1, 4, 0, 12000}, dsk_tune{64, 4, 1, 2, 0, 0},
                                dsk_tune{64, 4, 1, 2, 0, 9000}};
        for (int u : {2, 4}) c.push_back(dsk_tune{64, 8, 1, u, 0, 0});
        return c;
    }
    // every 100 GB/s from 5000 (the step-down below then lands exactly 100
    // under the best pace: the float32 256 x 512 x 1024 frame's best, 5400,
    // stepped down to 5200 while 5300 was missing)
    std::vector<dsk_tune> c{kDefaultTune};
    for (int pace : {0, 5000, 5100, 5200, 5300, 5400, 5500, 5600, 5800, 5900, 6000})
        c.push_back(dsk_tune{64, 4, 1, 2, 0, pace});
    // a 4-plane pipeline keeps more reads in flight where tiles are few (a
    // float32 stack of 256 x 512 x 1024 into 1793 columns: 0.308 ms at 5400
    // against 0.334 for the best 2-plane shape)
    for (int pace : {0, 5000, 5200, 5400, 5600, 5800, 6000})
        c.push_back(dsk_tune{64, 4, 1, 4, 0, pace});
    for (int pace : {0, 5000, 5200, 5400, 5600, 5800, 6000})
        c.push_back(dsk_tune{64, 8, 1, 2, 0, pace});
    return c;
}

// How the buffers tile is part of the key: it decides which vector kernel runs
// and where its pace's cliff lies (default_tune in deskew.hip: 5700 GB/s on
// 128-byte boundaries is past it elsewhere).
std::string fwd_key(const char *tiling, int in_is_f32, dsk_dims d, int64_t width, bool offs,
                    const float *vol, const float *psum, const float *pmax) {
    char buf[200];
    std::snprintf(buf, sizeof buf, "%s/k%d/fwd/%s/%dx%dx%d/w%lld/%s/%s%s%s/%s",
                  arch_name().c_str(), kTuneRevision, in_is_f32 ? "f32" : "u16", d.planes, d.rows,
                  d.cols, (long long)width, tiling, vol ? "v" : "", psum ? "s" : "",
                  pmax ? "m" : "", offs ? "offsets" : "uniform");
    return buf;
}

std::mutex g_memo_mu;
std::map<std::string, std::pair<dsk_tune, double>> g_memo;

// Times every candidate `reps` times, round-robin (a burst of kBurst
// back-to-back launches of each per round, so slow drifts of the device
// touch all alike, and each is timed the way a stream of stacks runs it),
// after one untimed round.  Score: the mean time per launch over all
// rounds -- back-to-back throughput -- so a pace at the cliff's edge that
// falls behind now and then pays for those launches.
constexpr int kBurst = 3;

int time_candidates(const std::vector<dsk_tune> &cand, int reps, const void *in, int in_is_f32,
                    dsk_dims d, const double *offs, double shift, int64_t origin, float *vol,
                    float *psum, float *pmax, int64_t width, hipStream_t s,
                    std::vector<double> *score) {
    const size_t nc = cand.size();
    std::vector<hipEvent_t> ev(nc + 1, nullptr);
    int st = DSK_OK;
    for (size_t i = 0; i <= nc && st == DSK_OK; ++i)
        if (hipEventCreate(&ev[i]) != hipSuccess) st = DSK_EHIP;
    std::vector<double> sum(nc, 0.0);
    for (int round = 0; round <= reps && st == DSK_OK; ++round) {
        if (hipEventRecord(ev[0], s) != hipSuccess) st = DSK_EHIP;
        for (size_t i = 0; i < nc && st == DSK_OK; ++i) {
            for (int k = 0; k < kBurst && st == DSK_OK; ++k)
                st = launch_forward(in, in_is_f32, d, offs, shift, origin, vol, psum, pmax,
                                    width, cand[i], s);
            if (st == DSK_OK && hipEventRecord(ev[i + 1], s) != hipSuccess) st = DSK_EHIP;
        }
        if (st == DSK_OK && hipEventSynchronize(ev[nc]) != hipSuccess) st = DSK_EHIP;
        for (size_t i = 0; i < nc && st == DSK_OK && round > 0; ++i) {
            float ms = 0.0f;
            if (hipEventElapsedTime(&ms, ev[i], ev[i + 1]) != hipSuccess) st = DSK_EHIP;
            sum[i] += ms / kBurst;
        }
    }
    for (hipEvent_t e : ev)
        if (e) (void)hipEventDestroy(e);
    if (st != DSK_OK) return st;
    score->assign(nc, 0.0);
    for (size_t i = 0; i < nc; ++i) (*score)[i] = sum[i] / reps;
    return DSK_OK;
}

// The choice: among the candidates within kMargin of the fastest, the one
// paced slowest (unpaced first) -- a gain inside the timing noise is not
// worth a faster pace.
constexpr double kMargin = 1.005;

size_t choose(const std::vector<dsk_tune> &cand, const std::vector<double> &score) {
    size_t best = 0;
    for (size_t i = 1; i < cand.size(); ++i)
        if (score[i] < score[best]) best = i;
    size_t pick = best;
    for (size_t i = 0; i < cand.size(); ++i)
        if (score[i] <= score[best] * kMargin && cand[i].pace_gbs < cand[pick].pace_gbs) pick = i;
    return pick;
}

// The same shape paced at least kStepDown GB/s lower and at most kPaceCap
// (the highest such candidate pace), or cand.size() for an unpaced shape or
// when none qualifies.  The chosen pace is stepped down once more: a pace
// the device holds for every launch while tuning can fail in the runs that
// follow, on some devices for every launch, on others for some launches
// only (on the 512x2048 frame, 6000 GB/s: 0.827 ms in the tuner's runs and
// 0.90-0.97 ms after; 5900 GB/s: 0.839 ms on two devices, on a third a
// third of its launches at 0.93-0.98 ms; 5800 held in back-to-back runs
// on every device measured, 0.824 ms, but lost a fifth of the launches of
// longer timed runs to the cliff, 5700 none).  Falling off costs 10-15%,
// the step about 1.5%; the cap keeps the pick at or below the pace that
// held everywhere.
constexpr int kStepDown = 100;
// 5800 held the 512 x 512 x 2048 frame's long timed runs once each row's
// tiles start on 128-byte boundaries (at most 1 of 40 launches a few us
// behind; 6000 lost a third of them); the default stays at 5700, which
// holds on more frames
constexpr int kPaceCap = 5800;

size_t step_down(const std::vector<dsk_tune> &cand, const dsk_tune &t) {
    size_t pick = cand.size();
    if (t.pace_gbs <= 0) return pick;
    const int top = std::min(t.pace_gbs - kStepDown, kPaceCap);
    for (size_t i = 0; i < cand.size(); ++i) {
        const dsk_tune &c = cand[i];
        if (c.block != t.block || c.per_thread != t.per_thread || c.unroll != t.unroll ||
            c.nt_store != t.nt_store || c.wg_per_cu != t.wg_per_cu || c.pace_gbs <= 0 ||
            c.pace_gbs > top)
            continue;
        if (pick == cand.size() || c.pace_gbs > cand[pick].pace_gbs) pick = i;
    }
    return pick;
}

// Steady-state check of the front runners.  Short bursts of a shape that
// follow other shapes can hold a pace that a long run of that shape alone
// cannot (the run settles and then falls off the cliff), and a stream of
// stacks is a long run.  The candidates within kSteadyBand of the best
// burst score are each run kSteady times back to back, kSteadyRounds
// rounds in turn, and re-scored by their mean time per launch.
constexpr double kSteadyBand = 1.03;
constexpr int kSteady = 12, kSteadyRounds = 2, kSteadyMax = 4;

int steady_scores(const std::vector<dsk_tune> &cand, const std::vector<double> &score,
                  const void *in, int in_is_f32, dsk_dims d, const double *offs, double shift,
                  int64_t origin, float *vol, float *psum, float *pmax, int64_t width,
                  hipStream_t s, std::vector<dsk_tune> *fc, std::vector<double> *fs) {
    double lo = score[0];
    for (double v : score) lo = v < lo ? v : lo;
    std::vector<size_t> idx;
    for (size_t i = 0; i < cand.size(); ++i)
        if (score[i] <= lo * kSteadyBand) idx.push_back(i);
    std::sort(idx.begin(), idx.end(), [&](size_t x, size_t y) { return score[x] < score[y]; });
    if (idx.size() > (size_t)kSteadyMax) idx.resize(kSteadyMax);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int st = DSK_OK;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) st = DSK_EHIP;
    std::vector<double> sum(idx.size(), 0.0);
    for (int round = 0; round < kSteadyRounds && st == DSK_OK; ++round) {
        for (size_t j = 0; j < idx.size() && st == DSK_OK; ++j) {
            const dsk_tune &t = cand[idx[j]];
            // one untimed launch settles the shape after the previous one
            st = launch_forward(in, in_is_f32, d, offs, shift, origin, vol, psum, pmax, width, t, s);
            if (st == DSK_OK && hipEventRecord(e0, s) != hipSuccess) st = DSK_EHIP;
            for (int k = 0; k < kSteady && st == DSK_OK; ++k)
                st = launch_forward(in, in_is_f32, d, offs, shift, origin, vol, psum, pmax, width,
                                    t, s);
            if (st == DSK_OK && hipEventRecord(e1, s) != hipSuccess) st = DSK_EHIP;
            if (st == DSK_OK && hipEventSynchronize(e1) != hipSuccess) st = DSK_EHIP;
            float ms = 0.0f;
            if (st == DSK_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) st = DSK_EHIP;
            sum[j] += ms / kSteady;
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (st != DSK_OK) return st;
    fc->clear();
    fs->clear();
    for (size_t j = 0; j < idx.size(); ++j) {
        fc->push_back(cand[idx[j]]);
        fs->push_back(sum[j] / kSteadyRounds);
    }
    return DSK_OK;
}

}  // namespace

extern "C" int dsk_deskew_autotune(const void *in, int in_is_f32, dsk_dims d,
                                   const double *offsets_dev, double shift_px, int64_t origin,
                                   float *vol, float *psum, float *pmax, int64_t out_width,
                                   int reps, hipStream_t stream, dsk_tune *tune, double *ms) {
    if (!tune || out_width <= 0 || reps < 3 || reps > 64) return DSK_EINVAL;
    if (!in || !dims_ok(d) || (!vol && !psum && !pmax)) return DSK_EINVAL;
    if (!offsets_dev && !std::isfinite(shift_px)) return DSK_EINVAL;
    auto key_of = [&](const char *tiling) {
        return fwd_key(tiling, in_is_f32 ? 1 : 0, d, out_width, offsets_dev != nullptr, vol, psum,
                       pmax);
    };
    const std::string key = key_of(tiling_name(in, in_is_f32 ? 1 : 0, d, vol, out_width));
    auto remembered = [&](const std::string &k) {
        std::lock_guard<std::mutex> lk(g_memo_mu);
        auto it = g_memo.find(k);
        if (it == g_memo.end()) return false;
        *tune = it->second.first;
        if (ms) *ms = it->second.second;
        return true;
    };
    if (remembered(key)) return DSK_OK;
    // a stream under capture cannot be timed: there the shape that another
    // tiling of the frame was given serves
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
        (void)hipGetLastError();   // not the next launch's error
        cap = hipStreamCaptureStatusNone;
    }
    if (cap != hipStreamCaptureStatusNone)
        for (const char *tiling : {"lines", "aligned", "general", "scalar"})
            if (remembered(key_of(tiling))) return DSK_OK;
    dsk_tune best{};
    double best_ms = 0.0;
    if (!tune_cache_lookup(key, &best, &best_ms, nullptr)) {
        const std::vector<dsk_tune> cand = fwd_candidates(vol != nullptr);
        std::vector<double> score;
        const int st = time_candidates(cand, reps, in, in_is_f32 ? 1 : 0, d, offsets_dev,
                                       shift_px, origin, vol, psum, pmax, out_width, stream,
                                       &score);
        if (st != DSK_OK) return st;
        std::vector<dsk_tune> front;
        std::vector<double> fscore;
        const int st2 = steady_scores(cand, score, in, in_is_f32 ? 1 : 0, d, offsets_dev,
                                      shift_px, origin, vol, psum, pmax, out_width, stream,
                                      &front, &fscore);
        if (st2 != DSK_OK) return st2;
        const size_t bi = choose(front, fscore);
        best = front[bi];
        best_ms = fscore[bi];
        // a pace stays clear of its cliff only where wavefronts write
        const size_t di = vol ? step_down(cand, best) : cand.size();
        if (di < cand.size()) {
            best = cand[di];
            best_ms = score[di];
        }
        tune_cache_store(key, best, best_ms, 0);
    }
    {
        std::lock_guard<std::mutex> lk(g_memo_mu);
        g_memo[key] = {best, best_ms};
    }
    *tune = best;
    if (ms) *ms = best_ms;
    return DSK_OK;
}
