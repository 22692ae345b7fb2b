// Autotuner: times the launch shapes of a kernel on the caller's buffers and
// remembers the fastest per (GPU architecture, kernel, lattice, precision,
// batch).  Choices live
// in a process-wide table; when HISQ_TUNE_CACHE names a file they are also
// loaded from and saved to it (a flat JSON object of integers).
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

#include "dslash_core.hpp"

namespace hisq {

static std::mutex g_mu;
static std::map<std::string, int> g_table;
static bool g_loaded = false;
// entries of kind "dslash_form", -1 until the file has been read: the small-lattice Dslash, a few microseconds in
// all, looks for its own entry only where there is one
static std::atomic<int> g_forms{ -1 };

// Architecture of the current device (e.g. "gfx950"), part of every key, so
// that a cache file written on one GPU model is not applied to another.
static std::string device_arch()
{
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return "unknown";
    std::string a = prop.gcnArchName;
    const size_t colon = a.find(':');  // drop feature suffixes such as ":sramecc+:xnack-"
    return colon == std::string::npos ? a : a.substr(0, colon);
}

static std::string key_of(const char *kind, const Geom &g, int prec, int n)
{
    static const std::string arch = device_arch();
    char buf[192];
    std::snprintf(buf, sizeof buf, "%s:%s:p%d:n%d:%dx%dx%dx%d", arch.c_str(), kind, prec, n, g.L[0], g.L[1], g.L[2],
                  g.L[3]);
    return buf;
}

static void load_locked()
{
    if (g_loaded) return;
    g_loaded = true;
    const char *path = std::getenv("HISQ_TUNE_CACHE");
    if (!path) return;
    FILE *f = std::fopen(path, "r");
    if (!f) return;
    // entries look like "key": value
    char line[512];
    while (std::fgets(line, sizeof line, f)) {
        char *q1 = std::strchr(line, '"');
        if (!q1) continue;
        char *q2 = std::strchr(q1 + 1, '"');
        if (!q2) continue;
        char *colon = std::strchr(q2, ':');
        if (!colon) continue;
        g_table[std::string(q1 + 1, q2)] = std::atoi(colon + 1);
    }
    std::fclose(f);
}

static void save_locked()
{
    const char *path = std::getenv("HISQ_TUNE_CACHE");
    if (!path) return;
    std::string tmp = std::string(path) + ".tmp";
    FILE *f = std::fopen(tmp.c_str(), "w");
    if (!f) return;
    std::fprintf(f, "{\n");
    size_t i = 0;
    for (auto &kv : g_table) std::fprintf(f, "  \"%s\": %d%s\n", kv.first.c_str(), kv.second, ++i < g_table.size() ? "," : "");
    std::fprintf(f, "}\n");
    std::fclose(f);
    std::rename(tmp.c_str(), path);
}

int tuned_choice(const char *kind, const Geom &g, int prec, int n, int fallback)
{
    std::lock_guard<std::mutex> lk(g_mu);
    load_locked();
    auto it = g_table.find(key_of(kind, g, prec, n));
    return it == g_table.end() ? fallback : it->second;
}

static void store_locked(const std::string &key, int v)
{
    g_table[key] = v;
    save_locked();
}

void set_tuned_choice(const char *kind, const Geom &g, int prec, int n, int v)
{
    std::lock_guard<std::mutex> lk(g_mu);
    load_locked();
    store_locked(key_of(kind, g, prec, n), v);
}

static void count_forms_locked()
{
    int n = 0;
    for (auto &kv : g_table) n += kv.first.find(":dslash_form:") != std::string::npos;
    g_forms.store(n);
}

DslashForm dslash_form(const Geom &g, int prec)
{
    if (g_forms.load() == 0) return DslashForm::rule;
    std::lock_guard<std::mutex> lk(g_mu);
    load_locked();
    if (g_forms.load() < 0) count_forms_locked();
    auto it = g_table.find(key_of("dslash_form", g, prec, 1));
    if (it == g_table.end()) return DslashForm::rule;
    return it->second == (int)DslashForm::set ? DslashForm::set
           : it->second == (int)DslashForm::tuned ? DslashForm::tuned
                                                  : DslashForm::rule;
}

void set_dslash_choice(const Geom &g, int prec, int shape, DslashForm form)
{
    std::lock_guard<std::mutex> lk(g_mu);
    load_locked();
    const std::string key = key_of("dslash_form", g, prec, 1);
    if (form == DslashForm::rule) g_table.erase(key);
    else g_table[key] = (int)form;
    store_locked(key_of("dslash", g, prec, 1), shape);
    count_forms_locked();
}

// Untuned default.  Shape 2 has workgroups of one tile; 3 and 4 have every term
// and four terms in flight, 10 two, 0 one, all with workgroups of four tiles,
// which leave a round of the 1024 tiles that the CUs take nearly empty just
// beyond each multiple of 1024.  Microseconds (three states in turn, so that
// nothing is left in a cache from the call before), shapes as headed:
//   tiles         1337       1625       2048       2808       3072       3822       4608       5120       5440       7168       13122
//   F64   10, 2   44.2 36.6  47.8 42.7  52.6 51.1  74.4 73.1  79.2 80.5  101  98    122  119   130  134   139  139   180  185   341  353
//   F32   3, 2    21.5 18.0  23.4 20.9  26.7 26.0  37.8 36.7  39.8 40.6  49.3 49.6  59.8 59.0  65.3 67.0  70.4 70.5  89.7 93.2  171  182
//   F32C  3, 2    19.7 17.3  21.1 19.0  23.5 21.7  33.1 30.9  34.0 33.9  43.7 43.4  53.1 51.7  54.9 56.5  62.0 61.5  77.4 81.0  148  154
//   I16S  4, 2                                     25.2 21.9  26.8 23.7  31.3 29.6  37.7 37.5  39.4 40.7  50.3 44.3  58.3 56.7  101  109
//   I16SC 4, 2                                     22.1 20.5  22.6 21.9  28.5 27.5  35.3 35.0  39.0 38.2  40.9 41.4  50.7 52.1  95.5 99.8
// (F16S within 6 % of I16S.)  Shape 0 is slower than the one chosen but for
// 1-2 % at single sizes (F32C 3021: 33.7 against 34.2).  Why four terms in
// flight lose to one above 5120 tiles with 16-bit links, 45.3 against 50.3 at
// 5440, was not found.  F64C takes two terms at every size (2: 1.5 times as slow).
static int default_dslash_shape(const Geom &g, int prec)
{
    const int n = g.ntiles;
    switch (prec) {
    case HISQ_F64: return n > 1024 && n <= 2816 ? 2 : 10;
    case HISQ_F64C: return 10;
    case HISQ_F32: return n <= 2816 ? 2 : 3;
    case HISQ_F32C: return n <= 4608 ? 2 : 3;
    case HISQ_I16SC: return n <= 5120 ? 2 : 4;
    default: return n <= 4608 || (n > 5120 && n <= 7168) ? 2 : 4;
    }
}

int tuned_dslash_shape(const Geom &g, int prec)
{
    const int def = default_dslash_shape(g, prec);
    int v = tuned_choice("dslash", g, prec, 1, def);
    return (v >= 0 && v < N_DSLASH_SHAPES) ? v : def;
}

// Times `launch()` with HIP events on stream s: 2 warm-up launches, then
// `reps` launches; returns microseconds per launch or a negative value.
template <class F>
static double time_launches(F launch, int reps, hipStream_t s)
{
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return -1;
    if (hipEventCreate(&b) != hipSuccess) { hipEventDestroy(a); return -1; }
    double us = -1;
    bool ok = true;
    for (int i = 0; i < 2 && ok; ++i) ok = launch() == hipSuccess;
    if (ok && hipEventRecord(a, s) == hipSuccess) {
        for (int i = 0; i < reps && ok; ++i) ok = launch() == hipSuccess;
        if (ok && hipEventRecord(b, s) == hipSuccess && hipEventSynchronize(b) == hipSuccess) {
            float ms = 0;
            if (hipEventElapsedTime(&ms, a, b) == hipSuccess) us = 1e3 * ms / reps;
        }
    }
    hipEventDestroy(a);
    hipEventDestroy(b);
    return us;
}

template <class P>
static int tune_dslash_impl(const Geom &g, const void *fat, const void *lng, const void *src, void *dst, int reps,
                            int *best, double *us_out, hipStream_t s)
{
    double best_us = 1e300, plain_us = 1e300;
    int best_i = 0, plain_i = -1;
    for (int i = 0; i < N_DSLASH_SHAPES; ++i) {
        double us = time_launches([&]() { return launch_dslash_shape<P>(i, g, fat, lng, src, dst, 1, s); }, reps, s);
        if (us_out) us_out[i] = us;
        if (us < 0) return fail(HISQ_EHIP, "autotune: timing failed");
        if (us < best_us) { best_us = us; best_i = i; }
        if (DSLASH_SHAPES[i].order == 0 && us < plain_us) { plain_us = us; plain_i = i; }
    }
    // FP64: the plain CG's fused kernels take the tile order of this choice, and inside the solve every blocked
    // order is slower than the plain one (32^4, m = 0.01: 1.80-1.86 s against 1.76 s per solve, the same in
    // three alternating rounds), while the bare Dslash times the orders within 2 % of each other either way.
    // A blocked shape is kept only when it beats the best plain-order shape by more than 3 %.
    if (P::prec == HISQ_F64 && plain_i >= 0 && DSLASH_SHAPES[best_i].order != 0 && best_us > 0.97 * plain_us) {
        best_i = plain_i;
        best_us = plain_us;
    }
    DslashForm form = DslashForm::rule;
    if (split_tiles(g, P::prec)) {
        const double us = time_launches([&]() { return launch_dslash_tiles<P>(g, fat, lng, src, dst, 1, s); }, reps, s);
        if (us < 0) return fail(HISQ_EHIP, "autotune: timing failed");
        if (best_us < us) form = DslashForm::tuned;
    }
    set_dslash_choice(g, P::prec, best_i, form);
    if (best) *best = best_i;
    return HISQ_OK;
}

}  // namespace hisq

using namespace hisq;

extern "C" int hisq_tune_dslash(const void *fat, const void *lng, const void *src, void *dst, const int dims[4],
                                int prec, int reps, int *best_shape, double *us_per_shape, void *stream)
{
    Geom g;
    int rc = make_geom(dims, g);
    if (rc) return rc;
    if (!fat || !lng || !src || !dst) return fail(HISQ_EINVAL, "hisq_tune_dslash: NULL pointer");
    if (!aligned16({fat, lng, src, dst}))
        return fail(HISQ_EINVAL, "hisq_tune_dslash: device pointers must be 16-byte aligned");
    if (src == dst) return fail(HISQ_EALIAS, "hisq_tune_dslash: src and dst alias");
    if (reps <= 0) reps = 20;
    hipStream_t s = (hipStream_t)stream;
    switch (prec) {
    case HISQ_F64: return tune_dslash_impl<PF64>(g, fat, lng, src, dst, reps, best_shape, us_per_shape, s);
    case HISQ_F32: return tune_dslash_impl<PF32>(g, fat, lng, src, dst, reps, best_shape, us_per_shape, s);
    case HISQ_F16S: return tune_dslash_impl<PF16S>(g, fat, lng, src, dst, reps, best_shape, us_per_shape, s);
    case HISQ_I16S: return tune_dslash_impl<PI16S>(g, fat, lng, src, dst, reps, best_shape, us_per_shape, s);
    case HISQ_F64C: return tune_dslash_impl<PF64C>(g, fat, lng, src, dst, reps, best_shape, us_per_shape, s);
    case HISQ_F32C: return tune_dslash_impl<PF32C>(g, fat, lng, src, dst, reps, best_shape, us_per_shape, s);
    case HISQ_I16SC: return tune_dslash_impl<PI16SC>(g, fat, lng, src, dst, reps, best_shape, us_per_shape, s);
    default: return fail(HISQ_EINVAL, "hisq_tune_dslash: unknown precision");
    }
}

extern "C" int hisq_dslash_shape(const int dims[4], int prec, int shape)
{
    Geom g;
    int rc = make_geom(dims, g);
    if (rc) return rc;
    if (prec < HISQ_F64 || prec > HISQ_I16SC) return fail(HISQ_EINVAL, "hisq_dslash_shape: unknown precision");
    if (shape == -2) return N_DSLASH_SHAPES;
    if (shape < -2 || shape >= N_DSLASH_SHAPES) return fail(HISQ_EINVAL, "hisq_dslash_shape: no such shape");
    if (shape >= 0) set_dslash_choice(g, prec, shape, DslashForm::set);
    return tuned_dslash_shape(g, prec);
}
