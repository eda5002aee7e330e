// Tile planning (paper section 3, step 2: choose the number of blocks and
// batches from the input length, the device memory and the precision the FFT
// needs).  Here a job is cut into key chunks (the paper's blocks/batches, Eq.
// 4-5) and, when the output is long, output windows; every tile of a plan uses
// one FFT length class.
#include "planner.hpp"

#include "pa.h"

#include <dlfcn.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

namespace pa {

namespace {
double g_kappa = 1.0;

int prec_index(int prec) { return prec == PREC_FP32 ? 0 : prec == PREC_FP64 ? 1 : 2; }

uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }
uint64_t round_up64(uint64_t a) { return (a + 63) & ~uint64_t(63); }
}  // namespace

// Smallest class; PA_MIN_LOG2_LEN (12..24) raises it (with PA_MAX_LOG2_LEN it
// pins the class, e.g. to exercise one kernel family).
int min_logL(int) {
    int lo = 12;
    if (const char* e = getenv("PA_MIN_LOG2_LEN")) {
        int v = atoi(e);
        if (v > lo && v <= 24) lo = v;
    }
    return lo;
}

// Largest class; PA_MAX_LOG2_LEN (12..24) lowers it, e.g. to force key
// chunking and output windows on small inputs.
int max_logL(int prec) {
    (void)prec;
    int cap = 24;
    if (const char* e = getenv("PA_MAX_LOG2_LEN")) {
        int v = atoi(e);
        if (v >= 12 && v < cap) cap = v;
    }
    return cap;
}

int ceil_log2(uint64_t L) {
    int k = 0;
    while ((1ull << k) < L) ++k;
    return k;
}

bool class_geometry(int prec, int cls, ClassGeom* g) {
    if (!class_id_valid(cls)) return false;
    const uint64_t L = class_len(cls);
    g->prec = prec;
    g->cls = cls;
    g->L = L;
    if (cls >= 32) {   // mixed-radix class L = P 2^k (FP32 and FP64 only)
        if (prec != PREC_FP32 && prec != PREC_FP64) return false;
        // power-of-two rows, 4096 points from 2^20 on;
        // the columns carry the factor P (radix-P stage, 4P points per thread)
        const int P = smooth_P(cls), k = smooth_k(cls);
        // rows of the three-pass geometry of 2^k (its short lengths run as
        // one-kernel tiles, whose row is the whole length)
        const int n2log = std::max(k - 13, std::min(prec == PREC_FP64 ? 11 : 10, k / 2));
        g->n1 = L >= (1ull << 20) ? 4096 : 1 << (k - n2log);
        g->n2 = (int)(L / (uint64_t)g->n1);
        return true;
    }
    const int logL = cls;
    if (prec == PREC_NTT) {
        const int n2log = std::min(11, logL / 2);
        g->n2 = 1 << n2log;
        g->n1 = 1 << (logL - n2log);
        return true;
    }
    if (logL >= 15) {  // wave-level classes
        const bool f32 = prec != PREC_FP64;
        // rows of 4096: the row pass then has two workgroups per CU in FP32, and
        // registers to spare in FP64.  FP32 2^24 keeps 8192 (its wave-level column
        // passes take at most 2048 points), FP64 2^24 takes workgroup-wide ones
        // (columns of 4096).  Below 2^20 a row is one wave's 512 points: many small
        // workgroups, no barriers
        const int n1log = logL < 20 ? 9 : f32 && logL == 24 ? 13 : 12;
        g->n1 = 1 << n1log;
        g->n2 = 1 << (logL - n1log);
        return true;
    }
    if (logL <= 13) {   // one-kernel tiles: the whole length in one workgroup
        g->n1 = 1 << logL;
        g->n2 = 1;
        return true;
    }
    int n2cap = prec == PREC_FP64 ? 11 : 10;
    int n2log = std::max(logL - 13, std::min(n2cap, logL / 2));
    g->n2 = 1 << n2log;
    g->n1 = 1 << (logL - n2log);
    return true;
}

static uint64_t env_u64(const char* name) {
    const char* e = getenv(name);
    return e ? strtoull(e, nullptr, 10) : 0;
}

int class_ids(int prec, int* ids, int cap_logL) {
    const uint64_t lo = 1ull << min_logL(prec), hi = 1ull << std::min(max_logL(prec), cap_logL);
    const uint64_t only = env_u64("PA_ONLY_LEN");
    const bool pow2 = env_u64("PA_POW2_ONLY") != 0;
    int count = 0;
    for (int id = kMinClassId; id <= kMaxClassId; ++id) {
        ClassGeom g;
        if (!class_geometry(prec, id, &g)) continue;
        if (g.L < lo || g.L > hi || (only && g.L != only) || (pow2 && id >= 32)) continue;
        ids[count++] = id;
    }
    std::sort(ids, ids + count, [](int a, int b) { return class_len(a) < class_len(b); });
    return count;
}

uint64_t class_filter_key() {
    return (uint64_t)min_logL(0) | ((uint64_t)max_logL(0) << 8) | ((env_u64("PA_POW2_ONLY") != 0 ? 1ull : 0ull) << 16) |
           (env_u64("PA_ONLY_LEN") << 20);
}

void set_error_kappa(double kappa) { g_kappa = kappa; }
double error_kappa() { return g_kappa; }

static double unit_roundoff(int prec) {
    return prec == PREC_FP32 ? std::ldexp(1.0, -24) : prec == PREC_FP64 ? std::ldexp(1.0, -53) : 0.0;
}

// Low-frequency term.  The key chunk is a 0/1 sequence on [0, Bi) padded with
// zeros, so its mean (1/2 per bit) gives it the spectrum of a box,
// |X_k| ~ D_k / 2 with the Dirichlet kernel D_k = |sin(pi Bi k / L) / sin(pi k / L)|,
// which reaches L / (2 pi k) at the lowest frequencies.  With the two sequences
// packed in one complex transform, an absolute error of about u |X_k| leaks
// into the separated W_k, and the product picks up about u |X_k|^2 there.  The
// inverse transform spreads these few bins over every output as a smooth
// wave of rms u sqrt(sum_k 2 (D_k / 2)^4) / L; the sum converges like k^-4 and
// 16 terms hold it (the rest is below 10^-4 of it).  The maximum over a tile
// is about 2-4 times the rms.
static double box_leak_rms(int prec, uint64_t Lc, uint64_t Bi) {
    const double L = (double)Lc;
    const uint64_t twoL = 2 * Lc;
    // sin(pi Bi k / L) and sin(pi k / L) for k = 1, 2, ... by rotation
    const double a = M_PI * (double)(Bi % twoL) / L, b = M_PI / L;
    const double sa = std::sin(a), ca = std::cos(a), sb = std::sin(b), cb = std::cos(b);
    double sak = sa, cak = ca, sbk = sb, cbk = cb, s4 = 0;
    for (uint64_t k = 1; k <= 16 && (double)k < L / 2; ++k) {
        const double d = std::fabs(sak / sbk) / 2;
        s4 += 2 * d * d * d * d;
        const double s1 = sak * ca + cak * sa, c1 = cak * ca - sak * sa;
        const double s2 = sbk * cb + cbk * sb, c2 = cbk * cb - sbk * sb;
        sak = s1, cak = c1, sbk = s2, cbk = c2;
    }
    return unit_roundoff(prec) * std::sqrt(s4) / L;
}

// The noise term: the packed transform carries the seed's norm sqrt(L) beside
// the chunk's sqrt(Bi), so even a one-bit chunk sees u sqrt(L log L).
static double noise_error(int prec, uint64_t Lc, uint64_t Bi) {
    const double L = (double)Lc;
    return 6.0 * g_kappa * unit_roundoff(prec) * std::sqrt(std::log2(L) * ((double)Bi + L));
}
static double leak_error(int prec, uint64_t L, uint64_t Bi) { return 5.0 * box_leak_rms(prec, L, Bi); }

double error_bound(int prec, uint64_t Lc, uint64_t Bi) {
    return prec == PREC_NTT ? 0.0 : noise_error(prec, Lc, Bi) + leak_error(prec, Lc, Bi);
}

// The same for the sum of the products of c chunks: the noise is independent from
// chunk to chunk, but the low-frequency error is not.  Every chunk has about the
// same box spectrum, so its roots' rounding leaves about the same wave, and the
// waves add in full: measured maxima grow as a sqrt(c) + b c, with b 0.22 to 0.35
// of the low-frequency term from 2^15 to 2^23.
static double group_error(int prec, uint64_t L, uint64_t Bi, uint64_t c) {
    return prec == PREC_NTT ? 0.0 : noise_error(prec, L, Bi) * std::sqrt((double)c) + leak_error(prec, L, Bi) * (double)c;
}

// Worst-case bound of Percival's form (Math. Comp. 72, 2003): an FFT
// convolution of a and b whose 3k radix-2 levels each add a relative error of
// at most (1+u) for the additions, (1+u sqrt5) for a complex product and
// (1+beta) for the twiddle (beta = 2u: table roots rounded once, four-step
// roots an FP64 product rounded once) has max error at most
// ||a|| ||b|| ((1+u)^3k (1+u sqrt5)^(3k+1) (1+beta)^3k - 1).  Read for this
// pipeline: radix-4/8/16 stages count as their radix-2 levels, a radix-3/5/7
// stage as ceil(log2 P) + 1 levels (k = ceil(log2 L) + 1 for a mixed-radix
// length), the spectrum separation and the half-length Hermitian inverse add
// two levels (3k+2), and the two sequences share one transform, so
// ||a|| ||b|| is replaced by (||x|| + ||w||)^2 with ||x|| <= sqrt(Bi) (0/1
// chunk) and ||w|| = sqrt(Bi+Bo-1) (+-1 seed slice).  It holds for every
// input bit pattern.  A group of c chunks adds c products of these norms before
// the inverse: c - 1 additions, each with a relative error of at most u.
double rigorous_bound(int prec, uint64_t L, uint64_t Bi, uint64_t Bo, uint64_t c) {
    if (prec == PREC_NTT || prec == PREC_DIRECT) return 0.0;
    const int levels = ceil_log2(L) + ((L & (L - 1)) ? 1 : 0);
    const double u = unit_roundoff(prec), lv = 3.0 * levels + 2.0, beta = 2.0 * u;
    const double g = (lv + (double)(c - 1)) * std::log1p(u) + (lv + 1) * std::log1p(u * std::sqrt(5.0)) + lv * std::log1p(beta);
    const double norms = std::sqrt((double)Bi) + std::sqrt((double)(Bi + Bo - 1));
    return (double)c * norms * norms * std::expm1(g);
}

CostModel::CostModel() {
    launch_s = 12e-6;
    // 32 bit products on the matrix cores at 2.9e15 per second (measured on
    // MI355X at n = 12,345,679, m = 20,000)
    direct_s = 1.1e-14;
    direct_launch_s = 12e-6;
    for (int p = 0; p < 3; ++p)
        for (int id = 0; id < 64; ++id) {
            const uint64_t Lc = class_len(id);
            chunk_s[p][id] = alone_s[p][id] = run_s[p][id] = few_s[p][id] = 0;
            if (Lc == 0) {
                tile_s[p][id] = 1.0;
                continue;
            }
            const double L = (double)Lc, lg = std::log2(L);
            // bytes moved by the three passes and a VALU estimate
            const double bytes = (p == 1 ? 48.0 : 24.0) * L;
            const double instr = L * (5.0 * lg + 40.0) * (p == 2 ? 3.0 : 1.0);
            const double t_mem = bytes / 5.0e12, t_alu = instr / 20.0e12;
            // the long mixed-radix classes run workgroup-wide Stockham column
            // passes, slower per point than the wave-level ones (measured on
            // MI355X: about 1.8x in FP32 and 1.4x in FP64)
            const double generic = (id >= 32 && Lc >= (1ull << 20)) ? (p == 1 ? 1.4 : 1.8) : 1.0;
            tile_s[p][id] = generic * std::max(t_mem, t_alu) + 1e-6;
            first_s[p][id] = launch_s;
        }
}

double CostModel::chunk(int prec, int cls) const {
    const double c = chunk_s[prec_index(prec)][cls];
    return c > 0 ? c : 0.7 * tile(prec, cls);
}
void CostModel::set_chunk(int prec, int cls, double s) { chunk_s[prec_index(prec)][cls] = s; }
double CostModel::tile_of(int prec, int cls, uint64_t groups) const {
    return std::max(tile(prec, cls), few_s[prec_index(prec)][cls] * 12.0 / (double)std::max<uint64_t>(groups, 12));
}
double CostModel::alone(int prec, int cls) const {
    const double a = alone_s[prec_index(prec)][cls];
    return a > 0 ? a : chunk(prec, cls);
}
double CostModel::run(int prec, int cls) const {
    const double r = run_s[prec_index(prec)][cls];
    return r > 0 ? r : alone(prec, cls);
}
double CostModel::chunk_of(int prec, int cls, uint64_t groups, uint64_t chunks, uint64_t tiles) const {
    const double cached = 240e6, bytes = (double)tiles * (double)class_len(cls) * (prec == PREC_FP64 ? 16 : 8);
    const double base = bytes > cached ? chunk(prec, cls) : least_chunk(prec, cls);
    double a = alone(prec, cls);
    if (chunks > 8) a = (7 * a + (double)(chunks - 8) * run(prec, cls)) / (double)(chunks - 1);
    return base + std::max(a - base, 0.0) / (double)groups;
}
void CostModel::set_run(int prec, int cls, double s) { run_s[prec_index(prec)][cls] = s; }
void CostModel::set_few(int prec, int cls, double s) { few_s[prec_index(prec)][cls] = s; }
void CostModel::set_alone(int prec, int cls, double s) { alone_s[prec_index(prec)][cls] = s; }
double CostModel::tile(int prec, int cls) const { return tile_s[prec_index(prec)][cls]; }
double CostModel::first(int prec, int cls) const { return first_s[prec_index(prec)][cls]; }
void CostModel::set(int prec, int cls, double s) { tile_s[prec_index(prec)][cls] = s; }
void CostModel::set_first(int prec, int cls, double s) { first_s[prec_index(prec)][cls] = s; }

static const char* prec_key(int prec) { return prec == PREC_FP32 ? "fp32" : prec == PREC_FP64 ? "fp64" : "ntt"; }

// Minimal reader of the table pa_tune writes:
//   {"launch": s, "direct": s, "direct_launch": s,
//    "fp32": {"<L>": [tile_s, first_s], ...}, "fp64": {...}, "fp32_few": {"<L>": few_s, ...},
//    "fp32_chunk": {"<L>": chunk_s, ...}, "fp32_chunk_alone": {"<L>": alone_s, ...},
//    "fp32_chunk_run": {"<L>": run_s, ...}}
// (a plain number instead of the pair sets tile_s only).
int load_tune_table(CostModel& cm, const char* path) {
    FILE* f = fopen(path, "r");
    if (!f) return -1;
    std::string text;
    char buf[4096];
    size_t got;
    while ((got = fread(buf, 1, sizeof buf, f)) > 0) text.append(buf, got);
    fclose(f);
    int loaded = 0;
    const size_t la = text.find("\"launch\":");
    if (la != std::string::npos) {
        const double v = strtod(text.c_str() + la + 9, nullptr);
        if (v >= 0 && v < 1.0) cm.launch_s = v;
    }
    const size_t di = text.find("\"direct\":");
    if (di != std::string::npos) {
        const double v = strtod(text.c_str() + di + 9, nullptr);
        if (v > 0 && v < 1e-6) {
            cm.direct_s = v;
            ++loaded;
        }
    }
    const size_t dl = text.find("\"direct_launch\":");
    if (dl != std::string::npos) {
        const double v = strtod(text.c_str() + dl + 16, nullptr);
        if (v >= 0 && v < 1e-2) cm.direct_launch_s = v;
    }
    for (int prec : {PREC_FP32, PREC_FP64, PREC_NTT}) {
        // "<prec>_few", "<prec>_chunk", "<prec>_chunk_alone", "<prec>_chunk_run":
        // {"<L>": seconds, ...} (absent in older tables)
        struct Section {
            const char* kind;
            void (CostModel::*set)(int, int, double);
            bool found;
        } sections[] = {{"_few", &CostModel::set_few, false},
                        {"_chunk", &CostModel::set_chunk, false},
                        {"_chunk_alone", &CostModel::set_alone, false},
                        {"_chunk_run", &CostModel::set_run, false}};
        for (Section& sec : sections) {
            const size_t ca = text.find(std::string("\"") + prec_key(prec) + sec.kind + "\"");
            if (ca == std::string::npos) continue;
            sec.found = true;
            const size_t o = text.find('{', ca), e = text.find('}', ca);
            if (o == std::string::npos || e == std::string::npos || e < o) return -1;
            const std::string body = text.substr(o + 1, e - o - 1);
            for (int k = kMinClassId; k <= kMaxClassId; ++k) {
                ClassGeom g;
                if (!class_geometry(prec, k, &g)) continue;
                const std::string key = "\"" + std::to_string(g.L) + "\":";
                const size_t p = body.find(key);
                if (p == std::string::npos) continue;
                const double v = strtod(body.c_str() + p + key.size(), nullptr);
                if (v > 0 && v < 10.0) (cm.*sec.set)(prec, k, v);
            }
        }
        const std::string tag = std::string("\"") + prec_key(prec) + "\"";
        const size_t at = text.find(tag);   // (the closing quote keeps "fp32_chunk" out)
        if (at == std::string::npos) continue;
        const size_t open = text.find('{', at), close = text.find('}', at);
        if (open == std::string::npos || close == std::string::npos || close < open) return -1;
        const std::string body = text.substr(open + 1, close - open - 1);
        for (int k = kMinClassId; k <= kMaxClassId; ++k) {
            ClassGeom g;
            if (!class_geometry(prec, k, &g)) continue;
            const std::string key = "\"" + std::to_string(g.L) + "\":";
            const size_t p = body.find(key);
            if (p == std::string::npos) continue;
            const char* q = body.c_str() + p + key.size();
            while (*q == ' ') ++q;
            const bool pair = *q == '[';
            char* end = nullptr;
            const double v = strtod(pair ? q + 1 : q, &end);
            if (!(v > 0 && v < 10.0)) continue;
            cm.set(prec, k, v);
            ++loaded;
            // an older table has one cost for all launches: not beside other tables' ends
            for (const Section& sec : sections)
                if (!sec.found) (cm.*sec.set)(prec, k, 0);
            if (pair && end) {
                while (*end == ' ' || *end == ',') ++end;
                const double w = strtod(end, nullptr);
                if (w >= 0 && w < 1.0) cm.set_first(prec, k, w);
            }
        }
    }
    return loaded;
}

const CostModel& default_cost_model() {
    static const CostModel cm = [] {
        CostModel m;
        const char* e = getenv("PA_TUNE_DEFAULT");
        if (e && e[0] == '0') return m;
        Dl_info info;
        if (dladdr((const void*)&load_tune_table, &info) && info.dli_fname) {
            std::string dir(info.dli_fname);
            const size_t slash = dir.rfind('/');
            dir = slash == std::string::npos ? std::string(".") : dir.substr(0, slash);
            (void)load_tune_table(m, (dir + "/tune_mi355x.json").c_str());
        }
        return m;
    }();
    return cm;
}

double direct_cost(uint64_t n, uint64_t m, const CostModel& cm) {
    const double outs = (double)(ceil_div(m, 256) * 256), words = (double)(ceil_div(ceil_div(n, 32), 4) * 4);
    return 1.1 * (cm.direct_launch_s + cm.direct_s * outs * words);
}

bool choose_direct(uint32_t flags, uint64_t n, uint64_t m, const CostModel& cm, const TilePlan& fft) {
    const uint32_t p = flags & PA_PREC_MASK;
    if (p == PA_PREC_DIRECT) return true;
    return p == PA_PREC_AUTO && direct_cost(n, m, cm) < fft.cost;
}

bool choose_direct_shared(uint32_t flags, uint64_t n, uint64_t m, const CostModel& cm, const TilePlan& fft, uint64_t jobs) {
    const uint32_t p = flags & PA_PREC_MASK;
    if (p == PA_PREC_DIRECT) return true;
    if (p != PA_PREC_AUTO) return false;
    TilePlan beside;
    if (!plan_at_class(n, m, fft.prec, fft.cls, cm, &beside, 0, jobs)) beside = fft;
    return kDirectShared * (direct_cost(n, m, cm) - 1.1 * cm.direct_launch_s) < beside.cost - cm.first(fft.prec, fft.cls);
}

// Classes whose row pass sums the products of several chunks: those with
// wave-level rows (powers of two from 2^15, mixed-radix lengths from 2^20 on).
static bool class_sums(int prec, int cls) {
    return prec != PREC_NTT && (cls < 32 ? cls >= 15 : class_len(cls) >= (1ull << 20));
}

// Classes with shared spectra (ClassKernels::shared1).
static bool class_shared(int prec, int cls) { return prec == PREC_FP32 && cls >= 21 && cls <= 23; }

// Modeled error of one product of shared spectra: the noise term of error_bound
// (the sequences of a pack are of equal size, so no box leaks into a seed).
static double shared_error(int prec, uint64_t L, uint64_t Bi) {
    return noise_error(prec, L, Bi);
}

// Chunks of one group: at most kMaxGroup, in equal groups, and for FP32 no more
// than keep the modeled error of the sum within the limit of groups.
constexpr uint64_t kMaxGroup = 64;
// The largest c with noise sqrt(c) + leak c within the limit.
static uint64_t most_chunks(double noise, double leak) {
    const double r = 2 * kGroupErrorLimit / (noise + std::sqrt(noise * noise + 4 * leak * kGroupErrorLimit));
    return std::min<uint64_t>(kMaxGroup, (uint64_t)std::max(1.0, std::floor(r * r)));
}
// Chunks that make one group whatever their length: the noise at Bi = L, and each
// |X_k| at most L / (2 pi k) (1% for the sines and the rounding).  kMaxGroup up to
// 2^17, so that the scan of a class's windows seldom asks the model.
static uint64_t any_chunks(int prec, uint64_t L) {
    if (prec != PREC_FP32) return kMaxGroup;
    return most_chunks(1.01 * noise_error(prec, L, L), 1.01 * 5.0 * unit_roundoff(prec) * (double)L * std::sqrt(2 * 1.0824) / (4 * M_PI * M_PI));
}
static uint64_t group_chunks(int prec, uint64_t L, uint64_t Bi, uint64_t nchunks, uint64_t any) {
    if (nchunks <= any) return nchunks;
    const uint64_t most = any < kMaxGroup ? most_chunks(noise_error(prec, L, Bi), leak_error(prec, L, Bi)) : kMaxGroup;
    return ceil_div(nchunks, ceil_div(nchunks, most));
}

// The plan of job (n, m) with shared spectra at class `cls`: chunks and windows
// of L / 2, the chunks in as many equal groups as the workspace and the error
// model ask for.  Only jobs of several windows gain (each chunk meets several).
static bool plan_shared(uint64_t n, uint64_t m, int prec, int cls, const CostModel& cm, uint64_t shared_bytes,
                        TilePlan* out) {
    if (!class_shared(prec, cls)) return false;
    TilePlan p;
    p.prec = prec;
    p.cls = cls;
    p.L = class_len(cls);
    p.shared = true;
    p.Bi = p.Bo = p.L / 2;
    p.nchunks = ceil_div(n, p.Bi);
    p.nouts = ceil_div(m, p.Bo);
    if (p.nouts < 2 || p.nchunks < 2 || p.tiles() > (1u << 20)) return false;
    const uint64_t tile_bytes = 8 * p.L + p.L / 4;
    const double err = shared_error(prec, p.L, p.Bi);
    uint64_t groups = 1;
    for (;; ++groups) {
        p.cgroup = ceil_div(p.nchunks, groups);
        p.bound = err * std::sqrt((double)p.cgroup);
        if (p.bound <= kGroupErrorLimit && p.packs(p.cgroup) * tile_bytes + p.nouts * 8 * p.L <= shared_bytes) break;
        if (p.cgroup <= 4) return false;   // little left to share
    }
    groups = ceil_div(p.nchunks, p.cgroup);
    // Measured per 1000 points (2^21 to 2^23; 6, 16 and 40 chunks, 2 to 16 windows): a
    // pack takes 6.1 to 7.1 ns up to four windows, with more 8.0 to 8.7 ns up to eight
    // and 9.6 to 10.7 up to sixteen (its spectrum is read once per eight), a
    // window's inverse and columns 1.5 to 1.9 ns.  Further reads cost less: 11.8 ns with
    // 24 windows, 12.3 with 32 and 13.1 with 47 (keys of 140 to 150 M bits).
    const double reads = (double)ceil_div(p.nouts, 8);
    const double pack = p.nouts <= 4 ? 6.3e-12 : 6.6e-12 + 1.75e-12 * std::min(reads, 3.0) + 0.5e-12 * std::max(reads - 3.0, 0.0);
    p.cost = (double)p.L * (double)groups * ((double)p.packs(p.cgroup) * pack + (double)p.nouts * 1.9e-12);
    p.rigorous = rigorous_bound(prec, p.L, p.Bi, p.Bo, p.cgroup);
    *out = p;
    return true;
}

bool plan_at_class(uint64_t n, uint64_t m, int prec, int cls, const CostModel& cm, TilePlan* out,
                   uint64_t shared_bytes, uint64_t jobs) {
    ClassGeom g;
    if (n == 0 || m == 0 || !class_geometry(prec, cls, &g)) return false;
    const uint64_t L = g.L;
    // largest chunk the error model admits at this length
    uint64_t bi_cap = n;
    if (prec != PREC_NTT) {
        const double per = 6.0 * g_kappa * unit_roundoff(prec) * std::sqrt(std::log2((double)L));
        const double cap = std::floor((kPlanErrorLimit / per) * (kPlanErrorLimit / per) - (double)L);
        if (cap < (double)bi_cap) bi_cap = (uint64_t)std::max(0.0, cap);
    }
    const bool sums = class_sums(prec, cls);
    const uint64_t any = sums ? any_chunks(prec, L) : 1;
    const double tile = cm.tile(prec, cls), chunk = sums ? cm.least_chunk(prec, cls) : tile;
    TilePlan best;
    bool found = false;
    const uint64_t max_outs = std::min<uint64_t>(ceil_div(m, 64), 1u << 14);
    uint64_t last_bo = 0;
    const uint64_t min_chunks = ceil_div(n, std::min<uint64_t>(L, bi_cap == 0 ? 1 : bi_cap));
    // fewer than ceil(m / L) windows cannot fit a window in L
    const double per_tile = (tile + (double)(kMaxGroup - 1) * chunk) / (double)kMaxGroup;   // in the largest groups
    for (uint64_t w = std::max<uint64_t>(1, ceil_div(m, L)); w <= std::max<uint64_t>(1, max_outs); ++w) {
        // every later candidate has >= w windows of >= min_chunks chunks
        if (found && (double)w * (tile + (double)(min_chunks - 1) * chunk) >= 1.03 * best.cost) break;
        // and >= w n / (L + 1 - m / w) tiles, which grows with w from w = 2 m / (L + 1)
        // on, in >= w groups of at most kMaxGroup
        const double room = (double)(L + 1) - (double)m / (double)w, tiles = (double)w * (double)n / room;
        if (found && chunk <= tile && 2 * room >= (double)(L + 1) &&
            (1 - 1e-9) * std::max((double)w * (tile - chunk) + tiles * chunk, tiles * per_tile) >= 1.03 * best.cost)
            break;
        uint64_t Bo = (w == 1) ? m : round_up64(ceil_div(m, w));
        if (Bo == last_bo) continue;
        last_bo = Bo;
        if (Bo > L) continue;
        TilePlan p;
        p.nouts = ceil_div(m, Bo);
        const uint64_t bi_max = std::min<uint64_t>(L - Bo + 1, bi_cap);
        if (bi_max == 0) continue;
        p.nchunks = ceil_div(n, bi_max);
        p.Bo = Bo;
        // a tie within the noise of the measured costs goes to fewer tiles (less workspace)
        const double limit = found ? (p.tiles() < best.tiles() ? 1.03 : 1.0) * best.cost : HUGE_VAL;
        auto groups_of = [&](uint64_t cgroup) { return ceil_div(p.nchunks, cgroup) * p.nouts; };
        const double least = (double)groups_of(kMaxGroup) * tile + (double)(p.tiles() - groups_of(kMaxGroup)) * chunk;
        // (the error model, the dearest step here, only where the largest groups would win)
        if (!sums || chunk > tile || least < limit) {
            p.Bi = ceil_div(n, p.nchunks);
            p.cgroup = sums ? group_chunks(prec, L, p.Bi, p.nchunks, any) : 1;
            const uint64_t groups = groups_of(p.cgroup);
            p.cost = (double)groups * cm.tile_of(prec, cls, groups * jobs);
            if (p.cgroup > 1)
                p.cost += (double)(p.tiles() - groups) * cm.chunk_of(prec, cls, groups * jobs, p.cgroup, p.tiles() * jobs);
            if (p.cost < limit) {
                found = true;
                best = p;
            }
        }
        if (best.nouts == 1 && best.nchunks == 1) break;
    }
    if (!found) return false;
    best.prec = prec;
    best.cls = cls;
    best.L = L;
    // the errors of a group's summed products add up, in the worst case in full
    best.bound = group_error(prec, L, best.Bi, best.cgroup);
    best.rigorous = rigorous_bound(prec, L, best.Bi, best.Bo, best.cgroup);
    if (best.bound > kPlanErrorLimit) return false;   // not reached by FP32 up to 2^24
    TilePlan sh;
    if (shared_bytes && plan_shared(n, m, prec, cls, cm, shared_bytes, &sh) && sh.cost < best.cost) best = sh;
    best.cost += cm.first(prec, cls);
    *out = best;
    return true;
}

bool plan_job(uint64_t n, uint64_t m, int policy, const CostModel& cm, TilePlan* out, int cap_logL,
              uint64_t shared_bytes) {
    if (n == 0 || m == 0) return false;
    const int prec = policy;
    int ids[kMaxClassId + 1];
    const int nid = class_ids(prec, ids, cap_logL);
    // Classes come in increasing length.  A plan that moves more points (tiles
    // x L) replaces the best so far only when its modeled cost is lower by
    // more than the noise of the measured costs (2%), so near-ties keep the
    // plan with fewer bytes.
    auto better = [](const TilePlan& p, const TilePlan& best) {
        const double pts = p.points(), bpts = best.points();
        return pts <= bpts ? p.cost < best.cost : p.cost < 0.98 * best.cost;
    };
    if (prec == PREC_FP64 || prec == PREC_NTT) {
        // one tile: the shortest class that holds the whole product, unless a
        // longer class is cheaper by more than the noise of a tile's measured time,
        // which its cost is (1%)
        bool one = false;
        TilePlan best1;
        for (int q = 0; q < nid; ++q) {
            TilePlan p;
            if (n + m - 1 > class_len(ids[q]) || !plan_at_class(n, m, prec, ids[q], cm, &p, shared_bytes)) continue;
            if (!one || p.cost < (p.points() > best1.points() ? 0.99 : 1.0) * best1.cost) {
                best1 = p;
                one = true;
            }
        }
        if (one) {
            *out = best1;
            return true;
        }
    }
    bool found = false;
    TilePlan best;
    for (int q = 0; q < nid; ++q) {
        TilePlan p;
        if (!plan_at_class(n, m, prec, ids[q], cm, &p, shared_bytes)) continue;
        if (!found || better(p, best)) {
            best = p;
            found = true;
        }
    }
    if (found) *out = best;
    return found;
}

bool plan_batch_groups(const std::vector<uint64_t>& ns, const std::vector<uint64_t>& ms, int policy,
                       const CostModel& cm, std::vector<BatchGroup>* groups, const std::vector<TilePlan>* own,
                       uint64_t shared_bytes) {
    if (ns.empty() || ns.size() != ms.size() || (own && own->size() != ns.size())) return false;
    // plans of job i at class id k, computed once: memo[i * NK + k], state 0
    // unknown, 1 found, -1 none
    constexpr int NK = kMaxClassId + 1;
    std::vector<TilePlan> memo(ns.size() * NK);
    std::vector<signed char> known(ns.size() * NK, 0);
    auto at_class = [&](size_t i, int k, TilePlan* p) {
        if (k < 0 || k >= NK) return false;
        const size_t x = i * NK + (size_t)k;
        if (!known[x]) known[x] = plan_at_class(ns[i], ms[i], policy, k, cm, &memo[x], shared_bytes, ns.size()) ? 1 : -1;
        if (known[x] < 0) return false;
        *p = memo[x];
        return true;
    };
    std::map<int, BatchGroup> by_class;
    for (size_t i = 0; i < ns.size(); ++i) {
        TilePlan p;
        if (own) p = (*own)[i];
        else if (!plan_job(ns[i], ms[i], policy, cm, &p)) return false;
        TilePlan beside;   // among the other jobs' groups its further chunks may cost less
        if (at_class(i, p.cls, &beside)) p = beside;
        BatchGroup& g = by_class[p.cls];
        g.cls = p.cls;
        g.jobs.push_back(i);
        g.plans.push_back(p);
        g.cost += p.cost - cm.first(policy, p.cls);
    }
    // A job's own class is the cheapest for a launch of its own, in which the fixed
    // cost of a launch and a device partly idle count for much.  The jobs of a group go
    // together to another class where that is cheaper by more than the noise of the
    // costs (3%); a few of them choose it.
    int ids[kMaxClassId + 1];
    const int nid = class_ids(policy, ids);
    std::map<int, BatchGroup> merged;
    for (auto& kv : by_class) {
        BatchGroup& g = kv.second;
        const double first = cm.first(policy, g.cls);
        const size_t step = (g.jobs.size() + 3) / 4;
        double least = HUGE_VAL;
        int to = g.cls;
        for (int q = 0; q < nid && g.jobs.size() > 1; ++q) {
            double c = 0;
            size_t sampled = 0;
            for (size_t j = 0; j < g.jobs.size() && c < HUGE_VAL; j += step, ++sampled) {
                TilePlan p;
                c += at_class(g.jobs[j], ids[q], &p) ? p.cost - cm.first(policy, ids[q]) : HUGE_VAL;
            }
            c = c * (double)g.jobs.size() / (double)sampled + cm.first(policy, ids[q]);
            if (c < least) {
                least = c;
                to = ids[q];
            }
        }
        BatchGroup moved;
        moved.cls = to;
        for (size_t j = 0; j < g.jobs.size() && to != g.cls; ++j) {
            TilePlan p;
            moved.cost += at_class(g.jobs[j], to, &p) ? p.cost - cm.first(policy, to) : HUGE_VAL;
            moved.plans.push_back(p);
        }
        if (to != g.cls && moved.cost + cm.first(policy, to) < 0.97 * (g.cost + first)) {
            moved.jobs = std::move(g.jobs);
            g = std::move(moved);
        }
        BatchGroup& m = merged[g.cls];
        m.cls = g.cls;
        m.cost += g.cost;
        m.jobs.insert(m.jobs.end(), g.jobs.begin(), g.jobs.end());
        m.plans.insert(m.plans.end(), g.plans.begin(), g.plans.end());
    }
    std::vector<BatchGroup> gs;
    for (auto& kv : merged) {
        kv.second.cost += cm.first(policy, kv.second.cls);
        gs.push_back(std::move(kv.second));
    }
    // fold groups while that saves more than it costs
    for (;;) {
        double best_gain = 0;
        size_t bg = 0, bh = 0;
        std::vector<TilePlan> best_plans;
        for (size_t g = 0; g < gs.size(); ++g)
            for (size_t h = 0; h < gs.size(); ++h) {
                if (g == h) continue;
                std::vector<TilePlan> moved(gs[g].jobs.size());
                double c = 0;
                bool ok = true;
                for (size_t q = 0; q < gs[g].jobs.size() && ok; ++q) {
                    const size_t i = gs[g].jobs[q];
                    ok = at_class(i, gs[h].cls, &moved[q]);
                    c += moved[q].cost - cm.first(policy, gs[h].cls);
                }
                if (!ok) continue;
                const double gain = gs[g].cost - c;   // the launch of g disappears
                if (gain > best_gain) {
                    best_gain = gain;
                    bg = g;
                    bh = h;
                    best_plans = std::move(moved);
                }
            }
        if (best_gain <= 0) break;
        BatchGroup& h = gs[bh];
        for (size_t q = 0; q < gs[bg].jobs.size(); ++q) {
            h.jobs.push_back(gs[bg].jobs[q]);
            h.plans.push_back(best_plans[q]);
            h.cost += best_plans[q].cost - cm.first(policy, h.cls);
        }
        gs.erase(gs.begin() + (long)bg);
    }
    std::sort(gs.begin(), gs.end(),
              [](const BatchGroup& a, const BatchGroup& b) { return class_len(a.cls) < class_len(b.cls); });
    *groups = std::move(gs);
    return true;
}

bool plan_batch(const std::vector<uint64_t>& ns, const std::vector<uint64_t>& ms, int policy,
                const CostModel& cm, int* cls_out, std::vector<TilePlan>* plans, int cap_logL, uint64_t shared_bytes) {
    if (ns.empty() || ns.size() != ms.size()) return false;
    bool found = false;
    double best_cost = 0;
    std::vector<TilePlan> tmp(ns.size());
    int ids[kMaxClassId + 1];
    const int nid = class_ids(policy, ids, cap_logL);
    for (int q = 0; q < nid; ++q) {
        const int k = ids[q];
        double cost = cm.first(policy, k);
        bool ok = true;
        for (size_t i = 0; i < ns.size() && ok; ++i) {
            ok = plan_at_class(ns[i], ms[i], policy, k, cm, &tmp[i], shared_bytes, ns.size());
            if (ok) cost += tmp[i].cost - cm.first(policy, k);
        }
        if (!ok) continue;
        if (!found || cost < best_cost) {
            found = true;
            best_cost = cost;
            *cls_out = k;
            *plans = tmp;
        }
    }
    return found;
}

}  // namespace pa
