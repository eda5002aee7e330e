// Tile planning: FFT length class, key-chunk and output-window sizes, and the
// rounding-error model that bounds them.  Pure host code.
#pragma once
#include <cstddef>
#include <algorithm>
#include <cstdint>
#include <vector>

#include "pa_internal.hpp"

namespace pa {

enum Prec { PREC_FP32 = 32, PREC_FP64 = 64, PREC_NTT = 1, PREC_DIRECT = 2 };

struct ClassGeom {
    int prec, cls;        // precision, class id (pa_internal.hpp)
    uint64_t L;           // FFT length n1 * n2
    int n1, n2;
};

// Geometry of class `cls` in the given precision; false if none.
bool class_geometry(int prec, int cls, ClassGeom* g);
// ceil(log2 L)
int ceil_log2(uint64_t L);
int min_logL(int prec);
int max_logL(int prec);
// The class ids a plan of precision `prec` may use, in increasing FFT length:
// 2^min_logL <= L <= 2^min(max_logL, cap_logL).  Environment (tests and
// measurements): PA_MIN_LOG2_LEN / PA_MAX_LOG2_LEN bound L; PA_ONLY_LEN=<L>
// keeps the class of that length only; PA_POW2_ONLY=1 drops the mixed-radix
// classes.  Writes at most kMaxClassId + 1 ids; returns the count.
int class_ids(int prec, int* ids, int cap_logL = 24);
// A key of the environment settings above (plan caches depend on them).
uint64_t class_filter_key();

// Cost of a class's launches (seconds), by prec and class id: a launch of G
// groups with T tiles costs first_s + G tile + (T - G) chunk.  tile is the cost of
// a tile with its inverse, chunk that of a further chunk whose product joins the
// same inverse; first_s the rest of a one-tile launch (launch latency, ramp-up, and
// the part of the device one tile leaves idle).  Both have two measured ends:
// tile_s and chunk_s on a full device, few_s per tile of four and alone_s per
// further chunk, up to the eighth, of a launch's only group, whose chunks follow
// one another through the row pass (run_s beyond the eighth).  In between, the few
// groups of a launch share what they leave idle: max(tile_s, few_s) up to 12 groups
// and max(tile_s, 12 few_s / G) beyond (FP32 2^19: a tile takes 5.5 us of 4, 4.0 of 16
// and 3.3 of 64; 2^17 2.4, 1.7 and 0.9); of the further chunks of G groups one costs
// alone_s and the others chunk_s each, or the least of the three where the tiles
// stay in the last-level cache (256 MB; 2^15, 30 chunks: 0.7 us per chunk of one group, 0.84
// per pair of two, 0.9 per four of four; 2^19: a further chunk takes 2.9 us up to the
// eighth, 1.6 to 2.0 up to the sixtieth, and 2.8 with 64 groups).  With one cost each, measured with 16 tiles, batches of 64 and more
// jobs of 0.8 to 1.4 Mbit took 2^19 where 2^20 and 2^21 are up to 1.9 times as fast, and
// single keys took more chunks in a shorter class than paid, by up to 36%.  Filled
// from tuning data when present, else from the built-in model.
struct CostModel {
    double tile_s[3][64];   // [0] FP32, [1] FP64, [2] NTT; index class id
    double few_s[3][64];    // (0: tile_s)
    double first_s[3][64];  // extra cost of a launch (its first tile)
    double chunk_s[3][64];  // (0: 0.7 tile_s)
    double alone_s[3][64];  // (0: chunk_s)
    double run_s[3][64];    // (0: alone_s)
    double launch_s;        // launch cost of a class without its own first_s
    double direct_s;        // direct GF(2) path: seconds per output per 32-bit key word
    double direct_launch_s; // direct GF(2) path: fixed cost of a job (its launches)
    CostModel();
    double tile(int prec, int cls) const;
    double first(int prec, int cls) const;
    double chunk(int prec, int cls) const;
    // in a launch of `groups` groups, of `chunks` chunks and `tiles` tiles altogether
    double tile_of(int prec, int cls, uint64_t groups) const;
    double chunk_of(int prec, int cls, uint64_t groups, uint64_t chunks, uint64_t tiles) const;
    double alone(int prec, int cls) const;
    double run(int prec, int cls) const;
    double least_chunk(int prec, int cls) const { return std::min({alone(prec, cls), run(prec, cls), chunk(prec, cls)}); }
    void set_chunk(int prec, int cls, double s);
    void set_few(int prec, int cls, double s);
    void set_alone(int prec, int cls, double s);
    void set_run(int prec, int cls, double s);
    void set(int prec, int cls, double s);
    void set_first(int prec, int cls, double s);
};
// The model a context starts from: the built-in one, replaced class by class
// by the tuning table measured on MI355X that ships beside the library
// (tune_mi355x.json next to libpa.so; PA_TUNE_DEFAULT=0 skips it).
const CostModel& default_cost_model();
// Read a tuning table (pa_tune's JSON) into cm; returns the number of values
// taken, or -1 if the file cannot be read.
int load_tune_table(CostModel& cm, const char* path);

struct TilePlan {
    int prec = 0, cls = 0;
    uint64_t L = 0;        // FFT length of the class
    uint64_t Bi = 0, Bo = 0, nchunks = 0, nouts = 0;
    uint64_t cgroup = 1;   // chunks whose products are summed before one inverse
    bool shared = false;   // spectra of chunks and seed slices shared by the windows (Bi = Bo = L / 2)
    // tiles that a shared-spectra group of c chunks transforms, two sequences each
    uint64_t packs(uint64_t c) const { return (c + 1) / 2 + (c + nouts) / 2; }
    double bound = 0, cost = 0;
    double rigorous = 0;   // worst-case rounding bound of a group (any input bits)
    uint64_t tiles() const { return nchunks * nouts; }
    // points transformed (shared spectra: packs and windows)
    double points() const {
        if (!shared) return (double)tiles() * (double)L;
        const uint64_t groups = (nchunks + cgroup - 1) / cgroup;
        return (double)(groups * (packs(cgroup) + nouts)) * (double)L;
    }
};

// Error model of one floating-point tile, a predicted maximum of the output
// error for an FFT convolution of a +-1 sequence with a 0/1 chunk of Bi bits at
// length L: 6 sigma of the random rounding noise, sigma = kappa u
// sqrt(log2 L (Bi + L)), plus 5 times the rms of the low-frequency error that
// the chunk's zero padding causes (about 0.036 u L once Bi > L/3; the larger
// term from 2^22 on in FP32).
double error_bound(int prec, uint64_t L, uint64_t Bi);
// Worst-case (a-priori) bound of a tile's max error for any input bits:
// (||x|| + ||w||)^2 times the relative error growth of the forward FFT,
// product and inverse FFT, with ||x|| <= sqrt(Bi), ||w|| = sqrt(Bi+Bo-1); of a
// group of c chunks, c times that with the rounding of the sum.  A tile or group
// whose bound is below 0.5 rounds to the exact integers.
double rigorous_bound(int prec, uint64_t L, uint64_t Bi, uint64_t Bo, uint64_t c = 1);
constexpr double kRigorousLimit = 0.5;
void set_error_kappa(double kappa);
double error_kappa();

// The admissible error for a floating-point plan before the a-posteriori
// certificate (half the rounding margin of 0.5).
constexpr double kPlanErrorLimit = 0.25;

// The admissible modeled error of a group's sum of products: about that of the
// longest single tile (0.19 at 2^24).  Over 230 shapes of random bits the largest
// residual of such groups was 0.07 (0.21 to 0.46 of the model, the largest groups
// up to 0.41), against the 0.125 that the certificate rejects.
constexpr double kGroupErrorLimit = 0.2;

// Modeled time of the direct GF(2) path for one job: a fixed cost and a cost per
// output (in blocks of 256) and key word (ceil(n/32), rounded up to 4), plus 10%
// so that near-ties within the noise of the measured costs stay with the FFT
// (measured on MI355X at n = 10^6: m = 50,000 direct 40 us, FFT 57; m = 100,000
// 55 and 57; m = 200,000 84 and 64).
double direct_cost(uint64_t n, uint64_t m, const CostModel& cm);
// Whether the precision bits of `flags` put job (n, m) on the direct path:
// always for PA_PREC_DIRECT; for PA_PREC_AUTO when the direct path is modeled
// cheaper than the FFT plan `fft`.
bool choose_direct(uint32_t flags, uint64_t n, uint64_t m, const CostModel& cm, const TilePlan& fft);

// The same for a job of a batch or a serving launch of about `jobs` jobs, where both
// paths share their launches with other jobs: the costs beyond the launches are
// compared, the FFT plan's in that company.  The direct path has to be modeled 1.1
// times as fast: on 258 batches of 1 to 256 jobs of random sizes that choice took
// 0.6 to 1.1% longer than the faster path, 1.3 to 2.4% at 1.3, and 4 to 6% at 2.5.
constexpr double kDirectShared = 1.1;
bool choose_direct_shared(uint32_t flags, uint64_t n, uint64_t m, const CostModel& cm, const TilePlan& fft, uint64_t jobs);

// Workspace that a shared-spectra plan may count on: what a serving lane of a
// context with the default HBM budget has (a launch with less cuts the chunks
// into smaller groups).
constexpr uint64_t kSharedBytes = (8ull << 30) / 3;

// Best (Bi, Bo) for job (n, m) at a fixed class; false if impossible.
// `shared_bytes`: workspace for shared spectra (0: none); `jobs`: about as many
// share the launch.
bool plan_at_class(uint64_t n, uint64_t m, int prec, int cls, const CostModel& cm, TilePlan* out,
                   uint64_t shared_bytes = kSharedBytes, uint64_t jobs = 1);

// Best plan over classes for one job.  policy: PREC_FP32 (segmented, bound
// limited), PREC_FP64 and PREC_NTT (a single tile if one fits, else the
// cheapest plan over the classes).  Among plans whose modeled costs differ by
// less than 2% (1% where each is one tile) the one that moves fewer points wins.
// Classes longer than 2^cap_logL are not used.
bool plan_job(uint64_t n, uint64_t m, int policy, const CostModel& cm, TilePlan* out, int cap_logL = 24,
              uint64_t shared_bytes = kSharedBytes);

// Jobs of a batch that share one FFT length class (one pipeline launch).
struct BatchGroup {
    int cls = 0;
    std::vector<size_t> jobs;      // indices into the batch
    std::vector<TilePlan> plans;   // plan of each job in `jobs`, at class cls
    double cost = 0;               // launch (first_s) plus tiles
};

// Batch plan with one launch per length class: every job starts in its own
// cheapest class, then a group is folded into another group's class while that
// lowers the summed cost (tiles plus one launch per group).  Groups come out
// in increasing FFT length.  `own` (optional): each job's own best plan, already
// known to the caller.
bool plan_batch_groups(const std::vector<uint64_t>& ns, const std::vector<uint64_t>& ms, int policy,
                       const CostModel& cm, std::vector<BatchGroup>* groups,
                       const std::vector<TilePlan>* own = nullptr, uint64_t shared_bytes = kSharedBytes);

// One class for a whole batch, of at most 2^cap_logL points: minimises the summed
// cost of every job's tiles.
bool plan_batch(const std::vector<uint64_t>& ns, const std::vector<uint64_t>& ms, int policy,
                const CostModel& cm, int* cls, std::vector<TilePlan>* plans, int cap_logL = 24,
                uint64_t shared_bytes = kSharedBytes);

}  // namespace pa
