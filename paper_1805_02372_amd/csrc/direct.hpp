// Host entry points of the direct GF(2) path, the word XOR and the certificate
// read-back (direct.hip).
#pragma once
#include <stdint.h>

namespace pa {

// Reversed-key words of an n-bit key (scratch `kr` of launch_direct_select).
uint64_t direct_key_words(uint64_t n);
// Direct product of one job on `stream`: launch_direct_prep clears out when
// several workgroups share an output word (no launch otherwise), then
// launch_direct_main writes the m output bits.  Each returns 0, or -1 on a
// launch error, and adds its launches to *launches.
int launch_direct_prep(uint64_t n, uint64_t m, uint64_t* out, void* stream, uint64_t* launches);
int launch_direct_main(const uint64_t* seed, const uint64_t* key, uint64_t n, uint64_t m, uint64_t* out, void* stream,
                       uint64_t* launches);
// The same for many jobs in at most four launches (the clearing and one per
// tile width).  direct_batch_plan orders `jobs` (seed, key, out, n, m set) and
// fills their grids; it returns count, or less when they do not fit one batch
// (they are then launched one by one).  `many` is the device copy of the jobs.
struct DirectJob {
    const uint64_t* seed;
    const uint64_t* key;
    uint64_t* out;
    uint64_t n, m;
    uint32_t wg_begin, bx;   // batches: first workgroup, workgroups along the outputs
    uint32_t seg, merge;
};
struct DirectBatch {
    uint32_t first[3], jobs[3], wgs[3], clears;
};
uint64_t direct_batch_plan(DirectJob* jobs, uint32_t count, DirectBatch* plan);
int launch_direct_batch(const DirectBatch& plan, const DirectJob* many, uint32_t count, void* stream,
                        uint64_t* launches);
// Selected outputs: bit k of res (ceil(count/64) words) = y[idx[k]].
int launch_direct_select(const uint64_t* seed, const uint64_t* key, uint64_t n, uint64_t m, const uint64_t* idx,
                         uint32_t count, uint64_t* res, uint32_t* kr, void* stream);
// dst[k] ^= src[k] for k < words (stream order); src may be dst (clears it).
int launch_xor_words(uint64_t* dst, const uint64_t* src, uint64_t words, void* stream);

// Copies `count` 16-byte records to pinned host memory and then sets *flag (pinned
// host memory) to seq, after everything queued before it on the stream.
int launch_publish(const void* src, void* host, uint32_t count, uint32_t* flag, uint32_t seq, void* stream);

}  // namespace pa
