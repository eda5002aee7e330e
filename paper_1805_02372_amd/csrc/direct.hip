// Direct evaluation of the Toeplitz hash over GF(2), with no transform and no
// rounding: y_i = parity(popcount(AND of the seed window at i with the reversed
// key)), the definition of section 2.1 (Eq. 1).  With xr[t] = x[n-1-t] (the key
// reversed),
//
//     y_i = XOR_{t<n} ( s[i+t] AND xr[t] ).
//
// Whole outputs are computed as a bit contraction on the matrix cores
// (k_direct_mm); chosen outputs word-parallel on the vector units
// (k_direct_select): the 32-bit seed words at bit offsets i + 32k, each a
// funnel shift (v_alignbit) of two aligned words, AND-ed with reversed-key word
// k and XOR-accumulated.  Both share nothing with the FFT path, and the second
// serves as its verifier.
//
// Seed bits past n+m-1 (and reads past the seed's last word, which return 0)
// only ever meet reversed-key bits t >= n, which are zero.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "direct.hpp"

namespace pa {

constexpr int kDirectThreads = 256;
constexpr uint32_t kDirectChunk = 4096;   // reversed-key words per workgroup (multiple of 4)

// 32 key bits starting at bit p (p may be negative: bits below 0 are 0);
// p + 31 < n, so no bit at or beyond n is read.
__device__ __forceinline__ uint32_t key_bits32(const uint64_t* __restrict__ key, int64_t p) {
    if (p <= -32) return 0u;
    if (p < 0) {
        const uint32_t cnt = (uint32_t)(32 + p);   // 1..31 bits from position 0
        return (uint32_t)(key[0] & ((1ull << cnt) - 1ull)) << (uint32_t)(-p);
    }
    const uint64_t w = (uint64_t)p >> 6;
    const uint32_t s = (uint32_t)p & 63u;
    uint64_t v = key[w] >> s;
    if (s > 32) v |= key[w + 1] << (64 - s);
    return (uint32_t)v;
}

// Reversed key kr[w] (bit b = key bit n-1-32w-b, zero for t >= n), for
// w < kw4, and zeroed output words.
__global__ void __launch_bounds__(kDirectThreads)
k_direct_prep(const uint64_t* __restrict__ key, uint64_t n, uint32_t* __restrict__ kr, uint64_t kw4,
              uint64_t* __restrict__ zero, uint64_t nzero) {
    const uint64_t g = (uint64_t)blockIdx.x * kDirectThreads + threadIdx.x;
    if (g < kw4) {
        const int64_t p = (int64_t)n - 32 - 32 * (int64_t)g;
        kr[g] = __builtin_bitreverse32(key_bits32(key, p));
    }
    if (g < nzero) zero[g] = 0ull;
}

// ---- the product on the matrix cores
// Output i = i0 + r + 64 d of a tile (r < 64, d < 16 NB) is
//     y_i = XOR_p ( s[i0 + r + p] AND xr[p - 64 d] ),    p = t + 64 d,
// a contraction over p of A[r][p] = s[i0 + r + p] (64 shifts of one seed
// stream) with B[p][d] = xr[p - 64 d] (16 NB word shifts of one key stream).
// Both hold bits, so 4-bit floating operands (e2m1) carry them exactly and the
// FP32 accumulators hold the exact counts (a wave adds at most 127 * 128
// products, far below 2^24); y_i is the count's low bit.
//
// Operands.  A lane of v_mfma_f32_16x16x128_f8f6f4 holds 32 elements of one
// row (or column) for one of four K groups.  The K order is free as long as A
// and B share it, so the 32 elements of a lane are the bits of one word, taken
// as four masks: bits 0, 4, .. / 1, 5, .. / 2, 6, .. / 3, 7, .. of the word in
// place are nibbles of value 0.5, 1 and 2 in A, matched by 2, 1 and 0.5 in B, so
// that every product of set bits is 1.  Expanding a word costs 5 (A) or 7 (B)
// operations beside A's funnel shift, no table; the four row blocks of A share
// their words (k_direct_mm).  The four K groups of each
// wave walk their own consecutive words, so a lane loads one new seed word and
// NB key words per step.
//
// Bound by the matrix cores for NB = 4 (16 products of 16 cycles per step beside
// 44 vector operations of 4) and by the vector operations that prepare a step
// for NB = 1 (23, and 4 products; 32 with every row block expanded by itself: call
// 26.9 -> 26.0 us at n = 12,345,679, m = 1000).  Measured on MI355X, that job 12-16
// us (the word-parallel kernel before it, one output per lane: 55 us); n = 10^6, m =
// 200,000 3.1e15 bit products per second (2.2e14 before).
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kMmThreads = 512;                          // 8 waves
constexpr int kMmStreams = kMmThreads / 16;              // K groups of a workgroup
constexpr uint32_t kMmMaxSeg = 127;                      // words per K group and workgroup
constexpr uint32_t kMmMinSeg = 7;
constexpr uint32_t kMmMaxChunk = kMmStreams * kMmMaxSeg;

// A's nibbles of the bits of w: 0.5, 1, 2, 2 by bit position mod 4.
__device__ __forceinline__ v8i mm_expand_a(uint32_t w) {
    return v8i{(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u),
               (int)((w >> 1) & 0x44444444u), 0, 0, 0, 0};
}
// B's: 2, 1, 0.5, 0.5.
__device__ __forceinline__ v8i mm_expand_b(uint32_t w) {
    return v8i{(int)((w << 2) & 0x44444444u), (int)(w & 0x22222222u), (int)((w >> 2) & 0x11111111u),
               (int)((w >> 3) & 0x11111111u), 0, 0, 0, 0};
}
// The nibbles a half word after those of a, b being the next word's.
__device__ __forceinline__ v8i mm_half(v8i a, v8i b) {
    v8i h{};
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = (int)__builtin_amdgcn_alignbit((uint32_t)b[q], (uint32_t)a[q], 16);
    return h;
}

// Workgroup (x, y) of a job: outputs [1024 NB x, + 1024 NB) over words
// [kc y, + kc) of the p axis (p < n + 64 (16 NB - 1)), kc = 32 seg.  `merge`:
// XOR the words into out (several workgroups along y; out cleared before), else
// store.  njobs = 0: one job by value, x and y from the grid and its bases;
// else the workgroups of all jobs of `many` in a row (wg_begin), x fastest.
template <int NB>
__global__ void __launch_bounds__(kMmThreads)
k_direct_mm(DirectJob one, const DirectJob* __restrict__ many, uint32_t njobs, uint64_t x_base, uint64_t y_base) {
    constexpr uint32_t XO = 32 * NB;                     // key words before the chunk (>= 2 (16 NB - 1))
    __shared__ uint32_t S[kMmMaxChunk + 4];
    __shared__ uint32_t X[kMmMaxChunk + XO];
    __shared__ unsigned long long red[kMmThreads / 64][16 * NB];
    const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
    DirectJob jd = one;
    uint64_t bx = x_base + blockIdx.x, by = y_base + blockIdx.y;
    if (njobs) {
        uint32_t lo = 0, hi = njobs - 1;
        while (lo < hi) {   // last job with wg_begin <= blockIdx.x
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (many[mid].wg_begin <= blockIdx.x) lo = mid; else hi = mid - 1;
        }
        jd = many[lo];
        const uint32_t q = blockIdx.x - jd.wg_begin;
        bx = q % jd.bx;
        by = q / jd.bx;
    }
    const uint64_t n = jd.n, m = jd.m, sw32 = 2 * ((n + m - 1 + 63) >> 6);
    const uint32_t* __restrict__ seed32 = reinterpret_cast<const uint32_t*>(jd.seed);
    const uint64_t* __restrict__ key = jd.key;
    uint64_t* __restrict__ out = jd.out;
    const uint32_t seg = jd.seg;
    const uint32_t kc = kMmStreams * seg;
    const uint64_t w0 = by * kc;                         // first word of the chunk
    const uint64_t sbase = bx * (32 * NB) + w0;               // its seed word
    for (uint32_t q = tid; q < kc + 3; q += kMmThreads) {
        const uint64_t g = sbase + q;
        S[q] = g < sw32 ? seed32[g] : 0u;
    }
    const uint64_t kw = (n + 31) >> 5;
    for (uint32_t q = tid; q < kc + XO; q += kMmThreads) {
        const int64_t w = (int64_t)(w0 + q) - (int64_t)XO;   // reversed-key word; none outside [0, kw)
        X[q] = (w >= 0 && (uint64_t)w < kw)
                   ? __builtin_bitreverse32(key_bits32(key, (int64_t)n - 32 - 32 * w)) : 0u;
    }
    __syncthreads();

    const int r = l & 15, g = l >> 4;
    const uint32_t q0 = (uint32_t)(wv * 4 + g) * seg;         // this K group's words q0 .. q0 + seg - 1
    const uint32_t* __restrict__ xs = X + q0 + XO - 2 * r;    // column d = 16 b + r reads xs[h - 32 b]
    v4f acc[4][NB];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
    // Row 16 a + r of a step are the 32 seed bits from bit 16 a + r of its word on:
    // for a = 0 and 2 the nibbles of this and the next word at shift r, for a = 1
    // and 3 the same a half word further (16 bits are whole nibbles).  Two of the
    // four are the next step's, so a step expands one word and shifts it once.
    uint32_t s2 = S[q0 + 2];
    v8i e0 = mm_expand_a(__builtin_amdgcn_alignbit(S[q0 + 1], S[q0], r));
    v8i e1 = mm_expand_a(__builtin_amdgcn_alignbit(s2, S[q0 + 1], r));
    v8i e2, h0 = mm_half(e0, e1), h1;
    // a step from (a, ha, b): its fourth row hb and the word c after b
    auto step = [&](uint32_t h, const v8i& a, const v8i& ha, const v8i& b, v8i& hb, v8i& c) {
        const uint32_t s3 = S[q0 + h + 3];
        c = mm_expand_a(__builtin_amdgcn_alignbit(s3, s2, r));
        s2 = s3;
        hb = mm_half(b, c);
        const v8i A[4] = {a, ha, b, hb};
        v8i B[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) B[k] = mm_expand_b(xs[(int)h - 32 * k]);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int k = 0; k < NB; ++k)
                acc[q][k] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A[q], B[k], acc[q][k], 4, 4, 0, 0, 0, 0);
    };
    // seg is odd: one step, then pairs
    step(0, e0, h0, e1, h1, e2);
    for (uint32_t h = 1; h + 1 < seg; h += 2) {
        step(h, e1, h1, e2, h0, e0);
        step(h + 1, e2, h0, e0, h1, e1);
        const v8i t = e1;   // (word, half, next word) = (e0, h1, e1)
        e1 = e0;
        e2 = t;
    }
    // lane (r, g) holds rows 16 a + 4 g + v of column 16 b + r: the parities of
    // one column are the 64 bits of one output word
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        uint64_t word = 0;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                word |= (uint64_t)((uint32_t)acc[a][b][v] & 1u) << (16 * a + v);
        word <<= 4 * g;
        word ^= __shfl_xor(word, 16);
        word ^= __shfl_xor(word, 32);
        if (g == 0) red[wv][16 * b + r] = word;
    }
    __syncthreads();
    if (tid < 16 * NB) {
        uint64_t word = 0;
#pragma unroll
        for (int w = 0; w < kMmThreads / 64; ++w) word ^= red[w][tid];
        const uint64_t o = bx * (16 * NB) + (uint64_t)tid, ow = (m + 63) >> 6;
        if (o < ow) {
            if (o == ow - 1 && (m & 63)) word &= (1ull << (m & 63)) - 1ull;
            if (!jd.merge) out[o] = word;
            else if (word) atomicXor((unsigned long long*)&out[o], (unsigned long long)word);
        }
    }
}

// Selected outputs idx[g] (g < count), bit g of res: each thread walks the
// seed from its own offset (global reads), the key words come from LDS.
__global__ void __launch_bounds__(kDirectThreads)
k_direct_select(const uint32_t* __restrict__ seed32, uint64_t sw32, const uint32_t* __restrict__ kr, uint64_t kw4,
                uint64_t k_base, uint32_t kc, const uint64_t* __restrict__ idx, uint32_t count,
                uint64_t* __restrict__ res) {
    __shared__ __align__(16) uint32_t K[kDirectChunk];
    const int tid = threadIdx.x;
    const uint64_t k0 = k_base + (uint64_t)blockIdx.y * kc;
    const uint32_t nk = (uint32_t)(kw4 - k0 < kc ? kw4 - k0 : kc);
    for (uint32_t q = tid; q < nk; q += kDirectThreads) K[q] = kr[k0 + q];
    __syncthreads();
    const uint32_t g = blockIdx.x * kDirectThreads + (uint32_t)tid;
    const bool valid = g < count;
    const uint64_t i = valid ? idx[g] : 0ull;
    const uint64_t w0 = (i >> 5) + k0;
    const uint32_t sh = (uint32_t)i & 31u;
    auto ld = [&](uint64_t q) -> uint32_t { return q < sw32 ? seed32[q] : 0u; };
    uint32_t lo = ld(w0), acc = 0u;
    for (uint32_t kk = 0; kk < nk; kk += 4) {
        const uint32_t h0 = ld(w0 + kk + 1), h1 = ld(w0 + kk + 2), h2 = ld(w0 + kk + 3), h3 = ld(w0 + kk + 4);
        const uint4 kv = *reinterpret_cast<const uint4*>(&K[kk]);
        acc ^= __builtin_amdgcn_alignbit(h0, lo, sh) & kv.x;
        acc ^= __builtin_amdgcn_alignbit(h1, h0, sh) & kv.y;
        acc ^= __builtin_amdgcn_alignbit(h2, h1, sh) & kv.z;
        acc ^= __builtin_amdgcn_alignbit(h3, h2, sh) & kv.w;
        lo = h3;
    }
    const bool bit = valid && (__popc(acc) & 1);
    const unsigned long long bal = __ballot(bit);
    const uint32_t g0 = blockIdx.x * kDirectThreads + (uint32_t)(tid & ~63);
    if ((tid & 63) == 0 && bal) atomicXor((unsigned long long*)&res[g0 >> 6], bal);
}

__global__ void __launch_bounds__(kDirectThreads)
k_xor_words(uint64_t* dst, const uint64_t* src, uint64_t words) {   // src may be dst (clears it)
    const uint64_t g = (uint64_t)blockIdx.x * kDirectThreads + threadIdx.x;
    if (g < words) dst[g] ^= src[g];
}

// Certificates to pinned host memory, then the flag that the host polls: one
// small kernel in place of a copy (its own blit kernel), an event and the
// event's queries (3 empty kernels and the read-back: 22.5 us per call with the
// copy and the event, 17.8 with this).  It starts after the kernels before it on
// the stream have ended, so their results are in place when the flag is seen.
__global__ void __launch_bounds__(kDirectThreads)
k_publish(const uint4* __restrict__ src, uint4* __restrict__ host, uint32_t count, uint32_t* flag, uint32_t seq) {
    for (uint32_t k = threadIdx.x; k < count; k += kDirectThreads) host[k] = src[k];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

int launch_publish(const void* src, void* host, uint32_t count, uint32_t* flag, uint32_t seq, void* stream) {
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(kDirectThreads), 0, (hipStream_t)stream, (const uint4*)src, (uint4*)host,
                       count, flag, seq);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

static uint64_t cdiv(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

int launch_xor_words(uint64_t* dst, const uint64_t* src, uint64_t words, void* stream) {
    if (words == 0) return 0;
    hipLaunchKernelGGL(k_xor_words, dim3((uint32_t)cdiv(words, kDirectThreads)), dim3(kDirectThreads), 0,
                       (hipStream_t)stream, dst, src, words);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

uint64_t direct_key_words(uint64_t n) { return cdiv(cdiv(n, 32), 4) * 4; }

// Grid slabs: at most 2^20 workgroups along x and 2^15 along y per launch.
constexpr uint64_t kSlabX = 1ull << 20, kSlabY = 1ull << 15;
// Workgroups of one batched launch, at most: a launch counts the work-items along a
// dimension in 32 bits, and drops those beyond without an error.
constexpr uint64_t kMmBatchWgs = 0xFFFFFFFFull / kMmThreads;

// Column blocks of a tile: 1024 NB outputs.  A step of 128 key bits takes
// about 92, 128 and 256 cycles of a SIMD at NB = 1, 2, 4 (operand preparation
// bounds the first, the matrix cores the others).
static int mm_blocks(uint64_t m) {
    int best = 1;
    double cost = 1e300;
    for (int nb : {1, 2, 4}) {
        const double c = (double)cdiv(m, 1024 * nb) * (nb == 1 ? 92.0 : nb == 2 ? 128.0 : 256.0);
        if (c < cost) cost = c, best = nb;
    }
    return best;
}

// Grid of one job: K groups of `seg` words.  The number is odd, so that the LDS
// reads of a wave's K groups start on different banks.
static uint64_t mm_words(uint64_t n, int nb) { return cdiv(n, 32) + 2 * (16 * (uint64_t)nb - 1); }
static uint32_t mm_seg(uint64_t words_per_group) {
    return (uint32_t)std::min<uint64_t>(std::max<uint64_t>(kMmMinSeg, words_per_group) | 1, kMmMaxSeg);
}
static uint64_t mm_chunks(uint64_t n, int nb, uint32_t seg) { return cdiv(mm_words(n, nb), (uint64_t)seg * kMmStreams); }
// Workgroups that a launch aims at when the outputs alone do not fill the
// device, and at most: two of 8 waves per CU, one round of the device.
constexpr uint64_t kMmTarget = 512;

template <int NB>
static int mm_launch(dim3 grid, const DirectJob& one, const DirectJob* many, uint32_t njobs, uint64_t x0, uint64_t y0,
                     hipStream_t s, uint64_t* launches) {
    hipLaunchKernelGGL((k_direct_mm<NB>), grid, dim3(kMmThreads), 0, s, one, many, njobs, x0, y0);
    if (hipGetLastError() != hipSuccess) return -1;
    *launches += 1;
    return 0;
}
static int mm_launch_nb(int nb, dim3 grid, const DirectJob& one, const DirectJob* many, uint32_t njobs, uint64_t x0,
                        uint64_t y0, hipStream_t s, uint64_t* launches) {
    return nb == 1   ? mm_launch<1>(grid, one, many, njobs, x0, y0, s, launches)
           : nb == 2 ? mm_launch<2>(grid, one, many, njobs, x0, y0, s, launches)
                     : mm_launch<4>(grid, one, many, njobs, x0, y0, s, launches);
}

static DirectJob mm_single(const uint64_t* seed, const uint64_t* key, uint64_t n, uint64_t m, uint64_t* out, int* nb) {
    *nb = mm_blocks(m);
    const uint64_t bx = cdiv(m, 1024 * (uint64_t)*nb), want_y = std::max<uint64_t>(1, kMmTarget / bx);
    DirectJob j{};
    j.seed = seed;
    j.key = key;
    j.out = out;
    j.n = n;
    j.m = m;
    j.seg = mm_seg(cdiv(mm_words(n, *nb), want_y * kMmStreams));
    j.merge = mm_chunks(n, *nb, j.seg) > 1 ? 1u : 0u;
    return j;
}

int launch_direct_prep(uint64_t n, uint64_t m, uint64_t* out, void* stream, uint64_t* launches) {
    int nb;
    if (!mm_single(nullptr, nullptr, n, m, out, &nb).merge) return 0;
    if (launch_xor_words(out, out, cdiv(m, 64), stream)) return -1;
    *launches += 1;
    return 0;
}

int launch_direct_main(const uint64_t* seed, const uint64_t* key, uint64_t n, uint64_t m, uint64_t* out, void* stream,
                       uint64_t* launches) {
    int nb;
    const DirectJob j = mm_single(seed, key, n, m, out, &nb);
    const uint64_t bx = cdiv(m, 1024 * (uint64_t)nb), by = mm_chunks(n, nb, j.seg);
    for (uint64_t x0 = 0; x0 < bx; x0 += kSlabX)
        for (uint64_t y0 = 0; y0 < by; y0 += kSlabY) {
            const dim3 grid((uint32_t)std::min(kSlabX, bx - x0), (uint32_t)std::min(kSlabY, by - y0));
            if (mm_launch_nb(nb, grid, j, nullptr, 0, x0, y0, (hipStream_t)stream, launches)) return -1;
        }
    return 0;
}

// Clears the outputs of the jobs that several workgroups merge into.
__global__ void __launch_bounds__(kDirectThreads) k_direct_clear(const DirectJob* __restrict__ many) {
    const DirectJob jd = many[blockIdx.x];
    if (!jd.merge) return;
    const uint64_t ow = (jd.m + 63) >> 6;
    for (uint64_t o = threadIdx.x; o < ow; o += kDirectThreads) jd.out[o] = 0ull;
}

uint64_t direct_batch_plan(DirectJob* jobs, uint32_t count, DirectBatch* plan) {
    // order by column blocks; K groups sized so that all jobs together give
    // about four times the workgroups of a single job
    std::stable_sort(jobs, jobs + count, [](const DirectJob& a, const DirectJob& b) { return mm_blocks(a.m) < mm_blocks(b.m); });
    uint64_t total = 0;   // tile words
    for (uint32_t k = 0; k < count; ++k) {
        const int nb = mm_blocks(jobs[k].m);
        total += cdiv(jobs[k].m, 1024 * (uint64_t)nb) * mm_words(jobs[k].n, nb);
    }
    const uint32_t seg = mm_seg(cdiv(total, 4 * kMmTarget * kMmStreams));
    *plan = DirectBatch{};
    uint64_t taken = 0;
    for (int i = 0; i < 3; ++i) {
        uint64_t wgs = 0;
        plan->first[i] = (uint32_t)taken;
        for (; taken < count && mm_blocks(jobs[taken].m) == 1 << i; ++taken) {
            DirectJob& j = jobs[taken];
            const uint64_t bx = cdiv(j.m, 1024ull << i), by = mm_chunks(j.n, 1 << i, seg);
            if (bx > kSlabX || by > kSlabX || wgs + bx * by > kMmBatchWgs) return 0;
            j.seg = seg;
            j.bx = (uint32_t)bx;
            j.wg_begin = (uint32_t)wgs;
            j.merge = by > 1 ? 1u : 0u;
            plan->clears |= j.merge;
            wgs += bx * by;
        }
        plan->jobs[i] = (uint32_t)taken - plan->first[i];
        plan->wgs[i] = (uint32_t)wgs;
    }
    return taken;
}

int launch_direct_batch(const DirectBatch& plan, const DirectJob* many, uint32_t count, void* stream,
                        uint64_t* launches) {
    hipStream_t s = (hipStream_t)stream;
    if (plan.clears) {
        hipLaunchKernelGGL(k_direct_clear, dim3(count), dim3(kDirectThreads), 0, s, many);
        if (hipGetLastError() != hipSuccess) return -1;
        *launches += 1;
    }
    for (int i = 0; i < 3; ++i)
        if (plan.jobs[i] && mm_launch_nb(1 << i, dim3(plan.wgs[i]), DirectJob{}, many + plan.first[i], plan.jobs[i], 0, 0,
                                         s, launches))
            return -1;
    return 0;
}

int launch_direct_select(const uint64_t* seed, const uint64_t* key, uint64_t n, uint64_t m, const uint64_t* idx,
                         uint32_t count, uint64_t* res, uint32_t* kr, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const uint64_t kw4 = direct_key_words(n), rw = cdiv(count, 64), sw32 = 2 * cdiv(n + m - 1, 64);
    const uint64_t prep = std::max(kw4, rw);
    hipLaunchKernelGGL(k_direct_prep, dim3((uint32_t)cdiv(prep, kDirectThreads)), dim3(kDirectThreads), 0, s, key, n,
                       kr, kw4, res, rw);
    if (hipGetLastError() != hipSuccess) return -1;
    const uint64_t bx = cdiv(count, kDirectThreads);   // count <= 2^20
    const uint64_t want_y = std::max<uint64_t>(1, cdiv(2048, bx));
    uint64_t kc = std::max<uint64_t>(256, cdiv(kw4, want_y));
    kc = std::min<uint64_t>(cdiv(kc, 4) * 4, kDirectChunk);
    const uint64_t by = cdiv(kw4, kc);
    for (uint64_t y0 = 0; y0 < by; y0 += kSlabY) {
        const dim3 grid((uint32_t)bx, (uint32_t)std::min(kSlabY, by - y0));
        hipLaunchKernelGGL(k_direct_select, grid, dim3(kDirectThreads), 0, s, (const uint32_t*)seed, sw32,
                           (const uint32_t*)kr, kw4, y0 * kc, (uint32_t)kc, idx, count, res);
        if (hipGetLastError() != hipSuccess) return -1;
    }
    return 0;
}

}  // namespace pa
