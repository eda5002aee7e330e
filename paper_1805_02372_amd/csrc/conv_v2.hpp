// Tile pipeline of the power-of-two FFT length classes from 2^15 on and of the
// mixed-radix ones from 2^20 on: the same three passes as conv_kernels.hpp (see
// there for the mathematics), restructured around wave-level transforms
// (wave_fft.hpp):
//
//  * pass 1, rows of 4096 and 8192: a small kernel transposes the key and seed bits
//    into bit planes, and the columns are split into 3 to 8 parts whose first radix
//    level is looked up from the bits; each wave transforms G columns of a part in
//    registers (FP32 2^20 and 2^21: G whole columns, with the bits as inputs).  Rows
//    of 512: the bits are staged through LDS and each wave transforms G whole
//    columns.  An LDS transpose turns the column-major results into C-element row
//    segments for the stores.
//  * pass 2: a row of 4096 points is a radix-8 stage across the 8 waves
//    (decimation in frequency, registers only) followed by one 512-point transform
//    per wave; the inverse runs the same steps in reverse.  Two workgroup barriers
//    per row transform.  The products of a group's chunks are summed before the
//    inverse.  Rows of 512 are one wave's.
//  * pass 3: C columns are read as C-element row segments, transposed in LDS, each
//    wave inverts G columns, the output bits are gathered in an LDS array and stored
//    as C-bit groups.
#pragma once
#include <type_traits>

#include "conv_kernels.hpp"
#include "wave_fft.hpp"

namespace pa {

// Lengths below 2^20 are bound by latency (one tile fills a fraction of the
// device), so their rows are 512 points, one wave each and without barriers, and
// their column workgroups small.  Against workgroup-wide passes on 512 x 512 (64
// column workgroups, rows of 1-2 waves with barriers): FP64 2^18, one tile,
// passes 11.8 + 10.9 + 12.5 -> 10.0 + 7.6 + 7.8 us, call 41.4 -> 36.0 us; four
// FP32 tiles of 2^19, 18.9 + 17.6 + 14.9 -> 22.4 + 17.0 + 9.4 us (summed, one
// pass 3), call 62.7 -> 57.5 us.
//
// Column blocks.  A wave takes G columns (or one half of a column), a workgroup
// as many waves, up to 8, as make row segments of 128 bytes (rows of 512, whose
// launches seldom fill the device: 64 bytes, twice the workgroups).
template <typename T, int N1> constexpr int column_target() { return (N1 >= 4096 ? 128 : 64) / (int)sizeof(cx<T>); }
constexpr int column_waves(int target, int g) { return target <= g ? 1 : (target / g > 8 ? 8 : target / g); }

// Whole columns: a column is one transform.
template <typename T, int N1, int N2> struct P1Geom {
    static constexpr int P = 1, M = N2, G = 1024 / M;      // columns per wave
    static constexpr int WAVES = column_waves(column_target<T, N1>(), G);
    static constexpr int C = WAVES * G;                    // columns per workgroup
    static constexpr int THREADS = WAVES * 64;
    static_assert(M <= 1024 && C <= 64 && (C & (C - 1)) == 0, "column block");
};

template <typename T, int N1, int N2> struct P3Geom {
    static constexpr int M = N2 / 2;                       // Hermitian half
    static constexpr int G = 1024 / M;
    static constexpr int CT = N1 >= 4096 ? 16 : 8;         // output groups of 8 bits and more
    static constexpr int WAVES = (sizeof(T) == 4 && G == 1) ? 16 : column_waves(CT, G);
    static constexpr int C = WAVES * G;
    static constexpr int THREADS = WAVES * 64;
    static constexpr int CW = (C + 31) / 32;               // 32-bit words per output row
    static constexpr int SLOTS = (WAVES * kWaveSlots > M * C) ? WAVES * kWaveSlots : M * C;
    // LDS with the stage tables and Hermitian twiddles copied in (the twiddles
    // share space with the output bit array) vs without; copy them when a CU
    // still holds its waves, or as many workgroups as without them.
    static constexpr int WPE = sizeof(T) == 4 ? 4 : 2;     // waves per SIMD that the registers allow
    static constexpr size_t kBits = (size_t)WAVES * 64 * 4;   // 32 output bits per lane
    static constexpr size_t kHtw = (size_t)M * sizeof(cx<T>);
    static constexpr size_t kBase = (size_t)SLOTS * sizeof(cx<T>) + C * sizeof(T) + 64;
    static constexpr size_t kWithout = kBase + kBits;
    static constexpr size_t kWith = kBase + (kBits > kHtw ? kBits : kHtw) + wfft_lds_entries(M) * sizeof(cx<T>);
    static constexpr bool LDS_TAB =
        kWith <= 163840 && (kWith * (4 * WPE / WAVES) <= 180000 || (163840 / kWith) >= (163840 / kWithout));
};

// Transposition tile: row k2 of C elements, columns XOR-swizzled by the row.
template <int C> __device__ __forceinline__ int tslot(int k, int f) { return k * C + (f ^ (k & (C - 1))); }

// ------------------------------------------------------------------ FP64 roots
// Four-step twiddles are formed as FP64 products of two-level tables and
// rounded once to the working precision: w_L^e = fa64[e >> fshift] fb64[e & mask].
struct Root64 {
    double re, im;
};
__device__ __forceinline__ Root64 mul64(Root64 a, Root64 b) {
    return Root64{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ Root64 root64(const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64,
                                         int fshift, uint32_t e) {
    const cx<double> a = fa64[e >> fshift], b = fb64[e & ((1u << fshift) - 1u)];
    return Root64{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T> __device__ __forceinline__ cx<T> rounded(Root64 w) { return cx<T>{(T)w.re, (T)w.im}; }

// ------------------------------------------------------------------ pass 1
// What a tile transforms: two bit sequences, the real and the imaginary part.
// An ordinary tile has a key chunk and its seed slice; the tiles of a job with
// shared spectra (SharedJob) have two key chunks or two seed slices.
//
// Position t (mod L) of a sequence holds source bit j0 + ((t + off) mod L) when
// that index is below len: a key chunk (off = bi - 1: placed so that the kept
// window starts at index 0) or a seed slice (off = 0).  Key bits are the values
// 0 and 1, seed bits -1 and 1, and 0 from position len on.
struct BitSeq {
    const uint64_t* src;
    uint64_t nw, j0;       // source words, first bit
    uint32_t off, len;
    bool seed;
};
struct TileBits {
    BitSeq s[2];
};
__device__ __forceinline__ BitSeq key_seq(const JobDesc& jd, uint64_t j0, uint64_t bi) {
    return BitSeq{jd.key, (jd.n + 63) >> 6, j0, bi ? (uint32_t)(bi - 1) : 0u, (uint32_t)bi, false};
}
__device__ __forceinline__ BitSeq seed_seq(const JobDesc& jd, uint64_t j0, uint64_t len) {
    return BitSeq{jd.seed, (jd.n + jd.m - 1 + 63) >> 6, j0, 0u, (uint32_t)len, true};
}
// Tile lt of a shared-spectra launch: key packs (chunks 2 lt, 2 lt + 1 of the
// group), then seed packs (slices b0 + 2 q, b0 + 2 q + 1).
__device__ __forceinline__ TileBits shared_bits(const JobTable& jt, uint32_t lt) {
    const JobDesc& jd = jt.one;
    const SharedJob& sh = jt.shared;
    TileBits r;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (lt < sh.kpacks) {
            const uint32_t c = 2 * lt + h;
            uint64_t lo = 0, bi = 0;
            if (c < sh.chunks) {
                const uint64_t hi = jd.n - (uint64_t)(sh.chunk0 + c) * jd.Bi;
                lo = hi > jd.Bi ? hi - jd.Bi : 0;
                bi = hi - lo;
            }
            r.s[h] = key_seq(jd, lo, bi);
        } else {
            const uint64_t at = (uint64_t)(sh.chunk0 + 2 * (lt - sh.kpacks) + h) * jd.Bi, all = jd.n + jd.m - 1;
            const uint64_t left = at < all ? all - at : 0, most = 2 * jd.Bi - 1;
            r.s[h] = seed_seq(jd, left ? at : 0, left < most ? left : most);
        }
    }
    return r;
}
__device__ __forceinline__ TileBits tile_bits(const JobDesc& jd, const TileGeo& g) {
    TileBits r;
    r.s[0] = key_seq(jd, g.j0, g.bi);
    r.s[1] = seed_seq(jd, g.sigma, g.bi + g.bo - 1);
    return r;
}

// Bit planes.  Columns of N2 = P M rows are split into P transforms of M points
// (k2_pass1_split), on the bits of rows e, e + M, .. together, and a lane has
// points e = j + NJ i (i < 16, NJ = M / 16 lanes per column); read in place, each
// of its bits is in another word, N1 bits apart.  k2_bits transposes the two
// sequences of every tile into planes after the launch's tiles in the workspace:
// per column NJ words of 16 fields of FW (4 or 8) bits, bit FW i + q of word j of
// column t1 being position t1 + N1 (j + NJ i + M q).  A lane of pass 1 then loads
// one word of each plane, a wave consecutive ones.
// P = 4 or 8 leaves M = 64 .. 256, two radix stages for the wave (n2 = 4096, FP64
// 2^24: P = 4 and M = 1024, three stages).
// Whole columns (P = 1, M = N2, k2_pass1_whole): a lane's 16 points are 16 bits.
constexpr int column_parts(int n2) { return odd_part(n2) > 1 ? odd_part(n2) : n2 == 2048 ? 8 : 4; }
template <int N1, int N2, int P_ = column_parts(N2)> struct BitPlanes {
    static constexpr int P = P_, M = N2 / P, FW = P == 1 ? 1 : P <= 4 ? 4 : 8;
    static constexpr int NJ = M / 16, BITS = 16 * FW;   // bits of a lane
    struct alignas(BITS / 8) Wide {
        uint32_t w[BITS < 32 ? 1 : BITS / 32];
    };
    using Word = std::conditional_t<BITS == 16, uint16_t, Wide>;
    static constexpr size_t kColumn = (size_t)M * FW / 8, kPlane = kColumn * N1;
    // row of bit b of a column's plane bytes (N2 where the bit stands for none)
    __device__ static __forceinline__ uint32_t row(uint32_t b) {
        const uint32_t j = b / BITS, r = b % BITS, q = r % FW;
        return P == FW || q < (uint32_t)P ? j + NJ * (r / FW) + M * q : N2;
    }
    static constexpr size_t kTile = 2 * kPlane;
    template <typename T>
    __device__ static const uint8_t* base(const cx<T>* ws, uint32_t ntiles, uint32_t lt) {
        return reinterpret_cast<const uint8_t*>(ws + (size_t)ntiles * ((size_t)N1 * N2)) + (size_t)lt * kTile;
    }
};

// 64 bits of a sequence at positions p .. p + 63 (p a multiple of 64), LSB first:
// the part before the wrap to index 0, then (rarely) the part after it.  32-bit
// words throughout: on gfx950 a 64-bit shift whose amount is in the last VGPR of
// the wave's allocation takes a wrong amount now and then, when another wave is
// resident, and the compiler does not avoid that register.
struct alignas(8) Bits64 {
    uint32_t lo, hi;
};
__device__ __forceinline__ uint32_t low_mask32(int cnt) { return cnt >= 32 ? ~0u : cnt > 0 ? (1u << cnt) - 1u : 0u; }
__device__ __forceinline__ Bits64 low_bits(Bits64 x, int cnt) {
    return Bits64{x.lo & low_mask32(cnt), x.hi & low_mask32(cnt - 32)};
}
// A lane's loads of one group of 64: three words from word `at` on, clamped to
// the source, unconditional, so that a lane issues all its loads back to back.
struct Seq64 {
    uint32_t w[3], s;      // words, shift
    uint32_t u;            // index of the first bit
};
__device__ __forceinline__ Seq64 seq64(const BitSeq& q, const uint32_t* src, uint32_t last, uint32_t L, uint32_t p) {
    Seq64 r;
    r.u = p + q.off;
    if (r.u >= L) r.u -= L;
    const uint32_t b = r.u + ((uint32_t)q.j0 & 31u), at = b >> 5;
    r.s = b & 31u;
#pragma unroll
    for (uint32_t k = 0; k < 3; ++k) r.w[k] = src[at + k < last ? at + k : last];
    return r;
}
__device__ __forceinline__ Bits64 funnel(const uint32_t (&w)[3], uint32_t s) {
    return Bits64{__builtin_amdgcn_alignbit(w[1], w[0], s), __builtin_amdgcn_alignbit(w[2], w[1], s)};
}
__device__ __forceinline__ Bits64 shift_left(Bits64 x, uint32_t s) {   // 0 < s < 64
    if (s >= 32u) return Bits64{0u, x.lo << (s - 32u)};
    return Bits64{x.lo << s, __builtin_amdgcn_alignbit(x.hi, x.lo, 32u - s)};
}

// Value of lane l ^ k (k a power of two below 32).
template <int K> __device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
    if constexpr (K == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);         // quad_perm 1 0 3 2
    else if constexpr (K == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true);    // quad_perm 2 3 0 1
    else if constexpr (K == 4)   // l ^ 7, then l ^ 3
        return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else if constexpr (K == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xF, 0xF, true);   // rotate a row by 8
    else return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x401F);                                     // xor 16
}
// One step of a bit transpose: lanes l and l ^ K exchange the bits c with
// (c ^ l) & K set.
template <int K> __device__ __forceinline__ uint32_t transpose_step(uint32_t x, int lane) {
    constexpr uint32_t low = K == 1 ? 0x55555555u : K == 2 ? 0x33333333u : K == 4 ? 0x0F0F0F0Fu : K == 8 ? 0x00FF00FFu : 0xFFFFu;
    const uint32_t y = lane_xor<K>(x);
    const bool up = (lane & K) != 0;
    const uint32_t keep = up ? ~low : low, moved = __builtin_amdgcn_alignbit(y, y, up ? K : 32 - K);   // rotated by K
    return (x & keep) | (moved & ~keep);
}
// 64 x 64 bit transpose across a wave: lane r holds row r (bit c: column c) and
// gets column r (bit c: row c).
__device__ __forceinline__ Bits64 transpose64(Bits64 x, int lane) {
    // lanes l and l ^ 32: the upper half's low words for the lower half's high words
    const bool up = lane >= 32;
    const uint32_t got = __shfl_xor(up ? x.lo : x.hi, 32);
    if (up) x.lo = got;
    else x.hi = got;
    auto half = [&](uint32_t w) {
        w = transpose_step<16>(w, lane);
        w = transpose_step<8>(w, lane);
        w = transpose_step<4>(w, lane);
        w = transpose_step<2>(w, lane);
        return transpose_step<1>(w, lane);
    };
    return Bits64{half(x.lo), half(x.hi)};
}

// One wave: 64 plane bits of every column (a lane each) by kBitsCols groups of 64
// columns of one plane.  Each lane reads consecutive words of its bit's row; a
// transpose turns them into 8 plane bytes per column.  Bound by requests, as each
// lane's words and plane bytes are in lines of their own: one wide load per lane
// instead of three per column group (calls: c3 125.7 -> 124.3 us, 128 Mbit 1.821 ->
// 1.798 ms, eight stream blocks 1.546 -> 1.511 ms).
constexpr int kBitsCols = 4;
template <int N1, int N2, int P>
__global__ void __launch_bounds__(256) k2_bits(JobTable jt, uint8_t* __restrict__ planes) {
    using Pl = BitPlanes<N1, N2, P>;
    constexpr uint32_t L = (uint32_t)N1 * N2;
    constexpr int NRC = (int)Pl::kColumn / 8, NCC = N1 / 64 / kBitsCols;   // row and column blocks of a plane
    static_assert((2 * NRC * NCC) % 4 == 0 && N1 % (64 * kBitsCols) == 0, "blocks");
    const int lane = threadIdx.x & 63;
    const uint32_t wave = xcd_block() * 4 + (threadIdx.x >> 6);   // neighbours share lines on both sides
    const uint32_t rc = wave % NRC, cc = (wave / NRC) % NCC, pl = (wave / (NRC * NCC)) & 1u;
    const uint32_t lt = wave / (2 * NRC * NCC);
    TileBits tb;
    if (jt.shared.kpacks) {
        tb = shared_bits(jt, lt);
    } else {
        const JobDesc jd = find_job(jt, jt.tile0 + lt);
        tb = tile_bits(jd, tile_geo(jd, jt.tile0 + lt - jd.tile_begin));
    }
    const BitSeq q = pl ? tb.s[1] : tb.s[0];
    const uint32_t row = Pl::row(rc * 64 + lane), p0 = cc * (64 * kBitsCols) + (uint32_t)N1 * row;
    Bits64 v[kBitsCols];
    if (q.len == 0) {   // no such sequence (a pack of one)
#pragma unroll
        for (int c = 0; c < kBitsCols; ++c) v[c] = Bits64{0, 0};
    } else {
        const uint32_t* __restrict__ src = reinterpret_cast<const uint32_t*>(q.src) + (q.j0 >> 5);
        const uint64_t left = 2 * q.nw - 1 - (q.j0 >> 5);
        const uint32_t last = left < 0xFFFFFFFFull ? (uint32_t)left : 0xFFFFFFFFu;
        // the lane's 64 kBitsCols bits in consecutive words, where none of the wave's
        // lanes wraps or meets the end of the source; past the slice any words do
        constexpr uint32_t NW = 2 * kBitsCols + 1;
        struct Words {
            uint32_t w[NW];
        };
        uint32_t u = p0 + q.off;
        if (u >= L) u -= L;
        const uint32_t b = u + ((uint32_t)q.j0 & 31u), at = u < q.len && row < (uint32_t)N2 ? b >> 5 : 0u;
        const bool none = row >= (uint32_t)N2;
        const bool whole = last >= NW - 1 && (none || (at <= last - (NW - 1) && u + 64u * kBitsCols <= L));
        if (__all(whole)) {
            Words x;
            __builtin_memcpy(&x, src + at, sizeof(x));
#pragma unroll
            for (int c = 0; c < kBitsCols; ++c) {
                const uint32_t w[3] = {x.w[2 * c], x.w[2 * c + 1], x.w[2 * c + 2]};
                v[c] = low_bits(funnel(w, b & 31u), none ? 0 : (int)q.len - (int)u - 64 * c);
            }
        } else {
            Seq64 e[kBitsCols];
#pragma unroll
            for (int c = 0; c < kBitsCols; ++c) e[c] = seq64(q, src, last, L, p0 + 64u * c);
#pragma unroll
            for (int c = 0; c < kBitsCols; ++c) {
                const uint32_t fs = L - e[c].u;   // bits before the wrap
                const int left_u = (int)q.len - (int)e[c].u;
                v[c] = low_bits(funnel(e[c].w, e[c].s), left_u < (int)fs ? left_u : (int)fs);
                if (fs < 64u) {
                    const uint32_t h[3] = {src[0], src[1 < last ? 1 : last], src[2 < last ? 2 : last]};
                    const uint32_t cnt = 64u - fs < q.len ? 64u - fs : q.len;
                    const Bits64 y = shift_left(low_bits(funnel(h, (uint32_t)q.j0 & 31u), (int)cnt), fs);
                    v[c].lo |= y.lo;
                    v[c].hi |= y.hi;
                }
                if (Pl::P != Pl::FW && row >= (uint32_t)N2) v[c] = Bits64{0, 0};
            }
        }
    }
    uint8_t* dst = planes + (size_t)lt * Pl::kTile + (size_t)pl * Pl::kPlane + (size_t)rc * 8;
#pragma unroll
    for (int c = 0; c < kBitsCols; ++c)
        *reinterpret_cast<Bits64*>(dst + (size_t)(cc * (64 * kBitsCols) + 64 * c + lane) * Pl::kColumn) =
            transpose64(v[c], lane);
}

// C (at most 16) bits of a sequence at position p, a multiple of C: two words, and
// in the rare case of a wrap to index 0 the sequence's first.
struct FieldLoad {
    uint32_t w[2], s, u;
};
__device__ __forceinline__ FieldLoad field_load(const BitSeq& q, const uint32_t* src, uint32_t last, uint32_t L, uint32_t p) {
    FieldLoad r;
    r.u = p + q.off;
    if (r.u >= L) r.u -= L;
    const uint32_t b = r.u + ((uint32_t)q.j0 & 31u), at = b >> 5;
    r.s = b & 31u;
    r.w[0] = src[at < last ? at : last];
    r.w[1] = src[at + 1 < last ? at + 1 : last];
    return r;
}
template <int C>
__device__ __forceinline__ uint32_t field_bits(const BitSeq& q, const uint32_t* src, uint32_t last, uint32_t L,
                                               const FieldLoad& e) {
    const uint32_t fs = L - e.u;   // bits before the wrap
    const int left = (int)q.len - (int)e.u, cnt = left < (int)fs ? left : (int)fs;
    uint32_t x = __builtin_amdgcn_alignbit(e.w[1], e.w[0], e.s) & low_mask32(cnt < C ? cnt : C);
    if (fs < (uint32_t)C) {
        const uint32_t head = __builtin_amdgcn_alignbit(src[1 < last ? 1 : last], src[0], (uint32_t)q.j0 & 31u);
        const uint32_t most = C - fs < q.len ? C - fs : q.len;
        x |= (head & low_mask32((int)most)) << fs;
    }
    return x;
}

// What the column passes share.  LDS: the wave regions, used again as the
// transposition tile, and the stage tables.
template <typename T, typename Gm> struct ColumnSmem {
    static constexpr int SLOTS = (Gm::WAVES * kWaveSlots > Gm::M * Gm::C) ? Gm::WAVES * kWaveSlots : Gm::M * Gm::C;
    static_assert(Gm::G * 16 * sizeof(Root64) <= kWaveSlots * sizeof(cx<T>), "twiddle factors fit a wave region");
    alignas(16) cx<T> lds[SLOTS];
    alignas(16) cx<T> st[wfft_lds_entries(Gm::M)];
};
// Four-step twiddle w_L^{t1 k2}, k2 = P (j + NJ i) + h, as base * c_i with base =
// w_L^{t1 (P j + h)} and c_i = w_L^{P NJ t1 i}.  Each lane fetches its share of its
// column's 16 factors before the transform (latency hidden behind it); they are
// exchanged through LDS afterwards.
template <int NJ, int P> struct ColumnRoots {
    static constexpr int CPL = (16 + NJ - 1) / NJ;   // factors fetched per lane
    Root64 base, c[CPL];
    __device__ __forceinline__ ColumnRoots(uint32_t t1, uint32_t j, uint32_t h, const cx<double>* __restrict__ fa64,
                                           const cx<double>* __restrict__ fb64, int fshift) {
        base = root64(fa64, fb64, fshift, t1 * (P * j + h));
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            const uint32_t i = j + q * NJ;
            c[q] = root64(fa64, fb64, fshift, i < 16 ? (uint32_t)(P * NJ) * t1 * i : 0u);
        }
    }
};
// The M-point transform of a lane's column and the twiddles.
template <typename T, typename Gm, typename Roots>
__device__ __forceinline__ void column_transform(cx<T> (&v)[16], ColumnSmem<T, Gm>& S, const Roots& roots, int wv, int grp,
                                                 int j) {
    constexpr int M = Gm::M, NJ = M / 16;
    wave_fft_lds<T, -1, M>(v, S.lds + wv * kWaveSlots + grp * (M + M / 16), j, S.st);
    // exchange the factors through this wave's own region (its transform is done)
    Root64* cw = reinterpret_cast<Root64*>(S.lds + wv * kWaveSlots) + grp * 16;
    wave_sync();
#pragma unroll
    for (int q = 0; q < Roots::CPL; ++q) {
        const int i = j + q * NJ;
        if (i < 16) cw[i] = roots.c[q];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = cmul(v[i], rounded<T>(mul64(roots.base, cw[i])));
}
// Rows P k + h of the workgroup's columns, transposed through LDS for row-segment
// stores.
template <typename T, typename Gm, int N1>
__device__ __forceinline__ void column_store(const cx<T> (&v)[16], ColumnSmem<T, Gm>& S, int tid, int f, int j, uint32_t h,
                                             cx<T>* __restrict__ Y) {
    constexpr int C = Gm::C, NJ = Gm::M / 16;
    static_assert(Gm::M * C == Gm::THREADS * 16, "store tile");
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) S.lds[tslot<C>(j + i * NJ, f)] = v[i];
    __syncthreads();
    cx<T> o[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + q * Gm::THREADS;
        o[q] = S.lds[tslot<C>(idx / C, idx % C)];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + q * Gm::THREADS;
        Y[(size_t)((uint32_t)Gm::P * (uint32_t)(idx / C) + h) * N1 + (idx % C)] = o[q];
    }
}

// -1 or 1 for a seed bit (in bit 31).
template <typename T> __device__ __forceinline__ T sign_value(uint32_t top);
template <> __device__ __forceinline__ float sign_value<float>(uint32_t top) {
    return __uint_as_float((top & 0x80000000u) ^ 0xBF800000u);
}
template <> __device__ __forceinline__ double sign_value<double>(uint32_t top) {
    return __hiloint2double((int)((top & 0x80000000u) ^ 0xBFF00000u), 0);
}

// Column pass of the rows of 512: a workgroup of WAVES waves takes C columns, each
// wave transforming G of them in registers.  The bits are staged through LDS, per
// row the C key bits and the C seed bits in one word: a thread loads a row or a few
// (all their words in flight at once).  Each lane fetching its own 16 rows instead
// took four times the requests, every one to another line, and bound the pass in
// launches of many tiles: FP32 2^19, 48 tiles and more 10.6 -> 3.0 ns per 1000
// points, four tiles 22.4 -> 19.3 us.
template <typename T, int N1, int N2>
__global__ void __launch_bounds__((P1Geom<T, N1, N2>::THREADS))
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
k2_pass1(JobTable jt, cx<T>* __restrict__ ws, uint32_t* __restrict__ part, const cx<T>* __restrict__ stw,
         const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64, int fshift) {
    using Gm = P1Geom<T, N1, N2>;
    constexpr int C = Gm::C, G = Gm::G, M = Gm::M, NJ = M / 16;
    constexpr int NCB = N1 / C, ROWS = N2 / Gm::THREADS;   // rows staged by a thread
    constexpr uint32_t L = (uint32_t)N1 * N2;
    static_assert(C <= 16 && ROWS * Gm::THREADS == N2, "staged fields");
    static_assert(sizeof(cx<T>) * Gm::WAVES * kWaveSlots >= sizeof(uint32_t) * N2, "staged fields fit the wave regions");
    __shared__ ColumnSmem<T, Gm> S;
    __shared__ uint32_t wsum;

    const uint32_t blk = xcd_block(), lt = blk / NCB, cb = blk % NCB;
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63, grp = l / NJ, j = l % NJ, f = wv * G + grp;
    const uint32_t t1 = cb * C + (uint32_t)f, t = jt.tile0 + lt;
    const JobDesc jd = find_job(jt, t);
    const TileGeo g = tile_geo(jd, t - jd.tile_begin);
    const TileBits tb = tile_bits(jd, g);
    const uint32_t* src[2];
    uint32_t last[2];
    FieldLoad e[ROWS][2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        src[s] = reinterpret_cast<const uint32_t*>(tb.s[s].src) + (tb.s[s].j0 >> 5);
        const uint64_t left = 2 * tb.s[s].nw - 1 - (tb.s[s].j0 >> 5);
        last[s] = left < 0xFFFFFFFFull ? (uint32_t)left : 0xFFFFFFFFu;
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            e[r][s] = field_load(tb.s[s], src[s], last[s], L, cb * C + (uint32_t)N1 * (uint32_t)(tid + r * Gm::THREADS));
    }
    clear_window(g, cb, NCB, tid, Gm::THREADS);
    if (tid == 0) wsum = 0;
    wfft_load_lds<T, M>(S.st, stw, tid, Gm::THREADS);
    const ColumnRoots<NJ, 1> roots(t1, (uint32_t)j, 0, fa64, fb64, fshift);
    uint32_t* fld = reinterpret_cast<uint32_t*>(S.lds);
    uint32_t pc = 0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const uint32_t kb = field_bits<C>(tb.s[0], src[0], last[0], L, e[r][0]);
        fld[tid + r * Gm::THREADS] = kb | field_bits<C>(tb.s[1], src[1], last[1], L, e[r][1]) << 16;
        pc += (uint32_t)__popc(kb);
    }
    __syncthreads();  // the fields, the stage tables and the zeroed sum are in place
    atomicAdd(&wsum, pc);
    // rows of the slice in this column: ceil((len - t1) / N1)
    const uint32_t win = tb.s[1].len, rows = win > t1 ? (win - t1 + N1 - 1) / N1 : 0u;
    cx<T> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t row = (uint32_t)(j + i * NJ), w = fld[row] >> f;
        v[i] = cx<T>{(T)(w & 1u), row < rows ? sign_value<T>(w << 15) : T(0)};
    }
    __syncthreads();  // the wave regions are free
    column_transform<T, Gm>(v, S, roots, wv, grp, j);
    column_store<T, Gm, N1>(v, S, tid, f, j, 0, ws + (size_t)lt * N1 * N2 + cb * C);
    if (tid == 0) part[(size_t)lt * NCB + cb] = wsum;
}

// Column pass of FP32 2^20 and 2^21 (rows of 4096, columns of 256 and 512): whole
// columns from the bit planes, a wave transforming G of them in registers.  The
// transforms are short enough that the split below only adds to them: its lookups,
// a product per point for the split's twiddles and as many workgroups again for each
// part.  Against the split columns, per tile: 2^20 in launches of 128 tiles 3.4 ->
// 2.3 us, one tile 18.3 -> 15.0; 2^21 of 64 tiles 6.6 -> 4.7, one 24.0 -> 21.2; 2^22, whose
// columns of 1024 take three stages, 11.5 us split and 12.3 whole.
template <typename T, int N1, int N2>
__global__ void __launch_bounds__((P1Geom<T, N1, N2>::THREADS))
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
k2_pass1_whole(JobTable jt, cx<T>* __restrict__ ws, uint32_t* __restrict__ part, const cx<T>* __restrict__ stw,
               const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64, int fshift) {
    using Gm = P1Geom<T, N1, N2>;
    using Pl = BitPlanes<N1, N2, 1>;
    constexpr int C = Gm::C, G = Gm::G, M = Gm::M, NJ = M / 16;
    constexpr int NCB = N1 / C;
    __shared__ ColumnSmem<T, Gm> S;
    __shared__ uint32_t wsum;

    const uint32_t blk = xcd_block(), lt = blk / NCB, cb = blk % NCB;
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63, grp = l / NJ, j = l % NJ, f = wv * G + grp;
    const uint32_t t1 = cb * C + (uint32_t)f, t = jt.tile0 + lt;
    const uint16_t* __restrict__ pw =
        reinterpret_cast<const uint16_t*>(Pl::base(ws, jt.ntiles, lt)) + (size_t)t1 * NJ + j;
    const uint32_t key = pw[0], seed = pw[Pl::kPlane / sizeof(uint16_t)];
    const JobDesc jd = find_job(jt, t);
    const TileGeo g = tile_geo(jd, t - jd.tile_begin);
    clear_window(g, cb, NCB, tid, Gm::THREADS);
    if (tid == 0) wsum = 0;
    wfft_load_lds<T, M>(S.st, stw, tid, Gm::THREADS);
    const ColumnRoots<NJ, 1> roots(t1, (uint32_t)j, 0, fa64, fb64, fshift);
    // rows of the slice in this column; of this lane's rows j + NJ i the first `valid`
    const uint32_t len = (uint32_t)(g.bi + g.bo - 1), rows = len > t1 ? (len - t1 + N1 - 1) / N1 : 0u;
    const uint32_t valid = rows > (uint32_t)j ? (rows - (uint32_t)j + NJ - 1) / NJ : 0u;
    cx<T> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = cx<T>{(T)((key >> i) & 1u), sign_value<T>(seed << (31 - i))};
    if (__any(valid < 16u)) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((uint32_t)i >= valid) v[i].im = T(0);
    }
    __syncthreads();  // the stage tables and the zeroed sum are in place
    atomicAdd(&wsum, (uint32_t)__popc(key));
    column_transform<T, Gm>(v, S, roots, wv, grp, j);
    column_store<T, Gm, N1>(v, S, tid, f, j, 0, ws + (size_t)lt * N1 * N2 + cb * C);
    if (tid == 0) part[(size_t)lt * NCB + cb] = wsum;
}

// Column pass of the rows of 4096 and 8192: columns of N2 = P M rows by a radix-P
// split in decimation in frequency.  The outputs k2 = P k + h are the M-point
// transform of
//   w_N2^{h e} sum_q z(e + M q) w_P^{h q},
// and a workgroup makes them for one h and C columns, a wave transforming G
// columns in registers.  The sums need no arithmetic: the inputs are bits, so that
// P of them index a table of 2^P sums in LDS (of the roots in FP64, rounded once),
// one lookup per sequence; the signs +-1 of a seed are twice the sum of its bits
// less that of its rows.
// Against a workgroup-wide transform of whole columns (one workgroup of 8 waves
// per CU, 122 KB of LDS, bits staged through LDS, barriers at each stage): FP64
// L = 7 2^21, 162 -> 85 us with k2_bits (2.8 TB/s written); FP64 2^24, 171 -> 122
// us; FP32 L = 5 2^20 in groups of four tiles, 8.8 -> 5.2 ns per 1000 points with
// the row pass.  Against whole (or halved) columns a wave with the bits as inputs,
// powers of two: two FP32 tiles of 2^23, 55.6 -> 51.0 us; FP64 2^22 in fives, 130 ->
// 106 us.  Now bound by vector instructions (1,180 for 1024 FP32 points, 130 of
// them the FP64 products of the four-step twiddles: about 3/4 of the time).
template <typename T, int N1_, int N2> struct PSplitGeom {
    static constexpr int N1 = N1_, P = column_parts(N2), M = N2 / P, G = 1024 / M;
    static constexpr int WAVES = column_waves(column_target<T, N1>(), G);
    static constexpr int C = WAVES * G, THREADS = WAVES * 64;
    static_assert(P > 1 && P <= 8 && M >= 64 && M <= 1024 && C <= 64 && (C & (C - 1)) == 0, "column block");
};
// tw: w_NT^e.  SHARED: the tiles are packs of two chunks or two slices, else of a
// chunk and its slice (one kernel for both took 20 registers more, and spilled).
template <typename T, int N1, int N2, int NT, bool SHARED>
__global__ void __launch_bounds__((PSplitGeom<T, N1, N2>::THREADS))
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
k2_pass1_split(JobTable jt, cx<T>* __restrict__ ws, uint32_t* __restrict__ part, const cx<T>* __restrict__ tw,
               const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64,
               int fshift) {
    using Gm = PSplitGeom<T, N1, N2>;
    constexpr int P = Gm::P, C = Gm::C, G = Gm::G, M = Gm::M, NJ = M / 16;
    using Pl = BitPlanes<N1, N2>;
    constexpr uint32_t L = (uint32_t)N1 * N2, ALL = (1u << P) - 1u;
    constexpr int NCB = N1 / C;
    __shared__ ColumnSmem<T, Gm> S;
    __shared__ __align__(16) cx<T> sums[1 << P];
    __shared__ uint32_t wsum;

    const uint32_t blk = xcd_block(), h = blk % P, lb = blk / P;   // the P workgroups of a column block share its bits
    const uint32_t lt = lb / NCB, cb = lb % NCB;
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63, grp = l / NJ, j = l % NJ, f = wv * G + grp;
    const uint32_t t1 = cb * C + (uint32_t)f;
    const typename Pl::Word* __restrict__ pw =
        reinterpret_cast<const typename Pl::Word*>(Pl::base(ws, jt.ntiles, lt)) + (size_t)t1 * NJ + j;
    const typename Pl::Word bits[2] = {pw[0], pw[Pl::kPlane / sizeof(typename Pl::Word)]};
    uint32_t len[2] = {0, 0};
    const bool seeds = SHARED && lt >= jt.shared.kpacks;   // both sequences are slices
    if constexpr (SHARED) {
        const TileBits tb = shared_bits(jt, lt);
        len[0] = tb.s[0].len;
        len[1] = tb.s[1].len;
    } else {
        const uint32_t t = jt.tile0 + lt;
        const JobDesc jd = find_job(jt, t);
        const TileGeo g = tile_geo(jd, t - jd.tile_begin);
        if (h == 0) clear_window(g, cb, NCB, tid, Gm::THREADS);
        len[1] = (uint32_t)(g.bi + g.bo - 1);
    }
    if (tid == 0) wsum = 0;
    wfft_load_lds<T, M>(S.st, stw, tid, Gm::THREADS);
    // sums of w_P^{h q} over the bits q of the index
    for (uint32_t x = tid; x <= ALL; x += Gm::THREADS) {
        Root64 a{0, 0};
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const Root64 r = root64(fa64, fb64, fshift, (h * q) % P * (L / P));
            if ((x >> q) & 1u) a = Root64{a.re + r.re, a.im + r.im};
        }
        if (h && x == ALL) a = Root64{0, 0};
        sums[x] = rounded<T>(a);
    }
    const ColumnRoots<NJ, P> roots(t1, (uint32_t)j, h, fa64, fb64, fshift);
    cx<T> r[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) r[i] = tw[h * (uint32_t)(j + i * NJ) * (uint32_t)(NT / N2)];
    __syncthreads();  // the tables and the zeroed sum are in place
    constexpr uint32_t FM = (1u << Pl::FW) - 1u;
    constexpr int PER = 32 / Pl::FW;   // fields per 32-bit word
    // rows of a slice in this column; of the P rows of element e, the first q0, and
    // one more when e < e0.  A key's rows add nothing
    cx<T> in0[2], in1[2];
    uint32_t e0[2], pc = 0;
#pragma unroll
    for (int s = SHARED ? 0 : 1; s < 2; ++s) {
        const uint32_t rows = (!SHARED || seeds) && len[s] > t1 ? (len[s] - t1 + N1 - 1) / N1 : 0u, q0 = rows / M;
        e0[s] = rows % M;
        in0[s] = sums[(1u << q0) - 1u];
        in1[s] = sums[((1u << (q0 + 1)) - 1u) & ALL];
    }
    const T scale = !SHARED || seeds ? T(2) : T(1);
#pragma unroll
    for (int i = 0; i < Pl::BITS / 32; ++i)
        pc += (uint32_t)__popc(bits[0].w[i]) + (SHARED ? (uint32_t)__popc(bits[1].w[i]) : 0u);
    if (h == 0 && !seeds) atomicAdd(&wsum, pc);
    cx<T> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        cx<T> x[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const cx<T> a = sums[(bits[s].w[i / PER] >> (Pl::FW * (i % PER))) & FM];
            if (!SHARED && s == 0) {
                x[s] = a;
            } else {
                const cx<T> in = (uint32_t)(j + i * NJ) < e0[s] ? in1[s] : in0[s];
                x[s] = cx<T>{scale * a.re - in.re, scale * a.im - in.im};
            }
        }
        v[i] = cmul(cx<T>{x[0].re - x[1].im, x[0].im + x[1].re}, r[i]);   // first + i second
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // a few lookups in flight, not all (registers)
    }
    column_transform<T, Gm>(v, S, roots, wv, grp, j);
    column_store<T, Gm, N1>(v, S, tid, f, j, h, ws + (size_t)lt * L + cb * C);
    if (tid == 0 && h == 0) part[(size_t)lt * NCB + cb] = wsum;
}

// ------------------------------------------------------------------ pass 2
// Row pass.  A workgroup transforms rows of N1 points, PT per lane, in W =
// N1 / (64 PT) waves: a radix-W stage across the waves (decimation in frequency,
// registers only), one workgroup exchange, one transform of M = 64 PT points per
// wave; the inverse runs the same steps in reverse.  Two workgroup barriers per
// row transform.  Rows of 4096 take 8 points per lane (8 x 8 x 8 x 8: a mirror
// pair and the group's sum are 48 registers per lane in FP32, so that two
// workgroups of 8 waves share a CU, at 128 registers with 17 to 22 spilled); rows of 8192 take 16 (8 x 4 x 16 x 16), rows
// of 512 are one wave's (8 x 8 x 8, no barriers).
template <typename T, int N1> struct RowGeom {
    static constexpr int PT = N1 >= 8192 ? 16 : 8;
    static constexpr int W = N1 / (64 * PT), M = 64 * PT, S = PT / W, THREADS = N1 / PT;
    static constexpr int SLOTS = M + M / (PT == 16 ? 16 : 8);   // LDS slots of a wave's region
    static_assert(W >= 1 && W <= 8 && S * W == PT, "row geometry");
    __device__ static __forceinline__ int slot(int e) { return PT == 16 ? e + (e >> 4) : e + (e >> 3); }
};

// A lane's points of one row.
template <typename T, int N1> using RowVec = cx<T>[RowGeom<T, N1>::PT];

// Shared memory: the row exchange / wave regions; rows of 4096 the second
// stage's twiddles w_64^{k r} at st[8 (r - 1) + k]; rows of 8192 the stage tables
// of the 1024-point transforms.
template <typename T, int N1> struct RowSmem {
    using G = RowGeom<T, N1>;
    static_assert(G::PT == 8 || sizeof(T) == 4, "FP64 rows are 4096 points");
    cx<T> data[G::W * G::SLOTS];
    cx<T> st[G::PT == 16 ? wfft_lds_entries(1024) : 7 * 8];
};

// Twiddles of a lane held in registers for the whole pass (both directions use
// the same ones): first stage w_N1^{ka nb}, nb = tid + THREADS s, at tw1[s (W-1)
// + ka - 1]; rows of 4096 also the last stage, w_512^{l r} at t3[r - 1].
template <typename T, int N1> struct RowReg {
    using G = RowGeom<T, N1>;
    cx<T> tw1[G::W > 1 ? G::S * (G::W - 1) : 1];
    cx<T> t3[G::PT == 8 ? 7 : 1];
};

// The same twiddles in LDS (kernels whose registers are taken): a lane reads its own
// entries, 512 or 64 apart.
template <typename T, int N1> struct RowTwiddles {
    using G = RowGeom<T, N1>;
    cx<T> tw1[G::S * (G::W - 1) * G::THREADS], t3[7 * 64];
};
template <typename T, int STRIDE> struct LdsLane {
    const cx<T>* p;
    __device__ __forceinline__ cx<T> operator[](int i) const { return p[i * STRIDE]; }
};
template <typename T, int N1> struct RowLds {
    LdsLane<T, RowGeom<T, N1>::THREADS> tw1;
    LdsLane<T, 64> t3;
};

// tw: w_NT^e, NT = max(n1, n2)
template <typename T, int N1, int N2>
__device__ __forceinline__ void row_setup(RowSmem<T, N1>& S, RowReg<T, N1>& R, const cx<T>* __restrict__ tw,
                                          const cx<T>* __restrict__ stw, int tid) {
    using G = RowGeom<T, N1>;
    constexpr int STEP = cmax<N1, N2>() / N1;
#pragma unroll
    for (int s = 0; s < G::S; ++s)
#pragma unroll
        for (int ka = 1; ka < G::W; ++ka) R.tw1[s * (G::W - 1) + ka - 1] = tw[STEP * ka * (tid + G::THREADS * s)];
    if constexpr (G::PT == 8) {
        const int l = tid & 63;
#pragma unroll
        for (int r = 1; r < 8; ++r) R.t3[r - 1] = tw[STEP * l * r * (N1 / 512)];
        if (tid < 56) S.st[tid] = tw[STEP * (tid & 7) * ((tid >> 3) + 1) * (N1 / 64)];
    } else {
        wfft_load_lds<T, 1024>(S.st, stw, tid, G::THREADS);
    }
    __syncthreads();
}

// Transform of M points by one wave, register i holding element l + 64 i before
// and after; `reg` is the wave's own LDS region.  512 points: three Stockham
// stages of radix 8 (wave_fft.hpp holds the 1024-point transform).
template <typename T, int N1, int DIR, typename Reg>
__device__ __forceinline__ void row_wave_fft(RowVec<T, N1>& v, cx<T>* __restrict__ reg, int l,
                                             const RowSmem<T, N1>& S, const Reg& R) {
    if constexpr (RowGeom<T, N1>::PT == 16) {
        wave_fft_lds<T, DIR, 1024>(v, reg, l, S.st);
    } else {
        dft8<DIR>(v);
        wave_sync();
        // span 1: butterfly l writes 8 l + r (slot 9 l + r); lanes read l + 64 i
        cx<T>* __restrict__ w1 = reg + 9 * l;
        cx<T>* __restrict__ rd = reg + l + (l >> 3);
#pragma unroll
        for (int r = 0; r < 8; ++r) w1[r] = v[r];
        wave_sync();
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = rd[72 * i];
#pragma unroll
        for (int r = 1; r < 8; ++r) v[r] = twmul<DIR>(v[r], S.st[8 * (r - 1) + (l & 7)]);
        dft8<DIR>(v);
        wave_sync();
        // span 8: butterfly l writes 64 (l / 8) + l mod 8 + 8 r
        cx<T>* __restrict__ w2 = reg + 72 * (l >> 3) + (l & 7);
#pragma unroll
        for (int r = 0; r < 8; ++r) w2[9 * r] = v[r];
        wave_sync();
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = rd[72 * i];
#pragma unroll
        for (int r = 1; r < 8; ++r) v[r] = twmul<DIR>(v[r], R.t3[r - 1]);
        dft8<DIR>(v);
        wave_sync();
    }
}

// a[s W + na] = row[nb + M na], nb = tid + THREADS s
template <typename T, int N1>
__device__ __forceinline__ void row_load(RowVec<T, N1>& a, const cx<T>* __restrict__ row, int tid) {
    using G = RowGeom<T, N1>;
#pragma unroll
    for (int s = 0; s < G::S; ++s)
#pragma unroll
        for (int na = 0; na < G::W; ++na) a[s * G::W + na] = row[tid + G::THREADS * s + G::M * na];
}

// Forward transform of a row loaded by row_load: lane l of wave w ends with
// X[W k_b + w] in register i, k_b = l + 64 i.
template <typename T, int N1, typename Reg>
__device__ __forceinline__ void row_forward(RowVec<T, N1>& a, RowSmem<T, N1>& S, const Reg& R,
                                            int tid) {
    using G = RowGeom<T, N1>;
    const int wv = tid >> 6, l = tid & 63;
    if constexpr (G::W == 1) {   // one wave: the loaded order is the transform's
        row_wave_fft<T, N1, -1>(a, S.data, l, S, R);
        return;
    }
#pragma unroll
    for (int s = 0; s < G::S; ++s) {
        dft<G::W, -1>(&a[s * G::W]);
#pragma unroll
        for (int ka = 1; ka < G::W; ++ka) a[s * G::W + ka] = cmul(a[s * G::W + ka], R.tw1[s * (G::W - 1) + ka - 1]);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < G::S; ++s)
#pragma unroll
        for (int ka = 0; ka < G::W; ++ka) S.data[ka * G::SLOTS + G::slot(tid + G::THREADS * s)] = a[s * G::W + ka];
    __syncthreads();
    cx<T>* reg = S.data + wv * G::SLOTS;
#pragma unroll
    for (int i = 0; i < G::PT; ++i) a[i] = reg[G::slot(l) + G::slot(64) * i];
    wave_sync();
    row_wave_fft<T, N1, -1>(a, reg, l, S, R);
}

// Inverse transform of a row held as P[W k_b + w] (register i, k_b = l + 64 i);
// ends with a[t_b + M t_a] in a[s W + t_a], t_b = tid + THREADS s.
template <typename T, int N1, typename Reg>
__device__ __forceinline__ void row_inverse(RowVec<T, N1>& a, RowSmem<T, N1>& S, const Reg& R,
                                            int tid) {
    using G = RowGeom<T, N1>;
    const int wv = tid >> 6, l = tid & 63;
    cx<T>* reg = S.data + wv * G::SLOTS;
    if constexpr (G::W == 1) {
        wave_sync();
        row_wave_fft<T, N1, +1>(a, reg, l, S, R);
        return;
    }
    __syncthreads();  // every wave is done with its region
    row_wave_fft<T, N1, +1>(a, reg, l, S, R);
    wave_sync();   // the wave's own region: no other wave uses it until the barrier below
#pragma unroll
    for (int i = 0; i < G::PT; ++i) reg[G::slot(l) + G::slot(64) * i] = a[i];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < G::S; ++s) {
#pragma unroll
        for (int ka = 0; ka < G::W; ++ka) a[s * G::W + ka] = S.data[ka * G::SLOTS + G::slot(tid + G::THREADS * s)];
#pragma unroll
        for (int ka = 1; ka < G::W; ++ka) a[s * G::W + ka] = cmulc(a[s * G::W + ka], R.tw1[s * (G::W - 1) + ka - 1]);
        dft<G::W, +1>(&a[s * G::W]);
    }
}

// Replace X (row layout of row_forward) by the values at the mirrored
// frequency: -k mod N1 when `zero`, else N1 - 1 - k.
template <typename T, int N1>
__device__ __forceinline__ void row_mirror(RowVec<T, N1>& X, cx<T>* lds, int tid, bool zero) {
    using G = RowGeom<T, N1>;
    const int wv = tid >> 6, l = tid & 63;
    wave_sync();   // X was produced in the wave's own region, which no other wave touches
#pragma unroll
    for (int i = 0; i < G::PT; ++i) lds[wv * G::SLOTS + G::slot(l) + G::slot(64) * i] = X[i];
    if constexpr (G::W == 1) wave_sync();
    else __syncthreads();
    const int sw = zero ? ((G::W - wv) & (G::W - 1)) : (G::W - 1 - wv);
#pragma unroll
    for (int i = 0; i < G::PT; ++i) {
        const int kb = l + 64 * i;
        const int sb = (zero && wv == 0) ? ((G::M - kb) & (G::M - 1)) : (G::M - 1 - kb);
        X[i] = lds[sw * G::SLOTS + G::slot(sb)];
    }
}

// Store V row `row` (inverse four-step twiddle w_L^{-row t1}): t1 = x + M ta
// with x = tid + THREADS s, so w_L^{row t1} = w_L^{row x} w_L^{M row ta}, an FP64
// product rounded once.  `real`: keep the real part only.
template <typename T, int N1>
__device__ __forceinline__ void row_store(cx<T>* __restrict__ Yrow, RowVec<T, N1>& a, uint32_t row,
                                          bool real, int tid, const cx<double>* __restrict__ fa64,
                                          const cx<double>* __restrict__ fb64, int fshift) {
    using G = RowGeom<T, N1>;
    if constexpr (sizeof(T) == 8) {
        // FP64 (register-bound): one table product per point
#pragma unroll
        for (int s = 0; s < G::S; ++s)
#pragma unroll
            for (int ta = 0; ta < G::W; ++ta) {
                const uint32_t t1 = (uint32_t)(tid + G::THREADS * s + G::M * ta);
                cx<T> vv = cmulc(a[s * G::W + ta], rounded<T>(root64(fa64, fb64, fshift, row * t1)));
                if (real) vv.im = T(0);
                Yrow[t1] = vv;
            }
        return;
    }
    Root64 b[G::S];
#pragma unroll
    for (int s = 0; s < G::S; ++s) b[s] = root64(fa64, fb64, fshift, row * (uint32_t)(tid + G::THREADS * s));
#pragma unroll
    for (int ta = 0; ta < G::W; ++ta) {
        Root64 c{1.0, 0.0};
        if (ta) c = root64(fa64, fb64, fshift, (uint32_t)G::M * row * (uint32_t)ta);
#pragma unroll
        for (int s = 0; s < G::S; ++s) {
            cx<T> vv = cmulc(a[s * G::W + ta], rounded<T>(ta ? mul64(b[s], c) : b[s]));
            if (real) vv.im = T(0);
            Yrow[tid + G::THREADS * s + G::M * ta] = vv;
        }
    }
}

// Row units: units 0 .. ngroups (n2/2 - 1) - 1 are mirror pairs (row pr >= 1
// with n2 - pr), the last ngroups units the self rows 0 and n2/2 of each group.
// A unit transforms its rows of every tile of the group, sums their spectrum
// products and inverts the sum into the first tile's row pr.
template <typename T, int N1, int N2, int NCB1>
__device__ __forceinline__ void row_unit(uint32_t u, const JobTable& jt, cx<T>* __restrict__ ws,
                                         const uint32_t* __restrict__ part, TileMeta* __restrict__ meta,
                                         RowSmem<T, N1>& S, const RowReg<T, N1>& R, uint32_t& wsum,
                                         const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64,
                                         int fshift) {
    constexpr uint32_t L = (uint32_t)N1 * N2;
    constexpr int NP = N2 / 2, PT = RowGeom<T, N1>::PT;
    const int tid = threadIdx.x;
    const T quarter = T(0.25) / T(L);
    const uint32_t npairs = jt.ngroups * (uint32_t)(NP - 1);
    const bool pair = u < npairs;
    const uint32_t gl = pair ? u / (uint32_t)(NP - 1) : u - npairs;
    const uint32_t pr = pair ? 1u + u % (uint32_t)(NP - 1) : 0u;
    const JobDesc jd = find_group_job(jt, jt.group0 + gl);
    uint32_t first, gs;
    (void)group_geo(jd, jt.group0 + gl - jd.group_begin, &first, &gs);
    const uint32_t lt = jd.tile_begin + first - jt.tile0;
    cx<T>* __restrict__ Y = ws + (size_t)lt * L;
    if (pair) {
        cx<T> acc[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) acc[i] = cx<T>{T(0), T(0)};
        for (uint32_t c = 0; c < gs; ++c) {
            const cx<T>* __restrict__ Yc = Y + (size_t)c * L;
            cx<T> A[PT], B[PT];
            row_load<T, N1>(A, Yc + (size_t)pr * N1, tid);
            row_forward<T, N1>(A, S, R, tid);
            row_load<T, N1>(B, Yc + (size_t)(N2 - pr) * N1, tid);
            row_forward<T, N1>(B, S, R, tid);
            row_mirror<T, N1>(B, S.data, tid, false);
#pragma unroll
            for (int i = 0; i < PT; ++i) acc[i] = acc[i] + spectrum_product(A[i], B[i], quarter);
        }
        row_inverse<T, N1>(acc, S, R, tid);
        row_store<T, N1>(Y + (size_t)pr * N1, acc, pr, false, tid, fa64, fb64, fshift);
    } else {
        // weight of the group's chunks from the pass-1 partial sums; reset the certificate
        __syncthreads();
        if (tid == 0) wsum = 0;
        __syncthreads();
        uint32_t sum = 0;
        for (uint32_t c = tid; c < gs * NCB1; c += RowGeom<T, N1>::THREADS) sum += part[(size_t)lt * NCB1 + c];
        atomicAdd(&wsum, sum);
        __syncthreads();
        if (tid == 0) meta[jt.group0 + gl] = TileMeta{wsum, 0u, 0u, 0u};
        // rows 0 and n2/2 are their own mirrors and their V rows are real:
        // each goes to the real parts of its own row
#pragma nounroll
        for (int v = 0; v < 2; ++v) {
            const uint32_t row = v == 0 ? 0u : (uint32_t)NP;
            cx<T> acc[PT];
#pragma unroll
            for (int i = 0; i < PT; ++i) acc[i] = cx<T>{T(0), T(0)};
            for (uint32_t c = 0; c < gs; ++c) {
                cx<T> A[PT], B[PT];
                row_load<T, N1>(A, Y + (size_t)c * L + (size_t)row * N1, tid);
                row_forward<T, N1>(A, S, R, tid);
#pragma unroll
                for (int i = 0; i < PT; ++i) B[i] = A[i];
                row_mirror<T, N1>(B, S.data, tid, v == 0);
#pragma unroll
                for (int i = 0; i < PT; ++i) acc[i] = acc[i] + spectrum_product(A[i], B[i], quarter);
            }
            row_inverse<T, N1>(acc, S, R, tid);
            row_store<T, N1>(Y + (size_t)row * N1, acc, row, true, tid, fa64, fb64, fshift);
        }
    }
}

// The row pass of the rows of 512 in launches that leave the device idle: a unit is
// a team of 2 Q waves, Q chunks at a time, the two rows of a pair in parallel.  Row
// n2 - pr comes mirrored through LDS; the first wave adds the Q partial sums and
// inverts.  Against one wave per unit: four summed FP32 tiles of 2^19, 18.6 -> 11.7
// us (call 53.4 -> 46.2); 48 of 2^17, 49 -> 20; one FP64 tile of 2^18, 9.5 -> 8.0.
template <typename T, int N1, int N2, int NCB1, int Q>
__global__ void __launch_bounds__(128 * Q)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
k2_pass2_team(JobTable jt, cx<T>* __restrict__ ws, const uint32_t* __restrict__ part, TileMeta* __restrict__ meta,
              const cx<T>* __restrict__ tw, const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64,
              const cx<double>* __restrict__ fb64, int fshift) {
    using G = RowGeom<T, N1>;
    static_assert(G::W == 1, "one wave per row");
    constexpr uint32_t L = (uint32_t)N1 * N2;
    constexpr int NP = N2 / 2, PT = G::PT;
    __shared__ __align__(16) RowSmem<T, N1> S[2 * Q];
    __shared__ uint32_t wsum;
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63, side = wv & 1, q = wv >> 1;
    const uint32_t u = blockIdx.x;
    const T quarter = T(0.25) / T(L);
    RowReg<T, N1> R;
    row_setup<T, N1, N2>(S[wv], R, tw, stw, l);
    const uint32_t npairs = jt.ngroups * (uint32_t)(NP - 1);
    const bool pair = u < npairs;
    const uint32_t gl = pair ? u / (uint32_t)(NP - 1) : u - npairs;
    const uint32_t pr = pair ? 1u + u % (uint32_t)(NP - 1) : 0u;
    const JobDesc jd = find_group_job(jt, jt.group0 + gl);
    uint32_t first, gs;
    (void)group_geo(jd, jt.group0 + gl - jd.group_begin, &first, &gs);
    const uint32_t lt = jd.tile_begin + first - jt.tile0;
    cx<T>* __restrict__ Y = ws + (size_t)lt * L;
    // pair: rows pr and n2 - pr; else rows 0 and n2/2, their own mirrors, with real V
    const uint32_t row = pair ? (side ? (uint32_t)N2 - pr : pr) : (side ? (uint32_t)NP : 0u);
    if (!pair) {   // weight of the group's chunks; reset the certificate
        if (tid == 0) wsum = 0;
        __syncthreads();
        uint32_t sum = 0;
        for (uint32_t c = tid; c < gs * NCB1; c += 128 * Q) sum += part[(size_t)lt * NCB1 + c];
        atomicAdd(&wsum, sum);
        __syncthreads();
        if (tid == 0) meta[jt.group0 + gl] = TileMeta{wsum, 0u, 0u, 0u};
    }
    cx<T> acc[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) acc[i] = cx<T>{T(0), T(0)};
    for (uint32_t c0 = 0; c0 < gs; c0 += Q) {   // the same trips for every wave: barriers inside
        const uint32_t c = c0 + (uint32_t)q;
        const bool active = c < gs;
        cx<T> A[PT], B[PT];
        if (active) {
            row_load<T, N1>(A, Y + (size_t)c * L + (size_t)row * N1, l);
            row_forward<T, N1>(A, S[wv], R, l);
        }
        if (pair) {
            if (active && side) {
                wave_sync();
#pragma unroll
                for (int i = 0; i < PT; ++i) S[wv].data[G::slot(l) + G::slot(64) * i] = A[i];
            }
            __syncthreads();
            if (active && !side) {
#pragma unroll
                for (int i = 0; i < PT; ++i) B[i] = S[wv + 1].data[G::slot(G::M - 1 - l - 64 * i)];
#pragma unroll
                for (int i = 0; i < PT; ++i) acc[i] = acc[i] + spectrum_product(A[i], B[i], quarter);
            }
            __syncthreads();
        } else if (active) {
#pragma unroll
            for (int i = 0; i < PT; ++i) B[i] = A[i];
            row_mirror<T, N1>(B, S[wv].data, l, side == 0);
#pragma unroll
            for (int i = 0; i < PT; ++i) acc[i] = acc[i] + spectrum_product(A[i], B[i], quarter);
        }
    }
    const bool holds = !pair || side == 0;
    if constexpr (Q > 1) {
        if (holds && q > 0) {
            wave_sync();
#pragma unroll
            for (int i = 0; i < PT; ++i) S[wv].data[G::slot(l) + G::slot(64) * i] = acc[i];
        }
        __syncthreads();
        if (holds && q == 0)
#pragma unroll
            for (int k = 1; k < Q; ++k)
#pragma unroll
                for (int i = 0; i < PT; ++i) acc[i] = acc[i] + S[wv + 2 * k].data[G::slot(l) + G::slot(64) * i];
    }
    if (holds && q == 0) {
        row_inverse<T, N1>(acc, S[wv], R, l);
        row_store<T, N1>(Y + (size_t)row * N1, acc, row, !pair, l, fa64, fb64, fshift);
    }
}

// Waves per SIMD: 4 in FP32 (two workgroups of rows of 4096 per CU), 2 in FP64
// and for rows of 8192.
template <typename T, int N1> constexpr int row_waves_per_eu() { return sizeof(T) == 4 && N1 <= 4096 ? 4 : 2; }
template <typename T, int N1> constexpr int row_wgs_per_cu() { return row_waves_per_eu<T, N1>() * 4 / RowGeom<T, N1>::W; }
template <typename T, int N1, int N2, int NCB1>
__global__ void __launch_bounds__((RowGeom<T, N1>::THREADS))
__attribute__((amdgpu_waves_per_eu(row_waves_per_eu<T, N1>())))
k2_pass2(JobTable jt, cx<T>* __restrict__ ws, const uint32_t* __restrict__ part, TileMeta* __restrict__ meta,
         const cx<T>* __restrict__ tw, const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64,
         const cx<double>* __restrict__ fb64, int fshift) {
    __shared__ __align__(16) RowSmem<T, N1> S;
    __shared__ uint32_t wsum;
    const uint32_t units = jt.ngroups * (uint32_t)(N2 / 2);
    RowReg<T, N1> R;
    row_setup<T, N1, N2>(S, R, tw, stw, threadIdx.x);
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x)
        row_unit<T, N1, N2, NCB1>(u, jt, ws, part, meta, S, R, wsum, fa64, fb64, fshift);
}

// ------------------------------------------------------------------ shared spectra
// Jobs with several chunks and windows of equal length B = L / 2: chunk b and
// window o meet seed slice b + o, so every chunk and slice is transformed once
// (two to a tile, columns by pass 1, rows here) and the windows' spectra
//     P_o = (1 / L) sum_b X_b S_{b+o}
// are sums over the packs' spectra.  Packing two chunks, or two slices, separates
// sequences of equal size: the large low-frequency values of the zero-padded
// chunks do not leak into the seeds' spectra.
//
// Jobs of up to four windows: a workgroup takes one pair of mirror rows (unit 0: the
// self rows 0 and n2/2 one after the other) through every pack, walks the key packs
// with the slices that the windows meet sliding through registers, and inverts the
// windows' sums; no spectrum goes to memory.  The unit of row 0 sets the
// certificates.
//
// 64 registers of sums and 64 of slices beside the two rows of a pack leave two
// waves per SIMD (one workgroup per CU; the twiddles are in LDS), so the next row
// is loaded while one is transformed.  Bound by the latency of a row's steps: 3.5
// us per row and CU, 2.4 TB/s.  33 packs of 2^23, four windows: 936 us, against
// 1,620 us for the three kernels below on as many points; per further four windows
// the rows would be transformed again, while the sums below take 510 us per eight.
// All 256 registers are taken and 30 more spilled (124 bytes of scratch per lane, two
// or three of them reloaded per key pack); two rows at a time: 1,550 us with the
// spills.
constexpr int kSharedWins = 4;
template <typename T, int N1, int N2, int NCB1>
__global__ void __launch_bounds__((RowGeom<T, N1>::THREADS)) __attribute__((amdgpu_waves_per_eu(2)))
k2_shared_rows(JobTable jt, const cx<T>* __restrict__ ws, cx<T>* __restrict__ win, const uint32_t* __restrict__ part,
               TileMeta* __restrict__ meta, const cx<T>* __restrict__ tw,
               const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64,
               int fshift) {
    using G = RowGeom<T, N1>;
    constexpr uint32_t L = (uint32_t)N1 * N2;
    constexpr int NP = N2 / 2, PT = G::PT;
    static_assert(kSharedWins == 4, "four slices in registers");
    __shared__ __align__(16) RowSmem<T, N1> S;
    __shared__ uint32_t wsum;
    __shared__ RowTwiddles<T, N1> X;
    const int tid = threadIdx.x;
    {
        RowReg<T, N1> r;
        row_setup<T, N1, N2>(S, r, tw, stw, tid);
#pragma unroll
        for (int i = 0; i < G::S * (G::W - 1); ++i) X.tw1[i * G::THREADS + tid] = r.tw1[i];
        if (tid < 64)
#pragma unroll
            for (int i = 0; i < 7; ++i) X.t3[i * 64 + tid] = r.t3[i];
    }
    const RowLds<T, N1> R{{X.tw1 + tid}, {X.t3 + (tid & 63)}};
    const SharedJob sh = jt.shared;
    const T quarter = T(0.25) / T(L);
    const uint32_t nw = jt.one.nouts;   // at most kSharedWins
    for (uint32_t u = blockIdx.x; u < (uint32_t)NP; u += gridDim.x) {
        const bool pair = u > 0;
        if (!pair) {
            __syncthreads();
            if (tid == 0) wsum = 0;
            __syncthreads();
            uint32_t sum = 0;
            for (uint32_t c = tid; c < sh.kpacks * NCB1; c += G::THREADS) sum += part[c];
            atomicAdd(&wsum, sum);
            __syncthreads();
            if (tid < (int)nw) meta[jt.group0 + tid] = TileMeta{wsum, 0u, 0u, 0u};
        }
#pragma nounroll
        for (int v = 0; v < (pair ? 1 : 2); ++v) {
            const uint32_t row = pair ? u : v ? (uint32_t)NP : 0u;
            const cx<T>* __restrict__ ra = ws + (size_t)row * N1;
            const cx<T>* __restrict__ rb = ws + (size_t)(N2 - u) * N1;
            cx<T> raw[PT];   // the next row, in flight
            row_load<T, N1>(raw, ra + (size_t)sh.kpacks * L, tid);
            // 2 X_a = z + conj m, 2 X_b = -i (z - conj m) of the pack whose first row is
            // in flight; `next` comes after it
            auto split = [&](uint32_t pack, uint32_t next, cx<T> (&xa)[PT], cx<T> (&xb)[PT]) {
#pragma unroll
                for (int i = 0; i < PT; ++i) xa[i] = raw[i];
                row_load<T, N1>(raw, pair ? rb + (size_t)pack * L : ra + (size_t)next * L, tid);
                row_forward<T, N1>(xa, S, R, tid);
                if (pair) {
#pragma unroll
                    for (int i = 0; i < PT; ++i) xb[i] = raw[i];
                    row_load<T, N1>(raw, ra + (size_t)next * L, tid);
                    row_forward<T, N1>(xb, S, R, tid);
                } else {
#pragma unroll
                    for (int i = 0; i < PT; ++i) xb[i] = xa[i];
                }
                row_mirror<T, N1>(xb, S.data, tid, !pair && v == 0);
#pragma unroll
                for (int i = 0; i < PT; ++i) {
                    const cx<T> m = conj(xb[i]), d = xa[i] - m;
                    xa[i] = xa[i] + m;
                    xb[i] = cx<T>{d.im, -d.re};
                }
            };
            // the slices of seed pack q; past the last pack zero, and pack `next` (in
            // flight) stays the next one
            auto slices = [&](uint32_t q, uint32_t next, cx<T> (&sa)[PT], cx<T> (&sb)[PT]) {
                if (q < sh.spacks) {
                    split(sh.kpacks + q, next, sa, sb);
                } else {
#pragma unroll
                    for (int i = 0; i < PT; ++i) sa[i] = sb[i] = cx<T>{T(0), T(0)};
                }
            };
            // pack that follows: seed pack q, or `other` where there is none
            auto seed_or = [&](uint32_t q, uint32_t other) { return q < sh.spacks ? sh.kpacks + q : other; };
            cx<T> acc[kSharedWins][PT], s0[PT], s1[PT], s2[PT], s3[PT];
#pragma unroll
            for (int o = 0; o < kSharedWins; ++o)
#pragma unroll
                for (int i = 0; i < PT; ++i) acc[o][i] = cx<T>{T(0), T(0)};
            slices(0, seed_or(1, 0), s0, s1);
            slices(1, 0, s2, s3);
#pragma nounroll
            for (uint32_t q = 0; q < sh.kpacks; ++q) {
                const uint32_t sq = q + kSharedWins / 2, after = q + 1 < sh.kpacks ? q + 1 : 0;
                cx<T> xa[PT], xb[PT];
                split(q, seed_or(sq, after), xa, xb);
#pragma unroll
                for (int i = 0; i < PT; ++i) {
                    acc[0][i] = acc[0][i] + cmul(xa[i], s0[i]) + cmul(xb[i], s1[i]);
                    acc[1][i] = acc[1][i] + cmul(xa[i], s1[i]) + cmul(xb[i], s2[i]);
                    acc[2][i] = acc[2][i] + cmul(xa[i], s2[i]) + cmul(xb[i], s3[i]);
                    acc[3][i] = acc[3][i] + cmul(xa[i], s3[i]);
                    s0[i] = s2[i];
                    s1[i] = s3[i];
                }
                slices(sq, after, s2, s3);
#pragma unroll
                for (int i = 0; i < PT; ++i) acc[3][i] = acc[3][i] + cmul(xb[i], s2[i]);
            }
#pragma unroll
            for (int o = 0; o < kSharedWins; ++o) {
                if ((uint32_t)o >= nw) break;
#pragma unroll
                for (int i = 0; i < PT; ++i) acc[o][i] = cx<T>{acc[o][i].re * quarter, acc[o][i].im * quarter};
                row_inverse<T, N1>(acc[o], S, R, tid);
                row_store<T, N1>(win + (size_t)o * L + (size_t)row * N1, acc[o], row, !pair, tid, fa64, fb64, fshift);
            }
        }
    }
}

// Jobs of more windows: forward rows, sums and inverse rows by three kernels, the
// spectra in memory.  Forward rows in place: row k2 of a tile becomes Z[k2][p], p = w M + kb holding
// frequency k1 = W kb + w, so the mirror of position p is N1 - 1 - p (row 0, whose
// mirror is -k1 mod N1: M - p mod M within w = 0, else N1 + M - 1 - p).
template <typename T, int N1, int N2>
__global__ void __launch_bounds__((RowGeom<T, N1>::THREADS)) __attribute__((amdgpu_waves_per_eu(8)))
k2_rows(JobTable jt, cx<T>* __restrict__ ws, const cx<T>* __restrict__ tw, const cx<T>* __restrict__ stw) {
    using G = RowGeom<T, N1>;
    __shared__ __align__(16) RowSmem<T, N1> S;
    RowReg<T, N1> R;
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
    row_setup<T, N1, N2>(S, R, tw, stw, tid);
    const uint32_t units = jt.ntiles * (uint32_t)N2;
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x) {
        cx<T>* __restrict__ row = ws + (size_t)u * N1;   // tiles and rows are contiguous
        cx<T> a[G::PT];
        row_load<T, N1>(a, row, tid);
        row_forward<T, N1>(a, S, R, tid);
#pragma unroll
        for (int i = 0; i < G::PT; ++i) row[wv * G::M + l + 64 * i] = a[i];
    }
}

// Sums of the windows o0 .. o0 + NW - 1 (NW even, o0 even): a thread takes one
// position of row k2 <= n2 / 2 and its mirror and walks the key packs, with the
// NW + 2 slices that the windows meet sliding through registers.  Each spectrum
// is read once per NW windows.  Bound by these reads.
template <typename T, int N1, int N2, int NW>
__global__ void __launch_bounds__(256)
k2_mac(JobTable jt, const cx<T>* __restrict__ ws, cx<T>* __restrict__ win, uint32_t o0) {
    constexpr uint32_t L = (uint32_t)N1 * N2;
    constexpr int M = RowGeom<T, N1>::M;
    const uint32_t k2 = blockIdx.x / (N1 / 256), p = (blockIdx.x % (N1 / 256)) * 256 + threadIdx.x;   // k2 <= n2 / 2
    const uint32_t km = k2 ? (uint32_t)N2 - k2 : 0u;
    const uint32_t pm = k2 ? (uint32_t)N1 - 1u - p : (p < M ? (M - p) & (M - 1) : (uint32_t)(N1 + M - 1) - p);
    const size_t at = (size_t)k2 * N1 + p, am = (size_t)km * N1 + pm;
    const SharedJob sh = jt.shared;
    const T quarter = T(0.25) / T(L);
    // 2 X_a = z + conj m, 2 X_b = -i (z - conj m) of a pack
    auto split = [&](uint32_t pack, cx<T>& xa, cx<T>& xb) {
        const cx<T> z = ws[(size_t)pack * L + at], m = conj(ws[(size_t)pack * L + am]);
        xa = z + m;
        const cx<T> d = z - m;
        xb = cx<T>{d.im, -d.re};
    };
    auto slices = [&](uint32_t q, cx<T>& sa, cx<T>& sb) {
        if (q < sh.spacks) {
            split(sh.kpacks + q, sa, sb);
        } else {
            sa = cx<T>{T(0), T(0)};
            sb = sa;
        }
    };
    cx<T> acc[NW], s[NW + 2];
#pragma unroll
    for (int o = 0; o < NW; ++o) acc[o] = cx<T>{T(0), T(0)};
#pragma unroll
    for (int o = 0; o < NW; o += 2) slices(o0 / 2 + o / 2, s[o], s[o + 1]);
    for (uint32_t q = 0; q < sh.kpacks; ++q) {
        cx<T> xa, xb;
        split(q, xa, xb);
        slices(q + (o0 + NW) / 2, s[NW], s[NW + 1]);
#pragma unroll
        for (int o = 0; o < NW; ++o) acc[o] = acc[o] + cmul(xa, s[o]) + cmul(xb, s[o + 1]);
#pragma unroll
        for (int o = 0; o < NW; ++o) s[o] = s[o + 2];
    }
#pragma unroll
    for (int o = 0; o < NW; ++o)
        if (o0 + o < jt.one.nouts) win[(size_t)(o0 + o) * L + at] = cx<T>{acc[o].re * quarter, acc[o].im * quarter};
}

// Inverse rows 0 .. n2 / 2 of every window, in place: from the order above to
// rows of V (natural order) for pass 3; the unit of row 0 sets the certificate.
template <typename T, int N1, int N2, int NCB1>
__global__ void __launch_bounds__((RowGeom<T, N1>::THREADS))
__attribute__((amdgpu_waves_per_eu(row_waves_per_eu<T, N1>())))
k2_rows_inv(JobTable jt, cx<T>* __restrict__ win, const uint32_t* __restrict__ part, TileMeta* __restrict__ meta,
            const cx<T>* __restrict__ tw, const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64,
            const cx<double>* __restrict__ fb64, int fshift) {
    using G = RowGeom<T, N1>;
    constexpr uint32_t L = (uint32_t)N1 * N2, NR = N2 / 2 + 1;
    __shared__ __align__(16) RowSmem<T, N1> S;
    __shared__ uint32_t wsum;
    RowReg<T, N1> R;
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
    row_setup<T, N1, N2>(S, R, tw, stw, tid);
    const uint32_t units = jt.ngroups * NR;
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x) {
        const uint32_t o = u / NR, k2 = u % NR;
        cx<T>* __restrict__ row = win + (size_t)o * L + (size_t)k2 * N1;
        cx<T> a[G::PT];
#pragma unroll
        for (int i = 0; i < G::PT; ++i) a[i] = row[wv * G::M + l + 64 * i];
        row_inverse<T, N1>(a, S, R, tid);   // its barriers separate the loads from the stores below
        row_store<T, N1>(row, a, k2, k2 == 0 || k2 == N2 / 2, tid, fa64, fb64, fshift);
        if (k2 == 0) {
            __syncthreads();
            if (tid == 0) wsum = 0;
            __syncthreads();
            uint32_t sum = 0;
            for (uint32_t c = tid; c < jt.shared.kpacks * NCB1; c += G::THREADS) sum += part[c];
            atomicAdd(&wsum, sum);
            __syncthreads();
            if (tid == 0) meta[jt.group0 + o] = TileMeta{wsum, 0u, 0u, 0u};
        }
    }
}

// ------------------------------------------------------------------ pass 3
// rint(z) mod 4 for an integral r (FP32: |r| < 2^31; FP64: |r| < 2^51)
__device__ __forceinline__ uint32_t low2(float r) { return (uint32_t)(int)r & 3u; }
__device__ __forceinline__ uint32_t low2(double r) {
    const double q = r * 0.25;
    return (uint32_t)(int)((q - floor(q)) * 4.0) & 3u;
}

template <typename T, int N1, int N2>
__global__ void __launch_bounds__((P3Geom<T, N1, N2>::THREADS))
__attribute__((amdgpu_waves_per_eu(P3Geom<T, N1, N2>::WPE)))
k2_pass3(JobTable jt, const cx<T>* __restrict__ ws, TileMeta* __restrict__ meta, const cx<T>* __restrict__ tw,
         const cx<T>* __restrict__ stw) {
    using Gm = P3Geom<T, N1, N2>;
    constexpr int C = Gm::C, G = Gm::G, M = Gm::M, NJ = M / 16, CW = Gm::CW;
    constexpr uint32_t L = (uint32_t)N1 * N2;
    constexpr int NCB = N1 / C;
    constexpr bool LT = Gm::LDS_TAB;
    constexpr int NHT = LT ? M : 1;
    constexpr int NLB = Gm::WAVES * 64;
    __shared__ __align__(16) cx<T> lds[Gm::SLOTS];
    __shared__ __align__(16) cx<T> st[LT ? wfft_lds_entries(M) : 1];
    // Hermitian twiddles w_n2^k (k < n2/2) until the transform, then the
    // output bits of each lane: bit 2 i + e of lbits[w * 64 + g NJ + j] is the
    // output of column w G + g, row 2 (j + NJ i) + e
    __shared__ __align__(16) union {
        cx<T> htw[NHT];
        uint32_t lbits[NLB];
    } U;
    __shared__ T hrow[C];
    __shared__ uint32_t s_res, s_abs, s_bad;

    const uint32_t blk = xcd_block(), t = jt.group0 + blk / NCB;   // group; neighbours write to the same lines
    const uint32_t cb = blk % NCB;
    const JobDesc jd = find_group_job(jt, t);
    uint32_t first, gs;
    const TileGeo g = group_geo(jd, t - jd.group_begin, &first, &gs);
    const uint32_t lt = jd.tile_begin + first - jt.tile0;
    const cx<T>* __restrict__ V = ws + (size_t)lt * L;
    const int tid = threadIdx.x;
    if (tid == 0) { s_res = 0; s_abs = 0; s_bad = 0; }
    static_assert((M * C) % Gm::THREADS == 0, "load tile");
    constexpr int LPT = M * C / Gm::THREADS;
    {
        cx<T> in[LPT];
#pragma unroll
        for (int q = 0; q < LPT; ++q) {
            const int idx = tid + q * Gm::THREADS;
            in[q] = V[(size_t)(idx / C) * N1 + cb * C + (idx % C)];
        }
        if (tid < C) hrow[tid] = V[(size_t)M * N1 + cb * C + tid].re;   // H[n2/2], real
        if constexpr (LT) {
            wfft_load_lds<T, M>(st, stw, tid, Gm::THREADS);
            for (int k = tid; k < M; k += Gm::THREADS) U.htw[k] = tw[k * (cmax<N1, N2>() / N2)];
        }
#pragma unroll
        for (int q = 0; q < LPT; ++q) {
            const int idx = tid + q * Gm::THREADS;
            lds[tslot<C>(idx / C, idx % C)] = in[q];
        }
    }
    __syncthreads();

    const int wv = tid >> 6, l = tid & 63;
    const int gg = l / NJ, j = l % NJ;
    const int f = wv * G + gg;
    const uint32_t t1 = cb * C + (uint32_t)f;
    const int64_t weight = (int64_t)meta[t].popcnt;
    cx<T> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int k = j + i * NJ;
        const cx<T> h = lds[tslot<C>(k, f)];
        if (k == 0) {
            // H[0] and H[n2/2] are real; H[n2/2] sits in the real parts of row n2/2
            const T hh = hrow[f];
            v[i] = cx<T>{h.re + hh, h.re - hh};
        } else {
            const cx<T> hm = conj(lds[tslot<C>(M - k, f)]);
            const cx<T> e = h + hm;
            const cx<T> wk = LT ? U.htw[k] : tw[k * (cmax<N1, N2>() / N2)];
            const cx<T> o = cmulc(h - hm, wk);
            v[i] = cx<T>{e.re - o.im, e.im + o.re};
        }
    }
    __syncthreads();  // tile (and twiddles) consumed; LDS becomes wave regions
    cx<T>* reg = lds + wv * kWaveSlots + gg * (M + M / 16);
    if constexpr (LT) wave_fft_lds<T, +1, M>(v, reg, j, st);
    else wave_fft<T, +1, M>(v, reg, j, stw);

    // window, exact rounding and parity (branch-free): only the low two bits
    // of rint(z) + weight matter, bit = bit 1, parity check = bit 0
    const uint32_t wlow = meta[t].popcnt & 3u;
    const uint32_t bo = (uint32_t)g.bo;
    const uint32_t rows = (bo + (uint32_t)N1 - 1u) / (uint32_t)N1;  // rows t2 holding outputs
    float mres = 0.f, mabs = 0.f;
    uint32_t bad = 0;
    uint32_t mybits = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (2u * (uint32_t)(i * NJ) >= rows) continue;   // register i holds no output row (uniform)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t t2 = 2u * (uint32_t)(j + i * NJ) + (uint32_t)e;
            const bool valid = t1 + (uint32_t)N1 * t2 < bo;
            const T zz = e ? v[i].im : v[i].re;
            const T r = round_even(zz);
            const uint32_t s2 = low2(r) + wlow;
            // an odd sum, or a non-finite z (fmaxf below would drop a NaN)
            bad += (valid && ((s2 & 1u) || !(fabs(zz - r) <= T(0.5)))) ? 1u : 0u;
            mres = fmaxf(mres, valid ? (float)fabs(zz - r) : 0.f);
            mabs = fmaxf(mabs, valid ? (float)fabs(zz) : 0.f);
            mybits |= (valid ? ((s2 >> 1) & 1u) : 0u) << (2 * i + e);
        }
    }
    U.lbits[wv * 64 + l] = mybits;
    atomicMax(&s_res, __float_as_uint(mres));
    atomicMax(&s_abs, __float_as_uint(mabs));
    atomicAdd(&s_bad, bad);
    __syncthreads();
    // assemble and store each output row's C bits (32 per word, C < 32: one C-bit group)
    constexpr int WB = C < 32 ? C : 32;    // bits per stored word
    const uint64_t limit = g.dst_words * 64u;
    for (uint32_t idx = tid; idx < rows * CW; idx += Gm::THREADS) {
        const uint32_t t2 = idx / CW, c = idx % CW;
        const uint32_t k = t2 >> 1, sh = 2u * (k / NJ) + (t2 & 1u), jj = k % NJ;
        uint32_t word = 0;
#pragma unroll
        for (int q = 0; q < WB; ++q) {
            const int col = 32 * (int)c + q;
            word |= ((U.lbits[(col / G) * 64 + (col % G) * NJ + jj] >> sh) & 1u) << q;
        }
        const uint64_t off = (uint64_t)cb * C + 32u * c + (uint64_t)N1 * t2;
        if (off >= limit) continue;
        put_bits<WB>(g, off, word);
    }
    if (tid == 0) {
        atomicMax(&meta[t].maxres, s_res);
        atomicMax(&meta[t].maxabs, s_abs);
        if (s_bad) atomicAdd(&meta[t].badpar, s_bad);
    }
}

// Compute units of the current device.
int row_pass_workgroups();

template <typename T, int N1, int N2, int NCB1, int Q>
int launch_team(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
    hipLaunchKernelGGL((k2_pass2_team<T, N1, N2, NCB1, Q>), dim3(jt.ngroups * (N2 / 2)), dim3(128 * Q), 0,
                       (hipStream_t)stream, jt, (cx<T>*)ws, (const uint32_t*)part, meta, (const cx<T>*)tb.tw,
                       (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64, (const cx<double>*)tb.fb64, tb.fshift);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T, int N1, int N2, int NCB1>
int launch_row_pass(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
    const uint32_t units = jt.ngroups * (N2 / 2);
    const uint32_t wgs = (uint32_t)(row_pass_workgroups() * row_wgs_per_cu<T, N1>());
    if constexpr (RowGeom<T, N1>::W == 1) {
        // teams as large as the chunks of a group give work to, while the device holds
        // all their waves at once (wgs is its waves here)
        // (and a repeat as large as the first run's, whose order of summation it needs)
        const uint32_t groups = jt.as_groups ? jt.as_groups : jt.ngroups, waves = groups * (N2 / 2);
        const uint32_t chunks = ((jt.as_groups ? jt.as_tiles : jt.ntiles) + groups - 1) / groups;
        if (chunks > 2 && waves * 8 <= wgs) return launch_team<T, N1, N2, NCB1, 4>(jt, ws, part, meta, tb, stream);
        if (chunks > 1 && waves * 4 <= wgs) return launch_team<T, N1, N2, NCB1, 2>(jt, ws, part, meta, tb, stream);
        if (waves * 2 <= wgs) return launch_team<T, N1, N2, NCB1, 1>(jt, ws, part, meta, tb, stream);
    }
    hipLaunchKernelGGL((k2_pass2<T, N1, N2, NCB1>), dim3(units < wgs ? units : wgs),
                       dim3(RowGeom<T, N1>::THREADS), 0,
                       (hipStream_t)stream, jt, (cx<T>*)ws, (const uint32_t*)part, meta, (const cx<T>*)tb.tw,
                       (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64, (const cx<double>*)tb.fb64, tb.fshift);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int N1, int N2, int P> void launch_bits(const JobTable& jt, uint8_t* planes, void* stream) {
    constexpr int waves = 2 * ((int)BitPlanes<N1, N2, P>::kColumn / 8) * (N1 / 64 / kBitsCols);   // of a tile
    hipLaunchKernelGGL((k2_bits<N1, N2, P>), dim3(jt.ntiles * (waves / 4)), dim3(256), 0, (hipStream_t)stream, jt, planes);
}

// Pass 1 of the rows of 4096 and 8192: the bit planes, then the split columns.
template <typename T, int N1, int N2, int NT, bool SHARED = false>
int launch_split(const JobTable& jt, void* ws, uint32_t* part, const void* tw, const Tables& tb, void* stream) {
    using G = PSplitGeom<T, N1, N2>;
    uint8_t* planes = reinterpret_cast<uint8_t*>((cx<T>*)ws + (size_t)jt.ntiles * ((size_t)N1 * N2));
    launch_bits<N1, N2, G::P>(jt, planes, stream);
    hipLaunchKernelGGL((k2_pass1_split<T, N1, N2, NT, SHARED>), dim3(jt.ntiles * (N1 / G::C) * G::P), dim3(G::THREADS), 0,
                       (hipStream_t)stream, jt, (cx<T>*)ws, part, (const cx<T>*)tw, (const cx<T>*)tb.stw,
                       (const cx<double>*)tb.fa64, (const cx<double>*)tb.fb64, tb.fshift);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T, int N1, int N2>
struct ClassImpl2 {
    // bit planes; whole columns from them where the columns are short (k2_pass1_whole)
    static constexpr bool kPlanes = N1 >= 1024, kWhole = sizeof(T) == 4 && N2 <= 512, kSplit = kPlanes && !kWhole;
    using G1 = std::conditional_t<kSplit, PSplitGeom<T, N1, kSplit ? N2 : 256>, P1Geom<T, N1, kSplit ? 256 : N2>>;
    using G3 = P3Geom<T, N1, N2>;
    static constexpr int C1 = G1::C, C3 = G3::C;
    // workspace bytes per tile beyond its points: the bit planes
    static constexpr size_t kWsExtra = kPlanes ? BitPlanes<N1, kPlanes ? N2 : 256>::kTile : 0;
    static int pass1(const JobTable& jt, void* ws, uint32_t* part, TileMeta*, const Tables& tb, void* stream) {
        if constexpr (kSplit) {
            return launch_split<T, N1, N2, cmax<N1, N2>()>(jt, ws, part, tb.tw, tb, stream);
        } else if constexpr (kPlanes) {
            static_assert(BitPlanes<N1, N2, 1>::kTile == kWsExtra, "planes of either form");
            launch_bits<N1, N2, 1>(jt, reinterpret_cast<uint8_t*>((cx<T>*)ws + (size_t)jt.ntiles * ((size_t)N1 * N2)), stream);
            hipLaunchKernelGGL((k2_pass1_whole<T, N1, N2>), dim3(jt.ntiles * (N1 / C1)), dim3(G1::THREADS), 0,
                               (hipStream_t)stream, jt, (cx<T>*)ws, part, (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64,
                               (const cx<double>*)tb.fb64, tb.fshift);
        } else {
            hipLaunchKernelGGL((k2_pass1<T, N1, N2>), dim3(jt.ntiles * (N1 / C1)), dim3(G1::THREADS), 0, (hipStream_t)stream,
                               jt, (cx<T>*)ws, part, (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64,
                               (const cx<double>*)tb.fb64, tb.fshift);
        }
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    static int pass2(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
        return launch_row_pass<T, N1, N2, N1 / C1>(jt, ws, part, meta, tb, stream);
    }
    // Shared spectra (FP32): `ws` holds the packs, then their planes, then the
    // windows; the windows' column passes are pass3 on the windows.
    static constexpr size_t shared_bytes(uint32_t packs, uint32_t windows) {
        return (size_t)packs * ((size_t)N1 * N2 * sizeof(cx<T>) + kWsExtra) + (size_t)windows * N1 * N2 * sizeof(cx<T>);
    }
    static void* windows(const JobTable& jt, void* ws) {
        return (uint8_t*)ws + (size_t)jt.ntiles * ((size_t)N1 * N2 * sizeof(cx<T>) + kWsExtra);
    }
    static int shared_pass1(const JobTable& jt, void* ws, uint32_t* part, TileMeta*, const Tables& tb, void* stream) {
        static_assert(PSplitGeom<T, N1, N2>::C == C1, "partial weights of the packs");
        return launch_split<T, N1, N2, cmax<N1, N2>(), true>(jt, ws, part, tb.tw, tb, stream);
    }
    template <int NW>
    static void mac(const JobTable& jt, void* ws, uint32_t o0, void* stream) {
        hipLaunchKernelGGL((k2_mac<T, N1, N2, NW>), dim3((N2 / 2 + 1) * (N1 / 256)), dim3(256), 0, (hipStream_t)stream, jt,
                           (const cx<T>*)ws, (cx<T>*)windows(jt, ws), o0);
    }
    static int shared_pass2(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
        hipStream_t s = (hipStream_t)stream;
        if (jt.one.nouts <= kSharedWins) {
            const uint32_t cus = (uint32_t)row_pass_workgroups(), units = N2 / 2;
            hipLaunchKernelGGL((k2_shared_rows<T, N1, N2, N1 / C1>), dim3(units < cus ? units : cus),
                               dim3(RowGeom<T, N1>::THREADS), 0, s, jt, (const cx<T>*)ws, (cx<T>*)windows(jt, ws),
                               (const uint32_t*)part, meta, (const cx<T>*)tb.tw, (const cx<T>*)tb.stw,
                               (const cx<double>*)tb.fa64, (const cx<double>*)tb.fb64, tb.fshift);
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
        const uint32_t wgs = (uint32_t)(row_pass_workgroups() * row_wgs_per_cu<T, N1>());
        const uint32_t rows = jt.ntiles * N2, inv = jt.ngroups * (N2 / 2 + 1);
        // one row at a time takes 64 registers: four workgroups per CU
        hipLaunchKernelGGL((k2_rows<T, N1, N2>), dim3(rows < 2 * wgs ? rows : 2 * wgs), dim3(RowGeom<T, N1>::THREADS), 0, s, jt,
                           (cx<T>*)ws, (const cx<T>*)tb.tw, (const cx<T>*)tb.stw);
        // eight windows at a time, the rest in the narrowest sum that holds them
        uint32_t o0 = 0;
        for (; o0 + 4 < jt.one.nouts; o0 += 8) mac<8>(jt, ws, o0, stream);
        if (o0 + 2 < jt.one.nouts) mac<4>(jt, ws, o0, stream);
        else if (o0 < jt.one.nouts) mac<2>(jt, ws, o0, stream);
        hipLaunchKernelGGL((k2_rows_inv<T, N1, N2, N1 / C1>), dim3(inv < wgs ? inv : wgs), dim3(RowGeom<T, N1>::THREADS), 0,
                           s, jt, (cx<T>*)windows(jt, ws), (const uint32_t*)part, meta, (const cx<T>*)tb.tw,
                           (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64, (const cx<double>*)tb.fb64, tb.fshift);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    // `jt.one` describes the windows as one-chunk groups here
    static int shared_pass3(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
        JobTable w = jt;
        w.tile0 = w.one.tile_begin = 0;
        return pass3(w, windows(jt, ws), part, meta, tb, stream);
    }
    static int pass3(const JobTable& jt, void* ws, uint32_t*, TileMeta* meta, const Tables& tb, void* stream) {
        dim3 grid(jt.ngroups * (N1 / C3)), block(G3::THREADS);
        hipLaunchKernelGGL((k2_pass3<T, N1, N2>), grid, block, 0, (hipStream_t)stream, jt, (const cx<T>*)ws, meta,
                           (const cx<T>*)tb.tw, (const cx<T>*)tb.stw);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
};

// Classes with rows of 4096 and split columns (L = 4096 n2, n2 = P 2^b): the
// wave-level column and row passes above, and the workgroup-wide Stockham pass 3
// of conv_kernels.hpp, whose columns carry the radix-P stage (RC points per
// thread).
template <typename T, int N2, int B3, int RC>
struct ClassImplS {
    static constexpr int N1 = 4096, C1 = PSplitGeom<T, N1, N2>::C, NCB1 = N1 / C1;
    static constexpr size_t kWsExtra = BitPlanes<N1, N2>::kTile;
    static int pass1(const JobTable& jt, void* ws, uint32_t* part, TileMeta*, const Tables& tb, void* stream) {
        return launch_split<T, N1, N2, N2>(jt, ws, part, tb.tw2, tb, stream);
    }
    static int pass2(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
        return launch_row_pass<T, N1, N2, NCB1>(jt, ws, part, meta, tb, stream);
    }
    static int pass3(const JobTable& jt, void* ws, uint32_t*, TileMeta* meta, const Tables& tb, void* stream) {
        dim3 grid(jt.ngroups * (N1 / B3)), block(B3 * (N2 / 2 / RC));
        hipLaunchKernelGGL((k_pass3<T, N1, N2, B3, RC, N2, true>), grid, block, 0, (hipStream_t)stream, jt,
                           (const cx<T>*)ws, meta, (const cx<T>*)tb.tw2);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
};

}  // namespace pa
