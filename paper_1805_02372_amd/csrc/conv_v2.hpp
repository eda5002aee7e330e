// Tile pipeline for the long FFT length classes (L = 8192 * n2, n2 = 128..2048):
// the same three passes as conv_kernels.hpp (see there for the mathematics),
// restructured around wave-level transforms (wave_fft.hpp):
//
//  * pass 1: the workgroup stages the key/seed bits of its C columns in LDS
//    (one funnel-shifted word per row instead of one load per point), each
//    wave transforms G whole columns (n2 <= 1024) or one half of a column
//    after a radix-2 split (n2 = 2048), and an LDS transpose turns the
//    column-major results into C-element row segments for the stores.
//  * pass 2: a row of 8192 points is a radix-8 stage across the 8 waves
//    (decimation in frequency, registers only) followed by one 1024-point
//    transform per wave; the inverse runs the same steps in reverse.  Two
//    workgroup barriers per row transform.
//  * pass 3: C columns are read as C-element row segments, transposed in
//    LDS, each wave inverts G columns, output bits are OR-ed into an LDS bit
//    array and stored as C-bit groups.
#pragma once
#include <type_traits>

#include "conv_kernels.hpp"
#include "wave_fft.hpp"

namespace pa {

template <typename T, int N2> struct P1Geom {
    static constexpr int W = N2 > 1024 ? N2 / 1024 : 1;    // waves per column
    static constexpr int M = N2 > 1024 ? 1024 : N2;        // wave transform size
    static constexpr int G = 1024 / M;                     // columns per wave
    static constexpr int WAVES = (sizeof(T) == 4 && W > 1) ? 16 : 8;
    static constexpr int C = WAVES * G / W;                // columns per workgroup
    static constexpr int THREADS = WAVES * 64;
    static_assert(W <= 2, "column length up to 2048");
    static constexpr bool kPlanes = sizeof(T) == 4 && C == 8;   // bits from the planes of k2_bits
    static_assert(C <= 64 && (C & (C - 1)) == 0, "column block");
};

template <typename T, int N2> struct P3Geom {
    static constexpr int M = N2 / 2;                       // Hermitian half
    static constexpr int G = 1024 / M;
    static constexpr int WAVES = (sizeof(T) == 4 && G == 1) ? 16 : 8;   // >= 128 B row segments
    static constexpr int C = WAVES * G;
    static constexpr int THREADS = WAVES * 64;
    static constexpr int CW = (C + 31) / 32;               // 32-bit words per output row
    static constexpr int SLOTS = (WAVES * kWaveSlots > M * C) ? WAVES * kWaveSlots : M * C;
    // LDS with the stage tables and Hermitian twiddles copied in (the twiddles
    // share space with the output bit array) vs without; copy them only when
    // the workgroups per CU (160 KB of LDS) stay the same.
    static constexpr size_t kBits = (size_t)WAVES * 64 * 4;   // 32 output bits per lane
    static constexpr size_t kHtw = (size_t)M * sizeof(cx<T>);
    static constexpr size_t kBase = (size_t)SLOTS * sizeof(cx<T>) + C * sizeof(T) + 64;
    static constexpr size_t kWithout = kBase + kBits;
    static constexpr size_t kWith = kBase + (kBits > kHtw ? kBits : kHtw) + wfft_lds_entries(M) * sizeof(cx<T>);
    static constexpr bool LDS_TAB = kWith <= 163840 && (163840 / kWith) >= (163840 / kWithout);
    // workgroups per CU that the LDS allows; registers are capped to match
    static constexpr int MIN_WG = (163840 / (LDS_TAB ? kWith : kWithout)) >= 2 ? 2 : 1;
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

// XCD-aware workgroup order: the hardware deals consecutive workgroups to the
// 8 XCDs in turn; remap so that each XCD gets a contiguous range of logical
// blocks (neighbouring column blocks of pass 1 share bit words in its L2).
__device__ __forceinline__ uint32_t xcd_block() {
    const uint32_t b = blockIdx.x, n = gridDim.x;
    return (n & 7u) ? b : (b & 7u) * (n >> 3) + (b >> 3);
}

// ------------------------------------------------------------------ pass 1
// Bit planes.  A pass-1 workgroup of 8 columns needs one byte of key bits and
// one of seed bits from every row of the tile, rows 1 KB apart: read in place,
// each byte costs a cache line on its way to the compute unit, and staging
// them took a fifth of pass 1.  For the FP32 classes with 8 columns per
// workgroup a small kernel first transposes them, coalesced, into two planes
// per tile after the launch's tiles in the workspace: byte cb n2 + r of the
// key plane holds the placed key bits at positions 8 cb + 8192 r .. + 7 (bit
// q: position + q), the seed plane the seed bits there (zero from the window
// end on).  Pass 1 then reads n2 contiguous bytes of each.
template <int N1, int N2> struct BitPlanes {
    static constexpr size_t kPlane = (size_t)N2 * (N1 / 8);
    static constexpr size_t kTile = 2 * kPlane;   // key plane, then seed plane
    template <typename T>
    __device__ static const uint8_t* key(const cx<T>* ws, uint32_t ntiles, uint32_t lt) {
        return reinterpret_cast<const uint8_t*>(ws + (size_t)ntiles * ((size_t)N1 * N2)) + (size_t)lt * kTile;
    }
};

// 8 x 8 byte transpose: byte c of x[q] moves to byte q of x[c].
__device__ __forceinline__ void transpose8x8(uint64_t (&x)[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint64_t a = x[q], b = x[q + 4];
        x[q] = (a & 0xFFFFFFFFull) | (b << 32);
        x[q + 4] = (a >> 32) | (b & 0xFFFFFFFF00000000ull);
    }
    constexpr uint64_t m16 = 0x0000FFFF0000FFFFull, m8 = 0x00FF00FF00FF00FFull;
#pragma unroll
    for (int q = 0; q < 8; q += (q & 1) ? 3 : 1) {   // q = 0, 1, 4, 5
        const uint64_t a = x[q], b = x[q + 2];
        x[q] = (a & m16) | ((b & m16) << 16);
        x[q + 2] = ((a >> 16) & m16) | (b & ~m16);
    }
#pragma unroll
    for (int q = 0; q < 8; q += 2) {
        const uint64_t a = x[q], b = x[q + 1];
        x[q] = (a & m8) | ((b & m8) << 8);
        x[q + 1] = ((a >> 8) & m8) | (b & ~m8);
    }
}

// 64-bit extractions for k2_bits, split into the word loads and the shifts,
// so that a thread issues all its loads back to back: both words of every
// extraction are loaded (indices clamped to the array of nw words) and both
// are used whatever the shift, so no load sits behind a branch.  Same results
// as extract_bits / placed_key_bits<64>.
struct Ext64 {
    uint64_t w;     // first word
    uint32_t s;     // bit offset in it
    uint64_t mask;  // cnt low bits
};
__device__ __forceinline__ Ext64 ext64(uint64_t pos, uint32_t cnt) {
    return Ext64{pos >> 6, (uint32_t)(pos & 63), cnt >= 64 ? ~0ull : ((1ull << (cnt & 63)) - 1ull)};
}
__device__ __forceinline__ void ext64_load(const uint64_t* __restrict__ a, uint64_t nw, const Ext64& e,
                                           uint64_t& lo, uint64_t& hi) {
    lo = a[e.w < nw ? e.w : nw - 1];
    hi = a[e.w + 1 < nw ? e.w + 1 : nw - 1];
}
__device__ __forceinline__ uint64_t ext64_value(const Ext64& e, uint64_t lo, uint64_t hi) {
    return ((lo >> e.s) | ((hi << 1) << (63 - e.s))) & e.mask;   // s = 0: hi drops out
}
// The two extractions of the placed key bits at positions s0 .. s0 + 63
// (position t holds key bit j0 + ((t + bi - 1) mod L) when that index is < bi):
// the positions before the wrap to u = 0, then those after it, shifted by fs.
struct PlacedKey64 {
    Ext64 e1, e2;
    uint32_t fs;
};
__device__ __forceinline__ PlacedKey64 placed_key64(uint64_t j0, uint32_t bi, uint32_t L, uint32_t s0) {
    uint32_t u0 = s0 + bi - 1;
    if (u0 >= L) u0 -= L;
    const uint32_t fs = u0 + 64 <= L ? 64u : L - u0;
    const uint32_t c1 = u0 < bi ? (bi - u0 < fs ? bi - u0 : fs) : 0u;
    const uint32_t c2 = fs < 64 ? (bi < 64 - fs ? bi : 64 - fs) : 0u;
    return PlacedKey64{ext64(j0 + u0, c1), ext64(j0, c2), fs & 63u};   // c2 = 0 when fs = 64
}

// Workgroup: 128 rows x 8 word columns (64 positions each) of one tile, both
// planes, 256 threads.  Loads: 8 consecutive lanes take 8 consecutive words
// of one row (64 contiguous bytes of key or seed), 4 rows per lane, every
// load of a lane issued before the first wait.  The words go to LDS; then
// each lane of one half of the workgroup (key plane, seed plane) reads the
// word column of 8 consecutive rows, transposes the 8 x 8 bytes and stores
// one 64-bit word (8 rows) per byte column, so that 16 consecutive lanes write
// one whole 128-byte line.
constexpr int kBitsRows = 128, kBitsCols = 8;
// LDS slot of (row r, word w): bits 3..4 of r permute the rows within each
// 256-byte bank span and bits 3..5 of r are XOR-ed into the word, so that both
// the row-wise writes and the column-wise reads of 64 lanes touch every bank
// pair at most twice.
__device__ __forceinline__ int bits_slot(int r, int w) {
    return (r ^ ((r >> 3) & 3)) * kBitsCols + (w ^ ((r >> 3) & 7));
}
template <int N1, int N2>
__global__ void __launch_bounds__(256) k2_bits(JobTable jt, uint8_t* __restrict__ planes) {
    constexpr int R = kBitsRows, WC = kBitsCols, RPL = R * WC / 256;   // rows per lane
    constexpr int NRB = N2 / R, NWB = N1 / 64 / WC;
    constexpr uint32_t L = (uint32_t)N1 * N2;
    static_assert(N2 % R == 0 && (N1 / 64) % WC == 0 && RPL == 4 && WC * 16 * 2 == 256, "workgroup block");
    __shared__ uint64_t wbits[2][R * WC];   // key words, seed words
    const uint32_t b = blockIdx.x;
    const uint32_t lt = b / (NRB * NWB), rem = b % (NRB * NWB);
    const uint32_t rb = rem / NWB, wb = rem % NWB;
    const uint32_t t = jt.tile0 + lt;
    const JobDesc jd = find_job(jt, t);
    const TileGeo g = tile_geo(jd, t - jd.tile_begin);
    const uint32_t bi = (uint32_t)g.bi, win = (uint32_t)(g.bi + g.bo - 1);
    const uint64_t nkw = (jd.n + 63) >> 6, nsw = (jd.n + jd.m - 1 + 63) >> 6;   // key and seed words
    const int tid = threadIdx.x;
    {
        const int wl = tid & (WC - 1);
        const uint32_t wc = wb * WC + (uint32_t)wl;
        PlacedKey64 pk[RPL];
        Ext64 se[RPL];
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            const int rl = tid / WC + (256 / WC) * q;
            const uint32_t s0 = wc * 64 + (uint32_t)N1 * (rb * R + (uint32_t)rl);
            pk[q] = placed_key64(g.j0, bi, L, s0);
            const uint32_t nv = s0 < win ? ((win - s0) < 64u ? (win - s0) : 64u) : 0u;
            se[q] = ext64(g.sigma + s0, nv);
        }
        uint64_t kw[RPL][4], sw[RPL][2];
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            ext64_load(jd.key, nkw, pk[q].e1, kw[q][0], kw[q][1]);
            ext64_load(jd.key, nkw, pk[q].e2, kw[q][2], kw[q][3]);
            ext64_load(jd.seed, nsw, se[q], sw[q][0], sw[q][1]);
        }
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            const int sl = bits_slot(tid / WC + (256 / WC) * q, wl);
            wbits[0][sl] = ext64_value(pk[q].e1, kw[q][0], kw[q][1]) |
                           (ext64_value(pk[q].e2, kw[q][2], kw[q][3]) << pk[q].fs);
            wbits[1][sl] = ext64_value(se[q], sw[q][0], sw[q][1]);
        }
    }
    __syncthreads();
    const int pl = tid >> 7, p = tid & 15, wl = (tid >> 4) & (WC - 1);   // plane, rows 8 p .. 8 p + 7, word
    uint64_t x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = wbits[pl][bits_slot(8 * p + i, wl)];
    transpose8x8(x);
    uint8_t* dst = planes + (size_t)lt * BitPlanes<N1, N2>::kTile + (size_t)pl * BitPlanes<N1, N2>::kPlane +
                   (size_t)((wb * WC + (uint32_t)wl) * 8) * N2 + rb * R + 8 * p;
#pragma unroll
    for (int c = 0; c < 8; ++c) *reinterpret_cast<uint64_t*>(dst + (size_t)c * N2) = x[c];
}

template <typename T, int N1, int N2>
__global__ void __launch_bounds__((P1Geom<T, N2>::THREADS))
k2_pass1(JobTable jt, cx<T>* __restrict__ ws, uint32_t* __restrict__ part, const cx<T>* __restrict__ tw,
         const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64,
         int fshift) {
    using Gm = P1Geom<T, N2>;
    constexpr int C = Gm::C, G = Gm::G, W = Gm::W, M = Gm::M, NJ = M / 16;
    constexpr uint32_t L = (uint32_t)N1 * N2;
    constexpr int NCB = N1 / C;
    constexpr int SLOTS = (Gm::WAVES * kWaveSlots > N2 * C) ? Gm::WAVES * kWaveSlots : N2 * C;
    static_assert(2 * N2 * sizeof(uint64_t) <= SLOTS * sizeof(cx<T>), "bit rows fit the LDS union");
    static_assert(G * 16 * sizeof(Root64) <= kWaveSlots * sizeof(cx<T>), "twiddle factors fit a wave region");
    __shared__ __align__(16) cx<T> lds[SLOTS];
    __shared__ __align__(16) cx<T> st[wfft_lds_entries(M)];
    __shared__ uint32_t wsum;
    uint64_t* kbits = reinterpret_cast<uint64_t*>(lds);   // consumed before the wave regions are used
    uint64_t* sbits = kbits + N2;

    const uint32_t blk = xcd_block();
    const uint32_t lt = blk / NCB;
    const uint32_t cb = blk % NCB;
    const uint32_t t = jt.tile0 + lt;
    const JobDesc jd = find_job(jt, t);
    const TileGeo g = tile_geo(jd, t - jd.tile_begin);
    const int tid = threadIdx.x;
    const uint32_t bi = (uint32_t)g.bi, win = (uint32_t)(g.bi + g.bo - 1);
    if (tid == 0) wsum = 0;
    clear_window(g, cb, NCB, tid, Gm::THREADS);
    wfft_load_lds<T, M>(st, stw, tid, Gm::THREADS);
    __syncthreads();

    // stage the bits of this workgroup's C columns: rows r = tid + q * THREADS
    constexpr int RPT = (N2 + Gm::THREADS - 1) / Gm::THREADS;
    uint32_t pc = 0;
    uint64_t kb[RPT], sb[RPT];
    constexpr bool kPlanes = Gm::kPlanes;
    const uint8_t* kp = nullptr;
    if constexpr (kPlanes) kp = BitPlanes<N1, N2>::key(ws, jt.ntiles, lt) + (size_t)cb * N2;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = tid + q * Gm::THREADS;
        kb[q] = 0;
        sb[q] = 0;
        if (r < N2) {
            if constexpr (kPlanes) {
                kb[q] = kp[r];
                sb[q] = kp[BitPlanes<N1, N2>::kPlane + r];
            } else {
                const uint32_t s0 = cb * C + (uint32_t)N1 * (uint32_t)r;
                kb[q] = placed_key_bits<C>(jd.key, g.j0, bi, L, s0);
                const uint32_t nv = s0 < win ? ((win - s0) < (uint32_t)C ? (win - s0) : (uint32_t)C) : 0u;
                sb[q] = extract_bits(jd.seed, g.sigma + s0, nv);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = tid + q * Gm::THREADS;
        if (r < N2) {
            kbits[r] = kb[q];
            sbits[r] = sb[q];
            pc += (uint32_t)__popcll(kb[q]);
        }
    }
    atomicAdd(&wsum, pc);
    __syncthreads();

    const int wv = tid >> 6, l = tid & 63;
    int f, ka = 0, j, grp;
    if constexpr (W == 1) {
        grp = l / NJ;
        j = l % NJ;
        f = wv * G + grp;
    } else {
        f = wv / W;
        ka = wv % W;
        j = l;
        grp = 0;
    }
    const uint32_t t1 = cb * C + (uint32_t)f;
    // Four-step twiddle w_L^{t1 k2} = base * c_i with
    //   W = 1: k2 = j + NJ i,           base = w_L^{t1 j},          c_i = w_L^{NJ t1 i}
    //   W = 2: k2 = 2 (j + 64 i) + ka,  base = w_L^{t1 (2 j + ka)}, c_i = w_L^{128 t1 i}
    // Each lane fetches its share of its group's 16 factors now (latency hidden
    // behind the transform); they are exchanged through LDS afterwards.
    constexpr int LPG = W == 1 ? NJ : 64;            // lanes per transform group
    constexpr int CPL = (16 + LPG - 1) / LPG;        // factors fetched per lane
    constexpr uint32_t CSTEP = W == 1 ? (uint32_t)NJ : 128u;
    const Root64 base = root64(fa64, fb64, fshift, W == 1 ? t1 * (uint32_t)j : t1 * (uint32_t)(2 * j + ka));
    Root64 cf[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
        const int i = j + q * LPG;
        cf[q] = root64(fa64, fb64, fshift, i < 16 ? CSTEP * t1 * (uint32_t)i : 0u);
    }
    // bit f of row r from the 32-bit half holding it (unconditional reads, selects)
    const uint32_t* __restrict__ kb32 = reinterpret_cast<const uint32_t*>(kbits) + (f >> 5);
    const uint32_t* __restrict__ sb32 = reinterpret_cast<const uint32_t*>(sbits) + (f >> 5);
    const uint32_t fs = (uint32_t)f & 31u;
    auto z = [&](int r) -> cx<T> {
        const uint32_t kw = kb32[2 * r], sw = sb32[2 * r];
        const T xb = ((kw >> fs) & 1u) ? T(1) : T(0);
        const T sv = ((sw >> fs) & 1u) ? T(1) : T(-1);
        const T wb = (t1 + (uint32_t)N1 * (uint32_t)r < win) ? sv : T(0);
        return cx<T>{xb, wb};
    };
    cx<T> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int e = j + i * NJ;
        if constexpr (W == 1) {
            v[i] = z(e);
        } else {
            // radix-2 split of the 2048-point column: half ka, twiddle w_2048^{e ka}
            const cx<T> a = z(e), b = z(e + 1024);
            if (ka == 0) v[i] = a + b;
            else v[i] = cmul(a - b, tw[e * (N1 / 2048)]);
        }
    }
    __syncthreads();  // bits consumed; LDS becomes wave regions
    cx<T>* reg = lds + wv * kWaveSlots + (W == 1 ? grp * (M + M / 16) : 0);
    wave_fft_lds<T, -1, M>(v, reg, j, st);

    // exchange the factors through this wave's own region (its transform is done)
    Root64* cw = reinterpret_cast<Root64*>(lds + wv * kWaveSlots) + grp * 16;
    wave_sync();
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
        const int i = j + q * LPG;
        if (i < 16) cw[i] = cf[q];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = cmul(v[i], rounded<T>(mul64(base, cw[i])));
    __syncthreads();
    // transpose through LDS for row-segment stores.  With W = 2 the rows
    // k2 = 2 e + ka of each half go to a tile of their own (the second one 8
    // slots further, off the first's banks), so that a wave writes
    // consecutive rows e as in the W = 1 layout
    constexpr int HALF = M * C + 8;
    static_assert(W * HALF <= SLOTS, "transposition tiles fit the LDS union");
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int e = j + i * NJ;
        lds[ka * HALF + tslot<C>(e, f)] = v[i];
    }
    __syncthreads();
    cx<T>* __restrict__ Y = ws + (size_t)lt * L;
    static_assert((N2 * C) % Gm::THREADS == 0, "store tile");
    constexpr int SPT = N2 * C / Gm::THREADS;
    cx<T> o[SPT];
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const int idx = tid + q * Gm::THREADS, k2 = idx / C;
        o[q] = lds[(k2 % W) * HALF + tslot<C>(k2 / W, idx % C)];
    }
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const int idx = tid + q * Gm::THREADS;
        Y[(size_t)(idx / C) * N1 + cb * C + (idx % C)] = o[q];
    }
    if (tid == 0) part[(size_t)lt * NCB + cb] = wsum;
}

// Pass 1 for FP32 columns of 2048 points, as two halves.  Half ka (outputs
// k2 = 2 e + ka) is the 1024-point transform of z(e) + z(e + 1024) (ka = 0) or
// (z(e) - z(e + 1024)) w_2048^e (ka = 1): a radix-2 split in decimation in
// frequency.  A workgroup of eight waves takes one half of 8 columns (one
// column per wave), so it needs the LDS of one half (the block's bits, then
// the wave regions, then the transposition tile: 78 KB, two workgroups per
// CU) and the registers of one 1024-point column; the two halves of a column
// block read the same bit-plane bytes.
struct P1hArgs {
    JobDesc jd;
    TileGeo g;
    uint32_t lt, cb, ntiles;
};

template <typename T, int N1, int KA>
__device__ __forceinline__ uint32_t pass1_half_body(const P1hArgs& A, cx<T>* __restrict__ ws, cx<T>* lds,
                                                    const cx<T>* st, const cx<T>* __restrict__ tw,
                                                    const cx<double>* __restrict__ fa64,
                                                    const cx<double>* __restrict__ fb64, int fshift) {
    constexpr int N2 = 2048, M = 1024, C = 8, THREADS = 512, NJ = M / 16;
    constexpr uint32_t L = (uint32_t)N1 * N2;
    const int tid = threadIdx.x, wv = tid >> 6, j = tid & 63;
    const TileGeo& g = A.g;
    const uint32_t bi = (uint32_t)g.bi, win = (uint32_t)(g.bi + g.bo - 1);
    const int f = wv;   // this wave's column
    const uint32_t t1 = A.cb * C + (uint32_t)f;
    uint16_t* fld = reinterpret_cast<uint16_t*>(lds);   // per row: key bits (low byte), seed bits (high byte)
    uint32_t pc = 0;
    __syncthreads();   // the previous half's stores have read the LDS
    const uint8_t* kp = BitPlanes<N1, N2>::key(ws, A.ntiles, A.lt) + (size_t)A.cb * N2;
    for (int r = tid; r < N2; r += THREADS) {
        const uint32_t kb = kp[r];
        const uint32_t sb = kp[BitPlanes<N1, N2>::kPlane + r];
        fld[r] = (uint16_t)(kb | (sb << 8));
        pc += (uint32_t)__popc(kb);
    }
    __syncthreads();
    // four-step twiddle w_L^{t1 k2}, k2 = 2 (j + 64 i) + KA: base w_L^{t1 (2 j + KA)}
    // times c_i = w_L^{128 t1 i} (lane i < 16 fetches c_i; exchanged after the transform)
    const Root64 base = root64(fa64, fb64, fshift, t1 * (uint32_t)(2 * j + KA));
    const Root64 cf = root64(fa64, fb64, fshift, j < 16 ? 128u * t1 * (uint32_t)j : 0u);
    auto z = [&](int r) -> cx<T> {
        const uint32_t w = fld[r];
        const T xb = ((w >> f) & 1u) ? T(1) : T(0);
        const T sv = ((w >> (8 + f)) & 1u) ? T(1) : T(-1);
        return cx<T>{xb, (t1 + (uint32_t)N1 * (uint32_t)r < win) ? sv : T(0)};
    };
    cx<T> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int e = j + i * NJ;
        const cx<T> a = z(e), b = z(e + M);
        if constexpr (KA == 0) v[i] = a + b;
        else v[i] = cmul(a - b, tw[e * (N1 / N2)]);
    }
    __syncthreads();   // bits consumed; LDS becomes wave regions
    cx<T>* reg = lds + wv * kWaveSlots;
    wave_fft_lds<T, -1, M>(v, reg, j, st);
    Root64* cw = reinterpret_cast<Root64*>(reg);
    wave_sync();
    if (j < 16) cw[j] = cf;
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = cmul(v[i], rounded<T>(mul64(base, cw[i])));
    __syncthreads();
    // transpose through LDS for row-segment stores (rows k2 = 2 e + KA)
#pragma unroll
    for (int i = 0; i < 16; ++i) lds[tslot<C>(j + i * NJ, f)] = v[i];
    __syncthreads();
    cx<T>* __restrict__ Y = ws + (size_t)A.lt * L;
    constexpr int SPT = M * C / THREADS;
    cx<T> o[SPT];
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const int idx = tid + q * THREADS;
        o[q] = lds[tslot<C>(idx / C, idx % C)];
    }
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const int idx = tid + q * THREADS;
        Y[(size_t)(2 * (idx / C) + KA) * N1 + A.cb * C + (idx % C)] = o[q];
    }
    return pc;
}

// Each half in a workgroup of its own: logical block 2 b + KA
// takes half KA of column block b (the two read the same bit words, through
// the L2 of one XCD).  Half 0 clears the window and reports the weight.
template <typename T, int N1>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
k2_pass1s(JobTable jt, cx<T>* __restrict__ ws, uint32_t* __restrict__ part, const cx<T>* __restrict__ tw,
          const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64, const cx<double>* __restrict__ fb64,
          int fshift) {
    constexpr int M = 1024, C = 8, THREADS = 512;
    constexpr int NCB = N1 / C;
    constexpr int SLOTS = 8 * kWaveSlots;
    static_assert(M * C <= SLOTS && 2048 * (int)sizeof(uint16_t) <= SLOTS * (int)sizeof(cx<T>), "LDS union");
    __shared__ __align__(16) cx<T> lds[SLOTS];
    __shared__ __align__(16) cx<T> st[wfft_lds_entries(M)];
    __shared__ uint32_t wsum;
    const uint32_t blk = xcd_block();
    const uint32_t lb = blk >> 1;
    const bool second = (blk & 1u) != 0;
    P1hArgs A;
    A.lt = lb / NCB;
    A.cb = lb % NCB;
    A.ntiles = jt.ntiles;
    const uint32_t t = jt.tile0 + A.lt;
    A.jd = find_job(jt, t);
    A.g = tile_geo(A.jd, t - A.jd.tile_begin);
    const int tid = threadIdx.x;
    if (tid == 0) wsum = 0;
    if (!second) clear_window(A.g, A.cb, NCB, tid, THREADS);
    wfft_load_lds<T, M>(st, stw, tid, THREADS);
    if (second) {
        (void)pass1_half_body<T, N1, 1>(A, ws, lds, st, tw, fa64, fb64, fshift);
        return;
    }
    const uint32_t pc = pass1_half_body<T, N1, 0>(A, ws, lds, st, tw, fa64, fb64, fshift);
    atomicAdd(&wsum, pc);
    __syncthreads();
    if (tid == 0) part[(size_t)A.lt * NCB + A.cb] = wsum;
}

// ------------------------------------------------------------------ pass 2
// Row pass.  A workgroup transforms rows of N1 points, PT per lane, in W =
// N1 / (64 PT) waves: a radix-W stage across the waves (decimation in frequency,
// registers only), one workgroup exchange, one transform of M = 64 PT points per
// wave; the inverse runs the same steps in reverse.  Two workgroup barriers per
// row transform.  Rows of 4096 take 8 points per lane (8 x 8 x 8 x 8: a mirror
// pair and the group's sum are 48 registers per lane in FP32, so that two
// workgroups of 8 waves share a CU); rows of 8192 take 16 (8 x 4 x 16 x 16).
template <typename T, int N1> struct RowGeom {
    static constexpr int PT = N1 >= 8192 ? 16 : 8;
    static constexpr int W = N1 / (64 * PT), M = 64 * PT, S = PT / W, THREADS = N1 / PT;
    static constexpr int SLOTS = M + M / (PT == 16 ? 16 : 8);   // LDS slots of a wave's region
    static_assert(W == 8 && S * W == PT, "row geometry");
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
    cx<T> tw1[G::S * (G::W - 1)];
    cx<T> t3[G::PT == 8 ? 7 : 1];
};

template <typename T, int N1>
__device__ __forceinline__ void row_setup(RowSmem<T, N1>& S, RowReg<T, N1>& R, const cx<T>* __restrict__ tw,
                                          const cx<T>* __restrict__ stw, int tid) {
    using G = RowGeom<T, N1>;
#pragma unroll
    for (int s = 0; s < G::S; ++s)
#pragma unroll
        for (int ka = 1; ka < G::W; ++ka) R.tw1[s * (G::W - 1) + ka - 1] = tw[ka * (tid + G::THREADS * s)];
    if constexpr (G::PT == 8) {
        const int l = tid & 63;
#pragma unroll
        for (int r = 1; r < 8; ++r) R.t3[r - 1] = tw[l * r * (N1 / 512)];
        if (tid < 56) S.st[tid] = tw[(tid & 7) * ((tid >> 3) + 1) * (N1 / 64)];
    } else {
        wfft_load_lds<T, 1024>(S.st, stw, tid, G::THREADS);
    }
    __syncthreads();
}

// Transform of M points by one wave, register i holding element l + 64 i before
// and after; `reg` is the wave's own LDS region.  512 points: three Stockham
// stages of radix 8 (wave_fft.hpp holds the 1024-point transform).
template <typename T, int N1, int DIR>
__device__ __forceinline__ void row_wave_fft(RowVec<T, N1>& v, cx<T>* __restrict__ reg, int l,
                                             const RowSmem<T, N1>& S, const RowReg<T, N1>& R) {
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
template <typename T, int N1>
__device__ __forceinline__ void row_forward(RowVec<T, N1>& a, RowSmem<T, N1>& S, const RowReg<T, N1>& R,
                                            int tid) {
    using G = RowGeom<T, N1>;
    const int wv = tid >> 6, l = tid & 63;
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
template <typename T, int N1>
__device__ __forceinline__ void row_inverse(RowVec<T, N1>& a, RowSmem<T, N1>& S, const RowReg<T, N1>& R,
                                            int tid) {
    using G = RowGeom<T, N1>;
    const int wv = tid >> 6, l = tid & 63;
    cx<T>* reg = S.data + wv * G::SLOTS;
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
    __syncthreads();
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

// Workgroups per CU: rows of 4096 in FP32 two (16 waves), else one.
template <typename T, int N1> constexpr int row_wgs_per_cu() { return N1 == 4096 && sizeof(T) == 4 ? 2 : 1; }
template <typename T, int N1, int N2, int NCB1>
__global__ void __launch_bounds__((RowGeom<T, N1>::THREADS))
__attribute__((amdgpu_waves_per_eu(row_wgs_per_cu<T, N1>() * RowGeom<T, N1>::THREADS / 256)))
k2_pass2(JobTable jt, cx<T>* __restrict__ ws, const uint32_t* __restrict__ part, TileMeta* __restrict__ meta,
         const cx<T>* __restrict__ tw, const cx<T>* __restrict__ stw, const cx<double>* __restrict__ fa64,
         const cx<double>* __restrict__ fb64, int fshift) {
    __shared__ __align__(16) RowSmem<T, N1> S;
    __shared__ uint32_t wsum;
    const uint32_t units = jt.ngroups * (uint32_t)(N2 / 2);
    RowReg<T, N1> R;
    row_setup<T, N1>(S, R, tw, stw, threadIdx.x);
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x)
        row_unit<T, N1, N2, NCB1>(u, jt, ws, part, meta, S, R, wsum, fa64, fb64, fshift);
}

// ------------------------------------------------------------------ pass 3
// rint(z) mod 4 for an integral r (FP32: |r| < 2^31; FP64: |r| < 2^51)
__device__ __forceinline__ uint32_t low2(float r) { return (uint32_t)(int)r & 3u; }
__device__ __forceinline__ uint32_t low2(double r) {
    const double q = r * 0.25;
    return (uint32_t)(int)((q - floor(q)) * 4.0) & 3u;
}

template <typename T, int N1, int N2>
__global__ void __launch_bounds__((P3Geom<T, N2>::THREADS))
__attribute__((amdgpu_waves_per_eu(P3Geom<T, N2>::MIN_WG * P3Geom<T, N2>::WAVES / 4)))
k2_pass3(JobTable jt, const cx<T>* __restrict__ ws, TileMeta* __restrict__ meta, const cx<T>* __restrict__ tw,
         const cx<T>* __restrict__ stw) {
    using Gm = P3Geom<T, N2>;
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

    const uint32_t t = jt.group0 + blockIdx.x / NCB;   // group
    const uint32_t cb = blockIdx.x % NCB;
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
            for (int k = tid; k < M; k += Gm::THREADS) U.htw[k] = tw[k * (N1 / N2)];
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
            const cx<T> wk = LT ? U.htw[k] : tw[k * (N1 / N2)];
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

template <typename T, int N1, int N2, int NCB1>
int launch_row_pass(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
    const uint32_t units = jt.ngroups * (N2 / 2);
    const uint32_t wgs = (uint32_t)(row_pass_workgroups() * row_wgs_per_cu<T, N1>());
    hipLaunchKernelGGL((k2_pass2<T, N1, N2, NCB1>), dim3(units < wgs ? units : wgs),
                       dim3(RowGeom<T, N1>::THREADS), 0,
                       (hipStream_t)stream, jt, (cx<T>*)ws, (const uint32_t*)part, meta, (const cx<T>*)tb.tw,
                       (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64, (const cx<double>*)tb.fb64, tb.fshift);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T, int N1, int N2>
struct ClassImpl2 {
    using G1 = P1Geom<T, N2>;
    using G3 = P3Geom<T, N2>;
    static constexpr int C1 = G1::C, C3 = G3::C;
    // workspace bytes per tile beyond its points: the bit planes
    static constexpr size_t kWsExtra = G1::kPlanes ? BitPlanes<N1, N2>::kTile : 0;
    static int pass1(const JobTable& jt, void* ws, uint32_t* part, TileMeta*, const Tables& tb, void* stream) {
        dim3 grid(jt.ntiles * (N1 / C1)), block(G1::THREADS);
        if constexpr (G1::kPlanes) {
            uint8_t* planes = reinterpret_cast<uint8_t*>((cx<T>*)ws + (size_t)jt.ntiles * ((size_t)N1 * N2));
            hipLaunchKernelGGL((k2_bits<N1, N2>), dim3(jt.ntiles * (N2 / kBitsRows) * (N1 / 64 / kBitsCols)), dim3(256),
                               0, (hipStream_t)stream, jt, planes);
        }
        if constexpr (sizeof(T) == 4 && N2 == 2048) {
            static_assert(C1 == 8, "eight columns per workgroup");
            hipLaunchKernelGGL((k2_pass1s<T, N1>), dim3(2 * grid.x), dim3(512), 0, (hipStream_t)stream, jt, (cx<T>*)ws,
                               part, (const cx<T>*)tb.tw, (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64,
                               (const cx<double>*)tb.fb64, tb.fshift);
        } else {
            hipLaunchKernelGGL((k2_pass1<T, N1, N2>), grid, block, 0, (hipStream_t)stream, jt, (cx<T>*)ws, part,
                               (const cx<T>*)tb.tw, (const cx<T>*)tb.stw, (const cx<double>*)tb.fa64,
                               (const cx<double>*)tb.fb64, tb.fshift);
        }
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    static int pass2(const JobTable& jt, void* ws, uint32_t* part, TileMeta* meta, const Tables& tb, void* stream) {
        return launch_row_pass<T, N1, N2, N1 / C1>(jt, ws, part, meta, tb, stream);
    }
    static int pass3(const JobTable& jt, void* ws, uint32_t*, TileMeta* meta, const Tables& tb, void* stream) {
        dim3 grid(jt.ngroups * (N1 / C3)), block(G3::THREADS);
        hipLaunchKernelGGL((k2_pass3<T, N1, N2>), grid, block, 0, (hipStream_t)stream, jt, (const cx<T>*)ws, meta,
                           (const cx<T>*)tb.tw, (const cx<T>*)tb.stw);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
};

// Mixed-radix classes with rows of 4096 (L = 4096 n2, n2 = P 2^b): the
// wave-level row pass above (it does not depend on how n2 factors) between
// the workgroup-wide Stockham column passes of conv_kernels.hpp, whose columns
// carry the radix-P stage (RC points per thread).
template <typename T, int N2, int B1, int B3, int RC>
struct ClassImplS {
    static constexpr int N1 = 4096, NCB1 = N1 / B1;
    static int pass1(const JobTable& jt, void* ws, uint32_t* part, TileMeta*, const Tables& tb, void* stream) {
        dim3 grid(jt.ntiles * NCB1), block(B1 * (N2 / RC));
        hipLaunchKernelGGL((k_pass1<T, N1, N2, B1, RC, N2>), grid, block, 0, (hipStream_t)stream, jt, (cx<T>*)ws,
                           part, (const cx<T>*)tb.tw2, (const cx<T>*)tb.fa, (const cx<T>*)tb.fb, tb.fshift);
        return hipGetLastError() == hipSuccess ? 0 : -1;
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
