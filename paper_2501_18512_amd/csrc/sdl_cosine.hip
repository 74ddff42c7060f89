// Cosine similarity between the replicas' outer gradients (Appendix of the paper, paragraph on
// the outer gradients' cosine similarity) for gfx950 (MI355X).
//
// Four kernels.
//   sdl_gram_kernel   up to 8 replicas: streams g and the M replicas once and accumulates the Gram matrix of
//                     the outer gradients Delta_m = g - float(w_m).  A workgroup is one
//                     64-lane wavefront or four of them; a set of parameters gets a share G of
//                     the launch's workgroups in proportion to its size, and the set's
//                     W = G or 4G wavefronts walk its tiles of 512 consecutive parameters with
//                     a fixed stride (tile k, k + W, k + 2W, ...), lane l owning the eight
//                     parameters [8l, 8l+8) of a tile, so every load instruction of the
//                     wavefront covers one contiguous piece of an array (2 x 1 KiB of fp32,
//                     1 KiB of bf16 through 128-bit accesses).  Each lane keeps its M(M+1)/2
//                     sums in fp64 registers (products of fp32 values are exact in fp64); at
//                     the end the wavefront folds them, half of the sums at each exchange, and
//                     the workgroup writes one partial Gram matrix.  The next tile's loads are issued
//                     before the current tile is consumed.
//   sdl_gram_pair_kernel  the same for 9 to 16 replicas: two wavefronts with half of the matrix each, which
//                     exchange the outer gradients through LDS.
//   sdl_digit_sums_kernel  the same for 13 to 16 replicas and many parameters: the outer gradients as 8-bit digits, whose products
//                     the matrix cores add up exactly.
//   sdl_gram_finalize adds the partial matrices of a set in a fixed order (one thread per entry and
//                     slice of the matrices, then the slices as a tree; a set with many partial matrices in
//                     two launches) and derives cos and the mean over pairs.  The same kernel adds
//                     the Gram matrices of several sets (fragment from spans, unions of fragments).
// No atomics: the order of every sum depends on the sizes alone, so results are reproducible.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "sdl.h"
#include "sdl_device.h"

namespace {

using namespace sdl_device;

constexpr int kLaneElems = 8;                   // consecutive parameters a lane owns in a tile
constexpr int kTile = kLaneElems * kWave;       // 512
constexpr int kMaxSets = 224;                   // parameter sets per launch
constexpr int kWindows = 48;                    // windows per launch: a set holding a share of 4/48 or more is cut
constexpr int kMaxPieces = kMaxSets + kWindows;
// A launch takes more sets than kFewSets only while they have no more than kManyParams parameters: fewer launches, but each set gets a smaller
// share of the workgroups, and up to 8 replicas a lane's chains of additions are as long as its share (16 parameters at kManyParams, which
// adds nothing to the error of 1e-16).  Whole call with 48 sets a launch and each launch's sums finished by themselves, and now, M = 2 / 4 / 8 / 16:
// 194 sets of 100 to 30000 parameters, 2.5 M in all, 44 / 51 / 69 / 139 us and 20 / 21 / 29 / 52; 195 sets of 256 to 8 M, 35 M in all, 96 / 125 /
// 209 / 371 and 66 / 90 / 153 / 319.
constexpr uint32_t kFewSets = 48;
constexpr uint64_t kManyParams = 1ull << 23;
// Up to 8 replicas, the wavefronts of a workgroup and the workgroups of a launch, which are shared out among the sets. Four wavefronts, whose sums
// are added in LDS, leave a quarter of the matrices to write and to add up.  A launch's shares are rounded up, so as many fewer workgroups are dealt
// out as there are sets.  Whole call with 8192 workgroups of one wavefront and now, M = 1 / 2 / 4 / 8: 1 M parameters 8.6 / 9.7 / 12.5 / 18.0 and 7.7
// / 8.3 / 10.7 / 16.5 us, 4 M 13.6 / 15.3 / 19.9 / 32.8 and 11.4 / 13.1 / 17.8 / 32.6, 32 M 39.3 / 49.5 / 68.4 / 113.4 and 36.3 / 46.9 / 64.9 /
// 108.4, 53 M in 39 sets 57.6 / 74.3 / 103.9 / 172.1 and 55.1 / 72.5 / 100.5 / 168.2, 302 M in 48 sets 287.5 / 379.3 / 563 / 952 and 286.1 / 372.9 /
// 557 / 945; with arrays at odd elements 32 M 42.2 / 53.8 / 78.7 / 131.6 and 39.5 / 50.7 / 76.2 / 129.8, and up to 3 % slower at 2 and 4 M with 7 and
// 8 replicas (21.4 / 24.3 and 22.0 / 24.7; 28.7 / 34.0 and 28.7 / 34.7). 2048 of them are 8 for a compute unit, of which 8 / 7 / 5 / 5 / 4 / 3 / 3 /
// 2 fit it at once by their registers.  Beyond kFewFours 10, from which 2 replicas gain 2 to 4 %; the others lie within 3 % (39 equal sets and 8: 5 % slower).
// M = 1 / 2 / 3 / 4 / 6 / 8, 2048 / 2560: 72 M 71.1 72.4 / 99.5 96.1 / 115.9 117.4 / 137.8 138.4 / 182.0 181.9 / 228.4 228.3, 130 M 129.0 129.9 /
// 175.0 167.3 / 204.1 204.9 / 240.9 242.7 / 317.9 317.6 / 388.4 391.6, 170 M 167.3 168.0 / 223.7 215.3 / 264.6 267.6 / 314.1 318.4 / 403.6 399.5 /
// 514.2 507.0; 302 M in 48 sets, M = 1 / 2 / 4 / 8, 289.6 285.9 / 379.8 374.8 / 563.6 556.9 / 954.5 951.0; 82 M in 39 equal sets 89.9 92.2 / 120.8
// 117.3 / 143.0 144.7 / 171.5 171.3 / 227.2 229.0 / 283.3 297.5; at 8 M, M = 1 / 2 / 4 / 8, 14.9 16.4 / 17.6 19.1 / 24.3 25.3 / 40.6 43.3.
// One wavefront for 8 replicas in more than kFewSets sets (194 sets, 2.5 M parameters in all: 26.8 us, with four 28.8; 195 sets, 35 M 168.9 and
// 170.7). The addresses of the arrays have no say: they would change the order of the sums.
constexpr uint32_t kGramWaves = 4;
constexpr uint32_t kFours = 2048;               // workgroups of four wavefronts: 8 per compute unit
constexpr uint32_t kManyFours = 2560;           // beyond kFewFours parameters
constexpr uint64_t kFewFours = 64u << 20;
constexpr uint32_t kGroups = 8192;              // workgroups of one wavefront
constexpr uint32_t kMaxGroups = 8192;           // what the workspace is sized for


struct Set {
    uint64_t offset;     // first element in the flat arrays
    uint64_t numel;
    uint32_t first_wg;   // first workgroup of the launch that works on this set
    uint32_t G;          // workgroups of this set (>= 1)
};

// What the kernel walks are pieces: a set, or a window of a large set (tile aligned), with its own share of the set's workgroups.  13 bytes
// each, so that as many as possible fit the kernel arguments.
struct GramArgs {
    const float* g;
    const uint16_t* w[8];
    double* partial;               // [workgroup of the launch][M*M]
    uint32_t n_pieces;
    uint32_t waves;                // of a workgroup
    uint32_t group_wg[kMaxPieces / 16 - 1];   // first workgroup of the 16th, 32nd, ... piece
    uint32_t first_wg[kMaxPieces + 1];        // of each piece, then the number of workgroups; 0xffffffff behind it
    uint32_t offset[kMaxPieces];              // first element in the flat arrays, low 32 bits
    uint32_t numel[kMaxPieces];
    uint32_t high[kMaxPieces / 4];            // a byte each: bits 32 to 38 of the offset, and kFast
};
static_assert(sizeof(GramArgs) <= 4096 && kMaxPieces % 16 == 0, "kernel arguments");
constexpr uint32_t kFast = 0x80;              // every array is 16-byte aligned at the piece's start
constexpr uint64_t kMaxOffset = 1ull << 39;

// The lane's number, counted anew: what is computed from it is computed here, not ahead of a loop that needs the registers.  (The offsets
// of a ragged tile's accesses, computed ahead, took 20 to 30 of them: sdl_gram_kernel at 4 / 7 / 8 replicas 117 / 193 / 228 registers, 90 / 162 /
// 193 so; 302 M parameters, M = 7 875 us and 861, the others the same.)
__device__ __forceinline__ uint32_t lane_here()
{
    uint32_t all = ~0u;
    asm volatile("" : "+s"(all));
    return __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}

// Raw bits of one tile as a lane holds them: 8 fp32 of g, 8 bf16 of each replica.
template <int NW>
struct TileRegs {
    u32x4 g0, g1;
    u32x4 w[NW];
};

// valid = parameters of the tile that exist (512 except in a set's last tile).  Full tiles of
// aligned sets use 128-bit buffer loads, full tiles of sets that start at some other element
// 128-bit loads of element alignment; a ragged last tile goes element by element under the buffer
// range check, which returns 0 past the end (g = 0 and w = 0 give Delta = 0: no contribution).
template <int NW>
__device__ __forceinline__ void load_tile(TileRegs<NW>& t, const float* g, const uint16_t* (&w)[NW],
                                          uint64_t e0, uint32_t valid, bool fast, uint32_t lane)
{
    if (fast && valid == (uint32_t)kTile) {
        const __amdgpu_buffer_rsrc_t rg = rsrc(g + e0, kTile * 4);
        t.g0 = __builtin_amdgcn_raw_buffer_load_b128(rg, (int)(lane * 32), 0, 2);
        t.g1 = __builtin_amdgcn_raw_buffer_load_b128(rg, (int)(lane * 32 + 16), 0, 2);
#pragma unroll
        for (int m = 0; m < NW; ++m)
            t.w[m] = __builtin_amdgcn_raw_buffer_load_b128(rsrc(w[m] + e0, kTile * 2), (int)(lane * 16), 0, 2);
    } else if (valid == (uint32_t)kTile) {
        lane = lane_here();
        const u32x4_f32elem* pg = reinterpret_cast<const u32x4_f32elem*>(g + e0 + lane * kLaneElems);
        t.g0 = __builtin_nontemporal_load(pg);
        t.g1 = __builtin_nontemporal_load(pg + 1);
#pragma unroll
        for (int m = 0; m < NW; ++m)
            t.w[m] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_bf16elem*>(w[m] + e0 + lane * kLaneElems));
    } else {
        lane = lane_here();
        const __amdgpu_buffer_rsrc_t rg = rsrc(g + e0, valid * 4);
        uint32_t x[kLaneElems];
#pragma unroll
        for (int j = 0; j < kLaneElems; ++j)
            x[j] = __builtin_amdgcn_raw_buffer_load_b32(rg, (int)((lane * kLaneElems + j) * 4), 0, 0);
        t.g0 = u32x4{x[0], x[1], x[2], x[3]};
        t.g1 = u32x4{x[4], x[5], x[6], x[7]};
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            const __amdgpu_buffer_rsrc_t rw = rsrc(w[m] + e0, valid * 2);
            uint32_t h[kLaneElems];
#pragma unroll
            for (int j = 0; j < kLaneElems; ++j)
                h[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rw, (int)((lane * kLaneElems + j) * 2), 0, 0)
                       & 0xffffu;
            t.w[m] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
        }
    }
}

// Outer gradients of one replica for the lane's 8 parameters: one fp32 subtraction each.
__device__ __forceinline__ void deltas(const u32x4& g0, const u32x4& g1, const u32x4& w, float (&d)[kLaneElems])
{
    const uint32_t gb[kLaneElems] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    const uint32_t wb[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int j = 0; j < kLaneElems; ++j) {
        const uint32_t bits = (j & 1) ? (wb[j / 2] & 0xffff0000u) : (wb[j / 2] << 16);
        d[j] = u2f(gb[j]) - u2f(bits);
    }
}

// The wavefront's totals of the N sums that each lane holds in v, lane by lane fewer of them: at each of the six levels two
// lanes split the sums they both hold, so that N / 2, N / 4, ... exchanges take the place of N at every level.  Afterwards a lane
// holds halved(N) totals.  (sdl_gram_kernel, every sum by a butterfly of six exchanges and the pieces looked at one by one, and
// now, whole call: 8.1 M parameters in 96 sets M = 2 86 us and 51; 1.8 M M = 8 40 and 23, M = 4 18 and 14; 302 M in 48 sets M = 4 542 and 539.)
constexpr int halved(int n, int levels = 6) { for (int l = 0; l < levels; ++l) n = (n + 1) / 2; return n; }

template <int LEVEL> __device__ __forceinline__ double from_partner(double x)
{
    constexpr int kCtrl = LEVEL == 2 ? 0x140 : LEVEL == 3 ? 0x141 : LEVEL == 4 ? 0x4E : 0xB1;   // mirrors of 16 and 8, quad_perm
    const u32x2 u = __builtin_bit_cast(u32x2, x);
    const u32x2 r = {(uint32_t)__builtin_amdgcn_mov_dpp((int)u.x, kCtrl, 0xF, 0xF, true),
                     (uint32_t)__builtin_amdgcn_mov_dpp((int)u.y, kCtrl, 0xF, 0xF, true)};
    return __builtin_bit_cast(double, r);
}

// (levels LEVEL to END - 1 alone)
template <int N, int LEVEL, int END = 6, int MAX>
__device__ __forceinline__ void halve(double (&v)[MAX], uint32_t lane)
{
    if constexpr (LEVEL < END) {
        constexpr int half = (N + 1) / 2;
        const bool upper = (lane >> (5 - LEVEL)) & 1u;
#pragma unroll
        for (int i = 0; i < half; ++i) {
            double lo = v[i], hi = half + i < N ? v[half + i] : 0.0;
            if constexpr (LEVEL < 2) {
                const u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
                u32x2 x, y;
                if constexpr (LEVEL == 0) {
                    x = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
                    y = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
                } else {
                    x = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
                    y = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
                }
                lo = __builtin_bit_cast(double, u32x2{x.x, y.x});
                hi = __builtin_bit_cast(double, u32x2{x.y, y.y});
                v[i] = lo + hi;
            } else {
                v[i] = (upper ? hi : lo) + from_partner<LEVEL>(upper ? lo : hi);
            }
        }
        halve<half, LEVEL + 1, END>(v, lane);
    }
}

// Which of the N sums a lane has after halve, and how many: at each level the lower lane kept the first half of them.
template <int N> __device__ __forceinline__ void halves_of(uint32_t lane, uint32_t* first, uint32_t* count)
{
    *first = 0;
    *count = N;
    uint32_t n = N;
    for (int level = 0; level < 6; ++level) {
        const uint32_t half = (n + 1u) / 2u;
        if ((lane >> (5 - level)) & 1u) { *first += half; *count = *count > half ? *count - half : 0u; }
        else *count = *count < half ? *count : half;
        n = half;
    }
}

// Up to 8 replicas: every lane holds the whole upper triangle.
template <int M>
__global__ void __launch_bounds__(kGramWaves * kWave) sdl_gram_kernel(const GramArgs a)
{
    constexpr int kSums = M * (M + 1) / 2, kLeft = halved(kSums);
    __shared__ double wave_sums[kGramWaves][kSums];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    // the first workgroups of 16 pieces are one scalar load, those of every 16th piece come first
    constexpr int kGroupsOf16 = kMaxPieces / 16, kFew = 6;
    uint32_t base = 0, s = 15;
    if (a.n_pieces > 16u) {
#pragma unroll
        for (int i = 1; i < kFew; ++i)
            if (blockIdx.x >= a.group_wg[i - 1]) base = (uint32_t)(i * 16);
        if (a.n_pieces > (uint32_t)(kFew * 16)) {
#pragma unroll
            for (int i = kFew; i < kGroupsOf16; ++i)
                if (blockIdx.x >= a.group_wg[i - 1]) base = (uint32_t)(i * 16);
        }
    }
#pragma unroll
    for (int i = 15; i >= 1; --i)
        if (blockIdx.x < a.first_wg[base + i]) s = (uint32_t)(i - 1);
    s += base;
    const uint32_t k = blockIdx.x - a.first_wg[s], G = a.first_wg[s + 1u] - a.first_wg[s], high = a.high[s / 4u] >> (s % 4u * 8u);
    const bool fast = high & kFast;
    const uint64_t offset = (uint64_t)(high & (kFast - 1u)) << 32 | a.offset[s];
    const uint32_t numel = a.numel[s], n_tiles = numel / kTile + (numel % kTile ? 1u : 0u);

    const uint16_t* w[M];
#pragma unroll
    for (int m = 0; m < M; ++m) w[m] = a.w[m];

    double sum[kSums];               // the triangle, row by row
#pragma unroll
    for (int i = 0; i < kSums; ++i) sum[i] = 0.0;

    auto valid_of = [&](uint32_t t) -> uint32_t {
        const uint32_t rem = numel - t * kTile;
        return rem < (uint32_t)kTile ? rem : (uint32_t)kTile;
    };

    auto consume = [&](const TileRegs<M>& t) {
        float f[M][kLaneElems];
#pragma unroll
        for (int m = 0; m < M; ++m) deltas(t.g0, t.g1, t.w[m], f[m]);
#pragma unroll
        for (int j = 0; j < kLaneElems; ++j) {
            double d[M];
#pragma unroll
            for (int m = 0; m < M; ++m) d[m] = (double)f[m][j];
            int i = 0;
#pragma unroll
            for (int r = 0; r < M; ++r)
#pragma unroll
                for (int c = r; c < M; ++c, ++i) sum[i] = __builtin_fma(d[r], d[c], sum[i]);
        }
    };

    // the wavefront's tiles: first, first + step, ... below end; neighbouring tiles go to neighbouring workgroups
    const uint32_t first = wave * G + k, step = a.waves * G, end = n_tiles;
    auto load = [&](TileRegs<M>& r, uint32_t t) { load_tile<M>(r, a.g, w, offset + (uint64_t)t * kTile, valid_of(t), fast, lane); };
    if constexpr (M <= 3) {
        // Two sets of registers in turn, so that two tiles are on the way.  (A copy of what was loaded ahead, as below, has to wait for it.
        // 302 M parameters in 48 spans, M = 1 / 2 / 3: 296 / 404 / 475 us with the copy, 288 / 386 / 473 so; at 4 to 7 replicas there is no
        // difference, at 8 the registers end it: 982 and 1000.)
        TileRegs<M> even, odd;
        if (first < end) load(even, first);
        if (first + step < end) load(odd, first + step);
        for (uint32_t t = first; t < end; t += 2 * step) {
            consume(even);
            if (t + 2 * step < end) load(even, t + 2 * step);
            if (t + step >= end) break;
            consume(odd);
            if (t + 3 * step < end) load(odd, t + 3 * step);
        }
    } else {
        TileRegs<M> cur;
        if (first < end) load(cur, first);
        for (uint32_t t = first; t < end; t += step) {
            TileRegs<M> nxt = cur;
            const uint32_t tn = t + step;
            if (tn < end) load(nxt, tn);
            consume(cur);
            cur = nxt;
        }
    }

    halve<kSums, 0>(sum, lane);
    uint32_t held, count;
    halves_of<kSums>(lane, &held, &count);
#pragma unroll
    for (uint32_t v = 0; v < (uint32_t)kLeft; ++v)
        if (v < count) wave_sums[wave][held + v] = sum[v];
    __syncthreads();
    if (threadIdx.x < (uint32_t)kSums) {
        uint32_t r = 0, c = threadIdx.x;
        while (c >= M - r) { c -= M - r; ++r; }
        const uint32_t i = threadIdx.x;
        static_assert(kGramWaves == 4);
        double total = wave_sums[0][i];
        if (a.waves > 1u) total = (total + wave_sums[1][i]) + (wave_sums[2][i] + wave_sums[3][i]);
        a.partial[(uint64_t)blockIdx.x * M * M + r * M + r + c] = total;
    }
}

// 9 to 16 replicas, H = ceil(M / 2) of them to each of the two wavefronts of a workgroup.  One lane cannot hold up to 136 sums.
// Wavefront 0 has the rows i = replicas 0..H-1 and the columns j = replicas H..2H-1, wavefront 1 the rows H..2H-1 and the columns
// 1, 2, ... H-1, 0.  Each forms its rows' triangle and, of the block rows x columns, the entries with (j - i) mod H <
// ceil(H / 2): in the first wavefront's terms the second one forms those with (j - i) mod H >= H - ceil(H / 2), so all are there
// (for odd H one diagonal twice).  With odd M the replica 2H-1 does not exist: replica 0 is read in its place and nothing of it is
// stored.
//
// A wavefront loads its own replicas, forms their outer gradients and puts them into LDS, where both find what they need as
// fp32: each difference is formed once, and the tile on its way takes 2H + 4 registers.  Bound: fp64 FMAs, 136 for a parameter at
// 16 replicas where a matrix instruction forms all 256 entries (both run at 16 a cycle and SIMD, and neither overlaps with the
// other).  On random data an FMA takes 2.4 ns, not the 1.7 of 2.4 GHz: 52.9 M parameters at 16 replicas are 263 us of FMAs, the
// rest conversions and subtractions; with one chain of additions for all of a lane's parameters 310 us measured with the loads
// and the staging left out, 350 with the staging, 385 with loads from the caches, 456 to 462 in all, and 30 to 35 more with chains
// of 16 (see total below).  Whole call at 52.9 M parameters, M = 9 / 12 / 13 / 16: 295 / 401 / 500 / 509 us as two wavefronts that
// each load everything (M <= 12) or on the matrix cores, 253 / 312 / 416 / 495 now (HBM 164 / 209 / 223 / 268); arrays at
// odd elements 393 / 486 / 764 / 860 and 276 / 345 / 442 / 525; 2.1 M parameters 51 / 80 / 59 / 63 and 28 / 32 / 37 / 42.
// Four wavefronts with a quarter of the matrix each (more of them in flight, 48 conversions instead of 32) 503 at 16 replicas,
// the tile copied to LDS past the registers, up to three tiles ahead, 478, each beside 463 and with one chain.
template <int H>
struct PairRaw {
    f32x4_elem g;
    u32x2 w[H];
};
constexpr int kPairTile = 4 * kWave;      // parameters a workgroup takes at a time
constexpr int kPairChain = 4;             // tiles after which the sums start a new chain (16 parameters of a lane)

// A whole tile of a set whose arrays are all 16-byte aligned (FAST) or start at any element.
template <int H, bool FAST>
__device__ __forceinline__ void load_pair_raw(PairRaw<H>& t, const float* g, const uint16_t* const (&w)[H], uint64_t e0, uint32_t lane)
{
    if constexpr (FAST) {
        t.g = __builtin_bit_cast(f32x4_elem, __builtin_amdgcn_raw_buffer_load_b128(rsrc(g + e0, kPairTile * 4), (int)(lane * 16), 0, 0));
#pragma unroll
        for (int m = 0; m < H; ++m)
            t.w[m] = __builtin_amdgcn_raw_buffer_load_b64(rsrc(w[m] + e0, kPairTile * 2), (int)(lane * 8), 0, 2);
    } else {
        lane = lane_here();
        t.g = *reinterpret_cast<const f32x4_elem*>(g + e0 + lane * 4);
#pragma unroll
        for (int m = 0; m < H; ++m) {
            const u32x2_elem x = *reinterpret_cast<const u32x2_elem*>(w[m] + e0 + lane * 4);
            t.w[m] = u32x2{x.x, x.y};
        }
    }
}
// A set's ragged last tile: 0 past the end of g and of every replica.
template <int H>
__device__ __forceinline__ void load_pair_tail(PairRaw<H>& t, const float* g, const uint16_t* const (&w)[H], uint64_t e0, uint32_t valid,
                                               uint32_t lane)
{
    lane = lane_here();
    const __amdgpu_buffer_rsrc_t rg = rsrc(g + e0, valid * 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) t.g[j] = u2f(__builtin_amdgcn_raw_buffer_load_b32(rg, (int)((lane * 4 + j) * 4), 0, 0));
#pragma unroll
    for (int m = 0; m < H; ++m) {
        const __amdgpu_buffer_rsrc_t rw = rsrc(w[m] + e0, valid * 2);
        uint32_t h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            h[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rw, (int)((lane * 4 + j) * 2), 0, 0) & 0xffffu;
        t.w[m] = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
    }
}

// Everything but the LDS accesses of the workgroup may be moved across, and loads stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// What the kernel works on: the tiles of all sets one behind the other, shared out among the workgroups in order.  A workgroup
// writes one matrix for each set that it has tiles of.  Up to three shares of the launch, each with as many workgroups as there is
// room for on the chip at once: 85 % of the tiles, then 10.5 % and 4.5 % in smaller parts, which fill what the first ones leave
// free when they end.  In a smaller launch the parts get as small as a few tiles, and more matrices take longer to add up than the parts
// save: two shares, 93 and 7 %, up to kTwoShares parameters, one up to kOneShare.  Whole call, us, with one share / two / three:
//   replicas        9                    12                   16
//   0.3 M      18.4 18.2 18.4       19.0 19.0 18.9       21.6 23.8 23.7
//   1 M        20.9 21.6 22.5       23.0 23.7 24.7       27.6 28.9 31.2
//   4 M        32.8 33.7 35.9       37.3 38.9 41.9       47.5 47.3 49.8
//   8 M        52.8 52.2 55.6       62.7 62.2 65.5       79.0 76.6 80.7
//   18 M       94.5 89.4 90.3      113.4 110.1 112.1    140.9 137.3 139.8
//   26 M        131  125  124        158  157  153        200  195  192
//   302 M      1500 1447 1413       1836 1796 1765       2261 2207 2163
constexpr int kShares = 3;
constexpr uint64_t kOneShare = 6ull << 20, kTwoShares = 24ull << 20;
struct Share {
    uint32_t first_wg, first_tile, per_wg, extra;     // workgroup first_wg + i takes per_wg tiles, one more if i < extra
};
// Workgroups of a launch that are on the chip at once: 12 wavefronts on a compute unit with up to 168 registers, else 8.  (With 198 at 11 and
// 12 replicas, the offsets of a ragged tile among them: 52.9 M parameters 334 and 342 us, 306 and 312 with 12 wavefronts; 302 M 1867 and 1887,
// 1719 and 1754.)
constexpr uint32_t pair_resident(uint32_t M, bool digits) { return 256u * (M <= 12u || digits ? 6u : 4u); }
struct PairArgs {
    const float* g;
    const uint16_t* w[SDL_MAX_WORKERS];
    double* partial;
    uint32_t M;
    uint32_t group_tile[kMaxSets / 16 - 1];   // first tile of the 16th, 32nd, ... set
    uint32_t first_tile[kMaxSets + 1];   // of each set, then the number of tiles; 0xffffffff behind it
    Share shares[kShares];
    int32_t slot[kMaxSets];           // workgroup b's matrix of set s is partial[b + slot[s]]
    uint32_t offset[kMaxSets];        // first element in the flat arrays, low 32 bits
    uint32_t more[kMaxSets];          // bits 32 to 38 of the offset; kFast: every array is 16-byte aligned at the set's start (24 sets of 48 off
                                      // it, 52.9 M parameters, M = 9 / 16: 268.6 / 517 us with all sets on the path for any alignment,
                                      // 266.3 / 514 so); from bit 8 on the parameters of the last tile
};
static_assert(sizeof(PairArgs) <= 4096 && kMaxSets % 16 == 0, "kernel arguments");

// The set that tile t belongs to.
__device__ __forceinline__ uint32_t set_of(const PairArgs& a, uint32_t t)
{
    uint32_t group = 0;
#pragma unroll
    for (int i = 1; i < kMaxSets / 16; ++i)
        if (t >= a.group_tile[i - 1]) group = (uint32_t)(i * 16);
    uint32_t s = group;
#pragma unroll
    for (int i = 1; i < 16; ++i)
        if (t >= a.first_tile[group + i]) s = group + (uint32_t)i;
    return s;
}

template <int H>
__global__ void __launch_bounds__(2 * kWave) __attribute__((amdgpu_waves_per_eu(H <= 6 ? 3 : 2))) sdl_gram_pair_kernel(const PairArgs a)
{
    constexpr int kOff = (H + 1) / 2;                // entries of the block rows x columns per row
    constexpr int kTri = H * (H + 1) / 2, kSums = kTri + H * kOff, kLeft = halved(kSums);
    __shared__ float diff[2][2 * H][kPairTile];      // outer gradients of two tiles
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint32_t M = a.M;

    auto row = [&](uint32_t i) -> uint32_t { return wave * H + i; };
    auto col = [&](uint32_t j) -> uint32_t { return wave ? (j + 1u) % H : H + j; };
    const uint16_t* w[H];
#pragma unroll
    for (int i = 0; i < H; ++i) w[i] = a.w[row(i) < M ? row(i) : 0u];

    auto stage = [&](uint32_t buf, const PairRaw<H>& t) {
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const f32x4_elem d = {t.g.x - u2f(t.w[i].x << 16), t.g.y - u2f(t.w[i].x & 0xffff0000u), t.g.z - u2f(t.w[i].y << 16),
                                  t.g.w - u2f(t.w[i].y & 0xffff0000u)};
            *reinterpret_cast<f32x4_elem __attribute__((aligned(16)))*>(&diff[buf][row(i)][lane * 4]) = d;
        }
    };
    // every 64th parameter of the tile: lane l's part-th one is part * 64 + l
    float f[2 * H];
    auto read = [&](uint32_t buf, int part) {
        const float* mine = &diff[buf][row(0)][part * kWave + lane];
        const float* theirs = &diff[buf][col(0)][part * kWave + lane];
#pragma unroll
        for (int i = 0; i < H; ++i) f[i] = mine[i * kPairTile];
#pragma unroll
        for (int j = 0; j < H - 1; ++j) f[H + j] = theirs[j * kPairTile];
        f[2 * H - 1] = diff[buf][col(H - 1)][part * kWave + lane];
        __builtin_amdgcn_sched_barrier(0);
    };
    double sum[kSums];                               // the rows' triangle, then the block's entries
    // Whole chains, added over 4 lanes (8 at H = 8).  Products of short mantissas end alike, so where a sum has outgrown them its
    // roundings all go one way, and the error grows with the chain: for squares, and for two replicas that point the same way as well.
    // 52.9 M parameters with outliers, rms error in units of 1e-16 of sqrt(G[a][a] G[b][b]), a = b / a != b, replicas correlated by
    // 0.9, at 9 / 12 / 13 / 16 replicas: one chain for a lane's 690 parameters (the diagonal alone in chains of 16) 0.5/13 0.9/18
    // 1.1/19 0.9/19; chains of 64 1.8/2.3 1.9/2.2 2.1/2.1 2.4/2.2; of 32 1.0/1.5 1.3/1.5 1.1/1.3 1.3/1.4; of 16 0.9/1.1 1.1/1.0
    // 0.9/1.0 1.1/1.1.  Whole call: 240 / 320 / 392 / 461 us with one chain, 253 / 334 / 416 / 495 with chains of 16.  A third
    // exchange costs 1 % (three levels, which 16 replicas need, as two spill there), all six 5 %; added up through LDS, eight
    // values to a lane, 538 at 16 replicas; with sums that are set to 0 instead of begun by their first product 506.  One chain of products that
    // a factor of 28 bits fills up at the bottom: as exact, 262 / 346 / 424 / 498.
    constexpr int kFolds = H == 8 ? 3 : 2, kHeld = halved(kSums, kFolds);
    double total[kHeld];
    // the sums of one parameter, the first of its chain or a later one; once it is converted, the next one is read into the same
    // registers
    auto consume = [&](auto is_first, auto read_next) {
        constexpr bool FIRST = decltype(is_first)::value;
        double d[2 * H];
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) d[m] = (double)f[m];
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) asm volatile("" : "+v"(d[m]));    // converted here, not where it is first used
        read_next();
        int k = 0;
#pragma unroll
        for (int i = 0; i < H; ++i)
#pragma unroll
            for (int j = i; j < H; ++j, ++k) sum[k] = __builtin_fma(d[i], d[j], FIRST ? 0.0 : sum[k]);
#pragma unroll
        for (int i = 0; i < H; ++i)
#pragma unroll
            for (int j = 0; j < kOff; ++j, ++k) sum[k] = __builtin_fma(d[i], d[H + (i + j) % H], FIRST ? 0.0 : sum[k]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto end_chain = [&]() {
        halve<kSums, 0, kFolds>(sum, lane);
#pragma unroll
        for (int i = 0; i < kHeld; ++i) total[i] += sum[i];
    };

    const uint32_t b = blockIdx.x;
    Share share = a.shares[0];
#pragma unroll
    for (int i = 1; i < kShares; ++i)
        if (b >= a.shares[i].first_wg) share = a.shares[i];
    const uint32_t nth = b - share.first_wg;
    uint32_t t = share.first_tile + nth * share.per_wg + (nth < share.extra ? nth : share.extra);
    const uint32_t end = t + share.per_wg + (nth < share.extra ? 1u : 0u);
    while (t < end) {
        const uint32_t s = set_of(a, t);
        const uint32_t set_first = a.first_tile[s], set_end = a.first_tile[s + 1], stop = end < set_end ? end : set_end;
        const uint32_t more = a.more[s], in_last = more >> 8;
        const uint64_t offset = (uint64_t)(more & (kFast - 1u)) << 32 | a.offset[s];
        const uint32_t whole = set_end - set_first - (in_last == (uint32_t)kPairTile ? 0u : 1u), last = stop - set_first < whole ? stop - set_first : whole;
        uint32_t k = t - set_first;
#pragma unroll
        for (int i = 0; i < kHeld; ++i) total[i] = 0.0;

        // whole tiles k, k + 1, ...: while one is consumed the next one lies in the other half of diff, or will by the time of
        // the barrier, and the one after it is on its way into registers (behind the last tile: that tile again)
        auto walk = [&](auto is_fast) {
            constexpr bool FAST = decltype(is_fast)::value;
            PairRaw<H> raw;
            auto load = [&](uint32_t n) {
                load_pair_raw<H, FAST>(raw, a.g, w, offset + (uint64_t)(n < last ? n : last - 1u) * kPairTile, lane);
            };
            uint32_t buf = 0;
            load(k);
            lds_barrier();       // the tile before this set has been read
            stage(0, raw);
            load(k + 1u);
            lds_barrier();
            read(0, 0);
            while (k < last) {
                const uint32_t chain = last - k < (uint32_t)kPairChain ? last : k + kPairChain;
                auto tile = [&](auto is_first) {
                    consume(is_first, [&]() { read(buf, 1); });
                    consume(std::false_type{}, [&]() { read(buf, 2); });
                    stage(buf ^ 1u, raw);
                    load(k + 2u);
                    consume(std::false_type{}, [&]() { read(buf, 3); });
                    lds_barrier();
                    consume(std::false_type{}, [&]() { read(buf ^ 1u, 0); });
                    buf ^= 1u;
                    ++k;
                };
                tile(std::true_type{});
                while (k < chain) tile(std::false_type{});
                end_chain();
            }
        };
        if (k < last) {
            if (more & kFast) walk(std::true_type{});
            else walk(std::false_type{});
        }
        if (stop - set_first > whole) {
            PairRaw<H> raw;
            load_pair_tail<H>(raw, a.g, w, offset + (uint64_t)whole * kPairTile, in_last, lane);
            lds_barrier();
            stage(0, raw);
            lds_barrier();
#pragma unroll
            for (int i = 0; i < kSums; ++i) sum[i] = 0.0;
#pragma unroll 1
            for (int part = 0; part < kPairTile / kWave; ++part) {
                read(0, part);
                consume(std::false_type{}, []() {});
            }
            end_chain();
        }
        halve<kHeld, kFolds>(total, lane);

        uint32_t first, count, lane_here = lane;
        asm volatile("" : "+v"(lane_here));      // (computed ahead of the loop, this would hold registers that it needs)
        halves_of<kSums>(lane_here, &first, &count);
        double* out = a.partial + (uint64_t)(uint32_t)((int32_t)b + a.slot[s]) * M * M;
#pragma unroll
        for (uint32_t v = 0; v < (uint32_t)kLeft; ++v) {
            if (v >= count) continue;
            uint32_t i = 0, j = first + v;
            if (j < (uint32_t)kTri) {
                while (j >= H - i) { j -= H - i; ++i; }
                j = row(i + j);
            } else {
                i = (j - kTri) / kOff;
                const uint32_t o = (j - kTri) % kOff;
                if (H % 2 == 1 && o == kOff - 1 && wave == 1u) continue;     // the diagonal that both formed: once is enough
                j = col((i + o) % H);
            }
            i = row(i);
            if (i < M && j < M) out[i < j ? i * M + j : j * M + i] = total[v];
        }
        t = stop;
    }
}

// 13 to 16 replicas and many parameters (see takes_digits): the sums in whole numbers on the matrix cores.  A replica's outer gradients, times a power
// of two that brings the largest of them near 2^21, are multiples of 2^-22 as a rule and written as six signed digits of 8 bits; the
// products of two replicas' digits are whole numbers that v_mfma_i32_16x16x64_i8 adds up without rounding, 64 parameters of all 256
// entries at a time, and what 16384 parameters gave is converted and added up in fp64.
//
// The digits.  x is a difference, t = x * scale, |t| <= kRoom.  As the sum with kBias is in [2^23, 2^24), fma(x, scale, kBias)
// is the bit pattern of t rounded to a whole number, plus 0x408080: in each of the two low bytes, and in the seven bits above, a digit
// with 128 (64) added, which the exclusive or (and an addition of 64 ahead of it) takes off all four bytes of a register at
// once.  What the rounding left, at most 1/2, is exact as an fma; times 2^22 it gives three more digits in the same way.
// Weights of the digits: 2^16, 2^8, 1 and 2^-6, 2^-14, 2^-22.
// The products of the digits a < b are formed once and their transpose is added at the end: T + T^T is the matrix of sums if T has
// half of the squares.  The last digit is 0 for nearly all differences between weights and replicas (multiples of the last place of the smaller
// of two numbers), and a step without one leaves its six products out; four of them, whose weights are 2^-22 and less, are kept in fp64 (`low`),
// together with what the additions to the totals round off.
//
// Nothing is rounded ahead of a product.  A difference has 24 bits, so what is not below 2 / scale (`least`) is a multiple of 2^-22 / scale, and so is 0.
// If a step has others they are looked at, and if one is no such multiple, the step's 64 parameters are added up in fp64 by v_mfma_f64_16x16x4_f64.
// (With 0 among those that are looked at: a tenth of the differences 0, 52.9 M parameters and 16 replicas 427 us, now 414.)  In fp64 go infinities as
// well, and differences below 2^-98 where there are no larger ones (their scale would not be a normal number).
// NaN, as in a replica that has diverged, would send every step there: its entries are NaN whatever follows, so the step goes on with 0 for that replica.
//
// The scale of a replica is that of the wavefront's parameters so far: where a difference exceeds what it has room for, the
// sums so far are put into fp64 and a new one is taken, with room for twice as much and more.  That costs as much as a step, and 16 replicas whose largest
// differences grow one after the other would have it 16 times: they all make room at once for the largest difference of any of them, if it is not more than
// kAlike times their own.  (Each by itself, t3 / with outliers: M = 16, 2.1 M parameters 43 / 44 us, now 36 / 36, 52.9 M 428 / 425 and 392 / 390; M = 13, 35 M
// in 195 sets, most of them small, 375 / 381 and 332 / 334.)
//
// Error against exact sums, 1e-16 of sqrt(G[a][a] G[b][b]), a = b / a != b, rms of six replicas and 20 seeds, 20 M parameters, by FMAs (whose partial
// matrices a tree adds up) at 13 and at 16 replicas, and here: normal 0.77/0.01 0.91/0.01, 0.59/0.00 0.73/0.00; Student t3 0.67/0.02 0.76/0.01,
// 0.40/0.00 0.55/0.00; with outliers 0.98/0.01 0.86/0.01, 0.46/0.00 0.53/0.00; differences with all 24 bits 0.83/0.73 0.80/0.72, 0.38/0.40
// 0.59/0.52.  8 M: normal 0.97/0.01 0.93/0.01, 0.67/0.00 0.77/0.00; 24 bits 0.81/0.87 0.67/0.71, 0.46/0.49 0.53/0.56.  Four seeds: replicas that agree,
// outliers in the same places, 0.95/1.03 0.86/0.86, 0.46/0.42 0.46/0.60; sizes that vary by 2^40 from one parameter to the next 0.71/0.01
// 0.78/0.01, 0.57/0.01 0.56/0.01.
//
// Bound: vector instructions, 13 for a difference (two to form it, a half each to look at the largest and the smallest, four for the digits, 3.5 that
// bring each digit's bytes together and 2 for the signs) of four cycles each: they take 93 % of the SIMDs' cycles, the matrix instructions, 15 of
// 16 cycles for 64 parameters, 27 % beside them.  52.9 M parameters and 16 replicas: 300 us with neither loads nor matrix instructions, 329 without the
// loads, 357 without the matrix instructions, 322 the loads and the staging alone, 385 in all (HBM 268).  Whole call, FMAs and here, M = 13 / 14 / 15 / 16:
// 52.9 M parameters 413 / 416 / 492 / 496 and 361 / 367 / 377 / 381; at odd elements 433 / 439 / 513 / 521 and 393 / 397 / 418 / 423.  M = 16 with
// outliers 494 and 386, t3 495 and 389, 24 bits 500 and 389, a tenth of the differences 0 495 and 414, one replica NaN 510 and 439; steps in fp64
// all along (sizes that vary by 2^40) 504 and 759.
// (The time hardly depends on the replicas, as a matrix instruction has 16 rows whatever they are: at 12 replicas 306 and 354.)  Tried, each beside 390
// to 409 with 18 products at every step: a tile of 512 for each wavefront, 252 registers, 409; 256 parameters, two tiles in LDS 401; the digits' products one
// step behind, between the vector instructions of the next, which takes 220 registers 427; workgroups that take turns at the tiles 397; subtraction by
// v_dot2_f32_bf16, which does not round to nearest.
constexpr int kDigitTile = kTile;                 // parameters a workgroup takes at a time, 64 of them a step, the wavefronts in turn
constexpr int kDigitSteps = kDigitTile / kWave;
constexpr uint32_t kFlushTiles = 64;              // after so many a sum has three products of 2^14 for each of 16384 parameters: 2^30
// From how many parameters of a launch on.  Whole call, us, FMAs and here, normal differences / t3 / with outliers (a tenth of the differences 0: 2.1 M and 16
// replicas 38.0 36.5, 5.3 M and 13 / 14 56.8 58.2 / 54.6 57.0, 6 M 60.0 61.2 / 60.3 61.4, 8 M and 13 78.5 76.1):
//   replicas            13                                     14                                     16
//   1.5 M                                                                                     30.5 30.7  30.6 31.9  30.5 31.9
//   2.1 M                                                                                     35.8 34.8  35.9 35.8  35.8 35.5
//   3 M                                                                                       42.9 40.9  43.2 42.1  43.0 41.4
//   4.2 M     46.8 46.0  46.9 47.6  46.6 46.8   46.7 46.2  47.1 48.0  46.8 47.2
//   5 M       52.6 51.2  52.6 52.6  52.5 52.1   52.8 51.6  52.7 53.2  52.8 52.6
//   6 M       60.2 57.4  60.4 60.1  60.1 59.1   60.3 58.8  60.6 61.6  60.6 59.4
// and 15 replicas like 16.
constexpr bool takes_digits(uint32_t M, uint64_t params) { return params >= (M > 14u ? 4ull << 19 : M > 12u ? 10ull << 19 : ~0ull); }

constexpr float kBias = 12615808.0f;              // 2^23 + 0x408080
constexpr float kRoom = 4161407.0f;               // 2^23 - 1 - 0x408080
constexpr float kLoScale = 4194304.0f;            // 2^22
constexpr float kAlike = 64.0f;                   // what replicas' largest differences may differ by for one to take another's scale
constexpr float kFltMax = 3.402823466e+38f;

enum Digit { kHi2, kHi1, kHi0, kLo2, kLo1, kLo0, kDigits };
struct Product { int a, b, acc; };
struct DigitSum { double weight; };
constexpr int kDigitSums = 13;
constexpr double kHalf = 0.5;                     // of a digit's square
constexpr DigitSum kSumOf[kDigitSums] = {{kHalf * 0x1p32}, {0x1p24}, {0x1p16}, {kHalf * 0x1p16}, {0x1p8}, {kHalf}, {0x1p10},
                                         {0x1p2}, {0x1p-6}, {0x1p-14}, {kHalf * 0x1p-12}, {0x1p-20}, {kHalf * 0x1p-28}};
constexpr Product kProducts[] = {
    {kHi2, kHi2, 0}, {kHi2, kHi1, 1}, {kHi2, kHi0, 2}, {kHi1, kHi1, 3}, {kHi1, kHi0, 4}, {kHi0, kHi0, 5}, {kHi2, kLo2, 6},
    {kHi2, kLo1, 7}, {kHi1, kLo1, 8}, {kHi1, kLo2, 7}, {kHi0, kLo2, 8}, {kHi0, kLo1, 9}, {kLo2, kLo2, 10}, {kLo2, kLo1, 11}, {kLo1, kLo1, 12}};
constexpr Product kLastDigit[] = {{kHi2, kLo0, 8}, {kHi1, kLo0, 9}};     // the others of the last digit go past the sums
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr double kDblMax = 1.7976931348623157e+308;

__device__ __forceinline__ float from_lane(float x, uint32_t lane)
{
    return u2f((uint32_t)__builtin_amdgcn_ds_bpermute((int)(lane << 2), (int)f2u(x)));
}

// The largest of the four lanes l % 16, and of the 16 lanes of a quarter; NaN if any is.
__device__ __forceinline__ float max_of_quarters(float x)
{
    u32x2 y = __builtin_amdgcn_permlane32_swap(f2u(x), f2u(x), false, false);
    x = __builtin_elementwise_maximum(u2f(y.x), u2f(y.y));
    y = __builtin_amdgcn_permlane16_swap(f2u(x), f2u(x), false, false);
    return __builtin_elementwise_maximum(u2f(y.x), u2f(y.y));
}
template <int RING = 8> __device__ __forceinline__ float max_of_rows(float x)
{
    x = __builtin_elementwise_maximum(x, u2f((uint32_t)__builtin_amdgcn_mov_dpp((int)f2u(x), 0x120 + RING, 0xF, 0xF, true)));
    if constexpr (RING > 1) return max_of_rows<RING / 2>(x);
    return x;
}

// What a wavefront loads of a tile: half of the replicas, and of every lane's 8 parameters of g the first or the last four.
template <int H>
struct HalfTile {
    u32x4 g;
    u32x4 w[H];
};
template <int H>
__device__ __forceinline__ void load_half(HalfTile<H>& t, const float* g, uint32_t half, const uint16_t* (&w)[H], uint64_t e0,
                                          uint32_t valid, bool fast, uint32_t lane)
{
    if (fast && valid == (uint32_t)kDigitTile) {
        t.g = __builtin_amdgcn_raw_buffer_load_b128(rsrc(g + e0, kDigitTile * 4), (int)(lane * 32 + half * 16), 0, 2);
#pragma unroll
        for (int m = 0; m < H; ++m)
            t.w[m] = __builtin_amdgcn_raw_buffer_load_b128(rsrc(w[m] + e0, kDigitTile * 2), (int)(lane * 16), 0, 2);
    } else if (valid == (uint32_t)kDigitTile) {
        lane = lane_here();
        t.g = __builtin_nontemporal_load(reinterpret_cast<const u32x4_f32elem*>(g + e0 + lane * kLaneElems + half * 4));
#pragma unroll
        for (int m = 0; m < H; ++m)
            t.w[m] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_bf16elem*>(w[m] + e0 + lane * kLaneElems));
    } else {                                       // a set's ragged last tile: 0 past the end of g and of every replica
        lane = lane_here();
        const __amdgpu_buffer_rsrc_t rg = rsrc(g + e0, valid * 4);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            t.g[j] = __builtin_amdgcn_raw_buffer_load_b32(rg, (int)((lane * kLaneElems + half * 4 + j) * 4), 0, 0);
#pragma unroll
        for (int m = 0; m < H; ++m) {
            const __amdgpu_buffer_rsrc_t rw = rsrc(w[m] + e0, valid * 2);
            uint32_t h[kLaneElems];
#pragma unroll
            for (int j = 0; j < kLaneElems; ++j)
                h[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rw, (int)((lane * kLaneElems + j) * 2), 0, 0) & 0xffffu;
            t.w[m] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
        }
    }
}

template <int H>
__global__ void __launch_bounds__(2 * kWave) __attribute__((amdgpu_waves_per_eu(3))) sdl_digit_sums_kernel(const PairArgs a)
{
    // A tile in LDS: the replicas, then g, both as they are in memory.  In a step lane l = 16 q + r has 16 parameters of replica r (0 where
    // there is none), of the q-th quarter of the tile.  The distances make the 16 replicas' pieces, and the four quarters of g, lie in
    // different banks.
    constexpr int R = 2 * H, kRowWords = kDigitTile / 2 + 4, kQuarterWords = kDigitTile / 4 + 4;
    __shared__ __attribute__((aligned(16))) uint32_t stage[R * kRowWords + 4 * kQuarterWords];
    __shared__ double totals[2][256];                // T of each wavefront: [16 q + r][v] is its row 4 q + v, column r
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint32_t M = a.M, r = lane % 16u, q = lane / 16u;
    const u32x4* const my_w = reinterpret_cast<const u32x4*>(stage + (r < (uint32_t)R ? r : 0u) * kRowWords + q * (kDigitTile / 8));
    const u32x4* const my_g = reinterpret_cast<const u32x4*>(stage + R * kRowWords + q * kQuarterWords);
    const uint16_t* w[H];
#pragma unroll
    for (int i = 0; i < H; ++i) w[i] = a.w[wave * H + i < M ? wave * H + i : 0u];

    i32x4 sum[kDigitSums];                           // [v] is row 4 q + v, column r
    double low[4];                                   // what the totals had no room for
    float scale = 0.0f, limit = -1.0f, least = 0.0f; // of the lane's replica; what is not 0 and below `least` may have bits that the digits lack
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < kDigitSums; ++i) sum[i] = i32x4{0, 0, 0, 0};
    };
    // adds x to entry v of the total, the rounding to `low`
    auto add = [&](int v, double x) {
        double* const total = &totals[wave][4u * lane_here() + (uint32_t)v];
        const double before = *total, after = before + x, part = after - before;
        const double rounding = (before - (after - part)) + (x - part);
        low[v] += __builtin_fabs(after) <= kDblMax ? rounding : 0.0;
        *total = after;
    };
    // 1 / (scale of row 4 q + v * scale of the lane's column), 0 where a scale is
    auto unscale = [&](int v) -> double {
        const float inv = scale > 0.0f ? u2f((254u << 23) - f2u(scale)) : 0.0f;
        return (double)inv * (double)from_lane(inv, 4u * (lane_here() / 16u) + (uint32_t)v);
    };
    auto flush = [&]() {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double t = 0.0;
#pragma unroll
            for (int i = kDigitSums - 1; i >= 0; --i) t = __builtin_fma((double)sum[i][v], kSumOf[i].weight, t);
            add(v, t * unscale(v));
        }
        clear();
    };
    // A step that the limits do not cover: true if its products have been added up here.
    auto adjust = [&](float (&d)[16], float largest, float smallest) -> bool {
        const uint32_t l = lane_here(), r = l % 16u;
        bool digits = true;
        if (__builtin_amdgcn_ballot_w64(!(largest <= limit))) {
            float m = max_of_quarters(largest);
            if (__builtin_amdgcn_ballot_w64(m != m)) {       // NaN in the replica's entries, whatever else it holds: the others go on with digits
                const bool nan = m != m;
#pragma unroll
                for (int v = 0; v < 4; ++v) low[v] = nan ? (double)m : low[v];
#pragma unroll
                for (int j = 0; j < 16; ++j) d[j] = nan ? 0.0f : d[j];
                m = nan ? 0.0f : m;
                smallest = nan ? least : smallest;
            }
            const bool fits = m <= limit;
            digits = !__builtin_amdgcn_ballot_w64(!fits && (!(m <= kFltMax) || (m > 0.0f && m < 0x1p-98f)));
            if (digits && __builtin_amdgcn_ballot_w64(!fits)) {
                if (__builtin_amdgcn_ballot_w64(scale != 0.0f)) flush();
                const float want = __builtin_fminf(max_of_rows(m), m * kAlike);
                if (!(want <= limit)) {              // 2^20 <= want * scale < 2^21
                    const uint32_t e = f2u(want) >> 23;
                    scale = want > 0.0f ? u2f((127u + 127u + 20u - e) << 23) : 0.0f;
                    limit = want > 0.0f ? kRoom * u2f((e - 20u) << 23) : 0.0f;
                    limit = limit <= kFltMax ? limit : kFltMax;
                    least = want > 0.0f ? u2f((e - 19u) << 23) : 0.0f;
                }
            }
        }
        uint32_t smallest_but_0 = ~0u;               // twice its bits, less 1, which of 0 is the largest number
        if (digits && __builtin_amdgcn_ballot_w64(!(smallest >= least))) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint32_t x = (f2u(d[j]) << 1) - 1u;
                smallest_but_0 = x < smallest_but_0 ? x : smallest_but_0;
            }
        }
        if (digits && __builtin_amdgcn_ballot_w64(smallest_but_0 < (f2u(least) << 1) - 1u)) {
            const int last = (int)(f2u(scale) >> 23) - 127 + 22;     // of the last digit, 2^-last
            float left = 0.0f;
#pragma unroll
            for (int j = 0; j < 16; ++j) left = __builtin_fmaxf(left, __builtin_amdgcn_fractf(__builtin_ldexpf(d[j], last)));
            digits = !__builtin_amdgcn_ballot_w64(left != 0.0f);
        }
        if (digits) return false;
        // v_mfma_f64_16x16x4_f64: lane 16 k + i gives row (left) or column (right) i of the k-th parameter and has entries 4 v + k, i; with the
        // rows in this order they are 4 k + v, i
        f64x4 products = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float row = from_lane(d[e], (l & 48u) + r % 4u * 4u + r / 4u);
            products = __builtin_amdgcn_mfma_f64_16x16x4f64(0.5 * (double)row, (double)d[e], products, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) add(v, products[v]);
        return true;
    };
    // 64 parameters of every replica; read_next reads what the next step needs into the registers that wv and gv are in.
    auto step = [&](const u32x4 (&wv)[2], const u32x4 (&gv)[4], auto read_next) {
        float d[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const uint32_t x = wv[j / 8][(j % 8) / 2];
            d[j] = u2f(gv[j / 4][j % 4]) - u2f(j & 1 ? x & 0xffff0000u : x << 16);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) asm volatile("" : "+v"(d[j]));     // formed here, not where it is first used
        float largest = __builtin_fabsf(d[0]), smallest = largest;      // NaN if any is
#pragma unroll
        for (int j = 1; j < 15; j += 2) {
            largest = __builtin_elementwise_maximum(__builtin_elementwise_maximum(largest, __builtin_fabsf(d[j])), __builtin_fabsf(d[j + 1]));
            smallest = __builtin_elementwise_minimum(__builtin_elementwise_minimum(smallest, __builtin_fabsf(d[j])), __builtin_fabsf(d[j + 1]));
        }
        largest = __builtin_elementwise_maximum(largest, __builtin_fabsf(d[15]));
        smallest = __builtin_elementwise_minimum(smallest, __builtin_fabsf(d[15]));
        const bool added = __builtin_amdgcn_ballot_w64(!(largest <= limit) || !(smallest >= least)) && adjust(d, largest, smallest);
        read_next();
        if (added) return;
        i32x4 digit[kDigits];
        auto planes = [&](int k, const uint32_t (&h)[4], int top, int middle, int low) {
            const uint32_t x = __builtin_amdgcn_perm(h[1], h[0], 0x05010400u), y = __builtin_amdgcn_perm(h[3], h[2], 0x05010400u);
            const uint32_t u = __builtin_amdgcn_perm(h[1], h[0], 0x0c0c0602u), v = __builtin_amdgcn_perm(h[3], h[2], 0x0c0c0602u);
            digit[low][k] = (int)(__builtin_amdgcn_perm(y, x, 0x05040100u) ^ 0x80808080u);
            digit[middle][k] = (int)(__builtin_amdgcn_perm(y, x, 0x07060302u) ^ 0x80808080u);
            digit[top][k] = (int)((__builtin_amdgcn_perm(v, u, 0x05040100u) + 0x40404040u) ^ 0x80808080u);
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = d[4 * k + j], h = __builtin_fmaf(x, scale, kBias), rest = __builtin_fmaf(x, scale, kBias - h);
                hi[j] = f2u(h);
                lo[j] = f2u(__builtin_fmaf(rest, kLoScale, kBias));
            }
            planes(k, hi, kHi2, kHi1, kHi0);
            planes(k, lo, kLo2, kLo1, kLo0);
        }
#pragma unroll
        for (const Product& x : kProducts)
            sum[x.acc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(digit[x.a], digit[x.b], sum[x.acc], 0, 0, 0);
        if (__builtin_amdgcn_ballot_w64((digit[kLo0][0] | digit[kLo0][1] | digit[kLo0][2] | digit[kLo0][3]) != 0)) {
#pragma unroll
            for (const Product& x : kLastDigit)
                sum[x.acc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(digit[x.a], digit[x.b], sum[x.acc], 0, 0, 0);
            auto product = [&](int a) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(digit[a], digit[kLo0], i32x4{0, 0, 0, 0}, 0, 0, 0); };
            const i32x4 x = product(kHi0) * 64 + product(kLo2), y = product(kLo1) * 512 + product(kLo0);     // of 2^-28 and 2^-45, each below 2^30
#pragma unroll
            for (int v = 0; v < 4; ++v) low[v] = __builtin_fma(__builtin_fma((double)x[v], 0x1p-28, (double)y[v] * 0x1p-45), unscale(v), low[v]);
        }
    };

    const uint32_t b = blockIdx.x;
    Share share = a.shares[0];
#pragma unroll
    for (int i = 1; i < kShares; ++i)
        if (b >= a.shares[i].first_wg) share = a.shares[i];
    const uint32_t nth = b - share.first_wg;
    uint32_t t = share.first_tile + nth * share.per_wg + (nth < share.extra ? nth : share.extra);
    const uint32_t end = t + share.per_wg + (nth < share.extra ? 1u : 0u);
    while (t < end) {
        const uint32_t s = set_of(a, t);
        const uint32_t set_first = a.first_tile[s], set_end = a.first_tile[s + 1], stop = end < set_end ? end : set_end;
        const uint32_t more = a.more[s], in_last = more >> 8, final_tile = set_end - set_first - 1u;
        const uint64_t offset = (uint64_t)(more & (kFast - 1u)) << 32 | a.offset[s];
        const bool fast = more & kFast;
#pragma unroll
        for (int i = 0; i < 4; ++i) totals[wave][4u * lane_here() + i] = low[i] = 0.0;
        clear();
        scale = least = 0.0f;
        limit = -1.0f;

        HalfTile<H> raw;
        auto load = [&](uint32_t k) {
            load_half<H>(raw, a.g, wave, w, offset + (uint64_t)k * kDigitTile, k == final_tile ? in_last : (uint32_t)kDigitTile, fast, lane);
        };
        u32x4 wv[2], gv[4];
        auto read = [&](uint32_t j) {
#pragma unroll
            for (uint32_t i = 0; i < 2u; ++i) wv[i] = my_w[2u * j + i];
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i) gv[i] = my_g[4u * j + i];
        };
        const uint32_t last = stop - set_first;
        uint32_t k = t - set_first, tiles = 0;
        load(k);
#pragma unroll 1
        for (; k < last; ++k) {
            lds_barrier();       // the tile before has been read
            u32x4* const to = reinterpret_cast<u32x4*>(stage + wave * H * kRowWords) + lane;
#pragma unroll
            for (int i = 0; i < H; ++i) to[i * (kRowWords / 4)] = raw.w[i];
            *reinterpret_cast<u32x4*>(stage + R * kRowWords + lane * 8u + q * 4u + wave * 4u) = raw.g;
            if (k + 1u < last) load(k + 1u);
            lds_barrier();
            read(wave);
#pragma unroll 1
            for (uint32_t j = wave; j < (uint32_t)kDigitSteps; j += 2u)
                step(wv, gv, [&]() { read((j + 2u) % kDigitSteps); });     // (behind the last: read and not used)
            if (++tiles == kFlushTiles || k + 1u == last) { flush(); tiles = 0; }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) totals[wave][4u * lane_here() + i] += low[i];
        __syncthreads();
        double* out = a.partial + (uint64_t)(uint32_t)((int32_t)b + a.slot[s]) * M * M;
        for (uint32_t i = wave * kWave + lane_here(); i < 256u; i += 2 * kWave) {
            const uint32_t x = i / 16u, y = i % 16u, at = (x / 4u * 16u + y) * 4u + x % 4u, turned = (y / 4u * 16u + x) * 4u + y % 4u;
            if (x <= y && y < M) out[x * M + y] = (totals[0][at] + totals[1][at]) + (totals[0][turned] + totals[1][turned]);
        }
        __syncthreads();
        t = stop;
    }
}

// What each output of the finalize kernel adds up.
constexpr uint32_t kFinThreads = 1024;                                     // most threads of a workgroup

// Threads that share an entry (beyond 64 the tree over them costs more than it saves), and the matrices that one first-level
// output adds: 8 for each of them.
__host__ __device__ constexpr uint32_t fin_slices(uint32_t M)
{
    const uint32_t s = kFinThreads / (M * (M + 1u) / 2u);
    return s < 64u ? s : 64u;
}
constexpr uint32_t fin_chunk(uint32_t M) { return 8u * fin_slices(M); }
constexpr uint32_t kFewSlices = 13;                                       // from so many replicas on 11 threads and fewer

// matrices of a launch, without one for each set
constexpr uint32_t mats_per_launch(uint32_t M) { return M > 8u ? kShares * pair_resident(M, M > 12u) : kGroups; }

// A launch over n sets leaves at most mats_per_launch + n matrices, so at most (mats_per_launch + n) / fin_chunk + n
// first-level outputs: kFirstLevel and one for each set, of which the workspace has room.
constexpr uint32_t kFirstLevel = kMaxGroups / 64 + 2;
constexpr uint32_t kMaxFin = 896;                                         // outputs per finalize launch
constexpr uint32_t kBatch = 11 * kFewSets;                                // sets that are finished together
static_assert(kBatch < kMaxFin, "the last level is one launch");
constexpr bool sums_fit()
{
    for (uint32_t M = 1; M <= SDL_MAX_WORKERS; ++M)
        if (mats_per_launch(M) > kMaxGroups || (mats_per_launch(M) + kMaxSets) / fin_chunk(M) > kFirstLevel) return false;
    return true;
}
static_assert(sums_fit(), "matrices per launch, matrices per first-level output and the workspace go together");

struct FinArgs {
    const double* in;              // matrices of M*M doubles (only a <= b is read), stride_k doubles apart
    double* out;                   // output o at out + o * out_stride
    double* last_out;              // if not null, where the last output goes instead
    uint64_t stride_k;
    uint64_t out_stride;
    uint32_t M;
    uint32_t emit;                 // 1: G, cos, mean (2*M*M + 1 doubles); 0: G only (M*M doubles)
    uint32_t first[kMaxFin + 1];   // output o adds the matrices first[o] .. first[o + 1] - 1; one that goes to last_out those of all before it
};
static_assert(sizeof(FinArgs) <= 4096, "kernel arguments");

// One workgroup per output.  A thread adds every S-th matrix's value of one entry a <= b (neighbouring threads read
// neighbouring entries), then the S sums of an entry are added as a tree.  Latency bound: a range should give a thread a
// handful of matrices, so long ranges go through a first level of fin_chunk matrices per output, and its loads are on the way eight at a
// time, the last few as well (one after the other those took 2 us: whole call, 1 M parameters, M = 2 / 4 / 9 / 16 13.0 / 14.7 / 20.7 / 27.1 us,
// now 11.7 / 13.2 / 19.5 / 25.4).  (One wavefront per entry
// and a butterfly of lane exchanges took 5 us at 4 replicas and 25 us at 16, entry after entry.)
__global__ void __launch_bounds__(kFinThreads) sdl_gram_finalize(const FinArgs f)
{
    __shared__ double G[SDL_MAX_WORKERS * SDL_MAX_WORKERS];
    __shared__ double C[SDL_MAX_WORKERS * SDL_MAX_WORKERS];
    __shared__ double part[kFinThreads];
    const bool all = f.last_out && blockIdx.x + 1u == gridDim.x;
    const uint32_t first = f.first[all ? 0u : blockIdx.x], count = f.first[blockIdx.x + (all ? 0u : 1u)] - first;
    const uint32_t M = f.M, entries = M * (M + 1u) / 2u, S = fin_slices(M);
    const double* base = f.in + (uint64_t)first * f.stride_k;
    const uint32_t entry = threadIdx.x % entries, slice = threadIdx.x / entries;
    uint32_t a = 0, b = entry;             // entry number -> (a, b), row by row of the upper triangle
    while (b >= M - a) { b -= M - a; ++a; }
    b += a;
    if (slice < S) {
        double s = 0.0;
        const double* const mine = base + a * M + b;
        for (uint32_t k = slice; k < count; k += 8u * S) {
            double x[8];
#pragma unroll
            for (uint32_t i = 0; i < 8u; ++i) {
                const bool there = k + i * S < count;
                x[i] = mine[(uint64_t)(there ? k + i * S : k) * f.stride_k];
                x[i] = there ? x[i] : 0.0;
            }
#pragma unroll
            for (uint32_t i = 0; i < 8u; ++i) s += x[i];
        }
        part[threadIdx.x] = s;
    }
    __syncthreads();
    if (M >= kFewSlices) {
        // up to 11 slices, one after the other, and what the additions round off at the end: no slower than a tree with its barriers (1 M
        // parameters, M = 13 / 16 24.0 / 26.3 us, now 23.6 / 26.2), and one rounding.  (By the tree the sums of digits, which are exact but leave
        // more matrices, were no closer to the exact sum than those of FMAs: 8 M parameters, M = 16 rms 1.02e-16 and 0.94e-16, now 0.80e-16.)
        if (threadIdx.x < entries) {
            double s = part[threadIdx.x], rest = 0.0;
            for (uint32_t k = 1; k < S; ++k) {
                const double x = part[threadIdx.x + k * entries], t = s + x, y = t - s;
                rest += (s - (t - y)) + (x - y);
                s = t;
            }
            if (__builtin_fabs(s) <= kDblMax) s += rest;
            G[a * M + b] = s;
            G[b * M + a] = s;
        }
    } else {
        // the slices, pair by pair (a sum in sequence would lose a digit that the partial matrices still have)
        for (uint32_t n = S; n > 1u;) {
            const uint32_t half = (n + 1u) / 2u;
            if (slice + half < n) part[threadIdx.x] += part[threadIdx.x + half * entries];
            n = half;
            __syncthreads();
        }
        if (threadIdx.x < entries) {
            G[a * M + b] = part[threadIdx.x];
            G[b * M + a] = part[threadIdx.x];
        }
    }
    __syncthreads();
    double* o = all ? f.last_out : f.out + (uint64_t)blockIdx.x * f.out_stride;
    if (!f.emit) {
        for (uint32_t i = threadIdx.x; i < M * M; i += blockDim.x) o[i] = G[i];
        return;
    }
    for (uint32_t i = threadIdx.x; i < M * M; i += blockDim.x) {
        const uint32_t a = i / M, b = i % M;
        const double den = __builtin_sqrt(G[a * M + a]) * __builtin_sqrt(G[b * M + b]);
        const double c = den > 0.0 ? G[i] / den : 0.0;
        C[i] = c;
        o[i] = G[i];
        o[M * M + i] = c;
    }
    __syncthreads();
    // the mean over the pairs a < b, by the threads of the first slice, as a tree (pair after pair in one thread: 2 us at 16 replicas)
    if (threadIdx.x < entries) part[threadIdx.x] = a < b ? C[a * M + b] : 0.0;
    __syncthreads();
    for (uint32_t n = entries; n > 1u;) {
        const uint32_t half = (n + 1u) / 2u;
        if (threadIdx.x + half < n) part[threadIdx.x] += part[threadIdx.x + half];
        n = half;
        __syncthreads();
    }
    if (threadIdx.x == 0) o[2 * M * M] = M > 1u ? part[0] / (double)(entries - M) : 0.0;
}

// ------------------------------------------------------------------ host side

int launch_kernel(uint32_t M, const GramArgs& a, hipStream_t st)
{
    const dim3 grid(a.first_wg[a.n_pieces]), one(a.waves * kWave);
    switch (M) {
    case 1: hipLaunchKernelGGL((sdl_gram_kernel<1>), grid, one, 0, st, a); break;
    case 2: hipLaunchKernelGGL((sdl_gram_kernel<2>), grid, one, 0, st, a); break;
    case 3: hipLaunchKernelGGL((sdl_gram_kernel<3>), grid, one, 0, st, a); break;
    case 4: hipLaunchKernelGGL((sdl_gram_kernel<4>), grid, one, 0, st, a); break;
    case 5: hipLaunchKernelGGL((sdl_gram_kernel<5>), grid, one, 0, st, a); break;
    case 6: hipLaunchKernelGGL((sdl_gram_kernel<6>), grid, one, 0, st, a); break;
    case 7: hipLaunchKernelGGL((sdl_gram_kernel<7>), grid, one, 0, st, a); break;
    case 8: hipLaunchKernelGGL((sdl_gram_kernel<8>), grid, one, 0, st, a); break;
    default: return SDL_ERR_INVALID_ARG;
    }
    return hipGetLastError() == hipSuccess ? SDL_OK : SDL_ERR_DEVICE;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool all_aligned16(const float* g, const void* const* w, uint32_t M, uint64_t offset)
{
    bool fast = aligned16(g + offset);
    for (uint32_t m = 0; m < M; ++m) fast = fast && aligned16(static_cast<const uint16_t*>(w[m]) + offset);
    return fast;
}

// Shares the launch's workgroups of so many wavefronts out among the sets in proportion to their tiles (at least
// one each); returns the total, at most groups + n_sets.
uint32_t share_groups(Set* sets, uint32_t n_sets, uint32_t groups, uint32_t waves)
{
    uint64_t total_tiles = 0;
    for (uint32_t s = 0; s < n_sets; ++s) total_tiles += (sets[s].numel + kTile - 1) / kTile;
    uint32_t next = 0;
    for (uint32_t s = 0; s < n_sets; ++s) {
        const uint64_t tiles = (sets[s].numel + kTile - 1) / kTile;
        uint64_t G = total_tiles ? (tiles * groups + total_tiles - 1) / total_tiles : 1;
        if (G > (tiles + waves - 1) / waves) G = (tiles + waves - 1) / waves;
        if (G < 1) G = 1;
        sets[s].first_wg = next;
        sets[s].G = (uint32_t)G;
        next += (uint32_t)G;
    }
    return next;
}

// Partial Gram matrices of up to kMaxSets sets (already given their workgroups) into
// `partial`, one M x M matrix per workgroup of the launch.
int launch_gram(const float* g, const void* const* w, uint32_t M, const Set* sets, uint32_t n_sets, uint32_t waves, double* partial,
                hipStream_t st)
{
    GramArgs a{};
    a.waves = waves;
    a.g = g;
    a.partial = partial;
    for (uint32_t& x : a.group_wg) x = 0xffffffffu;
    for (uint32_t& x : a.first_wg) x = 0xffffffffu;
    // cut the sets into windows: about `windows` pieces per launch, shared out like the workgroups
    const uint32_t windows = kWindows;
    uint64_t total_G = 0;
    for (uint32_t s = 0; s < n_sets; ++s) total_G += sets[s].G;
    for (uint32_t s = 0; s < n_sets; ++s) {
        const uint64_t tiles = (sets[s].numel + kTile - 1) / kTile;
        // only a set that holds a large share of the launch is cut (measured: cutting the spans
        // of a many-span fragment in two or three costs a few per cent, one large span gains 10 %)
        uint64_t nsub = total_G ? (uint64_t)windows * sets[s].G / total_G : 1;
        if (nsub < 4) nsub = 1;
        if (nsub > sets[s].G) nsub = sets[s].G;
        if (nsub > tiles) nsub = tiles;
        if (nsub < 1) nsub = 1;
        const uint64_t tiles_per = (tiles + nsub - 1) / nsub;
        for (uint64_t j = 0; j < nsub; ++j) {
            const uint32_t number = a.n_pieces++;
            const uint64_t e0 = j * tiles_per * kTile;
            const uint64_t e1 = (j + 1) * tiles_per * kTile < sets[s].numel ? (j + 1) * tiles_per * kTile : sets[s].numel;
            const uint64_t offset = sets[s].offset + (e0 < sets[s].numel ? e0 : sets[s].numel), numel = e1 > e0 ? e1 - e0 : 0;
            if (offset >= kMaxOffset || numel > 0xffffffffull) return SDL_ERR_UNSUPPORTED;     // more than any memory holds
            const uint32_t first = sets[s].first_wg + (uint32_t)((uint64_t)sets[s].G * j / nsub);
            a.first_wg[number] = first;
            if (number % 16u == 0u && number) a.group_wg[number / 16u - 1u] = first;
            a.offset[number] = (uint32_t)offset;
            a.numel[number] = (uint32_t)numel;
            const uint32_t high = (uint32_t)(offset >> 32) | (all_aligned16(g, w, M, offset) ? kFast : 0u);
            a.high[number / 4u] |= high << (number % 4u * 8u);
        }
    }
    a.first_wg[a.n_pieces] = sets[n_sets - 1].first_wg + sets[n_sets - 1].G;
    for (uint32_t m = 0; m < M; ++m) a.w[m] = static_cast<const uint16_t*>(w[m]);
    return launch_kernel(M, a, st);
}

// Partial Gram matrices of more than 8 replicas; sets[s].first_wg and .G become the numbers of set s's first matrix and of its
// matrices.  n_mats = all of them.
int launch_pair(const float* g, const void* const* w, uint32_t M, Set* sets, uint32_t n_sets, double* partial, uint32_t* n_mats,
                hipStream_t st)
{
    const uint32_t H = (M + 1u) / 2u;
    PairArgs a{};
    a.g = g;
    a.partial = partial;
    a.M = M;
    for (uint32_t m = 0; m < M; ++m) a.w[m] = static_cast<const uint16_t*>(w[m]);
    uint64_t tiles = 0, params = 0;
    for (uint32_t s = 0; s < n_sets; ++s) params += sets[s].numel;
    const bool digits = takes_digits(M, params);
    const uint64_t tile = digits ? kDigitTile : kPairTile;
    for (uint32_t s = 0; s < n_sets; ++s) {
        a.first_tile[s] = (uint32_t)tiles;
        if (s % 16u == 0u && s) a.group_tile[s / 16u - 1u] = (uint32_t)tiles;
        a.offset[s] = (uint32_t)sets[s].offset;
        const uint64_t rest = sets[s].numel % tile;
        a.more[s] = (uint32_t)(sets[s].offset >> 32) | (all_aligned16(g, w, M, sets[s].offset) ? kFast : 0u) | (uint32_t)(rest ? rest : tile) << 8;
        tiles += (sets[s].numel + tile - 1) / tile;
        if (tiles >= 0xffffffffull || sets[s].offset >= kMaxOffset) return SDL_ERR_UNSUPPORTED;     // more than any memory holds
    }
    a.first_tile[n_sets] = (uint32_t)tiles;
    for (uint32_t i = (n_sets + 15u) / 16u; i < (uint32_t)kMaxSets / 16u; ++i)
        if (i) a.group_tile[i - 1u] = 0xffffffffu;
    for (uint32_t s = n_sets + 1u; s <= (uint32_t)kMaxSets; ++s) a.first_tile[s] = 0xffffffffu;
    const uint32_t resident = pair_resident(M, digits);
    uint32_t mats = 0, n_wg = 0, at = 0;
    constexpr uint32_t kPercents[kShares][kShares] = {{100, 0, 0}, {93, 100, 0}, {85, 70, 100}};      // of what is left
    const uint32_t* const percent = kPercents[params <= kOneShare ? 0 : params <= kTwoShares ? 1 : 2];
    for (int i = 0; i < kShares; ++i) {
        const uint32_t left = (uint32_t)tiles - at, n = (uint32_t)((uint64_t)left * percent[i] / 100u);
        const uint32_t wgs = n < resident ? n : resident;
        a.shares[i] = Share{n_wg, at, wgs ? n / wgs : 0u, wgs ? n % wgs : 0u};
        n_wg += wgs;
        at += n;
    }
    auto wg_of = [&](uint32_t t) {
        int i = kShares - 1;
        while (i > 0 && t < a.shares[i].first_tile) --i;
        const Share& sh = a.shares[i];
        const uint32_t nth = t - sh.first_tile, longer = sh.extra * (sh.per_wg + 1u);
        return sh.first_wg + (nth < longer ? nth / (sh.per_wg + 1u) : sh.extra + (nth - longer) / sh.per_wg);
    };
    for (uint32_t s = 0; s < n_sets; ++s) {
        sets[s].first_wg = mats;
        sets[s].G = 0;
        if (a.first_tile[s + 1] == a.first_tile[s]) continue;
        const uint32_t b0 = wg_of(a.first_tile[s]), b1 = wg_of(a.first_tile[s + 1] - 1u);
        a.slot[s] = (int32_t)mats - (int32_t)b0;
        sets[s].G = b1 - b0 + 1u;
        mats += sets[s].G;
    }
    *n_mats = mats;
    if (!n_wg) return SDL_OK;
    const dim3 grid(n_wg), block(2 * kWave);
    if (digits) {
        if (H == 7u) hipLaunchKernelGGL((sdl_digit_sums_kernel<7>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((sdl_digit_sums_kernel<8>), grid, block, 0, st, a);
        return hipGetLastError() == hipSuccess ? SDL_OK : SDL_ERR_DEVICE;
    }
    switch (H) {
    case 5: hipLaunchKernelGGL((sdl_gram_pair_kernel<5>), grid, block, 0, st, a); break;
    case 6: hipLaunchKernelGGL((sdl_gram_pair_kernel<6>), grid, block, 0, st, a); break;
    case 7: hipLaunchKernelGGL((sdl_gram_pair_kernel<7>), grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL((sdl_gram_pair_kernel<8>), grid, block, 0, st, a); break;
    }
    return hipGetLastError() == hipSuccess ? SDL_OK : SDL_ERR_DEVICE;
}

int launch_finalize(const FinArgs& f, uint32_t n_out, hipStream_t st)
{
    // whole wavefronts for the entries and their slices: 64 threads at one replica, 192 at two (idle ones cost their barriers)
    const uint32_t threads = (f.M * (f.M + 1u) / 2u * fin_slices(f.M) + kWave - 1u) / kWave * kWave;
    hipLaunchKernelGGL(sdl_gram_finalize, dim3(n_out), dim3(threads), 0, st, f);
    return hipGetLastError() == hipSuccess ? SDL_OK : SDL_ERR_DEVICE;
}

// Partial Gram matrices of up to kMaxSets sets into `partial`; where they lie goes into the sets.  Up to 8 replicas by the rule at kGramWaves.
int launch_sums(const float* g, const void* const* w, uint32_t M, Set* sets, uint32_t n_sets, double* partial, uint32_t* n_mats,
                hipStream_t st)
{
    if (M > 8u) return launch_pair(g, w, M, sets, n_sets, partial, n_mats, st);
    uint64_t params = 0;
    for (uint32_t s = 0; s < n_sets; ++s) params += sets[s].numel;
    const bool one = M == 8u && n_sets > kFewSets;
    const uint32_t groups = one ? kGroups : params > kFewFours ? kManyFours : kFours;
    const uint32_t waves = one ? 1u : kGramWaves;
    *n_mats = share_groups(sets, n_sets, groups - n_sets, waves);
    return launch_gram(g, w, M, sets, n_sets, waves, partial, st);
}

// One result per set from the partial matrices of its workgroups (at partial + first_wg; the sets' matrices lie one behind the other) and, if
// union_out is not null, the result of all of them together.  Sets with many workgroups are first added up in chunks (into
// tmp), so that no thread of the finalize kernel walks a long range.
// Many is four chunks: a second launch costs 2 us, as much as a thread's 32 loads, eight at a time.  (At two chunks, 1 M parameters, M = 1 / 2 / 4
// 11.3 / 11.4 / 13.3 us, at four 9.4 / 9.5 / 12.5; at eight slower with 6 replicas and more.)
int finalize_sets(const double* partial, const Set* sets, uint32_t n_sets, uint32_t M, double* out, double* union_out,
                  double* tmp, hipStream_t st)
{
    const uint64_t mm = (uint64_t)M * M;
    const uint32_t chunk = fin_chunk(M);
    uint32_t total = 0;
    bool two_level = false;
    for (uint32_t s = 0; s < n_sets; ++s) {
        two_level = two_level || sets[s].G > 4 * chunk;
        total += sets[s].G;
    }
    two_level = two_level || (union_out && total > 4 * chunk);
    FinArgs last{};
    last.out = out;
    last.last_out = union_out;
    last.stride_k = mm;
    last.out_stride = SDL_COSINE_RESULT_DOUBLES(M);
    last.M = M;
    last.emit = 1;
    last.in = two_level ? tmp : partial;
    if (two_level) {
        FinArgs lvl1{};
        lvl1.in = partial;
        lvl1.stride_k = mm;
        lvl1.out_stride = mm;
        lvl1.M = M;
        uint32_t n = 0, done = 0;         // first-level outputs, and those of them that have been launched
        auto launch = [&](uint32_t end) {
            lvl1.first[n - done] = end;
            lvl1.out = tmp + (uint64_t)done * mm;
            const uint32_t count = n - done;
            done = n;
            return launch_finalize(lvl1, count, st);
        };
        for (uint32_t s = 0; s < n_sets; ++s) {
            last.first[s] = n;
            for (uint32_t c = 0; c < sets[s].G; c += chunk) {
                if (n - done == kMaxFin) {
                    const int rc = launch(sets[s].first_wg + c);
                    if (rc != SDL_OK) return rc;
                }
                lvl1.first[n++ - done] = sets[s].first_wg + c;
            }
        }
        last.first[n_sets] = n;
        if (n > done) {
            const int rc = launch(sets[0].first_wg + total);
            if (rc != SDL_OK) return rc;
        }
    } else {
        for (uint32_t s = 0; s < n_sets; ++s) last.first[s] = sets[s].first_wg;
        last.first[n_sets] = sets[0].first_wg + total;
    }
    return launch_finalize(last, n_sets + (union_out ? 1u : 0u), st);
}

// One result from the Gram matrices of `count` results that lie stride doubles apart.
int finalize_union(const double* results, uint64_t stride, uint32_t count, uint32_t M, double* out, hipStream_t st)
{
    FinArgs f{};
    f.in = results;
    f.out = out;
    f.stride_k = stride;
    f.out_stride = SDL_COSINE_RESULT_DOUBLES(M);
    f.M = M;
    f.emit = 1;
    f.first[0] = 0;
    f.first[1] = count;
    return launch_finalize(f, 1, st);
}

// Workspace layout, in M x M matrices: the partial matrices of every launch, then the
// first-level sums of the finalize step; then (plan-level call without span_results) one
// result per set.
size_t partial_mats(size_t n_sets)
{
    const size_t launches = (n_sets + kFewSets - 1) / kFewSets;     // or fewer
    return launches * kMaxGroups + n_sets;
}
size_t tmp_mats(size_t n_sets)
{
    const size_t launches = (n_sets + kFewSets - 1) / kFewSets;
    return launches * kFirstLevel + 2 * n_sets;
}

int check_common(const void* g, const void* const* w, uint32_t M, const void* workspace)
{
    if (!g || !w || M == 0 || M > SDL_MAX_WORKERS || !workspace) return SDL_ERR_INVALID_ARG;
    for (uint32_t m = 0; m < M; ++m)
        if (!w[m]) return SDL_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(workspace) & 7u) return SDL_ERR_ALIGNMENT;
    return SDL_OK;
}

}  // namespace

extern "C" {

size_t sdl_cosine_workspace_bytes(uint32_t M, uint32_t n_sets)
{
    if (M == 0 || M > SDL_MAX_WORKERS) return 0;
    return ((partial_mats(n_sets) + tmp_mats(n_sets)) * M * M + (size_t)n_sets * SDL_COSINE_RESULT_DOUBLES(M))
           * sizeof(double);
}

int sdl_outer_grad_cosine(const float* g, const void* const* w, uint32_t M, uint64_t numel, double* result,
                          void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_common(g, w, M, workspace);
    if (rc != SDL_OK) return rc;
    if (!result) return SDL_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(result) & 7u) return SDL_ERR_ALIGNMENT;
    if (workspace_bytes < sdl_cosine_workspace_bytes(M, 1)) return SDL_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Set set{0, numel, 0, 0};
    double* partial = static_cast<double*>(workspace);
    double* tmp = partial + partial_mats(1) * M * M;
    uint32_t n_mats = 0;
    rc = launch_sums(g, w, M, &set, 1, partial, &n_mats, st);
    if (rc != SDL_OK) return rc;
    return finalize_sets(partial, &set, 1, M, result, nullptr, tmp, st);
}

int sdl_outer_grad_cosine_plan(const sdl_plan_t* plan, uint32_t p, const float* g_base, const void* const* w_base,
                               uint32_t M, double* span_results, double* fragment_result, void* workspace,
                               size_t workspace_bytes, void* stream)
{
    int rc = check_common(g_base, w_base, M, workspace);
    if (rc != SDL_OK) return rc;
    if (!plan || !fragment_result) return SDL_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(fragment_result) & 7u) || (reinterpret_cast<uintptr_t>(span_results) & 7u))
        return SDL_ERR_ALIGNMENT;
    const sdl_span_t* spans = nullptr;
    uint32_t n_spans = 0;
    rc = sdl_plan_fragment_spans(plan, p, &spans, &n_spans);
    if (rc != SDL_OK) return rc;
    if (workspace_bytes < sdl_cosine_workspace_bytes(M, n_spans)) return SDL_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint64_t mm = (uint64_t)M * M, R = SDL_COSINE_RESULT_DOUBLES(M);
    double* partial = static_cast<double*>(workspace);
    double* tmp = partial + partial_mats(n_spans) * mm;
    double* per_span = span_results ? span_results : tmp + tmp_mats(n_spans) * mm;
    for (uint32_t b0 = 0; b0 < n_spans; b0 += kBatch) {
        const uint32_t n = n_spans - b0 < kBatch ? n_spans - b0 : kBatch;
        Set sets[kBatch];
        uint32_t used = 0;             // matrices so far
        for (uint32_t s0 = 0, s1 = 0; s0 < n; s0 = s1) {
            uint64_t params = 0;
            for (; s1 < n && s1 - s0 < (uint32_t)kMaxSets; ++s1) {
                params += spans[b0 + s1].numel;
                if (s1 - s0 >= kFewSets && params > kManyParams) break;
                sets[s1] = Set{spans[b0 + s1].offset, spans[b0 + s1].numel, 0, 0};
            }
            uint32_t n_mats = 0;
            rc = launch_sums(g_base, w_base, M, sets + s0, s1 - s0, partial + (uint64_t)used * mm, &n_mats, st);
            if (rc != SDL_OK) return rc;
            for (uint32_t s = s0; s < s1; ++s) sets[s].first_wg += used;
            used += n_mats;
        }
        // the spans of one batch give the fragment's result as well
        rc = finalize_sets(partial, sets, n, M, per_span + (uint64_t)b0 * R, n == n_spans ? fragment_result : nullptr, tmp, st);
        if (rc != SDL_OK) return rc;
        partial += (uint64_t)used * mm;
    }
    if (n_spans && n_spans <= kBatch) return SDL_OK;
    // the fragment: Gram matrices of its spans added in span order
    return finalize_union(per_span, R, n_spans, M, fragment_result, st);
}

int sdl_cosine_combine(const double* results, uint64_t stride_doubles, uint32_t n_sets, uint32_t M, double* result,
                       void* stream)
{
    if (!results || !result || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    if (n_sets && stride_doubles < SDL_COSINE_RESULT_DOUBLES(M)) return SDL_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(results) & 7u) || (reinterpret_cast<uintptr_t>(result) & 7u))
        return SDL_ERR_ALIGNMENT;
    return finalize_union(results, stride_doubles, n_sets, M, result, static_cast<hipStream_t>(stream));
}

}  // extern "C"
