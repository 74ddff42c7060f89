// Cosine similarity between the replicas' outer gradients (Appendix of the paper, paragraph on
// the outer gradients' cosine similarity) for gfx950 (MI355X).
//
// Four kernels.
//   sdl_gram_kernel   up to 8 replicas: streams g and the M replicas once and accumulates the Gram matrix of
//                     the outer gradients Delta_m = g - float(w_m).  A workgroup is one
//                     64-lane wavefront; a set of parameters gets a share G of the launch's
//                     workgroups in proportion to its size, and workgroup k of the set walks
//                     the set's tiles of 512 consecutive parameters with a fixed stride
//                     (tile k, k + G, k + 2G, ...), lane l owning the eight
//                     parameters [8l, 8l+8) of a tile, so every load instruction of the
//                     wavefront covers one contiguous piece of an array (2 x 1 KiB of fp32,
//                     1 KiB of bf16 through 128-bit accesses).  Each lane keeps its M(M+1)/2
//                     sums in fp64 registers (products of fp32 values are exact in fp64); at
//                     the end the wavefront folds them with a butterfly of lane exchanges and
//                     lane 0 writes one partial Gram matrix.  The next tile's loads are issued
//                     before the current tile is consumed.
//   sdl_gram_pair_kernel  the same for 9 to 12 replicas, two wavefronts with half of the matrix each.
//   sdl_gram_mfma_kernel  the same for 13 to 16 replicas, on the matrix cores.
//   sdl_gram_finalize adds the partial matrices of a set in a fixed order (one thread per entry and
//                     slice of the matrices, then the slices as a tree; a set with many partial matrices in
//                     two launches) and derives cos and the mean over pairs.  The same kernel adds
//                     the Gram matrices of several sets (fragment from spans, unions of fragments).
// No atomics: the order of every sum depends on the sizes alone, so results are reproducible.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "sdl.h"
#include "sdl_device.h"

namespace {

using namespace sdl_device;

constexpr int kLaneElems = 8;                   // consecutive parameters a lane owns in a tile
constexpr int kTile = kLaneElems * kWave;       // 512
constexpr int kMaxSets = 48;                    // parameter sets per launch
constexpr int kWindows = 48;                    // windows per launch: a set holding a share of 4/48 or more is cut
constexpr int kMaxPieces = kMaxSets + kWindows;
constexpr int kPairM = 12;                      // most replicas whose matrix two wavefronts share
constexpr uint32_t kGroups = 8192;              // workgroups per launch, shared out among the sets (32 per compute unit)
constexpr uint32_t kWideGroups = 4096;          // the same for the matrix cores, 4 wavefronts each (1024: 15-20 % slower, the
                                                // last round of workgroups is nearly empty; 8192: up to 5 %, twice the
                                                // partial matrices)
constexpr uint32_t kMaxGroups = 8192;           // what the workspace is sized for


struct Set {
    uint64_t offset;     // first element in the flat arrays
    uint64_t numel;
    uint32_t first_wg;   // first workgroup of the launch that works on this set
    uint32_t G;          // workgroups of this set (>= 1)
};

// What the kernel walks: a set, or a window of a large set (tile aligned), with its own
// share of the set's workgroups.
struct Piece {
    uint64_t offset;
    uint64_t numel;
    uint32_t first_wg;
    uint32_t G;
    uint32_t fast;       // every array is 16-byte aligned at the piece's start
    uint32_t pad_;
};

struct GramArgs {
    const float* g;
    const uint16_t* w[SDL_MAX_WORKERS];
    double* partial;               // [workgroup of the launch][M*M]
    uint32_t M;                    // side of the matrix
    uint32_t n_pieces;
    Piece pieces[kMaxPieces];
};
static_assert(sizeof(GramArgs) <= 4096, "kernel arguments");

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
        const u32x4_f32elem* pg = reinterpret_cast<const u32x4_f32elem*>(g + e0 + lane * kLaneElems);
        t.g0 = __builtin_nontemporal_load(pg);
        t.g1 = __builtin_nontemporal_load(pg + 1);
#pragma unroll
        for (int m = 0; m < NW; ++m)
            t.w[m] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_bf16elem*>(w[m] + e0 + lane * kLaneElems));
    } else {
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

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Up to 8 replicas: every lane holds the whole upper triangle.
template <int M>
__global__ void __launch_bounds__(kWave) sdl_gram_kernel(const GramArgs a)
{
    const uint32_t lane = threadIdx.x;
    uint32_t s = 0;
    while (s + 1 < a.n_pieces && blockIdx.x >= a.pieces[s + 1].first_wg) ++s;
    const Piece set = a.pieces[s];
    const uint32_t k = blockIdx.x - set.first_wg;
    const bool fast = set.fast != 0u;
    const uint64_t n_tiles = (set.numel + kTile - 1) / kTile;

    const uint16_t* w[M];
#pragma unroll
    for (int m = 0; m < M; ++m) w[m] = a.w[m];

    double acc[M][M];
#pragma unroll
    for (int r = 0; r < M; ++r)
#pragma unroll
        for (int c = 0; c < M; ++c) acc[r][c] = 0.0;

    auto valid_of = [&](uint64_t t) -> uint32_t {
        const uint64_t rem = set.numel - t * kTile;
        return rem < (uint64_t)kTile ? (uint32_t)rem : (uint32_t)kTile;
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
#pragma unroll
            for (int r = 0; r < M; ++r)
#pragma unroll
                for (int c = r; c < M; ++c) acc[r][c] = __builtin_fma(d[r], d[c], acc[r][c]);
        }
    };

    // workgroup k's tiles: first, first + step, ... below end; the next tile's loads are issued before the
    // current tile is consumed
    const uint64_t first = k, step = set.G, end = n_tiles;
    TileRegs<M> cur;
    if (first < end) load_tile<M>(cur, a.g, w, set.offset + first * kTile, valid_of(first), fast, lane);
    for (uint64_t t = first; t < end; t += step) {
        TileRegs<M> nxt = cur;
        const uint64_t tn = t + step;
        if (tn < end) load_tile<M>(nxt, a.g, w, set.offset + tn * kTile, valid_of(tn), fast, lane);
        consume(cur);
        cur = nxt;
    }

    double* out = a.partial + (uint64_t)blockIdx.x * M * M;
#pragma unroll
    for (int r = 0; r < M; ++r)
#pragma unroll
        for (int c = r; c < M; ++c) {
            const double v = wave_sum(acc[r][c]);
            if (lane == 0) out[r * M + c] = v;
        }
}

// 9 to 12 replicas, H = ceil(M / 2) per half, in one pass over memory (blocks of 8 x 8 need three).  One lane cannot hold 78 sums, the
// tile and the next one; the two wavefronts of a workgroup run the same code on the same tiles (the second finds them in L1
// / L2) and differ in which replicas they call "rows" and "columns":
//   wavefront 0   rows i = replicas 0..H-1,       columns j = replicas H..2H-1
//   wavefront 1   rows i = replicas H..2H-1,      columns j = replicas 1, 2, ... H-1, 0
// Each forms its rows' triangle and, of the block rows x columns, the entries with (j - i) mod H < ceil(H / 2): in the first
// wavefront's terms the second one forms those with (j - i) mod H >= H - ceil(H / 2), so all are there (for odd H one
// diagonal twice).  With odd M the replica 2H-1 does not exist: the lanes work on replica 0 in its place and nothing of it
// is stored.  Bound: both wavefronts form all 2H differences, and 166 / 198 registers leave 3 / 2 wavefronts on a SIMD to cover
// the loads.  52.9 M parameters, M = 9 / 10 / 12, whole call: 467 / 511 / 629 us as 8 x 8 blocks, 291 / 302 / 385 now (HBM 164 /
// 179 / 209, the matrix cores 475).  At 14 two wavefronts of 249 registers on a SIMD no longer cover
// the loads (494).
// Workgroups: as many as sdl_gram_kernel has, so that a lane's chain of additions is no longer than there.  With half as many
// M = 11 and 12 took 367 and 374 us (302 M parameters, M = 12: 2070, 1961 now), but the error of G[m][m] doubled: outliers
// 7.0e-16 where one wavefront at M = 8 has 3.4e-16, 3.7e-16 to 4.2e-16 now.
template <int H>
struct PairTile {
    f32x4_elem g;
    u32x2 w[2 * H];
};
constexpr int kPairTile = 4 * kWave;      // parameters a wavefront takes at a time

template <int H>
__device__ __forceinline__ void load_pair_tile(PairTile<H>& t, const float* g, const uint16_t* (&w)[2 * H], uint64_t e0,
                                               uint64_t left, bool fast, uint32_t lane)
{
    if (fast && left >= (uint64_t)kPairTile) {
        // normal cache policy: the other wavefront reads the same lines
        t.g = __builtin_bit_cast(f32x4_elem, __builtin_amdgcn_raw_buffer_load_b128(rsrc(g + e0, kPairTile * 4), (int)(lane * 16), 0, 0));
#pragma unroll
        for (int m = 0; m < 2 * H; ++m)
            t.w[m] = __builtin_amdgcn_raw_buffer_load_b64(rsrc(w[m] + e0, kPairTile * 2), (int)(lane * 8), 0, 0);
    } else if (left >= (uint64_t)kPairTile) {
        t.g = *reinterpret_cast<const f32x4_elem*>(g + e0 + lane * 4);
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) {
            const u32x2_elem x = *reinterpret_cast<const u32x2_elem*>(w[m] + e0 + lane * 4);
            t.w[m] = u32x2{x.x, x.y};
        }
    } else {
        // ragged tail: 0 past the end of g and of every replica
        const uint32_t valid = (uint32_t)left;
        const __amdgpu_buffer_rsrc_t rg = rsrc(g + e0, valid * 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) t.g[j] = u2f(__builtin_amdgcn_raw_buffer_load_b32(rg, (int)((lane * 4 + j) * 4), 0, 0));
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) {
            const __amdgpu_buffer_rsrc_t rw = rsrc(w[m] + e0, valid * 2);
            uint32_t h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                h[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rw, (int)((lane * 4 + j) * 2), 0, 0) & 0xffffu;
            t.w[m] = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
        }
    }
}

template <int H>
__global__ void __launch_bounds__(2 * kWave, 2) sdl_gram_pair_kernel(const GramArgs a)
{
    constexpr int kOff = (H + 1) / 2;     // entries of the block rows x columns per row
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    uint32_t s = 0;
    while (s + 1 < a.n_pieces && blockIdx.x >= a.pieces[s + 1].first_wg) ++s;
    const Piece set = a.pieces[s];
    const bool fast = set.fast != 0u;
    const uint32_t M = a.M;

    auto row = [&](int i) -> uint32_t { return wave ? (uint32_t)(H + i) : (uint32_t)i; };
    auto col = [&](int j) -> uint32_t { return wave ? (uint32_t)((j + 1) % H) : (uint32_t)(H + j); };
    const uint16_t* w[2 * H];
#pragma unroll
    for (int i = 0; i < H; ++i) {
        w[i] = a.w[row(i) < M ? row(i) : 0u];
        w[H + i] = a.w[col(i) < M ? col(i) : 0u];
    }

    double tri[H][H], off[H][kOff];
#pragma unroll
    for (int i = 0; i < H; ++i) {
#pragma unroll
        for (int j = 0; j < H; ++j) tri[i][j] = 0.0;
#pragma unroll
        for (int j = 0; j < kOff; ++j) off[i][j] = 0.0;
    }

    auto consume = [&](const PairTile<H>& t) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double d[2 * H];
#pragma unroll
            for (int m = 0; m < 2 * H; ++m) {
                const uint32_t u = t.w[m][e / 2];
                d[m] = (double)(t.g[e] - u2f((e & 1) ? (u & 0xffff0000u) : (u << 16)));   // one fp32 subtraction
            }
#pragma unroll
            for (int i = 0; i < H; ++i) {
#pragma unroll
                for (int j = i; j < H; ++j) tri[i][j] = __builtin_fma(d[i], d[j], tri[i][j]);
#pragma unroll
                for (int j = 0; j < kOff; ++j) off[i][j] = __builtin_fma(d[i], d[H + (i + j) % H], off[i][j]);
            }
        }
    };

    const uint64_t step = (uint64_t)set.G * kPairTile;
    uint64_t at = (uint64_t)(blockIdx.x - set.first_wg) * kPairTile;
    PairTile<H> cur;
    if (at < set.numel) load_pair_tile<H>(cur, a.g, w, set.offset + at, set.numel - at, fast, lane);
    for (; at < set.numel; at += step) {
        PairTile<H> nxt = cur;
        const uint64_t an = at + step;
        if (an < set.numel) load_pair_tile<H>(nxt, a.g, w, set.offset + an, set.numel - an, fast, lane);
        __builtin_amdgcn_sched_barrier(0);   // the loads stay ahead of the arithmetic
        consume(cur);
        cur = nxt;
    }

    double* out = a.partial + (uint64_t)blockIdx.x * M * M;
    auto store = [&](uint32_t x, uint32_t y, double v) {
        v = wave_sum(v);
        if (lane == 0 && x < M && y < M) out[x < y ? x * M + y : y * M + x] = v;
    };
#pragma unroll
    for (int i = 0; i < H; ++i) {
#pragma unroll
        for (int j = i; j < H; ++j) store(row(i), row(j), tri[i][j]);
#pragma unroll
        for (int j = 0; j < kOff; ++j)
            if (!(H % 2 == 1 && j == kOff - 1 && wave == 1u))    // the diagonal that both formed: once is enough
                store(row(i), col((i + j) % H), off[i][j]);
    }
}

// 13 to 16 replicas: the matrix cores form the whole matrix, v_mfma_f64_16x16x4_f64 taking four parameters of up to 16
// replicas at a time.  Lane l holds replica l % 16's value of parameter l / 16, which is the instruction's layout of the left
// operand and of the right one alike.  Bound: the matrix pipe, 256 fp64 FMAs per parameter (half of them for the lower
// triangle; rows behind the last replica repeat replica 0 and are not stored): 52.9 M parameters at the 77 TFLOP/s that a
// chain of this instruction reaches take 350 us, HBM 268 us at 16 replicas; the loads alone take 370 us in this layout, the
// arithmetic alone (the same few lines loaded again and again) 494: the conversions and additions between the chains are
// fp64 operations as well.  Whole call at 13 / 16 replicas: 698 / 935 us as 8 x 8 blocks in three launches, 502 / 510 now.
// A load covers 64 bytes of 16 arrays; the chunk of 64 parameters that a wavefront takes at a time is a whole line of each.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kMfmaWaves = 4;             // wavefronts per workgroup, which adds their matrices up before it writes one
constexpr int kMfmaChunk = 64;            // parameters: 16 per lane, as two pieces of 8

struct MfmaChunk {
    u32x4 g[2][2], w[2];
};

// g and w: the lane's first parameter of the chunk (w in the lane's replica).
__device__ __forceinline__ void load_chunk(MfmaChunk& c, const float* g, const uint16_t* w)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u32x4_f32elem* pg = reinterpret_cast<const u32x4_f32elem*>(g + 32 * h);
        c.g[h][0] = pg[0];
        c.g[h][1] = pg[1];
        c.w[h] = *reinterpret_cast<const u32x4_bf16elem*>(w + 32 * h);
    }
}

// The instruction rounds its sums towards zero, so a chain of it is kept to 4 (16 parameters); a chunk's four chains and the
// chunks are added by plain additions, which round to nearest, at two levels so that neither is long.  Root mean square of the
// error of G[m][m] against exact sums, M = 16, in units of 1e-16, for the recipes normal / student_t3 / outliers / an outer
// gradient with full mantissas: 0.26 M parameters 0.9 / 0.8 / 0.9 / 0.8, 8.4 M 1.0 / 0.9 / 0.9 / 0.8, 52.9 M 1.0 / 0.6 / 1.2 / 1.1;
// the plain FMAs of sdl_gram_kernel at M = 8 give 0.8 / 0.8 / 0.8 / 0.8, 1.0 / 0.8 / 0.9 / 0.5 and 0.9 / 0.4 / 3.5 / 3.7.  One
// chain for a chunk: outliers 2.4, full mantissas 1.8 at every size.  Chains of 8: 1.4 and 1.3, of 2: 0.7 and 0.8.  The whole
// call at 52.9 M parameters: 488 us with chains of 16, 495 with 8, 510 with 4, 550 with 2.
constexpr int kMfmaChain = 4;

struct MfmaSums {
    f64x4 total = {};     // whole chunks
    f64x4 part = {};      // the chains of a chunk
    f64x4 last = {};      // the latest chain, added one chain later, when its instructions have ended
};

__device__ __forceinline__ void add_chunk(const MfmaChunk& c, MfmaSums& s)
{
    f64x4 acc = {};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float f[kLaneElems];
        deltas(c.g[h][0], c.g[h][1], c.w[h], f);
#pragma unroll
        for (int j = 0; j < kLaneElems; ++j) {
            const int k = h * kLaneElems + j;
            const double d = (double)f[j];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(d, d, k % kMfmaChain ? acc : f64x4{}, 0, 0, 0);
            if (k % kMfmaChain != kMfmaChain - 1) continue;
            if (k / kMfmaChain == 0) {                // ends the chunk before this one
                s.part += s.last;
                s.total += s.part;
                asm volatile("" : "+v"(s.total));
            } else if (k / kMfmaChain == 1) {
                s.part = s.last;
            } else {
                s.part += s.last;
                asm volatile("" : "+v"(s.part));
            }
            s.last = acc;
            // Additions stay with their half of the chunk: moved to the end of the tile, they would keep every chain's sums
            // alive, more than the registers hold (spilled ones are read back behind the next chunk's loads).
            if (j == kLaneElems - 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// (four wavefronts per SIMD: left to itself the compiler takes registers for three, 539 us against 504)
__global__ void __launch_bounds__(kMfmaWaves * kWave) __attribute__((amdgpu_waves_per_eu(4)))
sdl_gram_mfma_kernel(const GramArgs a)
{
    __shared__ double mats[kMfmaWaves][16 * 16];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    uint32_t s = 0;
    while (s + 1 < a.n_pieces && blockIdx.x >= a.pieces[s + 1].first_wg) ++s;
    const Piece set = a.pieces[s];
    const uint32_t M = a.M, replica = lane % 16, quarter = lane / 16;
    const float* g = a.g + set.offset + quarter * kLaneElems;
    const uint16_t* w = a.w[replica < M ? replica : 0u] + set.offset + quarter * kLaneElems;

    MfmaSums sums;
    const uint64_t n_whole = set.numel / kTile, step = (uint64_t)set.G * kMfmaWaves;
    uint64_t t = (uint64_t)wave * set.G + (blockIdx.x - set.first_wg);
    MfmaChunk c[2];
    if (t < n_whole) load_chunk(c[0], g + t * kTile, w + t * kTile);
    for (; t < n_whole; t += step) {
#pragma unroll
        for (int k = 0; k < kTile / kMfmaChunk; ++k) {
            // the next chunk's loads go out before this one is consumed, and stay there (the compiler would move each down
            // to its first use)
            if (k + 1 < kTile / kMfmaChunk) {
                const uint64_t e = t * kTile + (k + 1) * kMfmaChunk;
                load_chunk(c[(k + 1) % 2], g + e, w + e);
            } else if (t + step < n_whole) {
                load_chunk(c[0], g + (t + step) * kTile, w + (t + step) * kTile);
            }
            __builtin_amdgcn_sched_barrier(0);
            add_chunk(c[k % 2], sums);
        }
    }
    if (t == n_whole && t * kTile < set.numel) {
        // ragged tail: g = 0 and w = 0 past the end give an outer gradient of 0
        const uint32_t left = (uint32_t)(set.numel - t * kTile);
        for (uint32_t at = 0; at < left; at += kMfmaChunk) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < kLaneElems; ++j) {
                    const bool there = at + 32 * h + quarter * kLaneElems + j < left;
                    const uint64_t e = t * kTile + at + 32 * h + j;
                    c[0].g[h][j / 4][j % 4] = there ? f2u(g[e]) : 0u;
                    const uint32_t x = there ? (uint32_t)w[e] : 0u;
                    c[0].w[h][j / 2] = j % 2 ? c[0].w[h][j / 2] | (x << 16) : x;
                }
            add_chunk(c[0], sums);
        }
    }
    const f64x4 total = sums.total + (sums.part + sums.last);
    // register i of lane l: row 4 i + l / 16, column l % 16
#pragma unroll
    for (int i = 0; i < 4; ++i) mats[wave][(4 * i + quarter) * 16 + replica] = total[i];
    __syncthreads();
    static_assert(kMfmaWaves * kWave == 16 * 16, "one thread per entry");
    const uint32_t row = threadIdx.x / 16, col = threadIdx.x % 16;
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < kMfmaWaves; ++k) v += mats[k][threadIdx.x];
    if (row <= col && col < M) a.partial[(uint64_t)blockIdx.x * M * M + row * M + col] = v;
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

constexpr uint32_t groups_per_launch(uint32_t M) { return M > (uint32_t)kPairM ? kWideGroups : kGroups; }

// A launch over n sets has at most groups_per_launch + n workgroups, so at most (groups_per_launch + n) / fin_chunk + n
// first-level outputs: kFirstLevel and one for each set, of which the workspace and the arguments have room.
constexpr uint32_t kFirstLevel = kMaxGroups / 64 + 2;
constexpr int kMaxFin = kFirstLevel + 2 * kMaxSets;                       // outputs per finalize launch
constexpr bool sums_fit()
{
    for (uint32_t M = 1; M <= SDL_MAX_WORKERS; ++M)
        if (groups_per_launch(M) > kMaxGroups || (groups_per_launch(M) + kMaxSets) / fin_chunk(M) > kFirstLevel) return false;
    return true;
}
static_assert(sums_fit(), "workgroups per launch, matrices per first-level output and the workspace go together");

struct FinArgs {
    const double* in;              // matrices of M*M doubles (only a <= b is read), stride_k doubles apart
    double* out;                   // output o at out + o * out_stride
    double* last_out;              // if not null, where the last output goes instead
    uint64_t stride_k;
    uint64_t out_stride;
    uint32_t M;
    uint32_t emit;                 // 1: G, cos, mean (2*M*M + 1 doubles); 0: G only (M*M doubles)
    uint32_t first[kMaxFin];       // output o adds the matrices first[o] .. first[o] + count[o] - 1
    uint32_t count[kMaxFin];
};

// One workgroup per output.  A thread adds every S-th matrix's value of one entry a <= b (neighbouring threads read
// neighbouring entries), then the S sums of an entry are added as a tree.  Latency bound: a range should give a thread a
// handful of matrices, so long ranges go through a first level of fin_chunk matrices per output.  (One wavefront per entry
// and a butterfly of lane exchanges took 5 us at 4 replicas and 25 us at 16, entry after entry.)
__global__ void __launch_bounds__(kFinThreads) sdl_gram_finalize(const FinArgs f)
{
    __shared__ double G[SDL_MAX_WORKERS * SDL_MAX_WORKERS];
    __shared__ double C[SDL_MAX_WORKERS * SDL_MAX_WORKERS];
    __shared__ double part[kFinThreads];
    const uint32_t M = f.M, count = f.count[blockIdx.x], entries = M * (M + 1u) / 2u, S = fin_slices(M);
    const double* base = f.in + (uint64_t)f.first[blockIdx.x] * f.stride_k;
    const uint32_t entry = threadIdx.x % entries, slice = threadIdx.x / entries;
    uint32_t a = 0, b = entry;             // entry number -> (a, b), row by row of the upper triangle
    while (b >= M - a) { b -= M - a; ++a; }
    b += a;
    if (slice < S) {
        double s = 0.0;
#pragma unroll 8
        for (uint32_t k = slice; k < count; k += S) s += base[(uint64_t)k * f.stride_k + a * M + b];
        part[threadIdx.x] = s;
    }
    __syncthreads();
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
    __syncthreads();
    double* o = f.last_out && blockIdx.x + 1u == gridDim.x ? f.last_out : f.out + (uint64_t)blockIdx.x * f.out_stride;
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
    if (threadIdx.x == 0) {
        double s = 0.0;
        uint32_t n = 0;
        for (uint32_t a = 0; a < M; ++a)
            for (uint32_t b = a + 1; b < M; ++b, ++n) s += C[a * M + b];
        o[2 * M * M] = n ? s / (double)n : 0.0;
    }
}

// ------------------------------------------------------------------ host side

int launch_kernel(uint32_t M, const GramArgs& a, hipStream_t st)
{
    const dim3 grid(a.pieces[a.n_pieces - 1].first_wg + a.pieces[a.n_pieces - 1].G), one(kWave);
    switch (M) {
    case 1: hipLaunchKernelGGL((sdl_gram_kernel<1>), grid, one, 0, st, a); break;
    case 2: hipLaunchKernelGGL((sdl_gram_kernel<2>), grid, one, 0, st, a); break;
    case 3: hipLaunchKernelGGL((sdl_gram_kernel<3>), grid, one, 0, st, a); break;
    case 4: hipLaunchKernelGGL((sdl_gram_kernel<4>), grid, one, 0, st, a); break;
    case 5: hipLaunchKernelGGL((sdl_gram_kernel<5>), grid, one, 0, st, a); break;
    case 6: hipLaunchKernelGGL((sdl_gram_kernel<6>), grid, one, 0, st, a); break;
    case 7: hipLaunchKernelGGL((sdl_gram_kernel<7>), grid, one, 0, st, a); break;
    case 8: hipLaunchKernelGGL((sdl_gram_kernel<8>), grid, one, 0, st, a); break;
    case 9: case 10: hipLaunchKernelGGL((sdl_gram_pair_kernel<5>), grid, dim3(2 * kWave), 0, st, a); break;
    case 11: case 12: hipLaunchKernelGGL((sdl_gram_pair_kernel<6>), grid, dim3(2 * kWave), 0, st, a); break;
    default: hipLaunchKernelGGL(sdl_gram_mfma_kernel, grid, dim3(kMfmaWaves * kWave), 0, st, a); break;
    }
    return hipGetLastError() == hipSuccess ? SDL_OK : SDL_ERR_DEVICE;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Shares the launch's workgroups out among the sets in proportion to their tiles (at least
// one each); returns the total, at most groups + n_sets.
uint32_t share_groups(Set* sets, uint32_t n_sets, uint32_t groups)
{
    uint64_t total_tiles = 0;
    for (uint32_t s = 0; s < n_sets; ++s) total_tiles += (sets[s].numel + kTile - 1) / kTile;
    uint32_t next = 0;
    for (uint32_t s = 0; s < n_sets; ++s) {
        const uint64_t tiles = (sets[s].numel + kTile - 1) / kTile;
        uint64_t G = total_tiles ? (tiles * groups + total_tiles - 1) / total_tiles : 1;
        if (G > tiles) G = tiles;
        if (G < 1) G = 1;
        sets[s].first_wg = next;
        sets[s].G = (uint32_t)G;
        next += (uint32_t)G;
    }
    return next;
}

// Partial Gram matrices of up to kMaxSets sets (already given their workgroups) into
// `partial`, one M x M matrix per workgroup of the launch.
int launch_gram(const float* g, const void* const* w, uint32_t M, const Set* sets, uint32_t n_sets, double* partial,
                hipStream_t st)
{
    GramArgs a{};
    a.g = g;
    a.partial = partial;
    a.M = M;
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
            Piece& pc = a.pieces[a.n_pieces++];
            const uint64_t e0 = j * tiles_per * kTile;
            const uint64_t e1 = (j + 1) * tiles_per * kTile < sets[s].numel ? (j + 1) * tiles_per * kTile : sets[s].numel;
            pc.offset = sets[s].offset + (e0 < sets[s].numel ? e0 : sets[s].numel);
            pc.numel = e1 > e0 ? e1 - e0 : 0;
            const uint32_t w0 = (uint32_t)((uint64_t)sets[s].G * j / nsub), w1 = (uint32_t)((uint64_t)sets[s].G * (j + 1) / nsub);
            pc.first_wg = sets[s].first_wg + w0;
            pc.G = w1 - w0;
            bool fast = aligned16(g + pc.offset);
            for (uint32_t m = 0; m < M; ++m)
                fast = fast && aligned16(static_cast<const uint16_t*>(w[m]) + pc.offset);
            pc.fast = fast ? 1u : 0u;
        }
    }
    for (uint32_t m = 0; m < M; ++m) a.w[m] = static_cast<const uint16_t*>(w[m]);
    return launch_kernel(M, a, st);
}

int launch_finalize(const FinArgs& f, uint32_t n_out, hipStream_t st)
{
    // whole wavefronts for the entries and their slices: 64 threads at one replica, 192 at two (idle ones cost their barriers)
    const uint32_t threads = (f.M * (f.M + 1u) / 2u * fin_slices(f.M) + kWave - 1u) / kWave * kWave;
    hipLaunchKernelGGL(sdl_gram_finalize, dim3(n_out), dim3(threads), 0, st, f);
    return hipGetLastError() == hipSuccess ? SDL_OK : SDL_ERR_DEVICE;
}

// One result per set from the partial matrices of its workgroups (the sets' workgroups lie one behind the other) and, if
// union_out is not null, the result of all of them together.  Sets with many workgroups are first added up in chunks (into
// tmp), so that no thread of the finalize kernel walks a long range.
int finalize_sets(const double* partial, const Set* sets, uint32_t n_sets, uint32_t M, double* out, double* union_out,
                  double* tmp, hipStream_t st)
{
    const uint64_t mm = (uint64_t)M * M;
    const uint32_t chunk = fin_chunk(M);
    uint32_t total = 0;
    bool two_level = false;
    for (uint32_t s = 0; s < n_sets; ++s) {
        two_level = two_level || sets[s].G > 2 * chunk;
        total += sets[s].G;
    }
    two_level = two_level || (union_out && total > 2 * chunk);
    FinArgs last{};
    last.out = out;
    last.last_out = union_out;
    last.stride_k = mm;
    last.out_stride = SDL_COSINE_RESULT_DOUBLES(M);
    last.M = M;
    last.emit = 1;
    last.in = partial;
    for (uint32_t s = 0; s < n_sets; ++s) { last.first[s] = sets[s].first_wg; last.count[s] = sets[s].G; }
    if (two_level) {
        FinArgs lvl1{};
        lvl1.in = partial;
        lvl1.out = tmp;
        lvl1.stride_k = mm;
        lvl1.out_stride = mm;
        lvl1.M = M;
        uint32_t n = 0;
        for (uint32_t s = 0; s < n_sets; ++s) {
            last.first[s] = n;
            for (uint32_t c = 0; c < sets[s].G; c += chunk) {
                lvl1.first[n] = sets[s].first_wg + c;
                lvl1.count[n] = sets[s].G - c < chunk ? sets[s].G - c : chunk;
                ++n;
            }
            last.count[s] = n - last.first[s];
        }
        const int rc = launch_finalize(lvl1, n, st);
        if (rc != SDL_OK) return rc;
        last.in = tmp;
        total = n;
    }
    if (union_out) { last.first[n_sets] = last.first[0]; last.count[n_sets] = total; }
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
    f.count[0] = count;
    return launch_finalize(f, 1, st);
}

// Workspace layout, in M x M matrices: the partial matrices of every launch, then the
// first-level sums of the finalize step; then (plan-level call without span_results) one
// result per set.
size_t partial_mats(size_t n_sets)
{
    const size_t launches = (n_sets + kMaxSets - 1) / kMaxSets;
    return launches * kMaxGroups + n_sets;
}
size_t tmp_mats(size_t n_sets)
{
    const size_t launches = (n_sets + kMaxSets - 1) / kMaxSets;
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
    share_groups(&set, 1, groups_per_launch(M));
    double* partial = static_cast<double*>(workspace);
    double* tmp = partial + partial_mats(1) * M * M;
    rc = launch_gram(g, w, M, &set, 1, partial, st);
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
    const uint32_t groups = groups_per_launch(M);
    const uint64_t mm = (uint64_t)M * M, R = SDL_COSINE_RESULT_DOUBLES(M);
    double* partial = static_cast<double*>(workspace);
    double* tmp = partial + partial_mats(n_spans) * mm;
    double* per_span = span_results ? span_results : tmp + tmp_mats(n_spans) * mm;
    uint64_t used = 0, used_tmp = 0;   // matrices handed out so far
    for (uint32_t s0 = 0; s0 < n_spans; s0 += kMaxSets) {
        const uint32_t ns = n_spans - s0 < (uint32_t)kMaxSets ? n_spans - s0 : (uint32_t)kMaxSets;
        Set sets[kMaxSets];
        for (uint32_t s = 0; s < ns; ++s) sets[s] = Set{spans[s0 + s].offset, spans[s0 + s].numel, 0, 0};
        const uint32_t n_wg = share_groups(sets, ns, groups);
        double* part = partial + used * mm;
        rc = launch_gram(g_base, w_base, M, sets, ns, part, st);
        if (rc != SDL_OK) return rc;
        // the spans of one launch give the fragment's result as well
        rc = finalize_sets(part, sets, ns, M, per_span + (uint64_t)s0 * R, ns == n_spans ? fragment_result : nullptr,
                           tmp + used_tmp * mm, st);
        if (rc != SDL_OK) return rc;
        used += n_wg;
        used_tmp += n_wg / fin_chunk(M) + ns;
    }
    if (n_spans && n_spans <= (uint32_t)kMaxSets) return SDL_OK;
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
