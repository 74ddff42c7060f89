// Device side of the library: the streaming kernels of the fragment outer step for
// gfx950 (MI355X), and the C entry points that launch them.
//
// One templated kernel serves every call: send side (quantize), receive side (decode + mean +
// Nesterov, with or without the merge), merge alone, and the fused outer step; the
// absolute-maximum pre-pass of the whole-span scale is a kernel of its own.
//
// Work decomposition (all modes).  A workgroup is one 64-lane wavefront and owns a
// tile of one or two rows of 256 consecutive parameters (the height is chosen per call and
// replica count, see tile_rows).  Lane l owns the four parameters [4l, 4l+4) of each row, so
//   - every memory instruction of the wavefront touches one contiguous piece of an
//     array (1 KiB of fp32 through 128-bit accesses, 512 B of bf16 through 64-bit
//     accesses): whole cache lines, nothing strided;
//   - eight neighbouring lanes own one 32-element scale block, and the block maximum
//     is three DPP exchanges (two inside the quad, one across the half row); wider
//     blocks add a row mirror and ds_bpermute exchanges.  No LDS storage is used.
// Tiles of runs that start on a multiple of four elements in 16-byte aligned arrays (long runs: of eight) use buffer
// instructions with non-temporal cache policy (every byte is touched once), ragged tails of a multiple
// of four elements among them; full tiles of other runs use vector accesses of element alignment in the same lane layout; other ragged tails use
// range-checked accesses of one element each.  A launch covers up to 272 contiguous runs of the flat
// model (160 of a whole-span format); every workgroup belongs to exactly one run, so scale blocks never straddle
// runs.
//
// Arithmetic contract (Algorithm 2 and Sections 2.1, 2.3, 2.4 of the paper, with the
// exchange formats documented in sdl.h): every fp32 operation is a single IEEE
// operation in the documented order; this file must be compiled with
// -ffp-contract=off and with fp32 denormals enabled (the hipcc default).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <mutex>

#include "sdl.h"
#include "sdl_device.h"

// Scale words of the allocation-free fused step (sdl_fragment_outer_step_plan_static): for the
// whole-span scale, one 4-byte word per span and replica, replica m's words at
// scratch + m * SDL_STATIC_MAX_SPANS.  Every GPU the library runs on holds its own copy of the
// array at its own address until the process ends.  In host code the name is only a handle for
// hipGetSymbolAddress: kernels and fills always get the per-device address kept below.
static __device__ __align__(256) uint32_t scratch[SDL_STATIC_MAX_SPANS * SDL_MAX_WORKERS];

namespace {

using namespace sdl_device;

constexpr int kVec = 4;                       // consecutive parameters a lane owns in one row
constexpr int kMaxRows = 2;                   // rows of the tallest tile
constexpr int kRow = kVec * kWave;            // parameters per row (256); a workgroup is one wavefront
constexpr int kPad = kRow * kMaxRows;          // message and staging layouts pad every piece to this many
                                              // parameters (512): a whole number of tiles of either height
constexpr int kRunGroup = 16;                 // runs whose first workgroups a workgroup compares at once
constexpr int kTableWords = 3 * 17 * kRunGroup;   // what a launch says about its runs (3.9 KB of kernel arguments in all)
constexpr int kCheckedRuns = 16;              // pieces over which a fragment's workgroups are added up for the check of its size
constexpr uint64_t kMaxRunElems = 1ull << 30;  // longest run of a launch (its numbers are 32-bit); longer ones are cut here

enum Mode { kQuantize = 0, kReduce = 1, kMerge = 2, kFused = 3, kReceive = 5 };   // kReceive = kReduce + kMerge

// Rows of a workgroup's tile, by call and compile-time replica count (0 = any M at run time).
// Rows are independent of each other (a scale block never leaves its row), so the height is a
// pure scheduling choice.  Measured on MI355X over 302 M parameters: one row instead of two gains
// 3-5 % on the fused kernel and the one-pass receive at M = 1, 2 and 4, 2-9 % on the receive side
// without the merge and 7 % on the merge at M = 1, and loses 2 % on the first two at M = 8, 1-3 % on
// the merge at M >= 2 and 3-12 % on the send side.  The whole-span scale keeps two rows: every tile reads its span's scale words, all
// tiles of a span the same few bytes, and twice the tiles cost it 8-14 %.
constexpr int tile_rows(int mode, int mt, int fmt)
{
    if (fmt == SDL_FMT_E3M0_SPAN) return 2;
    if (mode == kReduce) return mt > 0 ? 1 : 2;
    if (mode == kFused || mode == kReceive) return (mt == 1 || mt == 2 || mt == 4) ? 1 : 2;
    if (mode == kMerge) return mt == 1 ? 1 : 2;
    return 2;
}
// The compile-time replica count a call runs with: the kernels are built for 1, 2, 4 and 8 replicas
// plus one variant that takes any M; the message-writing fused kernel is a verification aid, for
// which the any-M variant is enough.
constexpr uint32_t variant_mt(int mode, uint32_t M, bool emit)
{
    const uint32_t mt = (mode == kFused && emit) ? 0u : M;
    return (mt == 1 || mt == 2 || mt == 4 || mt == 8) ? mt : 0u;
}

constexpr bool is_e3m0(int f) { return f == SDL_FMT_E3M0 || f >= SDL_FMT_E3M0_B64; }
constexpr bool is_scaled(int f) { return f == SDL_FMT_E4M3 || is_e3m0(f); }
constexpr bool is_span_scaled(int f) { return f == SDL_FMT_E3M0_SPAN; }
// elements that share a scale (0: the whole span)
constexpr int block_elems(int f)
{
    return f == SDL_FMT_E3M0_B64 ? 64 : f == SDL_FMT_E3M0_B128 ? 128 : f == SDL_FMT_E3M0_SPAN ? 0 : SDL_BLOCK;
}

// How the whole tiles of a run reach memory (a ragged last tile: the buffer path too if the run takes it and
// its length is a multiple of 4, else one access per element).
enum TilePath : uint32_t {
    kPathBuffer = 1,    // the call's arrays are 16-byte aligned and the run starts on a multiple of 4 elements, and if it is long
                        // on one of 8 (see Align)
    kPathVector = 2,    // any other run (messages of 4 and 8 bits may start at any byte)
};

// What a launch says about its runs, in 32-bit numbers relative to the launch's bases, three words a run so that as many as
// possible fit the kernel arguments: 272 runs (a fragment of 193 groups of 100 to 30000 parameters, M = 2: 20.8 us as two launches
// of 112 runs and 81, 17.5 as one).  Every run takes the workgroups of whole 512-element pieces, so the workgroup's number
// alone says where its tile lies in the messages and in staged g / mom, which hold the runs back to back in such pieces;
// where a tile has 256 parameters the last workgroup of a run may have nothing to do.  A whole-span format adds two words:
// the index of the run's scale word, and, since its runs are parts of what is staged, where it starts there.
constexpr int kRunWords = 3, kSpanRunWords = 5;
constexpr int run_words(int fmt) { return is_span_scaled(fmt) ? kSpanRunWords : kRunWords; }
constexpr int max_runs(int fmt) { return kTableWords / run_words(fmt) / kRunGroup * kRunGroup; }
// words of the table: the first workgroup of each run, ascending, 0xffffffff behind the last; then the runs
template <int FMT> constexpr uint32_t run_word(uint32_t r) { return (uint32_t)max_runs(FMT) + r * (uint32_t)(run_words(FMT) - 1); }
constexpr uint32_t kVectorBit = 1u << 31;      // in a run's number of elements: its whole tiles take kPathVector

struct Args {
    float* g;
    float* mom;
    const uint16_t* w_send[SDL_MAX_WORKERS];
    uint16_t* w_now[SDL_MAX_WORKERS];
    uint8_t* codes[SDL_MAX_WORKERS];
    uint8_t* scales[SDL_MAX_WORKERS];
    uint64_t offset0;    // what the runs' offsets count from, in the replicas and in g / mom
    uint64_t msg0;       // where the first run starts in the message arrays
    uint64_t soff0;      // and in staged g / mom
    uint32_t n_runs;
    uint32_t M;
    float lr, mu, alpha, one_minus_alpha;
    uint32_t aliased;    // w_send[m] == w_now[m]
    uint32_t emit;       // fused kernel: also write the messages
    uint32_t staged;     // g / mom point at a staging buffer that holds only this fragment
    uint32_t chunked;    // of the workgroups below this one each XCD takes kChunkRows consecutive rows (see chunked_tile)
    uint32_t group_wg[kTableWords / kRunWords / kRunGroup - 1];   // first workgroup of the 16th, 32nd, ... run
    uint32_t table[kTableWords];
};
static_assert(sizeof(Args) <= 4096, "kernel arguments");

// Cache policy bits of the buffer instructions on gfx950: 1 = sc0, 2 = nt, 16 = sc1.
constexpr int kAuxLoad = 2;      // loads: non-temporal (every byte is touched once)
constexpr int kAuxStore = 2;     // stores: non-temporal
constexpr int kAuxScale = 0;     // scale bytes: 16 per tile, 8 tiles per cache line -> let L2 combine them
constexpr int kWavesPerEu = 2;   // register budget: at least this many wavefronts per SIMD

// ------------------------------------------------------------------ bit helpers

// bf16 pair packed in one dword: element 0 in the low half.
__device__ __forceinline__ float bf16_lo(uint32_t u) { return u2f(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return u2f(u & 0xffff0000u); }

// Two fp32 -> packed bf16, round to nearest even, NaN stays a quiet NaN (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t bf16_pack(float lo, float hi)
{
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ void unpack_bf16(const uint32_t (&u)[2], float (&v)[kVec])
{
    v[0] = bf16_lo(u[0]); v[1] = bf16_hi(u[0]); v[2] = bf16_lo(u[1]); v[3] = bf16_hi(u[1]);
}

// Maximum over the LANES consecutive lanes that share a scale block (8, 16, 32 or all 64).
template <int LANES>
__device__ __forceinline__ uint32_t lanes_max(uint32_t v)
{
    uint32_t t = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);    // quad_perm 1,0,3,2
    v = v > t ? v : t;
    t = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);             // quad_perm 2,3,0,1
    v = v > t ? v : t;
    t = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);            // row_half_mirror: 7-i
    v = v > t ? v : t;
    if constexpr (LANES >= 16) {
        t = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true);        // row_mirror: 15-i
        v = v > t ? v : t;
    }
    if constexpr (LANES >= 32) {
        t = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(((threadIdx.x ^ 16u) & 63u) << 2), (int)v);   // lane ^ 16
        v = v > t ? v : t;
    }
    if constexpr (LANES >= 64) {
        t = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(((threadIdx.x ^ 32u) & 63u) << 2), (int)v);   // lane ^ 32
        v = v > t ? v : t;
    }
    return v;
}

// ------------------------------------------------------------------ exchange formats
// A message element is produced in two forms: its decoded fp32 value dq (what the
// receiver accumulates) and, when asked for, its code.

struct BlockScale {
    uint32_t sb;      // scale byte
    float inv;        // 2^(127-sb), or 0 for a degenerate block
    float scale;      // 2^(sb-127), NaN for a block that holds Inf/NaN
    bool degenerate;  // block maximum is zero, subnormal, Inf or NaN
};

template <int FMT>
__device__ __forceinline__ BlockScale block_scale_from_exponent(uint32_t e_a)
{
    // written with single comparisons and selects: this runs once per scale block and replica,
    // and as control flow it cost more than the codec of the block's elements
    // exponent of the code grid that the block maximum's binade is mapped to
    constexpr uint32_t emax = FMT == SDL_FMT_E4M3 ? 8u : FMT == SDL_FMT_E3M0_RN ? 3u : 4u;
    BlockScale b;
    const uint32_t sb = e_a > emax ? e_a - emax : 0u;
    const bool nan_block = e_a == 255u;
    b.degenerate = (e_a - 1u) >= 254u;                          // 0 (zero / subnormal maximum) or 255 (Inf / NaN)
    b.inv = b.degenerate ? 0.0f : u2f((254u - sb) << 23);
    const uint32_t scale_bits = (sb << 23) > 0x00400000u ? (sb << 23) : 0x00400000u;   // 2^-127 is an fp32 subnormal
    b.scale = u2f(nan_block ? 0x7fc00000u : scale_bits);
    b.sb = nan_block ? 255u : sb;
    return b;
}

__device__ __forceinline__ float scale_from_byte(uint32_t sb)
{
    float s = sb ? u2f(sb << 23) : u2f(0x00400000u);
    return sb == 255u ? u2f(0x7fc00000u) : s;
}

// Encode the lane's 4 outer gradients d of one row and one replica.  dq = decoded
// values.  Codes: E3M0 -> c[0] holds 4 nibbles (16 bits); E4M3 -> c[0] holds 4 bytes;
// BF16 -> c[0..1]; FP32 -> the bits of d.  sb = scale byte of the lane's block.
// span_amax: for the whole-span scale, the bit pattern of the span's absolute maximum.
template <int FMT>
__device__ __forceinline__ void encode(const float (&d)[kVec], float (&dq)[kVec], uint32_t (&c)[kVec],
                                       uint32_t& sb, bool want_codes, uint32_t span_amax)
{
    if constexpr (FMT == SDL_FMT_FP32) {
#pragma unroll
        for (int j = 0; j < kVec; ++j) { dq[j] = d[j]; c[j] = f2u(d[j]); }
        sb = 0;
    } else if constexpr (FMT == SDL_FMT_BF16) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            c[k] = bf16_pack(d[2 * k], d[2 * k + 1]);
            dq[2 * k] = bf16_lo(c[k]);
            dq[2 * k + 1] = bf16_hi(c[k]);
        }
        sb = 0;
    } else {
        uint32_t amax = 0;
#pragma unroll
        for (int j = 0; j < kVec; ++j) {
            const uint32_t m = f2u(d[j]) & 0x7fffffffu;
            amax = m > amax ? m : amax;
        }
        if constexpr (is_span_scaled(FMT)) amax = span_amax;
        else amax = lanes_max<block_elems(FMT) / kVec>(amax);
        const BlockScale b = block_scale_from_exponent<FMT>(amax >> 23);
        sb = b.sb;
        uint32_t packed = 0;
        if constexpr (FMT == SDL_FMT_E4M3) {
            // OCP FP8 E4M3 through the conversion instructions of gfx950 (round to nearest even,
            // subnormals, signed zero); they do not saturate, so clamp to +-448 first
            float y[kVec];
#pragma unroll
            for (int j = 0; j < kVec; ++j) y[j] = __builtin_amdgcn_fmed3f(d[j] * b.inv, 448.0f, -448.0f);
            packed = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false);
            packed = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], (int)packed, true);
            if (b.sb == 255u) {
                // a block that holds Inf / NaN keeps only the signs (0 * Inf made NaN codes above)
                packed = 0;
#pragma unroll
                for (int j = 0; j < kVec; ++j) packed |= ((f2u(d[j]) >> 24) & 0x80u) << (8 * j);
            }
            const f32x2_t lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)packed, false);
            const f32x2_t hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)packed, true);
            dq[0] = lo.x * b.scale; dq[1] = lo.y * b.scale; dq[2] = hi.x * b.scale; dq[3] = hi.y * b.scale;
        } else {
#pragma unroll
            for (int j = 0; j < kVec; ++j) {
                const float y = __builtin_fabsf(d[j]) * b.inv;     // exact power-of-two scaling
                const uint32_t yb = f2u(y);
                const uint32_t sign = f2u(d[j]) & 0x80000000u;
                // nearest power of two in the linear domain; a tie (mantissa exactly
                // 1.5) goes to the even exponent code, whose parity is that of the
                // biased fp32 exponent because the re-bias (124) is even
                const uint32_t rr = yb + 0x3fffffu + ((yb >> 23) & 1u);
                const float pw = __builtin_amdgcn_fmed3f(u2f(rr & 0x7f800000u), 0.25f, 16.0f);
                const float val = y > 0.125f ? pw : 0.0f;          // half of the smallest magnitude
                dq[j] = u2f(sign | f2u(val * b.scale));
                if (want_codes) {
                    // the code comes straight from a rounded bit pattern, not from val, so that a
                    // kernel that only writes messages does not carry the decode arithmetic: clamp
                    // to [1/4, 16] first (exact: everything below rounds up to 1/4 or is the zero
                    // code, everything above saturates), round as above with 4 added to the
                    // exponent field, and the three low bits of the field are the code
                    // (fields 125..131 -> 129..135 -> 1..7)
                    const uint32_t cb = f2u(__builtin_amdgcn_fmed3f(y, 0.25f, 16.0f));
                    const uint32_t rc = cb + 0x023fffffu + ((cb >> 23) & 1u);
                    const uint32_t E = y > 0.125f ? (rc >> 23) & 7u : 0u;
                    packed |= ((sign >> 28) | E) << (4 * j);
                }
            }
        }
        c[0] = packed;
    }
}

// Decode 4 E3M0 nibbles / 4 E4M3 bytes under the block scale.
__device__ __forceinline__ void decode_e3m0(uint32_t c0, float scale, float (&dq)[kVec])
{
#pragma unroll
    for (int j = 0; j < kVec; ++j) {
        const uint32_t nib = (c0 >> (4 * j)) & 15u;
        const uint32_t E = nib & 7u;
        const float val = E ? u2f((E + 124u) << 23) : 0.0f;
        dq[j] = u2f(((nib & 8u) << 28) | f2u(val * scale));
    }
}
// EXACT = false: the conversion instruction alone, which reads the byte values 0x7f / 0xff as
// NaN; the caller then repeats the decode with EXACT = true wherever a NaN shows up in the sum.
template <bool EXACT>
__device__ __forceinline__ void decode_e4m3(uint32_t c0, float scale, float (&dq)[kVec])
{
    // codes 0x7f / 0xff never come out of the encoder; read as a number (480) like every other
    // code rather than as the NaN the conversion instruction makes of them
    if (EXACT && (((c0 & 0x7f7f7f7fu) + 0x01010101u) & 0x80808080u)) {
#pragma unroll
        for (int j = 0; j < kVec; ++j) {
            const uint32_t byte = (c0 >> (8 * j)) & 255u;
            const uint32_t mag = byte & 0x7fu;
            const float val = mag >= 8u ? u2f((mag + 960u) << 20) : (float)mag * 0.001953125f;
            dq[j] = u2f(((byte & 0x80u) << 24) | f2u(val * scale));
        }
    } else {
        const f32x2_t lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)c0, false);
        const f32x2_t hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)c0, true);
        dq[0] = lo.x * scale; dq[1] = lo.y * scale; dq[2] = hi.x * scale; dq[3] = hi.y * scale;
    }
}

// A span's scale word, by a vector load that is under way with the tile's (a scalar one is waited for before the next instruction
// that needs any).
__device__ __forceinline__ uint32_t load_word(const uint8_t* words, uint32_t index)
{
    asm("" : "+v"(index));
    return reinterpret_cast<const uint32_t*>(words)[index];
}

// ------------------------------------------------------------------ tile I/O policies
// The arithmetic is written once against an I/O policy that moves a lane's 4 elements
// of row `row` of each array.
//   TileIOT<true>   a tile whose lanes start on the alignment of their accesses: buffer loads / stores through one
//              resource per array (scalar base, 32-bit lane offset) with explicit cache policy; PART: the ragged
//              last tile of a run whose length is a multiple of 4
//   TileIOT<false>  a whole tile of arrays that start at any element (a run behind a parameter
//              group of odd length, messages packed back to back): the same lane layout through
//              plain vector loads / stores of element alignment (byte alignment for the 4- and
//              8-bit codes)
//   TailIO     the other ragged last tiles, any alignment: one buffer access per element (per
//              byte of 4- and 8-bit codes) under the range check of the buffer instructions,
//              which returns 0 past the end and drops stores there -- no branches, so that all
//              of a tile's loads are in flight at once

template <bool ALIGNED, int ROWS, bool PART = false>
struct TileIOT {
    static constexpr int kTile = ROWS * kRow;   // parameters of the tile
    const Args& a;
    uint64_t t0;      // tile's first element in the flat arrays (workgroup uniform)
    uint64_t tb;      // tile's first element in the message arrays (a multiple of 512)
    uint32_t lane;
    uint32_t sidx;    // whole-span scale: index of the run's scale word
    uint64_t s0;      // tile's first element in g / mom (= t0 unless the state is staged)
    uint32_t left;    // PART: elements of the tile that exist (a multiple of 4, so that a lane has all four or none)

    // (a number in a whole tile: as a variable it moved the message loads of the one-pass receive at M = 8 behind each other, 2521 us
    // against 2772 for 302 M parameters)
    __device__ __forceinline__ uint32_t limit() const { return PART ? left : (uint32_t)kTile; }

    template <int B> __device__ __forceinline__ uint32_t scale_bytes() const { return (limit() + B - 1) / B; }
    // bit pattern of the span's absolute maximum (whole-span scale)
    __device__ __forceinline__ uint32_t span_amax(uint32_t m) const
    {
        return load_word(a.scales[m], sidx);
    }
    // the same by a scalar load
    __device__ __forceinline__ uint32_t span_amax_scalar(uint32_t m) const
    {
        return reinterpret_cast<const uint32_t*>(a.scales[m])[sidx];
    }
    template <int FMT> __device__ __forceinline__ float load_scale(uint32_t m, int row) const
    {
        if constexpr (is_span_scaled(FMT)) {
            // us, vector and scalar loads, 28 M parameters: one-pass receive M = 4 168 and 162, M = 8 256 and 244; without the merge M = 8
            // 94.8 and 93.4, M = 16 116.8 and 115.3, other counts the same; groups at odd elements, receive M = 8 380 and 385, without
            // the merge 125 and 127
            constexpr bool kScalar = ALIGNED && !PART;
            return block_scale_from_exponent<FMT>((kScalar ? span_amax_scalar(m) : span_amax(m)) >> 23).scale;
        } else {
            constexpr int B = block_elems(FMT);
            const uint32_t sb = __builtin_amdgcn_raw_buffer_load_b8(
                rsrc(a.scales[m] + tb / B, scale_bytes<B>()), (int)(row * (kRow / B) + lane / (B / kVec)), 0, kAuxScale);
            return scale_from_byte(sb);
        }
    }
    template <int FMT> __device__ __forceinline__ void store_scale(uint32_t m, int row, uint32_t sb) const
    {
        if constexpr (!is_span_scaled(FMT)) {
            constexpr int B = block_elems(FMT);
            if ((lane % (B / kVec)) == 0u)
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)sb, rsrc(a.scales[m] + tb / B, scale_bytes<B>()),
                                                     (int)(row * (kRow / B) + lane / (B / kVec)), 0, kAuxScale);
        }
    }
    // p = address of the tile's first element in the array
    __device__ __forceinline__ void ld_f32(const float* p, int row, float (&v)[kVec]) const
    {
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rsrc(p, limit() * 4),
                                                              (int)(row * kRow * 4 + lane * 16), 0, kAuxLoad);
        v[0] = u2f(x.x); v[1] = u2f(x.y); v[2] = u2f(x.z); v[3] = u2f(x.w);
    }
    __device__ __forceinline__ void st_f32(float* p, int row, const float (&v)[kVec]) const
    {
        const u32x4 x = {f2u(v[0]), f2u(v[1]), f2u(v[2]), f2u(v[3])};
        __builtin_amdgcn_raw_buffer_store_b128(x, rsrc(p, limit() * 4), (int)(row * kRow * 4 + lane * 16), 0,
                                               kAuxStore);
    }
    __device__ __forceinline__ void ld_bf16(const uint16_t* p, int row, uint32_t (&u)[2]) const
    {
        const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(rsrc(p, limit() * 2),
                                                             (int)(row * kRow * 2 + lane * 8), 0, kAuxLoad);
        u[0] = x.x; u[1] = x.y;
    }
    __device__ __forceinline__ void st_bf16(uint16_t* p, int row, const uint32_t (&u)[2]) const
    {
        const u32x2 x = {u[0], u[1]};
        __builtin_amdgcn_raw_buffer_store_b64(x, rsrc(p, limit() * 2), (int)(row * kRow * 2 + lane * 8), 0,
                                              kAuxStore);
    }

    // the model arrays: the buffer path above when the tile is 16-byte aligned in all of them,
    // element-aligned vectors (non-temporal as well) otherwise
    __device__ __forceinline__ void model_ld_f32(const float* p, int row, float (&v)[kVec]) const
    {
        if constexpr (ALIGNED) {
            ld_f32(p, row, v);
        } else {
            const f32x4_elem x =
                __builtin_nontemporal_load(reinterpret_cast<const f32x4_elem*>(p + row * kRow + lane * kVec));
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        }
    }
    __device__ __forceinline__ void model_st_f32(float* p, int row, const float (&v)[kVec]) const
    {
        if constexpr (ALIGNED) {
            st_f32(p, row, v);
        } else {
            const f32x4_elem x = {v[0], v[1], v[2], v[3]};
            __builtin_nontemporal_store(x, reinterpret_cast<f32x4_elem*>(p + row * kRow + lane * kVec));
        }
    }
    __device__ __forceinline__ void model_ld_bf16(const uint16_t* p, int row, uint32_t (&u)[2]) const
    {
        if constexpr (ALIGNED) {
            ld_bf16(p, row, u);
        } else {
            const u32x2_elem x =
                __builtin_nontemporal_load(reinterpret_cast<const u32x2_elem*>(p + row * kRow + lane * kVec));
            u[0] = x.x; u[1] = x.y;
        }
    }
    __device__ __forceinline__ void model_st_bf16(uint16_t* p, int row, const uint32_t (&u)[2]) const
    {
        if constexpr (ALIGNED) {
            st_bf16(p, row, u);
        } else {
            const u32x2_elem x = {u[0], u[1]};
            __builtin_nontemporal_store(x, reinterpret_cast<u32x2_elem*>(p + row * kRow + lane * kVec));
        }
    }
    __device__ __forceinline__ void load_g(int row, float (&v)[kVec]) const { model_ld_f32(a.g + s0, row, v); }
    __device__ __forceinline__ void load_mom(int row, float (&v)[kVec]) const { model_ld_f32(a.mom + s0, row, v); }
    __device__ __forceinline__ void store_g(int row, const float (&v)[kVec]) const { model_st_f32(a.g + s0, row, v); }
    __device__ __forceinline__ void store_mom(int row, const float (&v)[kVec]) const { model_st_f32(a.mom + s0, row, v); }
    __device__ __forceinline__ void load_ws(uint32_t m, int row, uint32_t (&u)[2]) const { model_ld_bf16(a.w_send[m] + t0, row, u); }
    __device__ __forceinline__ void load_wn(uint32_t m, int row, uint32_t (&u)[2]) const { model_ld_bf16(a.w_now[m] + t0, row, u); }
    __device__ __forceinline__ void store_wn(uint32_t m, int row, const uint32_t (&u)[2]) const { model_st_bf16(a.w_now[m] + t0, row, u); }

    // Where the lane's four codes of a row lie in a message array of NUM / DEN bytes per element.  Accesses at this address
    // (not ALIGNED) use the normal cache policy: lanes and tiles share lines, which L2 puts together.
    template <int NUM, int DEN> __device__ __forceinline__ uint64_t msg_byte(int row) const
    {
        return tb * NUM / DEN + (uint32_t)((row * kRow + (int)(lane * kVec)) * NUM / DEN);
    }

    // E4M3 only: with EXACT = false the two byte values the encoder never writes decode to NaN
    static constexpr bool kHasInexactDecode = true;
    template <int FMT, bool EXACT = true>
    __device__ __forceinline__ void load_message(uint32_t m, int row, float (&dq)[kVec]) const
    {
        const uint8_t* codes = a.codes[m];
        if constexpr (FMT == SDL_FMT_FP32) {
            if constexpr (ALIGNED) {
                ld_f32(reinterpret_cast<const float*>(codes) + tb, row, dq);
            } else {
                const f32x4_elem x = *(reinterpret_cast<const f32x4_elem*>(codes + msg_byte<4, 1>(row)));
                dq[0] = x.x; dq[1] = x.y; dq[2] = x.z; dq[3] = x.w;
            }
        } else if constexpr (FMT == SDL_FMT_BF16) {
            uint32_t u[2];
            if constexpr (ALIGNED) {
                ld_bf16(reinterpret_cast<const uint16_t*>(codes) + tb, row, u);
            } else {
                const u32x2_elem x = *(reinterpret_cast<const u32x2_elem*>(codes + msg_byte<2, 1>(row)));
                u[0] = x.x; u[1] = x.y;
            }
            unpack_bf16(u, dq);
        } else if constexpr (!ALIGNED) {
            const float scale = load_scale<FMT>(m, row);
            if constexpr (is_e3m0(FMT)) decode_e3m0(*reinterpret_cast<const u16_byte*>(codes + msg_byte<1, 2>(row)), scale, dq);
            else decode_e4m3<EXACT>(*reinterpret_cast<const u32_byte*>(codes + msg_byte<1, 1>(row)), scale, dq);
        } else {
            const float scale = load_scale<FMT>(m, row);
            if constexpr (is_e3m0(FMT)) {
                const uint32_t c0 = __builtin_amdgcn_raw_buffer_load_b16(rsrc(codes + tb / 2, limit() / 2),
                                                                         (int)(row * (kRow / 2) + lane * 2), 0,
                                                                         kAuxLoad);
                decode_e3m0(c0, scale, dq);
            } else {
                const uint32_t c0 = __builtin_amdgcn_raw_buffer_load_b32(rsrc(codes + tb, limit()),
                                                                         (int)(row * kRow + lane * 4), 0, kAuxLoad);
                decode_e4m3<EXACT>(c0, scale, dq);
            }
        }
    }
    template <int FMT>
    __device__ __forceinline__ void store_message(uint32_t m, int row, const uint32_t (&c)[kVec], uint32_t sb) const
    {
        uint8_t* codes = a.codes[m];
        if constexpr (!ALIGNED) {
            if constexpr (FMT == SDL_FMT_FP32) {
                *reinterpret_cast<u32x4_f32elem*>(codes + msg_byte<4, 1>(row)) = u32x4_f32elem{c[0], c[1], c[2], c[3]};
            } else if constexpr (FMT == SDL_FMT_BF16) {
                *reinterpret_cast<u32x2_elem*>(codes + msg_byte<2, 1>(row)) = u32x2_elem{c[0], c[1]};
            } else {
                store_scale<FMT>(m, row, sb);
                if constexpr (is_e3m0(FMT)) *reinterpret_cast<u16_byte*>(codes + msg_byte<1, 2>(row)) = (uint16_t)c[0];
                else *reinterpret_cast<u32_byte*>(codes + msg_byte<1, 1>(row)) = c[0];
            }
        } else if constexpr (FMT == SDL_FMT_FP32) {
            const u32x4 x = {c[0], c[1], c[2], c[3]};
            __builtin_amdgcn_raw_buffer_store_b128(x, rsrc(codes + tb * 4, limit() * 4),
                                                   (int)(row * kRow * 4 + lane * 16), 0, kAuxStore);
        } else if constexpr (FMT == SDL_FMT_BF16) {
            const u32x2 x = {c[0], c[1]};
            __builtin_amdgcn_raw_buffer_store_b64(x, rsrc(codes + tb * 2, limit() * 2),
                                                  (int)(row * kRow * 2 + lane * 8), 0, kAuxStore);
        } else {
            store_scale<FMT>(m, row, sb);
            if constexpr (is_e3m0(FMT)) {
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)c[0], rsrc(codes + tb / 2, limit() / 2),
                                                      (int)(row * (kRow / 2) + lane * 2), 0, kAuxStore);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(c[0], rsrc(codes + tb, limit()), (int)(row * kRow + lane * 4), 0,
                                                      kAuxStore);
            }
        }
    }
};

struct TailIO {
    const Args& a;
    uint64_t t0;           // tile's first element in the flat arrays
    uint64_t mb;           // tile's first element in the message arrays
    uint64_t s0;           // tile's first element in g / mom (= t0 unless the state is staged)
    uint32_t left;         // elements of the run from the tile's first on
    uint32_t lane;
    uint32_t sidx;         // whole-span scale: index of the run's scale word

    __device__ __forceinline__ uint32_t span_amax(uint32_t m) const
    {
        return load_word(a.scales[m], sidx);
    }
    // elements of a row that exist
    __device__ __forceinline__ uint32_t valid(int row) const
    {
        const uint32_t at = (uint32_t)(row * kRow);
        return left <= at ? 0u : left - at < (uint32_t)kRow ? left - at : (uint32_t)kRow;
    }
    // p = address of the tile's first element in the array
    __device__ __forceinline__ void ld_f32(const float* p, int row, float (&v)[kVec]) const
    {
        const __amdgpu_buffer_rsrc_t r = rsrc(p + row * kRow, valid(row) * 4);
#pragma unroll
        for (int j = 0; j < kVec; ++j) v[j] = u2f(__builtin_amdgcn_raw_buffer_load_b32(r, (int)(lane * 16 + 4 * j), 0, 0));
    }
    __device__ __forceinline__ void st_f32(float* p, int row, const float (&v)[kVec]) const
    {
        const __amdgpu_buffer_rsrc_t r = rsrc(p + row * kRow, valid(row) * 4);
#pragma unroll
        for (int j = 0; j < kVec; ++j) __builtin_amdgcn_raw_buffer_store_b32(f2u(v[j]), r, (int)(lane * 16 + 4 * j), 0, 0);
    }
    __device__ __forceinline__ void ld_bf16(const uint16_t* p, int row, uint32_t (&u)[2]) const
    {
        const __amdgpu_buffer_rsrc_t r = rsrc(p + row * kRow, valid(row) * 2);
        uint32_t h[kVec];
#pragma unroll
        for (int j = 0; j < kVec; ++j)
            h[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(lane * 8 + 2 * j), 0, 0) & 0xffffu;
        u[0] = h[0] | (h[1] << 16);
        u[1] = h[2] | (h[3] << 16);
    }
    __device__ __forceinline__ void st_bf16(uint16_t* p, int row, const uint32_t (&u)[2]) const
    {
        const __amdgpu_buffer_rsrc_t r = rsrc(p + row * kRow, valid(row) * 2);
#pragma unroll
        for (int j = 0; j < kVec; ++j)
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(u[j / 2] >> (16 * (j % 2))), r, (int)(lane * 8 + 2 * j), 0, 0);
    }
    // N codes of one byte each per lane (E4M3: 4; E3M0: 2, of two elements)
    template <int N> __device__ __forceinline__ __amdgpu_buffer_rsrc_t code_rsrc(uint8_t* codes, int row) const
    {
        return rsrc(codes + (mb + (uint32_t)(row * kRow)) * N / kVec, (valid(row) * N + kVec - 1) / kVec);
    }

    __device__ __forceinline__ void load_g(int row, float (&v)[kVec]) const { ld_f32(a.g + s0, row, v); }
    __device__ __forceinline__ void load_mom(int row, float (&v)[kVec]) const { ld_f32(a.mom + s0, row, v); }
    __device__ __forceinline__ void store_g(int row, const float (&v)[kVec]) const { st_f32(a.g + s0, row, v); }
    __device__ __forceinline__ void store_mom(int row, const float (&v)[kVec]) const { st_f32(a.mom + s0, row, v); }
    __device__ __forceinline__ void load_ws(uint32_t m, int row, uint32_t (&u)[2]) const { ld_bf16(a.w_send[m] + t0, row, u); }
    __device__ __forceinline__ void load_wn(uint32_t m, int row, uint32_t (&u)[2]) const { ld_bf16(a.w_now[m] + t0, row, u); }
    __device__ __forceinline__ void store_wn(uint32_t m, int row, const uint32_t (&u)[2]) const { st_bf16(a.w_now[m] + t0, row, u); }

    static constexpr bool kHasInexactDecode = false;
    template <int FMT, bool EXACT = true>
    __device__ __forceinline__ void load_message(uint32_t m, int row, float (&dq)[kVec]) const
    {
        uint8_t* codes = a.codes[m];
        if constexpr (FMT == SDL_FMT_FP32) {
            ld_f32(reinterpret_cast<const float*>(codes) + mb, row, dq);
        } else if constexpr (FMT == SDL_FMT_BF16) {
            uint32_t u[2];
            ld_bf16(reinterpret_cast<const uint16_t*>(codes) + mb, row, u);
            unpack_bf16(u, dq);
        } else {
            float scale;
            if constexpr (is_span_scaled(FMT)) {
                scale = block_scale_from_exponent<FMT>(span_amax(m) >> 23).scale;
            } else {
                constexpr int B = block_elems(FMT);
                const __amdgpu_buffer_rsrc_t r = rsrc(a.scales[m] + (mb + (uint32_t)(row * kRow)) / B, (valid(row) + B - 1) / B);
                scale = scale_from_byte(__builtin_amdgcn_raw_buffer_load_b8(r, (int)(lane / (B / kVec)), 0, kAuxScale));
            }
            constexpr int N = is_e3m0(FMT) ? 2 : 4;
            const __amdgpu_buffer_rsrc_t r = code_rsrc<N>(codes, row);
            uint32_t c0 = 0;
#pragma unroll
            for (int k = 0; k < N; ++k)
                c0 |= ((uint32_t)__builtin_amdgcn_raw_buffer_load_b8(r, (int)(lane * N + k), 0, 0) & 255u) << (8 * k);
            if constexpr (is_e3m0(FMT)) decode_e3m0(c0, scale, dq);
            else decode_e4m3<true>(c0, scale, dq);
        }
    }
    // elements beyond the end are zero outer gradients: they add nothing to a block maximum, and the unused nibble of a
    // last E3M0 byte is 0
    template <int FMT>
    __device__ __forceinline__ void store_message(uint32_t m, int row, const uint32_t (&c)[kVec], uint32_t sb) const
    {
        uint8_t* codes = a.codes[m];
        if constexpr (FMT == SDL_FMT_FP32) {
            float v[kVec];
#pragma unroll
            for (int j = 0; j < kVec; ++j) v[j] = u2f(c[j]);
            st_f32(reinterpret_cast<float*>(codes) + mb, row, v);
        } else if constexpr (FMT == SDL_FMT_BF16) {
            const uint32_t u[2] = {c[0], c[1]};
            st_bf16(reinterpret_cast<uint16_t*>(codes) + mb, row, u);
        } else {
            if constexpr (!is_span_scaled(FMT)) {
                constexpr int B = block_elems(FMT);
                if ((lane % (B / kVec)) == 0u)
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)sb, rsrc(a.scales[m] + (mb + (uint32_t)(row * kRow)) / B,
                                                                           (valid(row) + B - 1) / B),
                                                         (int)(lane / (B / kVec)), 0, kAuxScale);
            }
            constexpr int N = is_e3m0(FMT) ? 2 : 4;
            const __amdgpu_buffer_rsrc_t r = code_rsrc<N>(codes, row);
#pragma unroll
            for (int k = 0; k < N; ++k)
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(c[0] >> (8 * k)), r, (int)(lane * N + k), 0, 0);
        }
    }
};

// ------------------------------------------------------------------ the arithmetic of one lane
// MT > 0: number of replicas known at compile time; the replicas' words are loaded up
// front so that many loads are in flight.  MT == 0: any M at run time, taken in groups of four,
// two and one replicas whose loads are issued together (one replica at a time costs 6-8 %).

// One replica's contribution to the sum of one row: its message decoded (receive side), or its
// outer gradient encoded (send side and fused; ws = the replica's words at the send step, samax = its scale word unless
// it is asked for here).
template <int MODE, int FMT, bool EMIT, bool WORD_HERE = false, class IO>
__device__ __forceinline__ void add_replica(const IO& io, uint32_t m, int r, const uint32_t (&ws)[2],
                                            const float (&g)[kVec], float (&acc)[kVec], uint32_t samax)
{
    float dq[kVec];
    if constexpr (MODE == kReduce || MODE == kReceive) {
        io.template load_message<FMT, !(FMT == SDL_FMT_E4M3 && IO::kHasInexactDecode)>(m, r, dq);
    } else {
        float w[kVec], d[kVec];
        uint32_t c[kVec], sb;
        unpack_bf16(ws, w);
#pragma unroll
        for (int j = 0; j < kVec; ++j) d[j] = g[j] - w[j];
        constexpr bool want = MODE == kQuantize || EMIT;
        if constexpr (WORD_HERE) samax = io.span_amax_scalar(m);
        encode<FMT>(d, dq, c, sb, want, samax);
        if constexpr (want) io.template store_message<FMT>(m, r, c, sb);
    }
#pragma unroll
    for (int j = 0; j < kVec; ++j) acc[j] = acc[j] + dq[j];
}

// G replicas starting at m0, in ascending order, their loads issued before the first is consumed.
template <int MODE, int FMT, bool EMIT, int kRows, int G, class IO>
__device__ __forceinline__ void add_replica_group(const IO& io, uint32_t m0, const float (&g)[kRows][kVec],
                                                  float (&acc)[kRows][kVec])
{
    uint32_t ws[G][kRows][2] = {}, samax[G] = {};
    if constexpr (MODE == kQuantize || MODE == kFused) {
        if constexpr (is_span_scaled(FMT)) {
#pragma unroll
            for (int k = 0; k < G; ++k) samax[k] = io.span_amax(m0 + k);
        }
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int r = 0; r < kRows; ++r) io.load_ws(m0 + k, r, ws[k][r]);
    }
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int r = 0; r < kRows; ++r) add_replica<MODE, FMT, EMIT>(io, m0 + k, r, ws[k][r], g[r], acc[r], samax[k]);
}

// alpha-merge of the new global parameters into one row of one replica (wn = its words now).
template <class IO>
__device__ __forceinline__ void merge_replica(const Args& a, const IO& io, uint32_t m, int r, const uint32_t (&wn)[2],
                                              const float (&g)[kVec])
{
    float w[kVec];
    unpack_bf16(wn, w);
    uint32_t out[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
        out[k] = bf16_pack(a.alpha * w[2 * k] + a.one_minus_alpha * g[2 * k],
                           a.alpha * w[2 * k + 1] + a.one_minus_alpha * g[2 * k + 1]);
    io.store_wn(m, r, out);
}

template <int kRows, int G, class IO>
__device__ __forceinline__ void merge_replica_group(const Args& a, const IO& io, uint32_t m0, const float (&g)[kRows][kVec])
{
    uint32_t wn[G][kRows][2];
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int r = 0; r < kRows; ++r) io.load_wn(m0 + k, r, wn[k][r]);
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int r = 0; r < kRows; ++r) merge_replica(a, io, m0 + k, r, wn[k][r], g[r]);
}

// ALIASED: w_send[m] and w_now[m] are the same array (no overlap delay).  EMIT: the fused
// kernel also writes the messages.
template <int MODE, int FMT, int MT, bool ALIASED, bool EMIT, int kRows, class IO>
__device__ __forceinline__ void process(const Args& a, const IO& io)
{
    const uint32_t M = MT > 0 ? (uint32_t)MT : a.M;
    constexpr int MU = MT > 0 ? MT : 1;

    float g[kRows][kVec], mom[kRows][kVec], acc[kRows][kVec];
    uint32_t ws[MU][kRows][2] = {}, wn[MU][kRows][2], samax[MU] = {};

    // ---- loads that do not depend on anything; the scale words first: loads return in order, and the first replica cannot be encoded
    // without its own (28 M parameters, us, behind the tile's loads and ahead of them: fused, the whole call, M = 2 160.9 and 158.3;
    // send M = 4 134 and 128).  With 4 and 8 replicas compiled in, the fused step has enough on the way and takes scalar loads where it needs
    // the words (50 M parameters, whole call, M = 4: 418 so, 423 ahead of the tile, 425 by scalar loads ahead of it).  Of any M, the words
    // of a group of replicas go ahead of the group's loads as well: 28 M parameters, ahead and by scalar loads where needed, fused M = 3 / 6 / 12 /
    // 16 211 / 320 / 582 / 764 and 212 / 321 / 583 / 764; with messages M = 2 / 4 / 8 / 16 166 / 265.5 / 440 / 844 and 169 / 264 / 482 / 913;
    // send M = 3 / 12 107 / 330 and 110 / 342.  (Behind the group's loads: fused M = 3 222, M = 6 335.)
    constexpr bool kWordHere = MODE == kFused && MT >= 4 && is_span_scaled(FMT);
    if constexpr (MT > 0 && is_span_scaled(FMT) && (MODE == kQuantize || MODE == kFused) && !kWordHere) {
#pragma unroll
        for (int m = 0; m < MT; ++m) samax[m] = io.span_amax(m);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        io.load_g(r, g[r]);
        if constexpr (MODE == kReduce || MODE == kFused || MODE == kReceive) io.load_mom(r, mom[r]);
    }
    if constexpr (MT > 0) {
        if constexpr (MODE == kQuantize || MODE == kFused) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < kRows; ++r) io.load_ws(m, r, ws[m][r]);
        }
        if constexpr (MODE == kMerge || MODE == kReceive) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < kRows; ++r) io.load_wn(m, r, wn[m][r]);
        }
        if constexpr (MODE == kFused && !ALIASED) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < kRows; ++r) io.load_wn(m, r, wn[m][r]);
        }
    }

    // ---- outer gradients, messages, fp32 sum over replicas in ascending order
    if constexpr (MODE != kMerge) {
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int j = 0; j < kVec; ++j) acc[r][j] = 0.0f;
        if constexpr (MT > 0) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < kRows; ++r) add_replica<MODE, FMT, EMIT, kWordHere>(io, (uint32_t)m, r, ws[m][r], g[r], acc[r], samax[m]);
        } else {
            uint32_t m = 0;
            for (; m + 4u <= M; m += 4u) add_replica_group<MODE, FMT, EMIT, kRows, 4>(io, m, g, acc);
            if (M - m >= 2u) { add_replica_group<MODE, FMT, EMIT, kRows, 2>(io, m, g, acc); m += 2u; }
            for (; m < M; ++m) add_replica_group<MODE, FMT, EMIT, kRows, 1>(io, m, g, acc);
        }
    }

    // E4M3 messages were decoded by the conversion instruction alone.  It turns the two byte
    // values that the encoder never writes into NaN, which survives the sum: where any lane of
    // the wavefront sees a NaN (rare: a foreign message, or a block that really holds NaN), the
    // row is decoded again, exactly, from the messages in memory.
    if constexpr ((MODE == kReduce || MODE == kReceive) && FMT == SDL_FMT_E4M3 && IO::kHasInexactDecode) {
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float t = (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3]);
            if (__builtin_amdgcn_ballot_w64(t != t) != 0ull) {
#pragma unroll
                for (int j = 0; j < kVec; ++j) acc[r][j] = 0.0f;
                for (uint32_t m = 0; m < M; ++m) {
                    float dq[kVec];
                    io.template load_message<FMT, true>(m, r, dq);
#pragma unroll
                    for (int j = 0; j < kVec; ++j) acc[r][j] = acc[r][j] + dq[j];
                }
            }
        }
    }

    // ---- mean and Nesterov outer step
    if constexpr (MODE == kReduce || MODE == kFused || MODE == kReceive) {
        const float fm = (float)M;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
#pragma unroll
            for (int j = 0; j < kVec; ++j) {
                const float dbar = acc[r][j] / fm;
                const float m_new = a.mu * mom[r][j] + dbar;
                const float look = dbar + a.mu * m_new;
                mom[r][j] = m_new;
                g[r][j] = g[r][j] - a.lr * look;
            }
            io.store_g(r, g[r]);
            io.store_mom(r, mom[r]);
        }
    }

    // ---- alpha-merge into every replica
    if constexpr (MODE == kMerge || MODE == kFused || MODE == kReceive) {
        if constexpr (MT > 0) {
#pragma unroll
            for (int m = 0; m < MT; ++m) {
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    if constexpr (MODE == kFused && ALIASED) {
                        // same words as at the send step; hide that from the optimizer so that it
                        // re-expands the two packed registers instead of keeping four floats alive
                        uint32_t u[2] = {ws[m][r][0], ws[m][r][1]};
                        asm volatile("" : "+v"(u[0]), "+v"(u[1]));
                        merge_replica(a, io, (uint32_t)m, r, u, g[r]);
                    } else {
                        merge_replica(a, io, (uint32_t)m, r, wn[m][r], g[r]);
                    }
                }
            }
        } else {
            // (with w_send aliasing w_now these are the same words as at the send step, read again)
            uint32_t m = 0;
            for (; m + 4u <= M; m += 4u) merge_replica_group<kRows, 4>(a, io, m, g);
            if (M - m >= 2u) { merge_replica_group<kRows, 2>(a, io, m, g); m += 2u; }
            for (; m < M; ++m) merge_replica_group<kRows, 1>(a, io, m, g);
        }
    }
}

// ------------------------------------------------------------------ the kernel

// Workgroup -> tile.  The dispatcher deals workgroups round robin to the 8 XCDs.  Tiles in that order spread best over the
// memory channels, and it is what aligned arrays get.  Where the arrays start somewhere inside a cache line, every row
// shares its first and last line with its neighbours; on another XCD that line is fetched into a second L2 and written in
// two parts, so consecutive tiles go to one XCD, kChunkRows rows at a time (72 M parameters of odd groups, fused: M = 2
// 388 -> 329 us, M = 4 572 -> 483, M = 8 892 -> 869; half or twice the chunk is up to 2 % slower, and arrays that start on a
// line lose 3-8 % with it).  The rule (RunBuilder, flush) asks whether a run starts on a line in every array: groups of 1000 and
// 3 M parameters, which start on 16 bytes, without chunks and with: fused M = 2 374 and 342 us, M = 4 545 and 475, M = 8 856 and
// 826, send M = 4 179 and 174, receive M = 4 475 and 420, M = 2 332 and 294.  (One exception: kFoundBytes.)
constexpr int kXcds = 8;
constexpr int kChunkRows = 8;
template <int ROWS>
__device__ __forceinline__ uint32_t chunked_tile(uint32_t wg)
{
    constexpr uint32_t C = kChunkRows / ROWS, whole = kXcds * C;
    return wg / whole * whole + (wg % kXcds) * C + (wg / kXcds) % C;
}

// Has what a call's loads need in scalar registers from here on (the compiler would ask for each where it is first used, one
// wait after the other).
template <int MODE, int MT, bool ALIASED>
__device__ __forceinline__ void touch_arguments(const Args& a)
{
    asm volatile("" :: "s"(a.g), "s"(a.n_runs), "s"(a.chunked), "s"(a.staged), "s"(a.offset0), "s"(a.soff0));
    if constexpr (MODE != kMerge) asm volatile("" :: "s"(a.msg0));
    if constexpr (MODE == kReduce || MODE == kFused || MODE == kReceive) asm volatile("" :: "s"(a.mom));
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        if constexpr (MODE == kQuantize || MODE == kFused) asm volatile("" :: "s"(a.w_send[m]));
        if constexpr (MODE == kMerge || MODE == kReceive || (MODE == kFused && !ALIASED)) asm volatile("" :: "s"(a.w_now[m]));
        if constexpr (MODE == kReduce || MODE == kReceive) asm volatile("" :: "s"(a.codes[m]));
    }
}

template <int MODE, int FMT, int MT, bool ALIASED, bool EMIT>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(kWavesPerEu)))
void sdl_kernel(const Args a)
{
    // The start of a wavefront is a chain of dependent scalar loads, and with 8 wavefronts on a compute unit nothing
    // hides it: what does not depend on the run (the arrays' addresses, the first 16 first workgroups, the first run) is asked for
    // at once.
    uint32_t behind[kRunGroup - 1];                  // first workgroups of the 15 runs behind the first of the group
#pragma unroll
    for (int i = 1; i < kRunGroup; ++i) behind[i - 1] = a.table[i];
    uint32_t run = run_word<FMT>(0), first = 0, at = a.table[run], size = a.table[run + 1u], sidx = 0, soff = 0;
    if constexpr (is_span_scaled(FMT)) { sidx = a.table[run + 2u]; soff = a.table[run + 3u]; }
    touch_arguments<MODE, MT, ALIASED>(a);
    asm volatile("" :: "s"(at), "s"(size), "s"(sidx), "s"(soff), "s"(a.group_wg[0]), "s"(a.group_wg[1]), "s"(a.group_wg[2]), "s"(a.group_wg[3]),
                 "s"(a.group_wg[4]), "s"(a.group_wg[5]));
#pragma unroll
    for (int i = 1; i < kRunGroup; ++i) asm volatile("" :: "s"(behind[i - 1]));
    // Which run does this workgroup work on.  The first workgroups of 16 runs are one scalar load, compared all at once;
    // with more runs than that, those of every 16th run come first.  (Entry by entry it was a chain of scalar loads as long
    // as the list: 8.5 us for a launch of 16 small runs.  One vector load and a ballot are two dependent loads as well, but
    // the streams push the arguments out of the vector caches: 7 % slower on a fragment of 6 large runs.)  The scalar
    // instructions count as well: 16 groups compared where 6 would do, and three instructions to an entry, cost 5-6 % on 97 runs
    // with tiles of one row.
    constexpr int ROWS = tile_rows(MODE, MT, FMT);
    const uint32_t wg = blockIdx.x < a.chunked ? chunked_tile<ROWS>(blockIdx.x) : blockIdx.x;
    constexpr uint32_t kTile = ROWS * kRow;
    if (a.n_runs > 1u) {
        uint32_t base = 0, r = kRunGroup - 1;
        constexpr int kGroups = max_runs(FMT) / kRunGroup, kFew = kGroups < 7 ? kGroups : 7;
        if (a.n_runs > (uint32_t)kRunGroup) {
#pragma unroll
            for (int i = 1; i < kFew; ++i)
                if (wg >= a.group_wg[i - 1]) base = (uint32_t)(i * kRunGroup);
            if (a.n_runs > (uint32_t)(kFew * kRunGroup)) {
#pragma unroll
                for (int i = kFew; i < kGroups; ++i)
                    if (wg >= a.group_wg[i - 1]) base = (uint32_t)(i * kRunGroup);
            }
#pragma unroll
            for (int i = 1; i < kRunGroup; ++i) behind[i - 1] = a.table[base + i];
        }
#pragma unroll
        for (int i = kRunGroup - 1; i >= 1; --i)
            if (wg < behind[i - 1]) r = (uint32_t)(i - 1);
        r += base;
        run = run_word<FMT>(r);
        first = a.table[r];
        at = a.table[run];
        size = a.table[run + 1u];
        if constexpr (is_span_scaled(FMT)) { sidx = a.table[run + 2u]; soff = a.table[run + 3u]; }
        asm volatile("" :: "s"(first), "s"(at), "s"(size), "s"(sidx), "s"(soff));
    }
    const uint32_t numel = size & ~kVectorBit, tile = (wg - first) * kTile;   // first element of the tile in the run
    if (tile >= numel) return;
    const uint64_t t0 = a.offset0 + at + tile;
    const uint64_t tb = a.msg0 + (uint64_t)wg * kTile;
    const uint64_t s0 = !a.staged ? t0 : is_span_scaled(FMT) ? a.soff0 + soff + tile : a.soff0 + (uint64_t)wg * kTile;
    const uint32_t left = numel - tile;
    if (left < kTile && ((size & kVectorBit) || numel % kVec != 0u)) {
        const TailIO io{a, t0, tb, s0, left, threadIdx.x, sidx};
        process<MODE, FMT, 0, ALIASED, EMIT, ROWS>(a, io);
    } else if (left < kTile) {
        const TileIOT<true, ROWS, true> io{a, t0, tb, threadIdx.x, sidx, s0, left};
        process<MODE, FMT, MT, ALIASED, EMIT, ROWS>(a, io);
    } else if (!(size & kVectorBit)) {
        const TileIOT<true, ROWS> io{a, t0, tb, threadIdx.x, sidx, s0, kTile};
        process<MODE, FMT, MT, ALIASED, EMIT, ROWS>(a, io);
    } else {
        const TileIOT<false, ROWS> io{a, t0, tb, threadIdx.x, sidx, s0, kTile};
        process<MODE, FMT, MT, ALIASED, EMIT, ROWS>(a, io);
    }
}

// Pre-pass of the whole-span scale: the absolute maximum of every replica's outer gradient over
// each run, folded into the run's scale word with an integer atomic maximum (the words hold fp32
// bit patterns of non-negative values, which order like the values).  It has an argument block of
// its own, so that one launch covers up to 64 runs (a whole fragment as a rule).  The
// wavefronts are shared out among the runs; wavefront k of a run walks the run's tiles k, k + G, ...
// with 8 consecutive parameters per lane (128-bit loads, the next tile's loads issued before the
// current tile is consumed), keeps the running maxima in registers, and the scale words are touched
// once at the very end -- one atomic per workgroup (4 wavefronts) and replica instead of one per
// tile: atomics on one cache line are served one after the other, and the scale words of a launch
// share a few lines.
constexpr int kAbsmaxMaxRuns = 64;
constexpr int kAbsmaxWaves = 4;       // wavefronts per workgroup (50 to 113 VGPRs)
constexpr int kAbsmaxTile = 512;      // parameters a wavefront takes at a time: 8 per lane

struct AbsmaxRun {
    uint64_t offset;     // first element of the run in the flat arrays
    uint64_t numel;
    uint64_t soff;       // where the run starts in staged g (staged state only)
    uint32_t vec;        // g and every w_send are 16-byte aligned at the run start
    uint32_t sidx;       // index of the run's scale word
    uint32_t first;      // first workgroup of the launch that works on this run
    uint32_t G;          // workgroups of this run (>= 1)
};

struct AbsmaxArgs {
    const float* g;
    const uint16_t* w_send[SDL_MAX_WORKERS];
    uint8_t* scales[SDL_MAX_WORKERS];
    uint32_t M;
    uint32_t m0;         // first replica handled by this launch
    uint32_t staged;
    uint32_t n_runs;
    uint32_t look;       // a long launch: workgroups look at a word before the atomic on it
    uint32_t first[kAbsmaxMaxRuns];   // first workgroup of each run, ascending; 0xffffffff behind the last
    AbsmaxRun runs[kAbsmaxMaxRuns];
};
static_assert(sizeof(AbsmaxArgs) <= 4096, "kernel arguments");

template <int MB>
struct AbsmaxTile {
    u32x4 g0, g1;
    u32x4 w[MB];
};

template <int MB, bool KEEP>
__device__ __forceinline__ void absmax_load(AbsmaxTile<MB>& t, const AbsmaxArgs& a, uint64_t ge, uint64_t we,
                                            uint32_t valid, bool fast, uint32_t lane)
{
    constexpr int kAux = KEEP ? 0 : kAuxLoad;
    if (fast && valid == (uint32_t)kAbsmaxTile) {
        const __amdgpu_buffer_rsrc_t rg = rsrc(a.g + ge, kAbsmaxTile * 4);
        t.g0 = __builtin_amdgcn_raw_buffer_load_b128(rg, (int)(lane * 32), 0, kAux);
        t.g1 = __builtin_amdgcn_raw_buffer_load_b128(rg, (int)(lane * 32 + 16), 0, kAux);
#pragma unroll
        for (int m = 0; m < MB; ++m)
            t.w[m] = __builtin_amdgcn_raw_buffer_load_b128(rsrc(a.w_send[a.m0 + m] + we, kAbsmaxTile * 2),
                                                           (int)(lane * 16), 0, kAux);
    } else if (valid == (uint32_t)kAbsmaxTile) {
        // a whole tile of a run that starts at some other element: vectors of element alignment
        const u32x4_f32elem* pg = reinterpret_cast<const u32x4_f32elem*>(a.g + ge + lane * 8);
        t.g0 = KEEP ? pg[0] : __builtin_nontemporal_load(pg);
        t.g1 = KEEP ? pg[1] : __builtin_nontemporal_load(pg + 1);
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const u32x4_bf16elem* pw = reinterpret_cast<const u32x4_bf16elem*>(a.w_send[a.m0 + m] + we + lane * 8);
            t.w[m] = KEEP ? *pw : __builtin_nontemporal_load(pw);
        }
    } else {
        // ragged tail: element by element under the buffer range check, which returns 0 past the
        // end (g = 0 and w = 0 give an outer gradient of 0: no effect on a maximum)
        const __amdgpu_buffer_rsrc_t rg = rsrc(a.g + ge, valid * 4);
        uint32_t x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = __builtin_amdgcn_raw_buffer_load_b32(rg, (int)((lane * 8 + j) * 4), 0, 0);
        t.g0 = u32x4{x[0], x[1], x[2], x[3]};
        t.g1 = u32x4{x[4], x[5], x[6], x[7]};
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const __amdgpu_buffer_rsrc_t rw = rsrc(a.w_send[a.m0 + m] + we, valid * 2);
            uint32_t h[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                h[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rw, (int)((lane * 8 + j) * 2), 0, 0) & 0xffffu;
            t.w[m] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
        }
    }
}

// KEEP: normal cache policy, where the fused pass behind this one finds some of g and w_send in the memory-side cache.
template <int MB, bool KEEP>
__global__ __launch_bounds__(kWave * kAbsmaxWaves) void sdl_span_absmax_kernel(const AbsmaxArgs a)
{
    __shared__ uint32_t wave_max[kAbsmaxWaves][MB];
    // the wavefront's number is the same in all of its lanes: say so, or every address derived from it
    // is treated as different per lane and every buffer access is wrapped in a loop over lanes
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    uint32_t r = 0;
#pragma unroll
    for (int i = 1; i < kAbsmaxMaxRuns; ++i)       // four scalar loads, compared at once
        if (blockIdx.x >= a.first[i]) r = (uint32_t)i;
    const AbsmaxRun run = a.runs[r];
    // every wavefront of the run's workgroups walks its own tiles: k, k + G, ...; neighbouring
    // tiles go to neighbouring workgroups (which the dispatcher deals to different XCDs), not to
    // the wavefronts of one workgroup
    const uint32_t k = wave * run.G + (blockIdx.x - run.first), G = run.G * kAbsmaxWaves;
    const uint64_t n_tiles = (run.numel + kAbsmaxTile - 1) / kAbsmaxTile;
    const bool fast = run.vec != 0u;
    auto valid_of = [&](uint64_t t) -> uint32_t {
        const uint64_t rem = run.numel - t * kAbsmaxTile;
        return rem < (uint64_t)kAbsmaxTile ? (uint32_t)rem : (uint32_t)kAbsmaxTile;
    };
    auto g_elem = [&](uint64_t t) -> uint64_t { return (a.staged ? run.soff : run.offset) + t * kAbsmaxTile; };

    auto word = [&](uint32_t m) { return reinterpret_cast<uint32_t*>(a.scales[a.m0 + m]) + run.sidx; };
    uint32_t amax[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) amax[m] = 0u;

    AbsmaxTile<MB> cur;
    if (k < n_tiles) absmax_load<MB, KEEP>(cur, a, g_elem(k), run.offset + (uint64_t)k * kAbsmaxTile, valid_of(k), fast, lane);
    for (uint64_t t = k; t < n_tiles; t += G) {
        AbsmaxTile<MB> nxt = cur;
        const uint64_t tn = t + G;
        if (tn < n_tiles) absmax_load<MB, KEEP>(nxt, a, g_elem(tn), run.offset + tn * kAbsmaxTile, valid_of(tn), fast, lane);
        const uint32_t gb[8] = {cur.g0.x, cur.g0.y, cur.g0.z, cur.g0.w, cur.g1.x, cur.g1.y, cur.g1.z, cur.g1.w};
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const uint32_t wb[4] = {cur.w[m].x, cur.w[m].y, cur.w[m].z, cur.w[m].w};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float d = u2f(gb[j]) - ((j & 1) ? bf16_hi(wb[j / 2]) : bf16_lo(wb[j / 2]));
                const uint32_t mag = f2u(d) & 0x7fffffffu;
                amax[m] = mag > amax[m] ? mag : amax[m];
            }
        }
        cur = nxt;
    }
    // wavefront, then workgroup (all of whose wavefronts work on the same run), then one atomic
    // per workgroup and replica
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const uint32_t v = lanes_max<kWave>(amax[m]);
        if (lane == 0u) wave_max[wave][m] = v;
    }
    __syncthreads();
    if (threadIdx.x < (uint32_t)MB) {
        uint32_t v = 0u;
        for (int w = 0; w < kAbsmaxWaves; ++w) v = wave_max[w][threadIdx.x] > v ? wave_max[w][threadIdx.x] : v;
        // A look at the word first spares the atomic where the word already holds more, but it is itself served one after
        // the other, at memory that every XCD shares, and finds nothing while all workgroups end at once.  It pays only in
        // long launches, whose workgroups drift apart (28 M parameters, M = 2, 2048 workgroups: the whole call 197 us with
        // it, 167 without; 53 M 328 and 316; 302 M, M = 4, 2532 and 2539).
        uint32_t* const to = word(threadIdx.x);
        if (!a.look || v > __hip_atomic_load(to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            __hip_atomic_fetch_max(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Clears the scale words of a pre-pass launch's runs before the maximum is accumulated
// (thread = run * 16 + replica).
__global__ __launch_bounds__(SDL_MAX_WORKERS * kAbsmaxMaxRuns) void sdl_zero_span_scales(const AbsmaxArgs a)
{
    const uint32_t r = threadIdx.x / SDL_MAX_WORKERS, m = threadIdx.x % SDL_MAX_WORKERS;
    if (m < a.M && r < a.n_runs) reinterpret_cast<uint32_t*>(a.scales[m])[a.runs[r].sidx] = 0u;
}

// Streaming yardsticks for the HBM roofline, 16 bytes per lane: a plain copy, and the same copy, a
// read-only pass and a write-only pass with the non-temporal policy the method's kernels use.
constexpr int kCopyThreads = 256;
__global__ __launch_bounds__(kCopyThreads) void sdl_copy_kernel(uint4* __restrict__ dst,
                                                            const uint4* __restrict__ src, uint64_t n16)
{
    const uint64_t i = (uint64_t)blockIdx.x * kCopyThreads + threadIdx.x;
    if (i < n16) dst[i] = src[i];
}
template <int KIND>
__global__ __launch_bounds__(kCopyThreads) void sdl_probe_kernel(u32x4* __restrict__ dst,
                                                             const u32x4* __restrict__ src, uint64_t n16)
{
    const uint64_t i = (uint64_t)blockIdx.x * kCopyThreads + threadIdx.x;
    if (i >= n16) return;
    if constexpr (KIND == SDL_PROBE_COPY_NT) {
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
    } else if constexpr (KIND == SDL_PROBE_READ_NT) {
        // the data has to be used for the load to stay: one word of dst is written if the 16 bytes spell a
        // value that seeded or zeroed buffers never hold
        const u32x4 x = __builtin_nontemporal_load(src + i);
        if ((x.x ^ x.y ^ x.z ^ x.w) == 0x9e3779b9u && x.x == 0x7f4a7c15u) dst[0] = x;
    } else {
        const u32x4 x = {(uint32_t)i, 0u, 0u, 0u};
        __builtin_nontemporal_store(x, dst + i);
    }
}

// ------------------------------------------------------------------ host side

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

size_t code_align(sdl_format_t fmt)
{
    return fmt == SDL_FMT_FP32 ? 4 : fmt == SDL_FMT_BF16 ? 2 : 1;
}
size_t scale_align(sdl_format_t fmt) { return is_span_scaled(fmt) ? 4 : 1; }
// bytes of code per element (x2 for E3M0, which holds half a byte)
size_t code_bytes_at(sdl_format_t fmt, uint64_t elem)
{
    switch (fmt) {
    case SDL_FMT_FP32: return (size_t)elem * 4;
    case SDL_FMT_BF16: return (size_t)elem * 2;
    case SDL_FMT_E4M3: return (size_t)elem;
    default: return (size_t)(elem / 2);
    }
}

// Wavefronts that share a CU (0: as many as fit, 32).  Enough loads in flight, not so many that the access window in each array
// grows and DRAM page locality is lost: the knob that matters for a streaming kernel.  The kernels that write the replicas
// back want few, and fewer the more arrays they walk, but never less than 8 (6 cost 15-20 %); the receive side without the
// merge reads many small messages and writes two arrays, and wants more as decoding grows with the replicas; the send side
// wants all it can get, except where it writes whole words for many replicas.  Formats that run the codec want more than
// those that only round.  us in one process, the caps in turn on the same arrays, E3M0 unless named (between processes all
// of a row move by up to 4 %, with where the arrays lie; within one a figure repeats to 1 %):
//                                         M    none   21   16   11    8
//   fused, 105 M parameters               2     489  485  476  469  495
//                                         3     609  609  600  589  629
//                                         4     734  743  729  707  682
//                                         6     984  984  973  940  905
//                                         8    1228 1227 1250 1228 1190
//                                        12    1765 1765 1753 1682 1624
//   fused, w_send aliases w_now           2     417  412  406  404  471
//                                         4     582  577  565  552  596
//                                         8     914  912  914  882  866
//   one-pass receive, 53 M                2     216  214  209  227  240
//                                         3     268  261  258  262  290
//                                         5     365  364  350  342  356
//                                         6     409  412  399  384  389
//                                        12     708  716  696  668  650
//   merge, 67 M                           2     123  121  120  135  163
//                                         3     170  164  169  181  205
//                                         4     219  217  211  205  226
//                                         5     267  257  251  254  279
//                                         7     373  362  345  338  364
//                                        10     518  519  502  464  460
//                                        16     837  849  829  770  727
//   receive side without the merge, 67 M  3     200  190  183  189  217
//                                         9     230  225  224  250  304
//                                        10     236  232  228  258  316
//                                        12     253  247  254  297  366
//                                        16     280  277  302  362  444
//   send, FP32, 50 M                      5     296  306  298  285  281
//                                         6     355  367  358  345  336
//                                        12     706  728  719  699  679
//                                        16     940  969  961  938  922
//   messages written, BF16, 53 M          2     295  289  278  273  279
//                                         4     454  456  448  430  415
//                                         8     785  793  785  753  731
//   messages written, E3M0                3     318  318  318  344  398
//                                         6     517  517  517  508  538
//   messages written, E4M3                4     413  414  404  392  393
//                                         8     702  703  688  670  655
uint32_t waves_per_cu(int mode, uint32_t mt, uint32_t M, int fmt, bool aliased, bool emit)
{
    switch (mode) {
    case kFused:
        if (emit && is_scaled(fmt)) return M <= 4 ? 16 : 11;
        if (emit) return M <= 2 ? 16 : (M == 3 ? 11 : 8);
        if (mt == 0) return M == 3 ? 11 : 8;
        return mt == 1 ? 16 : (mt == 2 || (aliased && mt == 4) ? 11 : 8);
    case kReceive:
        if (mt == 0) return M <= 5 ? 11 : 8;
        return mt <= 2 ? 16 : 8;
    case kMerge:
        if (mt == 0) return M == 3 ? 21 : (M == 5 ? 16 : (M <= 7 ? 11 : 8));
        return mt == 1 ? 0 : (mt == 2 ? 16 : (mt == 4 ? 11 : 8));
    case kQuantize:
        return mt == 0 && M >= 5 && fmt == SDL_FMT_FP32 ? 8 : 0;
    case kReduce:
        if (mt == 0) return M <= 10 ? 16 : 21;
        return mt == 4 ? 16 : 0;
    default:
        return 0;
    }
}

// Launches that end within a few rounds of workgroups have no page locality to lose and want at least 16: up to 112 MiB moved.
// us on one card, states that rotate through more than the memory-side cache, as capped above and with 16 (fused, E3M0, but where named):
// M = 2, 29 MB 7.2 7.0, 59 MB 12.1 11.8, 117 MB 21.8 21.3, 235 MB 39.5 39.7; M = 4, 42 MB 9.9 9.5, 84 MB 16.7 16.6, 126 MB 22.9 23.5,
// 168 MB 29.6 30.4; w_send aliases w_now, M = 2, 25 MB 6.5 5.6; receive, M = 4, 64 MB 15.5 14.9; M = 5, 72 MB 18.2 17.2; M = 16, 160 MB
// 40.3 37.3; messages, BF16, M = 4, 88 MB 19.4 19.0, 280 MB 47.1 49.3; 193 groups of 100 to 30000 parameters, M = 2, 70 MB 16.1 15.4.
constexpr uint64_t kSmallLaunch = 112ull << 20;
constexpr uint32_t kSmallWaves = 16;
uint64_t bytes_per_param(int mode, uint32_t M, bool aliased, bool emit, int fmt)
{
    const uint64_t state = mode == kMerge ? 4 : mode == kQuantize ? 4 : 16;
    const uint64_t send = (mode == kQuantize || (mode == kFused && !aliased)) ? 2 : 0, merge = (mode == kReduce || mode == kQuantize) ? 0 : 4;
    const uint64_t code = fmt == SDL_FMT_FP32 ? 4 : fmt == SDL_FMT_BF16 ? 2 : 1;
    return state + M * (send + merge + (mode == kFused && !emit ? 0 : mode == kMerge ? 0 : code));
}

// The cap takes the form of dynamic LDS that nothing uses: 160 KiB per CU, given out in units of 1280 bytes (measured: 6826
// and 7680 bytes leave 21 wavefronts on a CU, 7681 leave 18, 12800 12, 13653 and 14080 11, 14081 10).
constexpr uint32_t kLdsPerCu = 163840, kLdsUnit = 1280;
constexpr uint32_t lds_cap_bytes(uint32_t waves) { return waves ? kLdsPerCu / waves / kLdsUnit * kLdsUnit : 0u; }
constexpr bool cap_is_kept(uint32_t waves) { return kLdsPerCu / lds_cap_bytes(waves) == waves; }
static_assert(cap_is_kept(8) && cap_is_kept(11) && cap_is_kept(16) && cap_is_kept(21), "the caps of waves_per_cu");

template <int MODE, int FMT, bool ALIASED, bool EMIT>
hipError_t launch_m(const Args& a, uint32_t n_wg, hipStream_t s)
{
    const dim3 grid(n_wg), block(kWave);
    const uint32_t mt = variant_mt(MODE, a.M, EMIT);   // the grid was sized for this variant's tile
    uint32_t waves = waves_per_cu(MODE, mt, a.M, FMT, ALIASED, EMIT);
    const uint64_t params = (uint64_t)n_wg * (uint64_t)(tile_rows(MODE, (int)mt, FMT) * kRow);
    if (waves && waves < kSmallWaves && params * bytes_per_param(MODE, a.M, ALIASED, EMIT, FMT) <= kSmallLaunch) waves = kSmallWaves;
    const uint32_t lds = lds_cap_bytes(waves);
    switch (mt) {
    case 1: if constexpr (!EMIT) hipLaunchKernelGGL((sdl_kernel<MODE, FMT, 1, ALIASED, EMIT>), grid, block, lds, s, a); break;
    case 2: if constexpr (!EMIT) hipLaunchKernelGGL((sdl_kernel<MODE, FMT, 2, ALIASED, EMIT>), grid, block, lds, s, a); break;
    case 4: if constexpr (!EMIT) hipLaunchKernelGGL((sdl_kernel<MODE, FMT, 4, ALIASED, EMIT>), grid, block, lds, s, a); break;
    case 8: if constexpr (!EMIT) hipLaunchKernelGGL((sdl_kernel<MODE, FMT, 8, ALIASED, EMIT>), grid, block, lds, s, a); break;
    default: hipLaunchKernelGGL((sdl_kernel<MODE, FMT, 0, ALIASED, EMIT>), grid, block, lds, s, a); break;
    }
    return hipGetLastError();
}

template <int MODE, int FMT>
hipError_t launch_f(const Args& a, uint32_t n_wg, hipStream_t s)
{
    if constexpr (MODE == kFused) {
        if (a.emit) return a.aliased ? launch_m<MODE, FMT, true, true>(a, n_wg, s) : launch_m<MODE, FMT, false, true>(a, n_wg, s);
        return a.aliased ? launch_m<MODE, FMT, true, false>(a, n_wg, s) : launch_m<MODE, FMT, false, false>(a, n_wg, s);
    } else {
        return launch_m<MODE, FMT, false, false>(a, n_wg, s);
    }
}

// Whole-span scale words of a list of runs: cleared, then the maximum of every replica's outer
// gradient over each run.  A launch's wavefronts are shared out among the runs in proportion to their tiles (whole
// workgroups, at least one each); up to 8 replicas per pass over g.  One wavefront for 16 tiles, 1024 to 8192 of them: the
// atomics at the end cost 8 ns for each workgroup and replica whatever the size (28 M parameters, M = 2: 160 us the whole
// call, 167 with 8192; 8 M parameters 50 and 60; 302 M the same).
constexpr uint32_t kAbsmaxMinGroups = 1024, kAbsmaxGroups = 8192, kAbsmaxTilesPerWave = 16;

// What the pre-pass reads stays in the 256 MiB memory-side cache for the pass behind it if it fits there (28 M parameters,
// 227 MB: the whole call 170 us with the normal cache policy, 183 non-temporal; 302 M, 3.6 GB: 2621 and 2604).
constexpr uint64_t kKeepBytes = 256ull << 20;

template <bool KEEP>
void launch_absmax(uint32_t mb, dim3 grid, hipStream_t s, const AbsmaxArgs& b)
{
    const dim3 block(kWave * kAbsmaxWaves);
    switch (mb) {
    case 8: hipLaunchKernelGGL((sdl_span_absmax_kernel<8, KEEP>), grid, block, 0, s, b); break;
    case 7: hipLaunchKernelGGL((sdl_span_absmax_kernel<7, KEEP>), grid, block, 0, s, b); break;
    case 6: hipLaunchKernelGGL((sdl_span_absmax_kernel<6, KEEP>), grid, block, 0, s, b); break;
    case 5: hipLaunchKernelGGL((sdl_span_absmax_kernel<5, KEEP>), grid, block, 0, s, b); break;
    case 4: hipLaunchKernelGGL((sdl_span_absmax_kernel<4, KEEP>), grid, block, 0, s, b); break;
    case 3: hipLaunchKernelGGL((sdl_span_absmax_kernel<3, KEEP>), grid, block, 0, s, b); break;
    case 2: hipLaunchKernelGGL((sdl_span_absmax_kernel<2, KEEP>), grid, block, 0, s, b); break;
    default: hipLaunchKernelGGL((sdl_span_absmax_kernel<1, KEEP>), grid, block, 0, s, b); break;
    }
}

struct SpanRun { uint64_t offset, numel, soff; bool vec; uint32_t sidx; };

hipError_t launch_span_prepass(const Args& a, const SpanRun* runs, uint32_t n_runs, hipStream_t s)
{
    for (uint32_t r0 = 0; r0 < n_runs; r0 += kAbsmaxMaxRuns) {
        AbsmaxArgs b{};
        std::memset(b.first, 0xff, sizeof(b.first));
        b.g = a.g;
        b.M = a.M;
        b.staged = a.staged;
        for (uint32_t m = 0; m < a.M; ++m) { b.w_send[m] = a.w_send[m]; b.scales[m] = a.scales[m]; }
        const uint32_t n = n_runs - r0 < (uint32_t)kAbsmaxMaxRuns ? n_runs - r0 : (uint32_t)kAbsmaxMaxRuns;
        uint64_t total_tiles = 0;
        for (uint32_t r = 0; r < n; ++r) total_tiles += (runs[r0 + r].numel + kAbsmaxTile - 1) / kAbsmaxTile;
        uint64_t groups = total_tiles / kAbsmaxTilesPerWave;
        if (groups < kAbsmaxMinGroups) groups = kAbsmaxMinGroups;
        if (groups > kAbsmaxGroups) groups = kAbsmaxGroups;
        b.look = total_tiles > 2u * kAbsmaxTilesPerWave * kAbsmaxGroups ? 1u : 0u;   // 134 M parameters
        uint32_t next = 0;
        for (uint32_t r = 0; r < n; ++r) {
            const SpanRun& in = runs[r0 + r];
            const uint64_t tiles = (in.numel + kAbsmaxTile - 1) / kAbsmaxTile;
            uint64_t waves = total_tiles ? (tiles * groups + total_tiles - 1) / total_tiles : 1;
            if (waves > tiles) waves = tiles;
            uint64_t G = (waves + kAbsmaxWaves - 1) / kAbsmaxWaves;
            if (G < 1) G = 1;
            b.first[r] = next;
            b.runs[r] = AbsmaxRun{in.offset, in.numel, in.soff, in.vec ? 1u : 0u, in.sidx, next, (uint32_t)G};
            next += (uint32_t)G;
        }
        b.n_runs = n;
        hipLaunchKernelGGL(sdl_zero_span_scales, dim3(1), dim3(SDL_MAX_WORKERS * kAbsmaxMaxRuns), 0, s, b);
        const dim3 grid(next);
        const bool keep = total_tiles * kAbsmaxTile * (4u + 2u * a.M) <= kKeepBytes;
        for (uint32_t m0 = 0; m0 < a.M;) {
            const uint32_t left = a.M - m0;
            const uint32_t mb = left < 8u ? left : 8u;
            b.m0 = m0;
            if (keep) launch_absmax<true>(mb, grid, s, b);
            else launch_absmax<false>(mb, grid, s, b);
            m0 += mb;
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

template <int MODE>
hipError_t launch(const Args& a, sdl_format_t fmt, uint32_t n_wg, hipStream_t s)
{
    if constexpr (MODE == kMerge) return launch_f<MODE, SDL_FMT_FP32>(a, n_wg, s);
    switch (fmt) {
    case SDL_FMT_FP32: return launch_f<MODE, SDL_FMT_FP32>(a, n_wg, s);
    case SDL_FMT_BF16: return launch_f<MODE, SDL_FMT_BF16>(a, n_wg, s);
    case SDL_FMT_E4M3: return launch_f<MODE, SDL_FMT_E4M3>(a, n_wg, s);
    case SDL_FMT_E3M0_B64: return launch_f<MODE, SDL_FMT_E3M0_B64>(a, n_wg, s);
    case SDL_FMT_E3M0_B128: return launch_f<MODE, SDL_FMT_E3M0_B128>(a, n_wg, s);
    case SDL_FMT_E3M0_SPAN: return launch_f<MODE, SDL_FMT_E3M0_SPAN>(a, n_wg, s);
    case SDL_FMT_E3M0_RN: return launch_f<MODE, SDL_FMT_E3M0_RN>(a, n_wg, s);
    default: return launch_f<MODE, SDL_FMT_E3M0>(a, n_wg, s);
    }
}

bool valid_format(sdl_format_t fmt) { return fmt >= SDL_FMT_FP32 && fmt <= SDL_FMT_E3M0_RN; }

// Alignment of a call's pointers (model: g, mom and the replicas; msg: the codes, scale bytes need none), and then of a run's
// first element: model asks for what the four elements of a lane need, wide for 16 bytes in every array, line for a cache line.
//
// The buffer path needs no more than model, but the whole tiles of a long run that is off 16 bytes are faster on the vector path (but for
// the send side).  us, on the buffer path and on the vector path:
//   runs of 3 and 4 M parameters, 42 M, half of them 4 elements off: reduce M = 2 bf16 143 and 130, receive M = 5 E4M3 312 and 295,
//   merge M = 8 296 and 289, with messages M = 2 bf16 247 and 225, fused M = 8 539 and 528, M = 2 201 and 200; send M = 1 47 and 49, M = 4 108 and
//   110, M = 8 196 and 202;
//   160004 each: reduce M = 2 112 and 106, with messages 186 and 178, receive M = 4 and fused M = 2 the same;
//   40004 each: reduce 87 and 83, with messages 145 and 143, the others the same;
//   10004 each: receive M = 8 E4M3 125 and 144, with messages M = 8 156 and 169, merge M = 4 46 and 49, reduce M = 2 44 and 42.
// So the line is kLongRun.
constexpr uint64_t kLongRun = 1u << 16;
struct Align {
    bool model = true, wide = true, line = true, msg = true;
    void add_model(const void* p)
    {
        model = wide = model && aligned(p, 16);
        line = line && aligned(p, 128);
    }
    Align at(uint64_t offset, uint64_t soff) const
    {
        const uint64_t low = offset | soff;
        return Align{model && low % kVec == 0, wide && low % 8 == 0, line && low % 64 == 0, msg};
    }
    TilePath path(int mode, uint64_t n) const
    {
        return (wide || (model && (mode == kQuantize || n < kLongRun))) && msg ? kPathBuffer : kPathVector;
    }
};

// Parameters per workgroup of the kernel variant that a call in this mode will run.
uint32_t tile_elems(int mode, const Args& a, sdl_format_t fmt)
{
    return (uint32_t)(tile_rows(mode, (int)variant_mt(mode, a.M, a.emit != 0u), (int)fmt) * kRow);
}

// Fills a launch's run table from a list of pieces.  A piece longer than kMaxRunElems takes several runs (they start at
// multiples of 512 elements, so scale blocks and tiles stay where they were).
struct RunBuilder {
    Args* a;
    uint64_t tile;       // parameters per workgroup
    int mode;
    uint32_t words, most;      // of a run; runs that the table has room for
    uint64_t n_wg = 0, n_unaligned = 0;
    RunBuilder(Args* args, int mode, uint32_t tile_elems, sdl_format_t fmt)
        : a(args), tile(tile_elems), mode(mode), words((uint32_t)run_words(fmt)), most((uint32_t)max_runs(fmt)) { reset(); }
    void reset()
    {
        a->n_runs = 0;
        n_wg = n_unaligned = 0;
        std::memset(a->table, 0xff, sizeof(uint32_t) * most);
        std::memset(a->group_wg, 0xff, sizeof(a->group_wg));
    }
    // Workgroups of a run: those of whole 512-element pieces.
    uint64_t wgs(uint64_t n) const { return (n + kPad - 1) / kPad * (kPad / tile); }
    // Whether a run of n elements still fits this launch: a free entry, numbers that fit 32 bits from the first run's,
    // and a grid that stays within the launch limit.
    bool fits(uint64_t offset, uint64_t n, uint64_t soff) const
    {
        if (a->n_runs == 0) return true;
        return a->n_runs < most && offset >= a->offset0 && offset - a->offset0 <= 0xffffffffull
               && (!a->staged || (soff >= a->soff0 && soff - a->soff0 <= 0xffffffffull)) && n_wg + wgs(n) <= 0x7fffffffull;
    }
    // msg and soff of a run are those of the run before it and its 512-element pieces (soff with a whole-span format is not).
    void add(uint64_t offset, uint64_t n, Align al, uint64_t msg, uint32_t sidx, uint64_t soff)
    {
        if (a->n_runs == 0) { a->offset0 = offset; a->msg0 = msg; a->soff0 = soff; }
        const uint32_t r = a->n_runs++;
        a->table[r] = (uint32_t)n_wg;
        if (r % kRunGroup == 0 && r) a->group_wg[r / kRunGroup - 1] = (uint32_t)n_wg;
        uint32_t* const run = a->table + most + r * (words - 1);
        run[0] = (uint32_t)(offset - a->offset0);
        run[1] = (uint32_t)n | (al.path(mode, n) == kPathVector ? kVectorBit : 0u);
        if (words == (uint32_t)kSpanRunWords) { run[2] = sidx; run[3] = (uint32_t)(soff - a->soff0); }
        n_wg += wgs(n);
        if (!al.line) n_unaligned += wgs(n);
    }
};

// The aliasing rule of the interface, checked: an array that a call writes must not overlap any other
// array of the call (w_send[m] being the very same pointer as w_now[m] is the one exception, and then
// only w_now[m] is listed).  model_elems / state_elems: elements of the replicas and of g / mom that the
// call may touch; code_bytes / scale_bytes: size of one replica's message arrays.
template <int MODE>
bool arrays_clash(const Args& a, sdl_format_t fmt, uint64_t model_elems, uint64_t state_elems, size_t code_bytes,
                  size_t scale_bytes)
{
    struct Range { uintptr_t lo, hi; bool written; };
    Range r[2 + 4 * SDL_MAX_WORKERS];
    int n = 0;
    auto add = [&](const void* p, uint64_t bytes, bool written) {
        if (p && bytes) { r[n].lo = reinterpret_cast<uintptr_t>(p); r[n].hi = r[n].lo + bytes; r[n].written = written; ++n; }
    };
    constexpr bool state_written = MODE == kReduce || MODE == kFused || MODE == kReceive;
    add(a.g, state_elems * 4, state_written);
    if constexpr (state_written) add(a.mom, state_elems * 4, true);
    const bool msg_written = MODE == kQuantize || (MODE == kFused && a.emit);
    const bool msg_used = msg_written || MODE == kReduce || MODE == kReceive;
    for (uint32_t m = 0; m < a.M; ++m) {
        if (MODE == kQuantize || (MODE == kFused && !a.aliased)) add(a.w_send[m], model_elems * 2, false);
        if (MODE == kMerge || MODE == kFused || MODE == kReceive) add(a.w_now[m], model_elems * 2, true);
        if (msg_used) add(a.codes[m], code_bytes, msg_written);
        if (msg_used || (MODE == kFused && is_span_scaled(fmt))) add(a.scales[m], scale_bytes, msg_written || MODE == kFused);
    }
    for (int i = 0; i < n; ++i)
        for (int j = i + 1; j < n; ++j)
            if ((r[i].written || r[j].written) && r[i].lo < r[j].hi && r[j].lo < r[i].hi) return true;
    return false;
}

// The pass behind the pre-pass of a whole-span scale finds g and w_send in the memory-side cache, if they are small.  A line that two
// XCDs fetch is cheap there, and chunks cost more than they save.  us, chunks and the order of the grid, one run 8 elements
// off a line, by what the pre-pass read: send M = 1 25 MB 19.0 17.2, 50 MB 26.9 24.6, 200 MB 75.0 73.7, M = 4 25 MB 18.1 17.4, 100 MB
// 42.7 42.0, 400 MB 158 160; fused M = 1 25 MB 31.1 29.5, 50 MB 50.0 48.7, M = 2 34 MB 35.1 33.2, 67 MB 59.5 59.2, 134 MB 104.6 105.3, M = 4
// 25 MB 29.7 27.9, 100 MB 80.1 81.2, M = 8 42 MB 41.1 39.9, 84 MB 71.4 72.4.  With many runs the pre-pass leaves them in another order:
// 193 runs of 100 to 30000 parameters, 30 MB, fused M = 4 50.1 51.2.
constexpr uint64_t kFoundBytes = 64ull << 20;
template <int MODE> constexpr bool after_prepass(sdl_format_t fmt)
{
    return (MODE == kQuantize || MODE == kFused) && is_span_scaled(fmt);
}

// Launches what the builder holds; false if the launch failed.
template <int MODE>
bool flush(RunBuilder& rb, sdl_format_t fmt, void* stream)
{
    if (rb.a->n_runs == 0) return true;
    // what most of the launch's tiles want (see chunked_tile)
    const uint32_t whole = kXcds * kChunkRows / (uint32_t)(rb.tile / kRow);
    const bool chunks = 2 * rb.n_unaligned > rb.n_wg && !(after_prepass<MODE>(fmt) && rb.a->n_runs == 1 && rb.n_wg * rb.tile * (4 + 2 * rb.a->M) <= kFoundBytes);
    rb.a->chunked = chunks ? (uint32_t)rb.n_wg / whole * whole : 0u;
    const hipError_t e = launch<MODE>(*rb.a, fmt, (uint32_t)rb.n_wg, (hipStream_t)stream);
    rb.reset();
    return e == hipSuccess;
}

// Adds one piece, cut to kMaxRunElems, launching whenever the launch is full.
template <int MODE>
bool add_piece(RunBuilder& rb, sdl_format_t fmt, uint64_t offset, uint64_t numel, Align al, uint64_t msg, uint32_t sidx,
               uint64_t soff, void* stream)
{
    for (uint64_t at = 0; at < numel; at += kMaxRunElems) {
        const uint64_t n = numel - at < kMaxRunElems ? numel - at : kMaxRunElems;
        if (!rb.fits(offset + at, n, soff + at) && !flush<MODE>(rb, fmt, stream)) return false;
        rb.add(offset + at, n, al, msg + at, sidx, soff + at);
    }
    return true;
}

// One span starting at the given pointers (offset 0).
template <int MODE>
int run_single_span(Args& a, uint64_t n, sdl_format_t fmt, Align al, void* stream)
{
    if (n == 0) return SDL_OK;
    const uint32_t tile = tile_elems(MODE, a, fmt);
    if (n > (uint64_t)0x7fffffff * (uint64_t)tile) return SDL_ERR_UNSUPPORTED;
    {
        size_t cb = 0, sb = 0;
        sdl_exchange_bytes(fmt, n, &cb, &sb);
        if (arrays_clash<MODE>(a, fmt, n, n, cb, sb)) return SDL_ERR_INVALID_ARG;
    }
    if constexpr (MODE == kQuantize || MODE == kFused) {
        if (is_span_scaled(fmt)) {
            // whole-span scale: clear the scale word, take the grid-wide maximum, then encode
            const SpanRun one{0, n, 0, al.wide, 0};
            if (launch_span_prepass(a, &one, 1, (hipStream_t)stream) != hipSuccess) return SDL_ERR_DEVICE;
        }
    }
    RunBuilder rb(&a, MODE, tile, fmt);
    return add_piece<MODE>(rb, fmt, 0, n, al, 0, 0, 0, stream) && flush<MODE>(rb, fmt, stream) ? SDL_OK : SDL_ERR_DEVICE;
}

}  // namespace

extern "C" {

int sdl_quantize_outer_grad(const float* g, const void* const* w_send, uint32_t M, uint64_t n,
                            sdl_format_t fmt, void* const* codes, void* const* scales, void* stream)
{
    if (!valid_format(fmt) || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    const bool scaled = is_scaled(fmt);
    if (n && (!g || !w_send || !codes || (scaled && !scales))) return SDL_ERR_INVALID_ARG;
    if (n == 0) return SDL_OK;
    Args a;
    std::memset(&a, 0, sizeof(a));
    a.g = const_cast<float*>(g);
    a.M = M;
    Align al;
    al.add_model(g);
    if (!aligned(g, 4)) return SDL_ERR_ALIGNMENT;
    for (uint32_t m = 0; m < M; ++m) {
        if (!w_send[m] || !codes[m] || (scaled && !scales[m])) return SDL_ERR_INVALID_ARG;
        if (!aligned(w_send[m], 2) || !aligned(codes[m], code_align(fmt))) return SDL_ERR_ALIGNMENT;
        if (scaled && !aligned(scales[m], scale_align(fmt))) return SDL_ERR_ALIGNMENT;
        al.add_model(w_send[m]);
        al.msg = al.msg && aligned(codes[m], 16);
        a.w_send[m] = static_cast<const uint16_t*>(w_send[m]);
        a.codes[m] = static_cast<uint8_t*>(codes[m]);
        a.scales[m] = scaled ? static_cast<uint8_t*>(scales[m]) : nullptr;
    }
    return run_single_span<kQuantize>(a, n, fmt, al, stream);
}

int sdl_dequant_reduce_nesterov(float* g, float* mom, const void* const* codes,
                                const void* const* scales, uint32_t M, uint64_t n, sdl_format_t fmt,
                                float lr, float mu, void* stream)
{
    if (!valid_format(fmt) || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    const bool scaled = is_scaled(fmt);
    if (n && (!g || !mom || !codes || (scaled && !scales))) return SDL_ERR_INVALID_ARG;
    if (n == 0) return SDL_OK;
    if (!aligned(g, 4) || !aligned(mom, 4)) return SDL_ERR_ALIGNMENT;
    Args a;
    std::memset(&a, 0, sizeof(a));
    a.g = g; a.mom = mom; a.M = M; a.lr = lr; a.mu = mu;
    Align al;
    al.add_model(g);
    al.add_model(mom);
    for (uint32_t m = 0; m < M; ++m) {
        if (!codes[m] || (scaled && !scales[m])) return SDL_ERR_INVALID_ARG;
        if (!aligned(codes[m], code_align(fmt))) return SDL_ERR_ALIGNMENT;
        if (scaled && !aligned(scales[m], scale_align(fmt))) return SDL_ERR_ALIGNMENT;
        al.msg = al.msg && aligned(codes[m], 16);
        a.codes[m] = static_cast<uint8_t*>(const_cast<void*>(codes[m]));
        a.scales[m] = scaled ? static_cast<uint8_t*>(const_cast<void*>(scales[m])) : nullptr;
    }
    return run_single_span<kReduce>(a, n, fmt, al, stream);
}

// Argument marshalling shared by the receive-side calls that also merge.
static int fill_receive_args(Args& a, float* g, float* mom, const void* const* codes, const void* const* scales,
                             void* const* w_now, uint32_t M, sdl_format_t fmt, float lr, float mu, float alpha,
                             Align* al)
{
    if (!valid_format(fmt) || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    const bool scaled = is_scaled(fmt);
    if (!g || !mom || !codes || !w_now || (scaled && !scales)) return SDL_ERR_INVALID_ARG;
    if (!aligned(g, 4) || !aligned(mom, 4)) return SDL_ERR_ALIGNMENT;
    std::memset(&a, 0, sizeof(a));
    a.g = g; a.mom = mom; a.M = M; a.lr = lr; a.mu = mu; a.alpha = alpha; a.one_minus_alpha = 1.0f - alpha;
    *al = Align{};
    al->add_model(g);
    al->add_model(mom);
    for (uint32_t m = 0; m < M; ++m) {
        if (!codes[m] || !w_now[m] || (scaled && !scales[m])) return SDL_ERR_INVALID_ARG;
        if (!aligned(codes[m], code_align(fmt)) || !aligned(w_now[m], 2)) return SDL_ERR_ALIGNMENT;
        if (scaled && !aligned(scales[m], scale_align(fmt))) return SDL_ERR_ALIGNMENT;
        al->add_model(w_now[m]);
        al->msg = al->msg && aligned(codes[m], 16);
        a.codes[m] = static_cast<uint8_t*>(const_cast<void*>(codes[m]));
        a.scales[m] = scaled ? static_cast<uint8_t*>(const_cast<void*>(scales[m])) : nullptr;
        a.w_now[m] = static_cast<uint16_t*>(w_now[m]);
    }
    return SDL_OK;
}

int sdl_receive_outer_step(float* g, float* mom, const void* const* codes, const void* const* scales,
                           void* const* w_now, uint32_t M, uint64_t n, sdl_format_t fmt, float lr, float mu,
                           float alpha, void* stream)
{
    if (n == 0) return (valid_format(fmt) && M >= 1 && M <= SDL_MAX_WORKERS) ? SDL_OK : SDL_ERR_INVALID_ARG;
    Args a;
    Align al;
    int rc = fill_receive_args(a, g, mom, codes, scales, w_now, M, fmt, lr, mu, alpha, &al);
    if (rc != SDL_OK) return rc;
    return run_single_span<kReceive>(a, n, fmt, al, stream);
}

int sdl_merge_overlap(const float* g_new, void* const* w_now, uint32_t M, uint64_t n, float alpha,
                      void* stream)
{
    if (M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    if (n && (!g_new || !w_now)) return SDL_ERR_INVALID_ARG;
    if (n == 0) return SDL_OK;
    if (!aligned(g_new, 4)) return SDL_ERR_ALIGNMENT;
    Args a;
    std::memset(&a, 0, sizeof(a));
    a.g = const_cast<float*>(g_new); a.M = M; a.alpha = alpha; a.one_minus_alpha = 1.0f - alpha;
    Align al;
    al.add_model(g_new);
    for (uint32_t m = 0; m < M; ++m) {
        if (!w_now[m]) return SDL_ERR_INVALID_ARG;
        if (!aligned(w_now[m], 2)) return SDL_ERR_ALIGNMENT;
        al.add_model(w_now[m]);
        a.w_now[m] = static_cast<uint16_t*>(w_now[m]);
    }
    return run_single_span<kMerge>(a, n, SDL_FMT_FP32, al, stream);
}

// Shared argument marshalling of the two fused entry points.
static int fill_fused_args(Args& a, float* g, float* mom, const void* const* w_send, void* const* w_now,
                           uint32_t M, sdl_format_t fmt, float lr, float mu, float alpha, Align* al)
{
    if (!valid_format(fmt) || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    if (!g || !mom || !w_send || !w_now) return SDL_ERR_INVALID_ARG;
    if (!aligned(g, 4) || !aligned(mom, 4)) return SDL_ERR_ALIGNMENT;
    std::memset(&a, 0, sizeof(a));
    a.g = g; a.mom = mom; a.M = M; a.lr = lr; a.mu = mu; a.alpha = alpha;
    a.one_minus_alpha = 1.0f - alpha;
    *al = Align{};
    al->add_model(g);
    al->add_model(mom);
    uint32_t same = 0;
    for (uint32_t m = 0; m < M; ++m) {
        if (!w_send[m] || !w_now[m]) return SDL_ERR_INVALID_ARG;
        if (!aligned(w_send[m], 2) || !aligned(w_now[m], 2)) return SDL_ERR_ALIGNMENT;
        al->add_model(w_send[m]);
        al->add_model(w_now[m]);
        same += (w_send[m] == w_now[m]);
        a.w_send[m] = static_cast<const uint16_t*>(w_send[m]);
        a.w_now[m] = static_cast<uint16_t*>(w_now[m]);
    }
    if (same != 0 && same != M) return SDL_ERR_INVALID_ARG;   // alias all replicas or none
    a.aliased = same == M;
    return SDL_OK;
}

// Optional message outputs of a fused call; the whole-span scale needs its scale words as
// workspace even when no message is written.
static int attach_fused_messages(Args& a, uint32_t M, sdl_format_t fmt, void* const* codes_or_null,
                                 void* const* scales_or_null, Align* al)
{
    if (codes_or_null) {
        const bool scaled = is_scaled(fmt);
        if (scaled && !scales_or_null) return SDL_ERR_INVALID_ARG;
        for (uint32_t m = 0; m < M; ++m) {
            if (!codes_or_null[m] || (scaled && !scales_or_null[m])) return SDL_ERR_INVALID_ARG;
            if (!aligned(codes_or_null[m], code_align(fmt))) return SDL_ERR_ALIGNMENT;
            al->msg = al->msg && aligned(codes_or_null[m], 16);
            a.codes[m] = static_cast<uint8_t*>(codes_or_null[m]);
            a.scales[m] = scaled ? static_cast<uint8_t*>(scales_or_null[m]) : nullptr;
        }
        a.emit = 1;
    }
    if (is_span_scaled(fmt)) {
        if (!scales_or_null) return SDL_ERR_INVALID_ARG;
        for (uint32_t m = 0; m < M; ++m) {
            if (!scales_or_null[m]) return SDL_ERR_INVALID_ARG;
            if (!aligned(scales_or_null[m], 4)) return SDL_ERR_ALIGNMENT;
            a.scales[m] = static_cast<uint8_t*>(scales_or_null[m]);
        }
    }
    return SDL_OK;
}

int sdl_fragment_outer_step(float* g, float* mom, const void* const* w_send, void* const* w_now,
                            uint32_t M, uint64_t n, sdl_format_t fmt, float lr, float mu, float alpha,
                            void* const* codes_or_null, void* const* scales_or_null, void* stream)
{
    if (n == 0) return (valid_format(fmt) && M >= 1 && M <= SDL_MAX_WORKERS) ? SDL_OK : SDL_ERR_INVALID_ARG;
    Args a;
    Align al;
    int rc = fill_fused_args(a, g, mom, w_send, w_now, M, fmt, lr, mu, alpha, &al);
    if (rc != SDL_OK) return rc;
    rc = attach_fused_messages(a, M, fmt, codes_or_null, scales_or_null, &al);
    if (rc != SDL_OK) return rc;
    return run_single_span<kFused>(a, n, fmt, al, stream);
}

}  // extern "C"

// The pieces of fragment p that one call processes, in model order: the joined runs, or, for the
// whole-span scale, the spans themselves (one scale word per parameter group).  Yields, for every
// non-empty piece, where it lies in the flat arrays, in the message arrays (pieces back to back,
// each padded to whole tiles) and in staged g / mom (the fragment's runs back to back, each padded
// to whole tiles).  Holds no storage of its own: the callers walk it once per pass.
struct PieceWalk {
    struct Piece { uint64_t offset, numel, msg, soff; Align al; uint32_t sidx; };
    const sdl_span_t* runs;
    const sdl_span_t* pieces;
    uint32_t n_runs, n_pieces;
    Align al;
    bool staged;
    uint32_t i = 0, run_i = 0;
    uint64_t msg = 0, run_start = 0;

    bool next(Piece* out)
    {
        for (; i < n_pieces; ++i) {
            if (pieces[i].numel == 0) continue;
            // the run that contains this piece, and where that run starts in the staged arrays
            while (run_i < n_runs && pieces[i].offset >= runs[run_i].offset + runs[run_i].numel) {
                run_start += (runs[run_i].numel + kPad - 1) / kPad * kPad;
                ++run_i;
            }
            const uint64_t soff = run_i < n_runs ? run_start + (pieces[i].offset - runs[run_i].offset) : 0;
            const Align piece_al = al.at(pieces[i].offset, staged ? soff : pieces[i].offset);
            *out = Piece{pieces[i].offset, pieces[i].numel, msg, soff, piece_al, i};
            msg += (pieces[i].numel + kPad - 1) / kPad * kPad;
            ++i;
            return true;
        }
        return false;
    }
};

// One mode over all runs of fragment p, on flat model arrays; the fragment's messages are
// the concatenation of its runs, each padded to a multiple of 512 elements.  No host or device
// memory is allocated on the way.
template <int MODE>
static int launch_fragment(Args& a, const sdl_plan_t* plan, uint32_t p, Align al, sdl_format_t fmt, void* stream)
{
    const sdl_span_t* runs = nullptr;
    const sdl_span_t* pieces = nullptr;
    uint32_t n_runs = 0, n_pieces = 0;
    int rc = sdl_plan_fragment_runs(plan, p, &runs, &n_runs);
    if (rc != SDL_OK) return rc;
    if (is_span_scaled(fmt) && MODE != kMerge) rc = sdl_plan_fragment_spans(plan, p, &pieces, &n_pieces);
    else { pieces = runs; n_pieces = n_runs; }
    if (rc != SDL_OK) return rc;
    const PieceWalk start{runs, pieces, n_runs, n_pieces, al, a.staged != 0u};
    PieceWalk::Piece pc;
    const uint32_t tile = tile_elems(MODE, a, fmt);
    {
        // refused before anything is launched: a fragment of which 16 consecutive pieces need more than 2^31 - 1 workgroups.  (Launches
        // are cut to the grid's limit by themselves, see RunBuilder::fits.)
        PieceWalk walk = start;
        uint64_t n_wg = 0;
        for (uint32_t in_group = 0; walk.next(&pc);) {
            n_wg += (pc.numel + tile - 1) / tile;
            if (n_wg > 0x7fffffffull) return SDL_ERR_UNSUPPORTED;
            if (++in_group == (uint32_t)kCheckedRuns) { in_group = 0; n_wg = 0; }
        }
    }
    {
        // the replicas are flat model arrays; g / mom too, unless they are a staging buffer of this fragment
        size_t cb = 0, sb = 0;
        if (MODE != kMerge) {
            rc = sdl_plan_message_bytes(plan, p, fmt, &cb, &sb);
            if (rc != SDL_OK) return rc;
        }
        const uint64_t model = sdl_plan_total_numel(plan);
        if (arrays_clash<MODE>(a, fmt, model, a.staged ? sdl_plan_staged_numel(plan, p) : model, cb, sb))
            return SDL_ERR_INVALID_ARG;
    }
    if (is_span_scaled(fmt) && (MODE == kQuantize || MODE == kFused)) {
        // whole-span scale: clear the scale words, take the grid-wide maxima, then encode
        SpanRun batch[kAbsmaxMaxRuns];
        uint32_t nb = 0;
        PieceWalk walk = start;
        for (bool more = walk.next(&pc); more || nb;) {
            if (more) batch[nb++] = SpanRun{pc.offset, pc.numel, pc.soff, pc.al.wide, pc.sidx};
            more = more && walk.next(&pc);
            if (nb == (uint32_t)kAbsmaxMaxRuns || !more) {
                if (launch_span_prepass(a, batch, nb, (hipStream_t)stream) != hipSuccess) return SDL_ERR_DEVICE;
                nb = 0;
            }
        }
    }
    RunBuilder rb(&a, MODE, tile, fmt);
    PieceWalk walk = start;
    while (walk.next(&pc))
        if (!add_piece<MODE>(rb, fmt, pc.offset, pc.numel, pc.al, pc.msg, pc.sidx, pc.soff, stream)) return SDL_ERR_DEVICE;
    if (!flush<MODE>(rb, fmt, stream)) return SDL_ERR_DEVICE;
    return SDL_OK;
}

extern "C" {

int sdl_plan_message_bytes(const sdl_plan_t* plan, uint32_t p, sdl_format_t fmt, size_t* code_bytes,
                           size_t* scale_bytes)
{
    if (!valid_format(fmt)) return SDL_ERR_INVALID_ARG;
    const sdl_span_t* runs = nullptr;
    uint32_t n_runs = 0;
    int rc = is_span_scaled(fmt) ? sdl_plan_fragment_spans(plan, p, &runs, &n_runs)
                                 : sdl_plan_fragment_runs(plan, p, &runs, &n_runs);
    if (rc != SDL_OK) return rc;
    uint64_t padded = 0;
    for (uint32_t i = 0; i < n_runs; ++i) padded += (runs[i].numel + kPad - 1) / kPad * kPad;
    sdl_exchange_bytes(fmt, padded, code_bytes, scale_bytes);
    if (is_span_scaled(fmt) && scale_bytes) *scale_bytes = (size_t)n_runs * 4;   // one word per span
    return SDL_OK;
}

static int fused_fragment(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                          const void* const* w_send_base, void* const* w_now_base, uint32_t M,
                          sdl_format_t fmt, float lr, float mu, float alpha, void* const* codes_or_null,
                          void* const* scales_or_null, void* stream, bool staged)
{
    if (!plan || p >= sdl_plan_num_fragments(plan)) return SDL_ERR_INVALID_ARG;
    // the whole-span scale needs scale words as workspace: only the calls that take them support it
    if (valid_format(fmt) && is_span_scaled(fmt) && !scales_or_null) return SDL_ERR_UNSUPPORTED;
    Args a;
    Align al;
    int rc = fill_fused_args(a, g_base, mom_base, w_send_base, w_now_base, M, fmt, lr, mu, alpha, &al);
    if (rc != SDL_OK) return rc;
    rc = attach_fused_messages(a, M, fmt, codes_or_null, scales_or_null, &al);
    if (rc != SDL_OK) return rc;
    a.staged = staged ? 1u : 0u;
    return launch_fragment<kFused>(a, plan, p, al, fmt, stream);
}

static int quantize_fragment(const sdl_plan_t* plan, uint32_t p, const float* g_base,
                             const void* const* w_send_base, uint32_t M, sdl_format_t fmt,
                             void* const* codes, void* const* scales, void* stream, bool staged)
{
    if (!plan || p >= sdl_plan_num_fragments(plan)) return SDL_ERR_INVALID_ARG;
    if (!valid_format(fmt) || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    const bool scaled = is_scaled(fmt);
    if (!g_base || !w_send_base || !codes || (scaled && !scales)) return SDL_ERR_INVALID_ARG;
    if (!aligned(g_base, 4)) return SDL_ERR_ALIGNMENT;
    Args a;
    std::memset(&a, 0, sizeof(a));
    a.g = const_cast<float*>(g_base);
    a.M = M;
    Align al;
    al.add_model(g_base);
    for (uint32_t m = 0; m < M; ++m) {
        if (!w_send_base[m] || !codes[m] || (scaled && !scales[m])) return SDL_ERR_INVALID_ARG;
        if (!aligned(w_send_base[m], 2) || !aligned(codes[m], code_align(fmt))) return SDL_ERR_ALIGNMENT;
        if (scaled && !aligned(scales[m], scale_align(fmt))) return SDL_ERR_ALIGNMENT;
        al.add_model(w_send_base[m]);
        al.msg = al.msg && aligned(codes[m], 16);
        a.w_send[m] = static_cast<const uint16_t*>(w_send_base[m]);
        a.codes[m] = static_cast<uint8_t*>(codes[m]);
        a.scales[m] = scaled ? static_cast<uint8_t*>(scales[m]) : nullptr;
    }
    a.staged = staged ? 1u : 0u;
    return launch_fragment<kQuantize>(a, plan, p, al, fmt, stream);
}

static int reduce_fragment(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                           const void* const* codes, const void* const* scales, uint32_t M,
                           sdl_format_t fmt, float lr, float mu, void* stream, bool staged)
{
    if (!plan || p >= sdl_plan_num_fragments(plan)) return SDL_ERR_INVALID_ARG;
    if (!valid_format(fmt) || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    const bool scaled = is_scaled(fmt);
    if (!g_base || !mom_base || !codes || (scaled && !scales)) return SDL_ERR_INVALID_ARG;
    if (!aligned(g_base, 4) || !aligned(mom_base, 4)) return SDL_ERR_ALIGNMENT;
    Args a;
    std::memset(&a, 0, sizeof(a));
    a.g = g_base; a.mom = mom_base; a.M = M; a.lr = lr; a.mu = mu;
    Align al;
    al.add_model(g_base);
    al.add_model(mom_base);
    for (uint32_t m = 0; m < M; ++m) {
        if (!codes[m] || (scaled && !scales[m])) return SDL_ERR_INVALID_ARG;
        if (!aligned(codes[m], code_align(fmt))) return SDL_ERR_ALIGNMENT;
        if (scaled && !aligned(scales[m], scale_align(fmt))) return SDL_ERR_ALIGNMENT;
        al.msg = al.msg && aligned(codes[m], 16);
        a.codes[m] = static_cast<uint8_t*>(const_cast<void*>(codes[m]));
        a.scales[m] = scaled ? static_cast<uint8_t*>(const_cast<void*>(scales[m])) : nullptr;
    }
    a.staged = staged ? 1u : 0u;
    return launch_fragment<kReduce>(a, plan, p, al, fmt, stream);
}

static int receive_fragment(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                            const void* const* codes, const void* const* scales, void* const* w_now_base,
                            uint32_t M, sdl_format_t fmt, float lr, float mu, float alpha, void* stream, bool staged)
{
    if (!plan || p >= sdl_plan_num_fragments(plan)) return SDL_ERR_INVALID_ARG;
    Args a;
    Align al;
    int rc = fill_receive_args(a, g_base, mom_base, codes, scales, w_now_base, M, fmt, lr, mu, alpha, &al);
    if (rc != SDL_OK) return rc;
    a.staged = staged ? 1u : 0u;
    return launch_fragment<kReceive>(a, plan, p, al, fmt, stream);
}

static int merge_fragment(const sdl_plan_t* plan, uint32_t p, const float* g_new_base, void* const* w_now_base,
                          uint32_t M, float alpha, void* stream, bool staged)
{
    if (!plan || p >= sdl_plan_num_fragments(plan)) return SDL_ERR_INVALID_ARG;
    if (M == 0 || M > SDL_MAX_WORKERS || !g_new_base || !w_now_base) return SDL_ERR_INVALID_ARG;
    if (!aligned(g_new_base, 4)) return SDL_ERR_ALIGNMENT;
    Args a;
    std::memset(&a, 0, sizeof(a));
    a.g = const_cast<float*>(g_new_base); a.M = M; a.alpha = alpha; a.one_minus_alpha = 1.0f - alpha;
    Align al;
    al.add_model(g_new_base);
    for (uint32_t m = 0; m < M; ++m) {
        if (!w_now_base[m]) return SDL_ERR_INVALID_ARG;
        if (!aligned(w_now_base[m], 2)) return SDL_ERR_ALIGNMENT;
        al.add_model(w_now_base[m]);
        a.w_now[m] = static_cast<uint16_t*>(w_now_base[m]);
    }
    a.staged = staged ? 1u : 0u;
    return launch_fragment<kMerge>(a, plan, p, al, SDL_FMT_FP32, stream);
}


int sdl_fragment_outer_step_plan(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                                 const void* const* w_send_base, void* const* w_now_base, uint32_t M,
                                 sdl_format_t fmt, float lr, float mu, float alpha, void* stream)
{
    return fused_fragment(plan, p, g_base, mom_base, w_send_base, w_now_base, M, fmt, lr, mu, alpha, nullptr, nullptr,
                          stream, false);
}
int sdl_fragment_outer_step_plan_ex(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                                    const void* const* w_send_base, void* const* w_now_base, uint32_t M,
                                    sdl_format_t fmt, float lr, float mu, float alpha, void* const* codes_or_null,
                                    void* const* scales_or_null, void* stream)
{
    return fused_fragment(plan, p, g_base, mom_base, w_send_base, w_now_base, M, fmt, lr, mu, alpha, codes_or_null,
                          scales_or_null, stream, false);
}

// Device address of `scratch` on the current device, looked up once per device.
static int static_scratch(uint32_t** out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mutex;
    static uint32_t* address[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SDL_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(mutex);
    if (!address[dev]) {
        uint32_t* ptr = nullptr;
        if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SDL_ERR_DEVICE;
        address[dev] = ptr;
    }
    *out = address[dev];
    return SDL_OK;
}

int sdl_fragment_outer_step_plan_static(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                                        const void* const* w_send_base, void* const* w_now_base, uint32_t M,
                                        sdl_format_t fmt, float lr, float mu, float alpha, void* stream)
{
    if (!plan || p >= sdl_plan_num_fragments(plan)) return SDL_ERR_INVALID_ARG;
    if (!valid_format(fmt) || M == 0 || M > SDL_MAX_WORKERS) return SDL_ERR_INVALID_ARG;
    if (!is_span_scaled(fmt))   // no other format needs memory beyond the model arrays
        return fused_fragment(plan, p, g_base, mom_base, w_send_base, w_now_base, M, fmt, lr, mu, alpha, nullptr,
                              nullptr, stream, false);
    const sdl_span_t* spans = nullptr;
    uint32_t n_spans = 0;
    int rc = sdl_plan_fragment_spans(plan, p, &spans, &n_spans);
    if (rc != SDL_OK) return rc;
    if (n_spans > SDL_STATIC_MAX_SPANS) return SDL_ERR_TOO_LARGE;
    uint32_t* base = nullptr;
    rc = static_scratch(&base);
    if (rc != SDL_OK) return rc;
    void* words[SDL_MAX_WORKERS];
    for (uint32_t m = 0; m < M; ++m) words[m] = base + (size_t)m * SDL_STATIC_MAX_SPANS;
    // the pre-pass clears the words of the fragment's spans with a fill kernel before it takes the
    // maxima, so what an earlier call left in the array does not matter
    return fused_fragment(plan, p, g_base, mom_base, w_send_base, w_now_base, M, fmt, lr, mu, alpha, nullptr, words,
                          stream, false);
}

int sdl_quantize_outer_grad_plan(const sdl_plan_t* plan, uint32_t p, const float* g_base,
                                 const void* const* w_send_base, uint32_t M, sdl_format_t fmt,
                                 void* const* codes, void* const* scales, void* stream)
{
    return quantize_fragment(plan, p, g_base, w_send_base, M, fmt, codes, scales, stream, false);
}
int sdl_dequant_reduce_nesterov_plan(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                                     const void* const* codes, const void* const* scales, uint32_t M,
                                     sdl_format_t fmt, float lr, float mu, void* stream)
{
    return reduce_fragment(plan, p, g_base, mom_base, codes, scales, M, fmt, lr, mu, stream, false);
}
int sdl_merge_overlap_plan(const sdl_plan_t* plan, uint32_t p, const float* g_new_base, void* const* w_now_base,
                           uint32_t M, float alpha, void* stream)
{
    return merge_fragment(plan, p, g_new_base, w_now_base, M, alpha, stream, false);
}

int sdl_receive_outer_step_plan(const sdl_plan_t* plan, uint32_t p, float* g_base, float* mom_base,
                                const void* const* codes, const void* const* scales, void* const* w_now_base,
                                uint32_t M, sdl_format_t fmt, float lr, float mu, float alpha, void* stream)
{
    return receive_fragment(plan, p, g_base, mom_base, codes, scales, w_now_base, M, fmt, lr, mu, alpha, stream, false);
}
int sdl_receive_outer_step_staged(const sdl_plan_t* plan, uint32_t p, float* g_frag, float* mom_frag,
                                  const void* const* codes, const void* const* scales, void* const* w_now_base,
                                  uint32_t M, sdl_format_t fmt, float lr, float mu, float alpha, void* stream)
{
    return receive_fragment(plan, p, g_frag, mom_frag, codes, scales, w_now_base, M, fmt, lr, mu, alpha, stream, true);
}

uint64_t sdl_plan_staged_numel(const sdl_plan_t* plan, uint32_t p)
{
    const sdl_span_t* runs = nullptr;
    uint32_t n_runs = 0;
    if (sdl_plan_fragment_runs(plan, p, &runs, &n_runs) != SDL_OK) return 0;
    uint64_t padded = 0;
    for (uint32_t i = 0; i < n_runs; ++i) padded += (runs[i].numel + kPad - 1) / kPad * kPad;
    return padded;
}
int sdl_fragment_outer_step_staged(const sdl_plan_t* plan, uint32_t p, float* g_frag, float* mom_frag,
                                   const void* const* w_send_base, void* const* w_now_base, uint32_t M,
                                   sdl_format_t fmt, float lr, float mu, float alpha, void* stream)
{
    return fused_fragment(plan, p, g_frag, mom_frag, w_send_base, w_now_base, M, fmt, lr, mu, alpha, nullptr, nullptr,
                          stream, true);
}
int sdl_fragment_outer_step_staged_ex(const sdl_plan_t* plan, uint32_t p, float* g_frag, float* mom_frag,
                                      const void* const* w_send_base, void* const* w_now_base, uint32_t M,
                                      sdl_format_t fmt, float lr, float mu, float alpha, void* const* codes_or_null,
                                      void* const* scales_or_null, void* stream)
{
    return fused_fragment(plan, p, g_frag, mom_frag, w_send_base, w_now_base, M, fmt, lr, mu, alpha, codes_or_null,
                          scales_or_null, stream, true);
}
int sdl_quantize_outer_grad_staged(const sdl_plan_t* plan, uint32_t p, const float* g_frag,
                                   const void* const* w_send_base, uint32_t M, sdl_format_t fmt,
                                   void* const* codes, void* const* scales, void* stream)
{
    return quantize_fragment(plan, p, g_frag, w_send_base, M, fmt, codes, scales, stream, true);
}
int sdl_dequant_reduce_nesterov_staged(const sdl_plan_t* plan, uint32_t p, float* g_frag, float* mom_frag,
                                       const void* const* codes, const void* const* scales, uint32_t M,
                                       sdl_format_t fmt, float lr, float mu, void* stream)
{
    return reduce_fragment(plan, p, g_frag, mom_frag, codes, scales, M, fmt, lr, mu, stream, true);
}
int sdl_merge_overlap_staged(const sdl_plan_t* plan, uint32_t p, const float* g_new_frag, void* const* w_now_base,
                             uint32_t M, float alpha, void* stream)
{
    return merge_fragment(plan, p, g_new_frag, w_now_base, M, alpha, stream, true);
}

int sdl_memory_probe(sdl_probe_t kind, void* dst, const void* src, uint64_t nbytes, void* stream)
{
    if (kind < SDL_PROBE_COPY || kind > SDL_PROBE_FILL_NT) return SDL_ERR_INVALID_ARG;
    if (nbytes == 0) return SDL_OK;
    if (!dst || (!src && kind != SDL_PROBE_FILL_NT) || nbytes % 16 != 0) return SDL_ERR_INVALID_ARG;
    if (!aligned(dst, 16) || !aligned(src, 16)) return SDL_ERR_ALIGNMENT;
    const uint64_t n16 = nbytes / 16, n_wg = (n16 + kCopyThreads - 1) / kCopyThreads;
    if (n_wg > 0x7fffffffull) return SDL_ERR_UNSUPPORTED;
    const dim3 grid((uint32_t)n_wg), block(kCopyThreads);
    hipStream_t s = (hipStream_t)stream;
    u32x4* d = static_cast<u32x4*>(dst);
    const u32x4* r = static_cast<const u32x4*>(src);
    switch (kind) {
    case SDL_PROBE_COPY:
        hipLaunchKernelGGL(sdl_copy_kernel, grid, block, 0, s, static_cast<uint4*>(dst), static_cast<const uint4*>(src), n16);
        break;
    case SDL_PROBE_COPY_NT: hipLaunchKernelGGL((sdl_probe_kernel<SDL_PROBE_COPY_NT>), grid, block, 0, s, d, r, n16); break;
    case SDL_PROBE_READ_NT: hipLaunchKernelGGL((sdl_probe_kernel<SDL_PROBE_READ_NT>), grid, block, 0, s, d, r, n16); break;
    default: hipLaunchKernelGGL((sdl_probe_kernel<SDL_PROBE_FILL_NT>), grid, block, 0, s, d, r, n16); break;
    }
    return hipGetLastError() == hipSuccess ? SDL_OK : SDL_ERR_DEVICE;
}

int sdl_copy_bytes(void* dst, const void* src, uint64_t nbytes, void* stream)
{
    return sdl_memory_probe(SDL_PROBE_COPY, dst, src, nbytes, stream);
}

}  // extern "C"
