// Multi-block tile passes: a sequence of fused blocks of <= 4 qubits applied
// to a state in ONE read and ONE write of HBM.
//
// The blocks of a pass act on a union U of at most TB positions.  A tile is
// the 2^TB amplitudes (TB = 13 or 14: 64 or 128 KiB of complex64 in LDS)
// spanned by U plus the lowest TB - |U| positions outside U (tile bit b <->
// position u_b, ascending), so it is made of contiguous runs of at least
// 2^(TB - |U|) amplitudes, longer when U holds low positions.  For every value of the remaining n - TB bits there
// is one tile; tiles are copied in and out with 16-byte accesses along those
// runs (tile bit 0 is always position 0).
//
// Inside the tile, block s (4 positions at tile bits t_s0 < .. < t_s3) is a
// complex GEMM Y = U_s X with X viewed as 16 rows (the block's tile bits) x
// 2^(TB-4) columns (the other tile bits): one MFMA chain per 32-column block,
// the real form A' = [[Ur,-Ui],[Ui,Ur]] interleaved by (re, im) as the A
// operand.  The operands of all blocks of the pass, expanded into each
// lane's A' fragments, and their column address tables are staged into LDS
// once per workgroup next to the tile.
// B operands and results are addressed in LDS as row(j) XOR column(c) (bit
// deposits, then an XOR swizzle against bank conflicts).  Each wave owns
// whole columns, so blocks update the tile in place with one barrier between
// blocks.
#include <hip/hip_runtime.h>

#include <cstring>
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace sv {
namespace dev {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float vf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Arithmetic of a tile pass: split products in BF16 or FP16 with FP32
// accumulation.  FP32 and BF16X3 passes run the same kernels (kPrecX3): three
// BF16 parts of the matrix and of the state, six products, which is closer to
// 64-bit values than FP32 MFMA (whose sums round 32 times) and does a block in
// 2.8 instead of 5.0 us per tile.
constexpr int kPrecX3 = kTileOperandF32, kPrecBF16 = kTileOperandBF16, kPrecF16 = kTileOperandF16;
// FP64 passes of complex128 states run the same tile loop: n qubits of
// complex128 lie in memory as n + 1 of complex64 whose position 0 chooses
// between re and im, so layouts, tiles (2^13 amplitudes) and 16-byte copies
// carry over; only the block arithmetic is their own (apply_block_f64).
constexpr int kPrecF64 = kTileOperandF64;
// Gate passes (apply_stage) in the same tile loop.
constexpr int kPrecGates32 = kTileOperandF64 + 1, kPrecGates64 = kTileOperandF64 + 2;

// LDS words per lane of one block's operand (the A' fragments of the 64
// lanes): 8 per matrix part where every part is expanded at staging, so that
// the block loop reads it as it is (FP16: two parts, BF16: three).  X3 expands
// the first part only and keeps the two others compact (4 words a lane each,
// expanded when read), so that as many blocks share a launch as with FP16;
// launches of fewer blocks have room for 24 words a lane (x3_whole).
constexpr int lane_words(int prec) { return prec == kPrecBF16 ? 24 : 16; }

// Where a lane's 16-byte chunk of X3's parts sits (words into the operand).
// The XORs put the chunks that one LDS access reads (8 lanes over 32 banks,
// 16 over 64) on distinct banks; the two lanes of a complex row read the same
// compact chunk.
__device__ __forceinline__ uint32_t x3_expanded_at(uint32_t lane, uint32_t i)
{
    return lane * 8 + 4 * (i ^ (((lane >> 2) ^ (lane >> 3)) & 1u));
}
// FP64 operands: entry (ci, j) of U sits at complex slot 16 ci + (j ^ f64_operand_swz(ci)),
// so that the eight rows and two columns of one access hit distinct banks.
__host__ __device__ constexpr uint32_t f64_operand_swz(uint32_t ci) { return 2u * (ci & 7u); }

template <class C>
__host__ __device__ constexpr bool x3_whole(int n_sub)
{
    return n_sub * 64 * 24 <= C::OP_AREA;
}
__device__ __forceinline__ uint32_t x3_compact_at(uint32_t part, uint32_t ci, uint32_t c)
{
    return 512 + (part - 1) * 256 + ci * 16 + 4 * (c ^ ((ci >> 1) & 3u));
}

// 16-byte chunk c of lane L's fragments sits at chunk c ^ frag_swz<LW>(L) of
// its LW words.  With 64-byte lanes (LW = 16) the lanes of one 16-byte LDS
// access (8 over 32 banks, or 16 over 64) would otherwise meet four to a
// bank group; the XOR with lane bits (1 ^ 3, 2) puts them on distinct banks.
// The 96-byte lanes of split BF16 (two to a group) stay in order: the same
// XOR there (lane bits 2 ^ 3) costs those kernels register spills.
template <int LW>
__device__ __forceinline__ uint32_t frag_swz(uint32_t lane)
{
    if constexpr (LW == 16) return (((lane >> 1) ^ (lane >> 3)) & 1u) | ((lane >> 1) & 2u);
    return 0u;
}

// Tile of 2^TB amplitudes held by a workgroup of WAVES waves: 2^TB / 16
// columns per 4-qubit block, in blocks of 32 split evenly over the waves.
// Shapes: (14, 8) and (14, 16) one 128 KiB tile per CU, with 2 or 4 waves
// per SIMD; (13, 4) two 64 KiB workgroups per CU, so one can copy while the
// other computes; (13, 8).  (12, 4), (11, 2) and (10, 1): small states
// (tile_shape_for), the last two as one tile.  MAX_SUB blocks' operands of LW words per lane
// fit in the LDS left beside the tile.
template <int TB, int WAVES, int LW = 24>
struct TileCfg {
    static constexpr int N = 1 << TB;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int COLS = N / 16;
    static constexpr int CBLOCKS = COLS / 32;  // 32-column blocks
    static constexpr int NB_PER_WAVE = CBLOCKS / WAVES;
    static constexpr int CHUNKS = N / 2 / THREADS;  // 16-byte copies per thread
    static constexpr int TABLE_WORDS = CBLOCKS + 32;
    // two (13, 4) workgroups share a CU; the others hold the CU alone
    static constexpr int LDS_BUDGET = (TB == 13 && WAVES == 4) || TB <= 12 ? 160 * 1024 / 2 : 160 * 1024;
    static constexpr int OPERAND_WORDS = 64 * LW;
    static constexpr int FIT = (LDS_BUDGET - N * 8 - 8 * WAVES) / (4 * (OPERAND_WORDS + TABLE_WORDS));
    static constexpr int MAX_SUB = FIT < kMaxTileSubBlocks ? FIT : kMaxTileSubBlocks;
    // X3 (LW = 16) keeps all three parts expanded where the launch's blocks leave room
    static constexpr int OP_AREA = LW == 16 ? (LDS_BUDGET - N * 8 - 8 * WAVES - 4 * MAX_SUB * TABLE_WORDS) / 16 * 4
                                            : MAX_SUB * OPERAND_WORDS;
    static_assert(THREADS <= 1024 && NB_PER_WAVE >= 1 && OP_AREA >= MAX_SUB * OPERAND_WORDS,
                  "tile shape");
};

__device__ __forceinline__ uint32_t deposit(uint32_t v, uint32_t mask)
{
    // scatter the low bits of v into the set bits of mask (ascending)
    uint32_t r = 0;
    for (uint32_t m = mask; m; m &= m - 1) {
        const uint32_t low = m & (~m + 1);
        if (v & 1) r |= low;
        v >>= 1;
    }
    return r;
}

// LDS placement of tile index i: S(i), linear over XOR, with image a.swz[b]
// of tile bit b (chosen per pass on the host, choose_swizzle).  S keeps bit 0,
// so the pair (2t, 2t + 1) stays one aligned 16-byte slot for the HBM copies,
// and permutes the tile's indices.
__device__ __forceinline__ uint32_t swz(uint32_t i, const TileArgs &a)
{
    uint32_t r = 0;
#pragma unroll
    for (int b = 0; b < kMaxTileBits; ++b)
        if ((i >> b) & 1) r ^= a.swz[b];
    return r;
}

__device__ __forceinline__ uint64_t tile_base(uint64_t T, const TileArgs &a)
{
    // the tile index's bits go to the positions outside the tile, ascending
    uint64_t x = 0;
    for (int i = 0; i < a.n_ext; ++i) x |= ((T >> i) & 1) << a.ext_pos[i];
    return x;
}

template <int TB>
__device__ __forceinline__ uint64_t global_off(uint32_t t, const TileArgs &a)
{
    uint64_t g = 0;
#pragma unroll
    for (int b = 0; b < TB; ++b)
        if ((t >> b) & 1) g += uint64_t(1) << a.ubit[b];
    return g;
}

// Swizzled LDS index of complex row j (compile-time after unrolling) of a
// block: the XOR of the per-row-bit values rb[0..3].
__device__ __forceinline__ uint32_t row_of(const uint32_t *rb, int j)
{
    uint32_t r = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
        if ((j >> b) & 1) r ^= rb[b];
    return r;
}

// HBM <-> LDS copies of one tile: thread tid moves float4 slots
// tid + i * THREADS, i.e. tile indices 2 * slot and 2 * slot + 1.
template <int TB, int WAVES>
struct TileCopy {
    static constexpr int kChunks = TileCfg<TB, WAVES>::CHUNKS;
    static constexpr int kThreads = TileCfg<TB, WAVES>::THREADS;
    uint64_t g_lo;               // global offset of tile index 2 * tid
    uint64_t g_hi[kChunks];      // uniform: offset of tile index 2 * i * THREADS
    uint32_t lds_slot;           // float4 slot of tile index 2 * tid: S(2 tid) / 2
    uint32_t lds_hi[kChunks];    // uniform: S(2 i THREADS) / 2, XORed onto lds_slot

    __device__ __forceinline__ void init(const TileArgs &args, int tid)
    {
        g_lo = global_off<TB>(uint32_t(2 * tid), args);
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            g_hi[i] = global_off<TB>(uint32_t(2 * i * kThreads), args);
            lds_hi[i] = swz(uint32_t(2 * i * kThreads), args) >> 1;
        }
        lds_slot = swz(uint32_t(2 * tid), args) >> 1;
    }
    __device__ __forceinline__ void load(vf4 *buf, const float *psi, uint64_t base) const
    {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) buf[i] = *reinterpret_cast<const vf4 *>(psi + 2 * (base + g_lo + g_hi[i]));
    }
    // The same tile of a basis state, read from nowhere: zeros, and 1 at tile
    // index t when the basis state lies in this tile (`here`).  Thread tid's
    // chunk i holds tile indices 2 (tid + i THREADS) and the next one.
    // (F64: tile index t holds the real part, a double.)
    template <bool F64>
    __device__ __forceinline__ void basis(vf4 *buf, bool here, uint32_t t, int tid) const
    {
        const uint32_t pair = t >> 1;
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            buf[i] = vf4{0.f, 0.f, 0.f, 0.f};
            if (here && pair == uint32_t(tid) + uint32_t(i) * kThreads) {
                if (F64)
                    buf[i].y = __uint_as_float(0x3FF00000u);  // the high word of 1.0
                else if (t & 1u)
                    buf[i].z = 1.f;
                else
                    buf[i].x = 1.f;
            }
        }
    }
    // The same with a scale for the values in LDS (exact powers of two): LDS =
    // buf * scale, out = LDS * unscale.
    __device__ __forceinline__ void to_lds_scaled(vf4 *X4, const vf4 *buf, float scale) const
    {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) X4[lds_slot ^ lds_hi[i]] = buf[i] * scale;
    }
    __device__ __forceinline__ void store_scaled(float *psi, uint64_t base, const vf4 *X4, float unscale) const
    {
#pragma unroll
        for (int i = 0; i < kChunks; ++i)
            *reinterpret_cast<vf4 *>(psi + 2 * (base + g_lo + g_hi[i])) = X4[lds_slot ^ lds_hi[i]] * unscale;
    }
    __device__ __forceinline__ void swap_scaled(float *psi, uint64_t base_out, vf4 *X4, const vf4 *buf, float scale,
                                                float unscale) const
    {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const vf4 o = X4[lds_slot ^ lds_hi[i]];
            X4[lds_slot ^ lds_hi[i]] = buf[i] * scale;
            *reinterpret_cast<vf4 *>(psi + 2 * (base_out + g_lo + g_hi[i])) = o * unscale;
        }
    }
    // sum of the squares of the values in buf
    __device__ __forceinline__ float sum_sq(const vf4 *buf) const
    {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < kChunks; ++i)
            a += buf[i].x * buf[i].x + buf[i].y * buf[i].y + buf[i].z * buf[i].z + buf[i].w * buf[i].w;
        return a;
    }
    __device__ __forceinline__ void to_lds(vf4 *X4, const vf4 *buf) const
    {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) X4[lds_slot ^ lds_hi[i]] = buf[i];
    }
    __device__ __forceinline__ void store(float *psi, uint64_t base, const vf4 *X4) const
    {
#pragma unroll
        for (int i = 0; i < kChunks; ++i)
            *reinterpret_cast<vf4 *>(psi + 2 * (base + g_lo + g_hi[i])) = X4[lds_slot ^ lds_hi[i]];
    }
    // Each slot: store the finished tile's value (at base_out) and put the
    // next tile's value in its place.  The thread owns its slots, so no
    // barrier is needed between the two.
    __device__ __forceinline__ void swap(float *psi, uint64_t base_out, vf4 *X4, const vf4 *buf) const
    {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const vf4 o = X4[lds_slot ^ lds_hi[i]];
            X4[lds_slot ^ lds_hi[i]] = buf[i];
            *reinterpret_cast<vf4 *>(psi + 2 * (base_out + g_lo + g_hi[i])) = o;
        }
    }
    // largest magnitude of the values in buf
    __device__ __forceinline__ float max_abs(const vf4 *buf) const
    {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < kChunks; ++i)
            a = fmaxf(a, fmaxf(fmaxf(fabsf(buf[i].x), fabsf(buf[i].y)), fmaxf(fabsf(buf[i].z), fabsf(buf[i].w))));
        return a;
    }
};

// FP16 passes scale the tile's values by 2^e where they are split, e chosen
// from the tile's largest magnitude m (at copy-in) so that m 2^e lies in
// [2^7, 2^8), and scale the products back by 2^-e (exact powers of two).  The
// blocks act unitarily on the tile, so no value can grow beyond the tile's
// 2-norm, which is at most sqrt(2^15) m: every scaled value stays below
// 2^15.5 < 65504 (the FP16 parts stay finite) while values many binades below
// m stay in FP16's normal range.
__device__ __forceinline__ void tile_scale(float m, float &scale, float &unscale)
{
    scale = unscale = 1.f;
    if (m > 0.f && m <= 3.0e38f) {
        int e;
        frexpf(m, &e);  // m in [2^(e-1), 2^e)
        int s = 8 - e;
        s = s > 120 ? 120 : (s < -120 ? -120 : s);
        scale = ldexpf(1.f, s);
        unscale = ldexpf(1.f, -s);
    }
}

// A scale for a whole pass of FP16 products from the state's 2-norm r (the
// blocks keep it): 2^e with r 2^e in [2^14, 2^15), so that no value, being at
// most r in magnitude, exceeds 2^15 once scaled.  Scale 1 if r is 0 or not
// finite.
__device__ __forceinline__ void norm_scale(double r, float &scale, float &unscale)
{
    scale = unscale = 1.f;
    if (r > 0.0 && r <= 1e300) {
        int e;
        frexp(r, &e);  // r in [2^(e-1), 2^e)
        int s = 15 - e;
        s = s > 120 ? 120 : (s < -120 ? -120 : s);
        scale = ldexpf(1.f, s);
        unscale = ldexpf(1.f, -s);
    }
}

// Per-block data staged in LDS: the A operand and the swizzled column terms
// of lane l32 and column block cb = w NBW + q of wave w: cq[cb] ^ cl[l32].
// Column index c (deposited into the block's column bits, ascending):
// c = (32 w + l32) NBW + q, which puts q on the lowest column bits, so that
// when tile bit 0 is a column bit the column blocks q and q + 1 of a lane share
// one 16-byte slot.
template <int TB, int WAVES, int LW>
struct TileShared {
    using C = TileCfg<TB, WAVES, LW>;
    vf4 X4[C::N / 2];
    alignas(16) uint32_t op[C::OP_AREA];  // the blocks' operands, C::op_words(n_sub) apart
    uint32_t cq[C::MAX_SUB][C::CBLOCKS];
    uint32_t cl[C::MAX_SUB][32];
    float red[WAVES];  // per-wave partial of a tile's scale (FP16 passes)
    float nrm[WAVES];  // per-wave sum of squares read so far (FP16 passes that report the norm)
};

// Stage the launch's blocks: each lane's A' fragments, expanded from the
// compact operands (pack_tile_operand) into lane_words(PREC) consecutive
// words per lane, and the column tables.  Lane (half, l32) takes row r = l32 of A' =
// [[Ur,-Ui],[Ui,Ur]] interleaved by (re, im): complex row ci = r / 2, part
// ri = r % 2.
//   word 8 p + 4 i + e (part p = 0..2, step i = 0, 1, e = 0..3) holds the
//   16-bit pair A'[r][16 i + 8 half + 2 e + {0, 1}] of part p: (Ur, -Ui)
//   for ri = 0, (Ui, Ur) for ri = 1, at complex column j = 8 i + 4 half + e.
template <int TB, int WAVES, int PREC>
__device__ __forceinline__ void stage_blocks(TileShared<TB, WAVES, lane_words(PREC)> &sh, const uint32_t *A,
                                             const TileArgs &args, int tid, bool whole)
{
    using C = TileCfg<TB, WAVES, lane_words(PREC)>;
    constexpr int CHUNKS = lane_words(PREC) / 4;  // 16-byte chunks per lane, each 4 consecutive compact words
    constexpr bool X3 = PREC == kPrecX3, F64 = PREC == kPrecF64, GATES = PREC == kPrecGates32 || PREC == kPrecGates64;
    constexpr int STRIDE = F64 ? kTileOperandWordsF64 : kTileOperandWords;
    const int nsub = args.n_sub;
    const int per_block = 64 * (whole ? 6 : CHUNKS);
    const int units = nsub * per_block;
    typedef uint32_t vu4 __attribute__((ext_vector_type(4)));
    // X3: units 0..127 of a block are the first part's fragments, the rest
    // the compact chunks of the two other parts, or their fragments
    struct Unit {
        int s, lane, c, part;
        bool expand;
    };
    auto unit_of = [&](int u) {
        Unit x;
        x.s = whole ? u / (64 * 6) : u / (64 * CHUNKS);
        const int r = u - x.s * per_block;
        x.expand = !F64 && (!X3 || whole || r < 128);
        if (F64) {
            x.lane = r;
            x.c = x.part = 0;
        } else if (X3) {
            x.lane = x.expand ? (r & 127) >> 1 : (r & 63) >> 2;  // compact: the complex row
            x.c = x.expand ? r & 1 : r & 3;
            x.part = x.expand ? r >> 7 : 1 + ((r - 128) >> 6);
        } else {
            x.lane = r / CHUNKS;
            x.c = r % CHUNKS;
            x.part = x.c >> 1;
        }
        return x;
    };
    // four loads in flight per thread (more where the threads are few): the
    // operands come from HBM, and word by word their latency alone was 2 us of a launch
    constexpr int DEPTH = C::THREADS >= 256 ? 4 : 16;
    for (int u0 = tid; u0 < units && !GATES; u0 += DEPTH * C::THREADS) {
        vu4 v[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int u = u0 + d * C::THREADS;
            if (u >= units) continue;
            const Unit x = unit_of(u);
            // X3: row 16 c + l16, columns 4 kg ..; else row l32, columns 8 i + 4 half ..
            const int at = F64 ? 4 * x.lane
                           : X3 ? (x.expand ? (8 * x.c + ((x.lane & 15) >> 1)) * 16 + 4 * (x.lane >> 4) : x.lane * 16 + 4 * x.c)
                              : ((x.lane & 31) >> 1) * 16 + 8 * (x.c & 1) + 4 * (x.lane >> 5);
            v[d] = *reinterpret_cast<const vu4 *>(A + size_t(x.s) * STRIDE + 256 * x.part + at);
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int u = u0 + d * C::THREADS;
            if (u >= units) continue;
            const Unit x = unit_of(u);
            vu4 w = v[d];
            if (x.expand) w = x.lane & 1 ? (w >> 16) | (w << 16) : w ^ 0x80000000u;
            uint32_t to;
            if (F64)
                to = 4 * uint32_t(x.lane);
            else if (!X3)
                to = uint32_t(x.lane) * lane_words(PREC) + 4 * (uint32_t(x.c) ^ frag_swz<lane_words(PREC)>(uint32_t(x.lane)));
            else if (x.expand)
                to = 512 * uint32_t(x.part) + x3_expanded_at(uint32_t(x.lane), uint32_t(x.c));
            else
                to = x3_compact_at(uint32_t(x.part), uint32_t(x.lane), uint32_t(x.c));
            *reinterpret_cast<vu4 *>(&sh.op[x.s * (4 * per_block) + to]) = w;
        }
    }
    for (int e = tid; e < nsub * (C::CBLOCKS + 32); e += C::THREADS) {
        const int s = e / (C::CBLOCKS + 32), r = e % (C::CBLOCKS + 32);
        uint32_t m = 0;
        for (int b = 0; b < 4; ++b) m |= 1u << args.tbit[s][b];
        const uint32_t cmask = ((1u << TB) - 1) & ~m;
        constexpr int NBW = C::NB_PER_WAVE;
        if (r < C::CBLOCKS)
            sh.cq[s][r] = swz(deposit(uint32_t((r / NBW) * 32 * NBW + r % NBW), cmask), args);
        else
            sh.cl[s][r - C::CBLOCKS] = swz(deposit(uint32_t(r - C::CBLOCKS) * NBW, cmask), args);
    }
}

// hi = RNE(v), lo = RNE(v - hi) and, with three parts, lo2 = RNE(v - hi - lo)
// of one (re, im) pair, as packed 16-bit pairs (H2 = bf16x2 or f16x2).  The
// differences are exact in FP32.  FP16 (two parts): lo = RNE(hi * m1 + v)
// with hi read as FP16 and m1 = -1 held in a register (minus_one()), one
// mixed-precision FMA per value (the compiler rounds some of them straight
// to FP16 in the same instruction): the same bits as a conversion back, a
// subtraction and a second conversion.
template <int NS, typename H2>
__device__ __forceinline__ void split_pair(float re, float im, H2 *parts, float m1)
{
    vf2 v;
    v.x = re;
    v.y = im;
    if constexpr (std::is_same<H2, f16x2>::value) {
        static_assert(NS == 2, "FP16 splits in two parts");
        parts[0] = __builtin_convertvector(v, H2);
        parts[1].x = static_cast<_Float16>(__builtin_fmaf(float(parts[0].x), m1, v.x));
        parts[1].y = static_cast<_Float16>(__builtin_fmaf(float(parts[0].y), m1, v.y));
    } else {
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            parts[j] = __builtin_convertvector(v, H2);
            if (j + 1 < NS) v -= __builtin_convertvector(parts[j], vf2);
        }
    }
}

// -1.0f in a scalar register, opaque to the compiler: with the literal it
// folds v + hi * (-1) back into a conversion and a subtraction.
__device__ __forceinline__ float minus_one()
{
    int bits;
    asm volatile("s_mov_b32 %0, 0xbf800000" : "=s"(bits));
    return __builtin_bit_cast(float, bits);
}

// One 32 x 32 x 16 product of 16-bit operands with FP32 accumulation.
__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma16(f16x8 a, f16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// One 16 x 16 x 32 product of 16-bit operands with FP32 accumulation.
__device__ __forceinline__ f32x4 mfma16x16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void lds_st4(char *Xb, uint32_t byte_off, float a, float b, float c, float d)
{
    vf4 v;
    v.x = a;
    v.y = b;
    v.z = c;
    v.w = d;
    *reinterpret_cast<vf4 *>(Xb + byte_off) = v;
}

// One block of the pass on the tile in LDS (BF16 and FP16; X3: apply_block_x3).
// D real row = 8 (v / 4) + 4 half
// + v % 4: acc[4 g + 2 e] and acc[4 g + 2 e + 1] are (re, im) of complex row
// 4 g + 2 half + e.  Each wave owns its columns, so its reads of the block
// precede its writes; the caller places the barrier.
//
// Every LDS access moves 16 bytes, two complex values that differ in tile bit 0.  If tile bit 0 is
// the block's row bit 0, these are rows (t, t + 1) of one column; otherwise
// tile bit 0 is the lowest column bit, i.e. column blocks (q, q + 1).
template <int TB, int WAVES, int PREC, int SCALE>
__device__ __forceinline__ void apply_block(TileShared<TB, WAVES, lane_words(PREC)> &sh, const TileArgs &args, int s,
                                            int w, int half, int l32, float scale, float unscale)
{
    using C = TileCfg<TB, WAVES, lane_words(PREC)>;
    using H2 = typename std::conditional<PREC == kPrecF16, f16x2, bf16x2>::type;  // packed 16-bit pair
    using H8 = typename std::conditional<PREC == kPrecF16, f16x8, bf16x8>::type;  // MFMA operand
    constexpr int NBW = C::NB_PER_WAVE;
    static_assert(NBW % 2 == 0, "column blocks come in pairs");
    char *Xb = reinterpret_cast<char *>(sh.X4);
    uint32_t rb[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) rb[b] = args.swz[args.tbit[s][b]];
    const uint32_t cl = sh.cl[s][l32];
    uint32_t lq[NBW], wq[NBW];  // lane byte terms of this lane's column in block q
#pragma unroll
    for (int q = 0; q < NBW; ++q) {
        const uint32_t col = cl ^ sh.cq[s][w * NBW + q];
        lq[q] = (col ^ (half ? rb[2] : 0u)) << 3;  // B rows 8 i + 4 half + t
        wq[q] = (col ^ (half ? rb[1] : 0u)) << 3;  // complex row bit 1 = half
    }
    f32x16 acc[NBW];
#pragma unroll
    for (int q = 0; q < NBW; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[q][v] = 0.f;
    const uint32_t *op = sh.op + s * C::OPERAND_WORDS;
    const uint32_t lane = uint32_t(half * 32 + l32);
    const vf4 *ap = reinterpret_cast<const vf4 *>(op + lane * lane_words(PREC));  // staged fragments
    const uint32_t fsw = frag_swz<lane_words(PREC)>(lane);                        // their chunk order
    // step i (K = 16 i .. 16 i + 15) with the operand's parts A_p
    // (BF16: three, FP16: two) and the tile values split into NS parts X_s:
    // every A_p X_0 and every A_0 X_s, the smaller terms accumulated first.
    // FP16: the values are scaled by `scale` before the split (SCALE 0: one
    // scale per tile; SCALE 1: the tile is held scaled in LDS with one scale
    // per pass), A_1 is held multiplied by 2^11 and meets X_0 2^-11 (so that
    // neither falls below FP16's normal range), and the sums are scaled back
    // by `unscale` (SCALE 0).
    constexpr bool F16 = PREC == kPrecF16;
    constexpr bool SCALE_HERE = F16 && SCALE == 0;
    constexpr int NP = F16 ? 2 : 3;
    constexpr int NS = 2;
    auto scaled = [&](vf4 v) { return SCALE_HERE ? v * scale : v; };
    auto out = [&](float v) { return SCALE_HERE ? v * unscale : v; };
    // X_0 2^-11 of a pair's X_0 (FP16 only; exact unless it falls below
    // FP16's normal range, where its product with A_1 is below 2^-35 of m)
    auto low_pair = [&](H2 x0) {
        vf2 c;
        c.x = 0x1p-11f;
        c.y = 0x1p-11f;
        return x0 * __builtin_convertvector(c, H2);  // a packed 16-bit multiply
    };
    const float m1 = F16 ? minus_one() : -1.f;
    auto fragment = [&](int p, int i) {
        H8 h;
        const vf4 f = ap[uint32_t(2 * p + i) ^ fsw];
        __builtin_memcpy(&h, &f, 16);
        return h;
    };
    auto products = [&](f32x16 c, const H8 *xa, const H8 *b) {
#pragma unroll
        for (int d = NP + NS - 2; d >= 0; --d)  // A_p X_s is about 2^(-8 (p + s)) of A X
#pragma unroll
            for (int sp = 0; sp < NS; ++sp) {
                const int p = d - sp;
                if (p >= 0 && p < NP && (sp == 0 || p == 0))
                    c = mfma16(xa[p], b[sp], c);
            }
        return c;
    };
    if (args.tbit[s][0] == 0) {  // uniform: rows (t, t + 1) share a slot
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            H8 xa[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) xa[p] = fragment(p, i);
#pragma unroll
            for (int q = 0; q < NBW; ++q) {
                vf4 raw[2];  // rows 8 i + 2 k2 + {0, 1} (plus 4 half)
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
                    raw[k2] = scaled(*reinterpret_cast<const vf4 *>(Xb + ((row_of(rb, 8 * i + 2 * k2) << 3) ^ lq[q])));
                H2 pp[4][NS];
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) {
                    split_pair<NS>(raw[k2].x, raw[k2].y, pp[2 * k2], m1);
                    split_pair<NS>(raw[k2].z, raw[k2].w, pp[2 * k2 + 1], m1);
                }
                H8 b[NS];
#pragma unroll
                for (int sp = 0; sp < NS; ++sp) {
                    H2 t[4] = {pp[0][sp], pp[1][sp], pp[2][sp], pp[3][sp]};
                    __builtin_memcpy(&b[sp], t, 16);
                }
                if constexpr (F16) {
                    H2 t[4] = {low_pair(pp[0][0]), low_pair(pp[1][0]), low_pair(pp[2][0]), low_pair(pp[3][0])};
                    H8 bs;
                    __builtin_memcpy(&bs, t, 16);
                    acc[q] = mfma16(xa[0], b[1], acc[q]);
                    acc[q] = mfma16(xa[1], bs, acc[q]);
                    acc[q] = mfma16(xa[0], b[0], acc[q]);
                } else {
                    acc[q] = products(acc[q], xa, b);
                }
            }
        }
        // rows 4 g + 2 half + {0, 1} are acc[4 g .. 4 g + 3]
#pragma unroll
        for (int q = 0; q < NBW; ++q)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                lds_st4(Xb, (row_of(rb, 4 * g) << 3) ^ wq[q], out(acc[q][4 * g]), out(acc[q][4 * g + 1]),
                        out(acc[q][4 * g + 2]), out(acc[q][4 * g + 3]));
    } else {  // column blocks (q, q + 1) share a slot
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            H8 xa[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) xa[p] = fragment(p, i);
#pragma unroll
            for (int q = 0; q < NBW; q += 2) {
                vf4 raw[4];  // row 8 i + t (plus 4 half): column blocks (q, q + 1)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    raw[t] = scaled(*reinterpret_cast<const vf4 *>(Xb + ((row_of(rb, 8 * i + t) << 3) ^ lq[q])));
                H2 p0[4][NS], p1[4][NS];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    split_pair<NS>(raw[t].x, raw[t].y, p0[t], m1);
                    split_pair<NS>(raw[t].z, raw[t].w, p1[t], m1);
                }
                H8 b0[NS], b1[NS];
#pragma unroll
                for (int sp = 0; sp < NS; ++sp) {
                    H2 t0[4] = {p0[0][sp], p0[1][sp], p0[2][sp], p0[3][sp]};
                    H2 t1[4] = {p1[0][sp], p1[1][sp], p1[2][sp], p1[3][sp]};
                    __builtin_memcpy(&b0[sp], t0, 16);
                    __builtin_memcpy(&b1[sp], t1, 16);
                }
                if constexpr (F16) {
                    H2 t0[4], t1[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        t0[t] = low_pair(p0[t][0]);
                        t1[t] = low_pair(p1[t][0]);
                    }
                    H8 bs0, bs1;
                    __builtin_memcpy(&bs0, t0, 16);
                    __builtin_memcpy(&bs1, t1, 16);
                    acc[q] = mfma16(xa[0], b0[1], acc[q]);
                    acc[q + 1] = mfma16(xa[0], b1[1], acc[q + 1]);
                    acc[q] = mfma16(xa[1], bs0, acc[q]);
                    acc[q + 1] = mfma16(xa[1], bs1, acc[q + 1]);
                    acc[q] = mfma16(xa[0], b0[0], acc[q]);
                    acc[q + 1] = mfma16(xa[0], b1[0], acc[q + 1]);
                } else {
                    acc[q] = products(acc[q], xa, b0);
                    acc[q + 1] = products(acc[q + 1], xa, b1);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < NBW; q += 2)
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    lds_st4(Xb, (row_of(rb, 4 * g + e) << 3) ^ wq[q], out(acc[q][4 * g + 2 * e]),
                            out(acc[q][4 * g + 2 * e + 1]), out(acc[q + 1][4 * g + 2 * e]),
                            out(acc[q + 1][4 * g + 2 * e + 1]));
    }
}

// X3's block on the tile in LDS, in 16 x 16 x 32 products: lane (kg, l16) holds
// the 8 consecutive K values (4 complex rows 4 kg + {0..3}) of column l16, so
// one product covers the whole contraction, and a step's accumulators are 8
// registers (16 with a column pair) instead of the 32 of two 32 x 32 blocks:
// with three parts of each value the latter spilled the prefetched tile.  D
// real row = 16 r + 4 kg + v (r = 0, 1): complex rows 8 r + 2 kg + {0, 1}.
// The columns of a wave, their LDS addresses and the 16-byte accesses are
// those of apply_block, 16 columns (g2) at a time.
template <int TB, int WAVES>
__device__ __forceinline__ void apply_block_x3(TileShared<TB, WAVES, lane_words(kPrecX3)> &sh, const TileArgs &args,
                                               int s, int w, int lane, bool whole)
{
    using C = TileCfg<TB, WAVES, lane_words(kPrecX3)>;
    constexpr int NBW = C::NB_PER_WAVE;
    typedef uint32_t vu4 __attribute__((ext_vector_type(4)));
    char *Xb = reinterpret_cast<char *>(sh.X4);
    const uint32_t kg = uint32_t(lane) >> 4, l16 = uint32_t(lane) & 15u;
    uint32_t rb[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) rb[b] = args.swz[args.tbit[s][b]] << 3;  // byte terms
    const uint32_t rterm = (kg & 1u ? rb[2] : 0u) ^ (kg & 2u ? rb[3] : 0u);
    const uint32_t wterm = (kg & 1u ? rb[1] : 0u) ^ (kg & 2u ? rb[2] : 0u);
    // A' fragments: row 16 r + l16 (complex row 8 r + l16 / 2), complex columns
    // 4 kg .. 4 kg + 3; compact words are turned by 16 bits (the low 5 bits of
    // `turn`) on odd rows and their high half negated on even ones
    const uint32_t turn = l16 << 4, negate = (l16 << 31) ^ 0x80000000u;
    const uint32_t *op = sh.op + s * (whole ? 64 * 24 : 64 * 16);
    bf16x8 xa[2][3];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const bool fragment = p == 0 || whole;
            const uint32_t at = fragment ? 512u * uint32_t(p) + x3_expanded_at(uint32_t(lane), uint32_t(r))
                                         : x3_compact_at(uint32_t(p), uint32_t(8 * r) + (l16 >> 1), kg);
            vu4 f = *reinterpret_cast<const vu4 *>(op + at);
            if (!fragment) {
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = __builtin_amdgcn_alignbit(f[e], f[e], turn) ^ negate;
            }
            __builtin_memcpy(&xa[r][p], &f, 16);
        }
    // acc[r] = sum of the products A_p X_s, the smaller first, of 4 complex values.
    // The matrix unit cuts off what lies below the largest term of a sum (0.1 ulp
    // towards zero on average where the small terms come in as its C operand),
    // which would add up over the blocks: the trace of a density matrix drifted by
    // -2.5e-7 in 100 blocks; added outside, rounded to nearest, +-3e-8.
    auto column = [&](const vf2 *x, f32x4 *acc) __attribute__((always_inline)) {
        bf16x2 pp[4][3];
#pragma unroll
        for (int t = 0; t < 4; ++t) split_pair<3>(x[t].x, x[t].y, pp[t], -1.f);
        bf16x8 b[3];
#pragma unroll
        for (int sp = 0; sp < 3; ++sp) {
            const bf16x2 t[4] = {pp[0][sp], pp[1][sp], pp[2][sp], pp[3][sp]};
            __builtin_memcpy(&b[sp], t, 16);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
            c = mfma16x16(xa[r][2], b[0], c);
            c = mfma16x16(xa[r][1], b[1], c);
            c = mfma16x16(xa[r][0], b[2], c);
            c = mfma16x16(xa[r][1], b[0], c);
            c = mfma16x16(xa[r][0], b[1], c);
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            acc[r] = mfma16x16(xa[r][0], b[0], zero) + c;
        }
    };
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2) {
        const uint32_t cl = sh.cl[s][l16 + 16u * uint32_t(g2)] << 3;
        if (args.tbit[s][0] == 0) {  // uniform: rows (t, t + 1) share a slot
#pragma unroll
            for (int q = 0; q < NBW; ++q) {
                const uint32_t col = cl ^ sh.cq[s][w * NBW + q] << 3, rd = col ^ rterm, wr = col ^ wterm;
                vf2 x[4];
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) {
                    const vf4 v = *reinterpret_cast<const vf4 *>(Xb + (row_of(rb, 2 * k2) ^ rd));
                    x[2 * k2] = vf2{v.x, v.y};
                    x[2 * k2 + 1] = vf2{v.z, v.w};
                }
                f32x4 acc[2];
                column(x, acc);
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    *reinterpret_cast<vf4 *>(Xb + (row_of(rb, 8 * r) ^ wr)) = acc[r];
            }
        } else {  // column blocks (q, q + 1) share a slot
#pragma unroll
            for (int q = 0; q < NBW; q += 2) {
                const uint32_t col = cl ^ sh.cq[s][w * NBW + q] << 3, rd = col ^ rterm, wr = col ^ wterm;
                vf2 x0[4], x1[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const vf4 v = *reinterpret_cast<const vf4 *>(Xb + (row_of(rb, t) ^ rd));
                    x0[t] = vf2{v.x, v.y};
                    x1[t] = vf2{v.z, v.w};
                }
                f32x4 a0[2], a1[2];
                column(x0, a0);
                column(x1, a1);
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        lds_st4(Xb, row_of(rb, 8 * r + e) ^ wr, a0[r][2 * e], a0[r][2 * e + 1],
                                a1[r][2 * e], a1[r][2 * e + 1]);
            }
        }
    }
}

// An FP64 block on the tile in LDS: 16 x 16 x 4 products, 2 row tiles x 8
// steps for 16 columns.  Lane (kq, l16) holds K = 4 t + kq (t = 0..7), part
// kq % 2 (re, im) of complex row 2 t + kq / 2 of column l16, and the products'
// D real row 16 r + 4 v + kq is K = 4 (4 r + v) + kq: each lane writes the eight
// 8-byte places it read.  Column c = (32 w + l16 + 16 g2) NBW + 2 q2 (its lowest
// bit is the virtual position 0).  The block is bound by the FP64 matrix units
// (3.4 us for a tile at their peak rate, 5.0 measured; the generic
// kernel takes a whole state pass, at least 30 us, a block), so 8 waves with 4 column
// groups each keep the operand (16 words a lane, read once a block) cheap.
template <int TB, int WAVES>
__device__ __forceinline__ void apply_block_f64(TileShared<TB, WAVES, lane_words(kPrecF64)> &sh, const TileArgs &args,
                                                int s, int w, int lane)
{
    using C = TileCfg<TB, WAVES, lane_words(kPrecF64)>;
    constexpr int NBW = C::NB_PER_WAVE;
    char *Xb = reinterpret_cast<char *>(sh.X4);
    const uint32_t kq = uint32_t(lane) >> 4, l16 = uint32_t(lane) & 15u;
    uint32_t rb[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) rb[b] = args.swz[args.tbit[s][b]] << 3;
    const uint32_t term = (kq & 2u ? rb[0] : 0u) | (kq & 1u) << 3;
    // A'[16 r + l16][4 t + kq]: complex row 8 r + l16 / 2, column 2 t + kq / 2
    double a[2][8];
    const double *op = reinterpret_cast<const double *>(sh.op + s * C::OPERAND_WORDS);
    const uint32_t ri = l16 & 1u, part = ri ^ (kq & 1u);
    const uint64_t flip = uint64_t(!ri && (kq & 1u)) << 63;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t ci = uint32_t(8 * r) + (l16 >> 1), j = uint32_t(2 * t) + (kq >> 1);
            const double v = op[2 * (ci * 16 + (j ^ f64_operand_swz(ci))) + part];
            a[r][t] = __longlong_as_double(__double_as_longlong(v) ^ flip);
        }
    // the next group's values are read before this one's are written (the
    // compiler keeps LDS reads behind writes that might be to the same place)
    uint32_t col[NBW];
#pragma unroll
    for (int g = 0; g < NBW; ++g)
        col[g] = ((sh.cl[s][l16 + 16u * uint32_t(g & 1)] ^ sh.cq[s][w * NBW + (g & ~1)]) << 3) ^ term;
    double b[2][8];
#pragma unroll
    for (int t = 0; t < 8; ++t) b[0][t] = *reinterpret_cast<const double *>(Xb + (row_of(rb, 2 * t) ^ col[0]));
#pragma unroll
    for (int g = 0; g < NBW; ++g) {
        if (g + 1 < NBW) {
#pragma unroll
            for (int t = 0; t < 8; ++t)
                b[(g + 1) & 1][t] = *reinterpret_cast<const double *>(Xb + (row_of(rb, 2 * t) ^ col[g + 1]));
        }
        f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 2; ++r)
                acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r][t], b[g & 1][t], acc[r], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *reinterpret_cast<double *>(Xb + (row_of(rb, 2 * (4 * r + v)) ^ col[g])) = acc[r][v];
    }
}

// ---------------------------------------------------------- gate passes
// Runs of gates of at most 3 qubits, applied one by one (SV_RULE_NONE, and
// small blocks left on their own by the other rules) with the arithmetic of
// the register kernel (apply.hip): per output amplitude the same chain of
// fused multiply-adds, in the state's own type.  One state pass per gate is
// bound by HBM (or the memory-side cache: 41 us a gate at 24 qubits, 6.5 TB/s);
// here a tile stays in LDS for all gates of a pass, and a STAGE of them, the
// gates on 4 tile positions, runs in registers: a thread loads the 16 rows of
// a column (complex64: of two columns, so that every LDS access is 16 bytes),
// applies the stage's gates in order and stores them back.  What is left is
// the FP32 (FP64) arithmetic: 8 multiply-adds an amplitude for one-qubit and
// 16 for two-qubit gates.  Measured at 24 qubits, 268 gates: 7
// passes of 271 us, 11.4 -> 1.9 ms in all.
struct GateOp {
    uint32_t code;  // which of the stage's row bits: gate_code()
    uint32_t mat;   // its canonical matrix: element offset (real type) from the operand's start
};

// Complex k-qubit product on local row bits B..., of NC columns.
template <typename T, int NC, int... B>
__device__ __forceinline__ void gate_rows(T (&re)[NC][16], T (&im)[NC][16], const T *m)
{
    constexpr int K = sizeof...(B), D = 1 << K;
    constexpr int bit[K] = {B...};
    constexpr int mask = ((1 << B) | ...);
    T mr[D][D], mi[D][D];
#pragma unroll
    for (int e = 0; e < D * D; ++e) {
        mr[e / D][e % D] = scalar_load(m, 2 * e);
        mi[e / D][e % D] = scalar_load(m, 2 * e + 1);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int base = 0; base < 16; ++base) {
            if (base & mask) continue;
            T vr[D], vi[D];
#pragma unroll
            for (int x = 0; x < D; ++x) {
                int r = base;
#pragma unroll
                for (int j = 0; j < K; ++j) r |= ((x >> j) & 1) << bit[j];
                vr[x] = re[c][r];
                vi[x] = im[c][r];
            }
#pragma unroll
            for (int x = 0; x < D; ++x) {
                T sr = 0, si = 0;
#pragma unroll
                for (int y = 0; y < D; ++y) {
                    sr = fma(mr[x][y], vr[y], sr);
                    sr = fma(-mi[x][y], vi[y], sr);
                    si = fma(mr[x][y], vi[y], si);
                    si = fma(mi[x][y], vr[y], si);
                }
                int r = base;
#pragma unroll
                for (int j = 0; j < K; ++j) r |= ((x >> j) & 1) << bit[j];
                re[c][r] = sr;
                im[c][r] = si;
            }
        }
}

template <typename T, int NC>
__device__ __forceinline__ void apply_gate_op(T (&re)[NC][16], T (&im)[NC][16], uint32_t code, const T *m)
{
    switch (code) {  // uniform
    case 0: gate_rows<T, NC, 0>(re, im, m); break;
    case 1: gate_rows<T, NC, 1>(re, im, m); break;
    case 2: gate_rows<T, NC, 2>(re, im, m); break;
    case 3: gate_rows<T, NC, 3>(re, im, m); break;
    case 4: gate_rows<T, NC, 0, 1>(re, im, m); break;
    case 5: gate_rows<T, NC, 0, 2>(re, im, m); break;
    case 6: gate_rows<T, NC, 0, 3>(re, im, m); break;
    case 7: gate_rows<T, NC, 1, 2>(re, im, m); break;
    case 8: gate_rows<T, NC, 1, 3>(re, im, m); break;
    case 9: gate_rows<T, NC, 2, 3>(re, im, m); break;
    case 10: gate_rows<T, NC, 0, 1, 2>(re, im, m); break;
    case 11: gate_rows<T, NC, 0, 1, 3>(re, im, m); break;
    case 12: gate_rows<T, NC, 0, 2, 3>(re, im, m); break;
    default: gate_rows<T, NC, 1, 2, 3>(re, im, m); break;
    }
}

// Stage s of the pass on the tile in LDS.  A = the pass's operand: the stages'
// op ranges (kMaxTileSubBlocks + 1 words), the ops, the matrices.  Column c of
// a lane: (32 w + l32) 4 + q; complex64 with tile bit 0 a column bit: the pair
// q = 2 half, 2 half + 1 (one slot), with tile bit 0 a row bit: q = half and
// half + 2 (rows t, t + 1 share a slot); complex128: q = 2 half.
template <int TB, int WAVES, typename T>
__device__ __forceinline__ void apply_stage(TileShared<TB, WAVES, lane_words(kPrecGates32)> &sh, const TileArgs &args,
                                            const uint32_t *A, int s, int w, int half, int l32)
{
    constexpr int NC = sizeof(T) == 4 ? 2 : 1;
    char *Xb = reinterpret_cast<char *>(sh.X4);
    uint32_t rb[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) rb[b] = args.swz[args.tbit[s][b]] << 3;
    const bool row_pairs = NC == 2 && args.tbit[s][0] == 0;  // uniform
    uint32_t col[2];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        col[c] = (sh.cl[s][l32] ^ sh.cq[s][w * 4 + (row_pairs ? half + 2 * c : 2 * half)]) << 3;
    T re[NC][16], im[NC][16];
    if constexpr (NC == 2) {
        if (row_pairs) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const vf4 v = *reinterpret_cast<const vf4 *>(Xb + (row_of(rb, r) ^ col[c]));
                    re[c][r] = v.x; im[c][r] = v.y; re[c][r + 1] = v.z; im[c][r + 1] = v.w;
                }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const vf4 v = *reinterpret_cast<const vf4 *>(Xb + (row_of(rb, r) ^ col[0]));
                re[0][r] = v.x; im[0][r] = v.y; re[1][r] = v.z; im[1][r] = v.w;
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const vd2 v = *reinterpret_cast<const vd2 *>(Xb + (row_of(rb, r) ^ col[0]));
            re[0][r] = v.x; im[0][r] = v.y;
        }
    }
    const uint32_t o0 = scalar_load(A, s), o1 = scalar_load(A, s + 1);
    for (uint32_t o = o0; o < o1; ++o) {
        const uint32_t code = scalar_load(A, kGateHeaderWords + 2 * o), mat = scalar_load(A, kGateHeaderWords + 2 * o + 1);
        apply_gate_op<T, NC>(re, im, code, reinterpret_cast<const T *>(A) + mat);
    }
    if constexpr (NC == 2) {
        if (row_pairs) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int r = 0; r < 16; r += 2)
                    lds_st4(Xb, row_of(rb, r) ^ col[c], re[c][r], im[c][r], re[c][r + 1], im[c][r + 1]);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) lds_st4(Xb, row_of(rb, r) ^ col[0], re[0][r], im[0][r], re[1][r], im[1][r]);
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const vd2 v = {re[0][r], im[0][r]};
            *reinterpret_cast<vd2 *>(Xb + (row_of(rb, r) ^ col[0])) = v;
        }
    }
}

// The tile loop of one workgroup: tiles T, T + step, .. below T_end of the
// state at psi.  A = the blocks' compact operands (pack_tile_operand), back to
// back.  The host splits U into 16-bit parts, U = A_0 + A_1 + A_2 for
// BF16 (8 more significand bits each, about FP32's 24 in all) and A_0 + A_1
// for FP16; each B operand (8 consecutive K values = 4 complex rows of one
// column) is split while it is read from LDS, into X_0 + X_1 (kPrecBF16,
// kPrecF16) or X_0 + X_1 + X_2 (kPrecX3), and the products
// sum_p A_p X_0 + sum_s A_0 X_s (plus A_1 X_1 for kPrecX3) run on
// 32 x 32 x 16 MFMA with FP32 accumulation.  The dropped terms are about
// 2^-17 (BF16: the state's third part, A_1 X_1), 2^-22 (FP16) and 2^-25
// (X3) relative to the result.  FP16 passes scale the values per tile
// (tile_scale; SCALE 0, SCALE 5, which holds the tile scaled in LDS, and SCALE 2,
// which is SCALE 0 and also reports the workgroup's sum of squares to norm.out)
// or per pass from the state's norm (norm_scale; SCALE 1, from the sums an
// earlier pass of the run reported; SCALE 3, the same scale with the state
// already held scaled in HBM, copied as it is).
template <int TB, int WAVES, int PREC, int SCALE, int WHOLE, bool SPREAD>
__device__ __forceinline__ void tile_loop(TileShared<TB, WAVES, lane_words(PREC)> &sh, float *__restrict__ psi,
                                          const uint32_t *__restrict__ A, const TileArgs &args, uint64_t T,
                                          uint64_t T_end, uint64_t step, const TileNorm &norm)
{
    using C = TileCfg<TB, WAVES>;
    constexpr bool F16 = PREC == kPrecF16;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;

    // X3: whether every part is staged expanded (WHOLE 1, 0; -1: by the blocks)
    const bool whole = PREC == kPrecX3 && (WHOLE < 0 ? x3_whole<TileCfg<TB, WAVES, lane_words(PREC)>>(args.n_sub) : WHOLE > 0);
    stage_blocks<TB, WAVES, PREC>(sh, A, args, tid, whole);
    TileCopy<TB, WAVES> cp;
    cp.init(args, tid);
    // the largest magnitude in buf over the workgroup: a wave maximum into
    // sh.red[w]; the caller's next barrier publishes it
    auto wave_max_to_red = [&](const vf4 *buf) {
        // xor butterflies inside each 32-lane half (ds_swizzle in bit-mask
        // mode: no lane-index registers), then the two halves via readlane
        int m = __float_as_int(cp.max_abs(buf));
        m = __float_as_int(fmaxf(__int_as_float(m), __int_as_float(__builtin_amdgcn_ds_swizzle(m, 0x041F))));
        m = __float_as_int(fmaxf(__int_as_float(m), __int_as_float(__builtin_amdgcn_ds_swizzle(m, 0x081F))));
        m = __float_as_int(fmaxf(__int_as_float(m), __int_as_float(__builtin_amdgcn_ds_swizzle(m, 0x101F))));
        m = __float_as_int(fmaxf(__int_as_float(m), __int_as_float(__builtin_amdgcn_ds_swizzle(m, 0x201F))));
        m = __float_as_int(fmaxf(__int_as_float(m), __int_as_float(__builtin_amdgcn_ds_swizzle(m, 0x401F))));
        const float wm = fmaxf(__int_as_float(__builtin_amdgcn_readlane(m, 0)),
                               __int_as_float(__builtin_amdgcn_readlane(m, 32)));
        if (lane == 0) sh.red[w] = wm;
    };
    auto red_max = [&]() {
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) m = fmaxf(m, sh.red[i]);
        // uniform over the workgroup: keep it (and the scales) in scalar registers
        return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, m)));
    };

    // FP16 with SCALE 1: one scale for the pass from the state's norm, the
    // sum of the workgroups' sums of squares that an earlier pass of the run
    // wrote (64 lanes' strided sums, then a butterfly: a fixed order; uniform,
    // in scalar registers).  The copy-in
    // multiplies by it unless the state is already held scaled in HBM, and
    // the copy-out divides by it unless the state is to stay scaled.  SCALE 3:
    // the state is held scaled in HBM before and after the pass, so the pass
    // copies it as it is.
    float pscale = 1.f, punscale = 1.f;
    if (F16 && SCALE == 1) {
        double r2 = 0.0;
        for (int i = lane; i < norm.n_in; i += 64) r2 += norm.in[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) r2 += __shfl_xor(r2, o, 64);
        norm_scale(sqrt(r2), pscale, punscale);
        if (norm.in_scaled) pscale = 1.f;
        if (norm.out_scaled) punscale = 1.f;
        pscale = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, pscale)));
        punscale = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, punscale)));
    }
    constexpr bool PER_TILE = F16 && (SCALE == 0 || SCALE == 2);  // scales from each tile's maximum
    // SCALE 5: the same scales, but multiplied in at copy-in and out at copy-out
    // instead of around every block (exact powers of two: the same bits), for a
    // barrier more a tile
    constexpr bool HELD = F16 && SCALE == 5;
    // SCALE 2: per-tile scales as SCALE 0, and the workgroup's sum of squares to norm.out
    constexpr bool want_norm = F16 && SCALE == 2;
    if (T >= T_end) {  // uniform over the workgroup
        if (want_norm && tid == 0) norm.out[blockIdx.x] = 0.0;
        return;
    }
    // the wave's sum of squares of what it reads (want_norm), kept in LDS
    auto wave_sum = [&](float v) {
        v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x041F));
        v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x081F));
        v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x101F));
        v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x201F));
        v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)) +
               __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    };
    if (want_norm && lane == 0) sh.nrm[w] = 0.f;
    // A finished tile is written to HBM at the top of the next round, before
    // that round's prefetch is issued: loads and stores may complete out of
    // order, so any wait for the prefetch also waits for earlier stores, and
    // these were issued a whole round of block work earlier.
    // a pass that starts the state from a basis state reads nothing: the
    // basis state lies in the tile whose outside positions match its bits,
    // at the tile index its tile-position bits form (split FP16, and X3 in a
    // variant of its own, SCALE 4: the extra registers make it spill)
    constexpr bool CAN_SYNTH = PREC == kPrecF16 || PREC == kPrecF64 || SCALE == 4;
    const bool synth = CAN_SYNTH && norm.basis >= 0;  // uniform
    uint64_t b_out = 0;
    uint32_t b_t = 0;
    if (synth) {
        const uint64_t b = uint64_t(norm.basis);
        uint64_t in_mask = 0;
        for (int j = 0; j < TB; ++j) {
            b_t |= uint32_t((b >> args.ubit[j]) & 1u) << j;
            in_mask |= uint64_t(1) << args.ubit[j];
        }
        b_out = b & ~in_mask;
    }
    auto fetch = [&](vf4 *into, uint64_t base) {
        if (synth)
            cp.template basis<PREC == kPrecF64>(into, base == b_out, b_t, tid);
        else
            cp.load(into, psi, base);
    };
    // Workgroups that start together copy together and compute together, tile
    // after tile: the memory idles while all of them compute.  A long pass
    // (SPREAD) spreads their starts over about one tile's period, 2 us apart.
    // Ladder circuits, without and with (lowest of four interleaved runs, which
    // differ by 0.5 %): FP16 3705 and 3649 us at 27 qubits, 32983 and 32870 at 30;
    // FP64 11554 and 11469 at 27; gate passes 16722 and 16577 at 28; split BF16
    // 3932 and 3918 at 27.  X3 passes gain nothing (4497 and 4519; 41977 and
    // 41958), and the workgroups of a batch do not start together.
    if (SPREAD && T_end - T > 16 * step)
        for (uint32_t i = 0; i < ((blockIdx.x >> 3) & 7u); ++i) __builtin_amdgcn_s_sleep(75);
    vf4 buf[C::CHUNKS];
    fetch(buf, tile_base(T, args));
    uint64_t prev = 0;
    for (bool first = true; T < T_end; T += step, first = false) {
        const uint64_t base = tile_base(T, args);
        float unscale_prev = punscale;
        if (HELD) {
            wave_max_to_red(buf);
            __syncthreads();
            tile_scale(red_max(), pscale, punscale);
            pscale = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, pscale)));
            punscale = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, punscale)));
        }
        if (F16 && (SCALE == 1 || HELD)) {
            if (first)
                cp.to_lds_scaled(sh.X4, buf, pscale);
            else
                cp.swap_scaled(psi, prev, sh.X4, buf, pscale, unscale_prev);
        } else {
            if (first)
                cp.to_lds(sh.X4, buf);
            else
                cp.swap(psi, prev, sh.X4, buf);
        }
        if (want_norm) {
            const float v = wave_sum(cp.sum_sq(buf));
            if (lane == 0) sh.nrm[w] += v;  // only this wave's lane 0 touches sh.nrm[w]
        }
        if (PER_TILE) wave_max_to_red(buf);  // this tile's largest magnitude, published by the barrier
        __syncthreads();  // the first one also publishes the staged blocks
        float scale = 1.f, unscale = 1.f;
        if (PER_TILE) {
            tile_scale(red_max(), scale, unscale);
            // uniform: held in scalar registers through the block loop
            scale = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, scale)));
            unscale = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, unscale)));
        }
        const uint64_t Tn = T + step;
        const bool more = Tn < T_end;  // uniform
        if (more) {
            // the next tile's loads go out at raised wave priority, ahead of
            // the other waves' block work on the SIMD (2-3 % per pass)
            __builtin_amdgcn_s_setprio(3);
            fetch(buf, tile_base(Tn, args));
            __builtin_amdgcn_s_setprio(0);
        }
        for (int s = 0; s < args.n_sub; ++s) {
            if constexpr (PREC == kPrecGates32)
                apply_stage<TB, WAVES, float>(sh, args, A, s, w, half, l32);
            else if constexpr (PREC == kPrecGates64)
                apply_stage<TB, WAVES, double>(sh, args, A, s, w, half, l32);
            else if constexpr (PREC == kPrecF64)
                apply_block_f64<TB, WAVES>(sh, args, s, w, lane);
            else if constexpr (PREC == kPrecX3)
                apply_block_x3<TB, WAVES>(sh, args, s, w, lane, whole);
            else
                apply_block<TB, WAVES, PREC, F16 && !PER_TILE ? 1 : 0>(sh, args, s, w, half, l32, scale, unscale);
            __syncthreads();
        }
        prev = base;
    }
    // the last tile of this workgroup
    if (F16 && (SCALE == 1 || HELD))
        cp.store_scaled(psi, prev, sh.X4, punscale);
    else
        cp.store(psi, prev, sh.X4);
    if (want_norm) {
        // the workgroup's sum of squares: the wave sums in wave order, in FP64
        // (the norm only has to be right to a factor of two)
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int i = 0; i < WAVES; ++i) t += double(sh.nrm[i]);
            norm.out[blockIdx.x] = t;
        }
    }
}

// One pass over one state (gridDim.y = 1) or over psi and psi2 alike
// (gridDim.y = 2): a persistent grid strides over the tiles of its state.
template <int TB, int WAVES, int PREC, int SCALE, int WHOLE = 0>
__global__ void __launch_bounds__(64 * WAVES) k_tile_pass(float *__restrict__ psi, const uint32_t *__restrict__ A,
                                                          const TileArgs args, float *__restrict__ psi2,
                                                          const TileNorm norm)
{
    __shared__ TileShared<TB, WAVES, lane_words(PREC)> sh;
    // Consecutive workgroups go to different XCDs.  The 2^g tiles that share
    // 128-byte lines (tiles of short runs: g positions below 4 lie outside
    // the tile) go to one, or each of its lines would be read by 2^g L2s (three
    // blocks on eleven high positions, 2^12 tiles of 16-byte runs at 20 qubits:
    // 19.5 to 11.7 us).
    uint32_t g = 0, T = blockIdx.x;
    if constexpr (TB < kMaxTileBits)
        for (int e = 0; e < 3 && e < args.n_ext; ++e) g += args.ext_pos[e] < 4;
    if (g && !(gridDim.x & ((8u << g) - 1))) T = (((T >> 3 >> g) * 8 + (T & 7u)) << g) | ((T >> 3) & ((1u << g) - 1));
    tile_loop<TB, WAVES, PREC, SCALE, WHOLE, PREC != kPrecX3>(sh, blockIdx.y ? psi2 : psi, A, args, T, args.n_tiles, gridDim.x, norm);
}

// Passes of many states in one grid: workgroup i takes tiles [t0, t1) of
// the pass units[i] names (states of a batch, each with its own tile layout,
// blocks and operands).
// START: the states' first passes, which read nothing and start from |0..0>.
// FP16 scales by each tile's maximum and holds the tile scaled in LDS (SCALE 5).
// One scale for a whole state, from its norm, would need no maximum, but leaves
// amplitudes below 2^-28 of the norm one part and those below 2^-38 nothing.
template <int TB, int WAVES, int PREC, bool START>
__global__ void __launch_bounds__(64 * WAVES) k_tile_batch(const TileUnit *__restrict__ units,
                                                           const TilePass *__restrict__ passes,
                                                           const uint32_t *__restrict__ pool, float *__restrict__ buf)
{
    __shared__ TileShared<TB, WAVES, lane_words(PREC)> sh;
    const TileUnit u = units[blockIdx.x];
    const TilePass &p = passes[u.pass];
    TileNorm norm;
    norm.basis = START ? 0 : -1;
    constexpr int SCALE = PREC == kPrecF16 ? 5 : START ? 4 : 0;
    tile_loop<TB, WAVES, PREC, SCALE, -1, false>(sh, buf + 2 * p.state_off, pool + p.op_off, p.args, u.t0, u.t1, 1, norm);
}

template <int TB, int WAVES>
hipError_t tile_launch(const TileArgs &a, const void *d_a, int prec, float *psi, float *psi2, hipStream_t st,
                       int cap, const TileNorm &norm, int *grid_out)
{
    uint64_t g = a.n_tiles;
    if (cap > 0 && g > uint64_t(cap)) g = cap;
    if (grid_out) *grid_out = int(g);
    const uint32_t *A = static_cast<const uint32_t *>(d_a);
    const dim3 grid(unsigned(g), psi2 ? 2 : 1);
    const dim3 block(64 * WAVES);
    TileNorm plain;  // the variants without the norm take only the basis start
    plain.basis = norm.basis;
    if (prec == kPrecF64) {
        if constexpr ((TB == kF64TileBits && WAVES == kF64TileWaves) || (TB == 13 && WAVES == 8) || TB == 12 || TB == 11)
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecF64, 0>), grid, block, 0, st, psi, A, a, psi2, plain);
        else
            return hipErrorInvalidValue;
    } else if (prec == kPrecBF16 || prec == kPrecF16) {
        if constexpr (TB < 12) return hipErrorInvalidValue;
        else if (prec == kPrecBF16)
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecBF16, 0>), grid, block, 0, st, psi, A, a, psi2, plain);
        else if (norm.in && norm.in_scaled && norm.out_scaled)
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecF16, 3>), grid, block, 0, st, psi, A, a, psi2, norm);
        else if (norm.in)
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecF16, 1>), grid, block, 0, st, psi, A, a, psi2, norm);
        else if (norm.out)
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecF16, 2>), grid, block, 0, st, psi, A, a, psi2, norm);
        else
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecF16, 0>), grid, block, 0, st, psi, A, a, psi2, plain);
    } else if (x3_whole<TileCfg<TB, WAVES, lane_words(kPrecX3)>>(a.n_sub)) {
        if (norm.basis >= 0)
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecX3, 4, 1>), grid, block, 0, st, psi, A, a, psi2, plain);
        else
            hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecX3, 0, 1>), grid, block, 0, st, psi, A, a, psi2, plain);
    } else if (norm.basis >= 0) {
        hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecX3, 4>), grid, block, 0, st, psi, A, a, psi2, plain);
    } else {
        hipLaunchKernelGGL((k_tile_pass<TB, WAVES, kPrecX3, 0>), grid, block, 0, st, psi, A, a, psi2, plain);
    }
    return hipGetLastError();
}

}  // namespace

// The shapes of small states, (12, 4), (11, 2) and (10, 1).
static bool small_shape(int tile_bits, int waves)
{
    return tile_bits >= kMinTileQubitsSmall && tile_bits <= 12 && waves == 1 << (tile_bits - 10);
}

bool tile_supported(int n, int union_bits) { return n >= kMinTileQubits && union_bits <= kMaxTileUnion; }

bool tile_shape_supported(int tile_bits, int waves)
{
    return (tile_bits == 14 && (waves == 8 || waves == 16)) || (tile_bits == 13 && (waves == 4 || waves == 8));
}

int tile_wgs_per_cu(int tile_bits, int waves)
{
    // LDS: a 64 KiB tile leaves room for a second workgroup; registers: two
    // 8-wave workgroups would need <= 128 VGPRs per lane
    return tile_bits == 13 && waves == 4 ? 2 : 1;
}

template <int LW>
static int max_blocks_of(int tile_bits, int waves)
{
    if (tile_bits == 14) return waves == 16 ? TileCfg<14, 16, LW>::MAX_SUB : TileCfg<14, 8, LW>::MAX_SUB;
    if (tile_bits == 12) return TileCfg<12, 4, LW>::MAX_SUB;
    if (tile_bits == 11) return TileCfg<11, 2, LW>::MAX_SUB;
    if (tile_bits == 10) return TileCfg<10, 1, LW>::MAX_SUB;
    return waves == 4 ? TileCfg<13, 4, LW>::MAX_SUB : TileCfg<13, 8, LW>::MAX_SUB;
}

int tile_max_blocks(int tile_bits, int waves, int prec)
{
    if (!tile_shape_supported(tile_bits, waves) && !small_shape(tile_bits, waves)) return 0;
    // BF16X3's limit is that of split BF16, though its operands are smaller
    if (prec == kTileOperandF64) return max_blocks_of<16>(kF64TileBits, kF64TileWaves);  // the fewest of its shapes
    return prec == kTileOperandBF16 || prec == kTileOperandBF16X3 ? max_blocks_of<24>(tile_bits, waves)
                                                                   : max_blocks_of<16>(tile_bits, waves);
}

static uint32_t f2bf_rne(float x)
{
    uint32_t u;
    std::memcpy(&u, &x, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

static float bf2f(uint32_t h)
{
    const uint32_t u = h << 16;
    float x;
    std::memcpy(&x, &u, 4);
    return x;
}

void pack_tile_operand(const cd *m, int prec, uint32_t *out)
{
    if (prec == kTileOperandF64) {
        double *d = reinterpret_cast<double *>(out);
        for (uint32_t r = 0; r < 16; ++r)
            for (uint32_t c = 0; c < 16; ++c) {
                const uint32_t at = r * 16 + (c ^ f64_operand_swz(r));
                d[2 * at] = m[r * 16 + c].real();
                d[2 * at + 1] = m[r * 16 + c].imag();
            }
        return;
    }
    std::memset(out, 0, sizeof(uint32_t) * kTileOperandWords);
    for (int r = 0; r < 16; ++r)
        for (int c = 0; c < 16; ++c) {
            const double re = m[r * 16 + c].real(), im = m[r * 16 + c].imag();
            // part p = RNE(x - parts 0..p-1), as (re, im) halves of one word:
            // three BF16 parts, two FP16 parts (the second held times 2^11,
            // which keeps it in FP16's normal range; the kernel pairs it with
            // X_0 2^-11)
            const int parts = prec == kTileOperandF16 ? 2 : 3;
            double xr = re, xi = im;
            for (int p = 0; p < parts; ++p) {
                uint32_t hr, hi;
                if (prec == kTileOperandF16) {
                    const double f = p ? 2048.0 : 1.0;
                    hr = half_bits(float(xr * f));
                    hi = half_bits(float(xi * f));
                    xr -= double(half_value(hr)) / f;
                    xi -= double(half_value(hi)) / f;
                } else {
                    hr = f2bf_rne(float(xr));
                    hi = f2bf_rne(float(xi));
                    xr -= double(bf2f(hr));
                    xi -= double(bf2f(hi));
                }
                out[256 * p + r * 16 + c] = hr | (hi << 16);
            }
        }
}

hipError_t make_tile_args(int n_sub, const int (*sub_pos)[4], int n, int tile_bits, int waves, int prec,
                          TileArgs *out)
{
    const int kTileBits = tile_bits;
    if (tile_bits < kMinTileQubitsSmall || tile_bits > kMaxTileBits || n_sub < 1 || n_sub > kMaxTileSubBlocks || n < kTileBits)
        return hipErrorInvalidValue;
    TileArgs &a = *out;
    std::memset(&a, 0, sizeof a);
    uint64_t umask = 0;
    for (int s = 0; s < n_sub; ++s)
        for (int i = 0; i < 4; ++i) {
            // row bit i of block s is its i-th lowest position
            if (sub_pos[s][i] < 0 || sub_pos[s][i] >= n || (i && sub_pos[s][i] <= sub_pos[s][i - 1]))
                return hipErrorInvalidValue;
            umask |= uint64_t(1) << sub_pos[s][i];
        }
    const int nu = __builtin_popcountll(umask);
    if (nu > kTileBits) return hipErrorInvalidValue;
    // tile positions: the union plus the lowest positions outside it
    uint64_t tmask = umask;
    for (int p = 0; p < n && __builtin_popcountll(tmask) < kTileBits; ++p) tmask |= uint64_t(1) << p;
    if (!(tmask & 1)) return hipErrorInvalidValue;  // unreachable: position 0 always joins
    int b = 0;
    for (int p = 0; p < n; ++p) {
        if ((tmask >> p) & 1) a.ubit[b++] = p;
        else a.ext_pos[a.n_ext++] = p;
    }
    a.n_sub = n_sub;
    for (int s = 0; s < n_sub; ++s)
        for (int i = 0; i < 4; ++i) {
            int t = 0;
            while (a.ubit[t] != sub_pos[s][i]) ++t;
            a.tbit[s][i] = t;
        }
    a.n_tiles = uint64_t(1) << (n - kTileBits);
    // lanes of a wave take columns l32 NBW + q, so a lane group's columns differ
    // from column bit log2(NBW) up
    if (waves <= 0 || (1 << (tile_bits - 9)) % waves) return hipErrorInvalidValue;
    choose_tile_placement(a, tile_bits, waves, prec);
    return hipSuccess;
}

hipError_t launch_tile_pass(int n_sub, const int (*sub_pos)[4], const void *d_a, int prec, void *psi, int n,
                            hipStream_t st, int grid_cap, int tile_bits, int waves, void *psi2, const TileNorm &norm,
                            int *grid_out)
{
    if ((norm.in || norm.out) && (prec != kTileOperandF16 || psi2 || (norm.in && norm.n_in < 1)))
        return hipErrorInvalidValue;
    if ((norm.in_scaled || norm.out_scaled) && !norm.in) return hipErrorInvalidValue;
    if (norm.basis >= 0 && (psi2 || n >= 63 || (uint64_t(norm.basis) >> n) != 0 || norm.in_scaled ||
                            (prec != kTileOperandF32 && prec != kTileOperandF16 && prec != kTileOperandF64)))
        return hipErrorInvalidValue;
    if (prec < kTileOperandF32 || prec > kTileOperandF64) return hipErrorInvalidValue;
    if (prec == kTileOperandF64) {
        // virtual position 0 is re / im: every position moves up by one
        if (n_sub < 1 || n_sub > tile_max_blocks(kF64TileBits, kF64TileWaves, prec)) return hipErrorInvalidValue;
        // n >= 10 and the virtual position: 11 tile bits at least
        if (tile_bits != kF64TileBits && tile_bits != 13 && !(tile_bits > 10 && small_shape(tile_bits, waves)))
            return hipErrorInvalidValue;
        int pos[kMaxTileSubBlocks][4];
        for (int s = 0; s < n_sub; ++s)
            for (int i = 0; i < 4; ++i) pos[s][i] = sub_pos[s][i] + 1;
        TileArgs a;
        const int w = tile_bits >= 13 ? 8 : waves;
        if (hipError_t e = make_tile_args(n_sub, pos, n + 1, tile_bits, w, prec, &a)) return e;
        if (a.ubit[0] != 0) return hipErrorInvalidValue;  // a union of 14 positions leaves no place for it
        TileNorm nv = norm;
        if (nv.basis >= 0) nv.basis <<= 1;
        float *p = static_cast<float *>(psi), *p2 = static_cast<float *>(psi2);
        if (tile_bits == 11) return tile_launch<11, 2>(a, d_a, prec, p, p2, st, grid_cap, nv, grid_out);
        if (tile_bits == 12) return tile_launch<12, 4>(a, d_a, prec, p, p2, st, grid_cap, nv, grid_out);
        if (tile_bits == 13) return tile_launch<13, 8>(a, d_a, prec, p, p2, st, grid_cap, nv, grid_out);
        return tile_launch<kF64TileBits, kF64TileWaves>(a, d_a, prec, p, p2, st, grid_cap, nv, grid_out);
    }
    if (!tile_shape_supported(tile_bits, waves) && !small_shape(tile_bits, waves)) return hipErrorInvalidValue;
    if (n_sub < 1 || n_sub > tile_max_blocks(tile_bits, waves, prec)) return hipErrorInvalidValue;
    TileArgs a;
    if (hipError_t e = make_tile_args(n_sub, sub_pos, n, tile_bits, waves, prec, &a)) return e;
    float *p = static_cast<float *>(psi), *p2 = static_cast<float *>(psi2);
    if (tile_bits == 10) return tile_launch<10, 1>(a, d_a, prec, p, p2, st, grid_cap, norm, grid_out);
    if (tile_bits == 11) return tile_launch<11, 2>(a, d_a, prec, p, p2, st, grid_cap, norm, grid_out);
    if (tile_bits == 12) return tile_launch<12, 4>(a, d_a, prec, p, p2, st, grid_cap, norm, grid_out);
    if (tile_bits == 14)
        return waves == 16 ? tile_launch<14, 16>(a, d_a, prec, p, p2, st, grid_cap, norm, grid_out)
                           : tile_launch<14, 8>(a, d_a, prec, p, p2, st, grid_cap, norm, grid_out);
    return waves == 4 ? tile_launch<13, 4>(a, d_a, prec, p, p2, st, grid_cap, norm, grid_out)
                      : tile_launch<13, 8>(a, d_a, prec, p, p2, st, grid_cap, norm, grid_out);
}

int gate_code(int k, const int *b)
{
    if (k == 1) return b[0];
    if (k == 2) return b[0] == 0 ? 3 + b[1] : b[0] == 1 ? 5 + b[1] : 9;
    return b[0] == 1 ? 13 : b[1] == 2 ? 12 : 8 + b[2];
}

hipError_t launch_gate_pass(int n_stages, const int (*pos)[4], const void *d_ops, int dtype, void *psi, int n,
                            hipStream_t st, int grid_cap, void *psi2)
{
    if (n_stages < 1 || n_stages > tile_max_blocks(14, 8, kTileOperandF32)) return hipErrorInvalidValue;
    const bool f64 = dtype != SV_C64;
    int p[kMaxTileSubBlocks][4];
    for (int s = 0; s < n_stages; ++s)
        for (int i = 0; i < 4; ++i) p[s][i] = pos[s][i] + (f64 ? 1 : 0);  // complex128: virtual position 0 is re / im
    TileArgs a;
    if (hipError_t e = make_tile_args(n_stages, p, n + (f64 ? 1 : 0), 14, 8, f64 ? kPrecF64 : kPrecX3, &a)) return e;
    if (f64 && a.ubit[0] != 0) return hipErrorInvalidValue;
    uint64_t g = a.n_tiles;
    if (grid_cap > 0 && g > uint64_t(grid_cap)) g = grid_cap;
    const dim3 grid(unsigned(g), psi2 ? 2 : 1), block(64 * 8);
    const uint32_t *A = static_cast<const uint32_t *>(d_ops);
    float *s = static_cast<float *>(psi), *s2 = static_cast<float *>(psi2);
    if (f64)
        hipLaunchKernelGGL((k_tile_pass<14, 8, kPrecGates64, 0>), grid, block, 0, st, s, A, a, s2, TileNorm{});
    else
        hipLaunchKernelGGL((k_tile_pass<14, 8, kPrecGates32, 0>), grid, block, 0, st, s, A, a, s2, TileNorm{});
    return hipGetLastError();
}

hipError_t launch_tile_batch(const TileUnit *units, int n_units, const TilePass *passes, const uint32_t *pool,
                             void *buf, hipStream_t st, int prec, bool start)
{
    if (n_units <= 0) return hipSuccess;
    const dim3 grid{unsigned(n_units)}, block{unsigned(64 * kBatchTileWaves)};
    float *b = static_cast<float *>(buf);
#define SV_TILE_BATCH(P, S) \
    hipLaunchKernelGGL((k_tile_batch<kBatchTileBits, kBatchTileWaves, P, S>), grid, block, 0, st, units, passes, pool, b)
    if (prec == kPrecBF16) {
        if (start) SV_TILE_BATCH(kPrecBF16, true);
        else SV_TILE_BATCH(kPrecBF16, false);
    } else if (prec == kPrecF16) {
        if (start) SV_TILE_BATCH(kPrecF16, true);
        else SV_TILE_BATCH(kPrecF16, false);
    } else {
        if (start) SV_TILE_BATCH(kPrecX3, true);
        else SV_TILE_BATCH(kPrecX3, false);
    }
#undef SV_TILE_BATCH
    return hipGetLastError();
}

}  // namespace dev
}  // namespace sv
