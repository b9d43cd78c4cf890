// XOR-PIR on the matrix cores (gfx950): the GF(2) product as an fp4 matrix
// product of 0/1 values, exact in fp32 accumulators.
//
// A request bit and a database bit meet in one multiply-accumulate; the
// answer bit is the low bit of the count. v_mfma_f32_32x32x64_f8f6f4 with
// 4-bit elements takes 64 buckets x 32 requests x 32 answer bits in 32 clocks
// of a SIMD, 2048 of them per clock and SIMD. Both operands stay packed (one
// bit per bit) in memory and are widened to 4-bit elements on the way to the
// matrix cores, so D moves as often as in any other kernel.
//
// Widening. An element is one nibble; E2M1 codes 1, 2 and 4 are 0.5, 1 and 2,
// so a word masked with 0x11111111 << b holds eight elements of weight
// 2^(b - 1): every masked word is an operand word as it stands.
//  * Requests: word w of a row (32 buckets) gives the four operand words
//    (w >> i) & 0x11111111, element j of word i being bucket 4j + i. They are
//    formed once per workgroup and kept in LDS.
//  * Database: the operand needs eight buckets of one bit column per word.
//    The words of buckets 4j + i (j < 8, one i) of a 32-bit column form an
//    8 x 8 matrix of nibbles; transposed, word q holds nibble q of the eight
//    buckets, and its mask b is bit column 4q + b. A transposition costs 4
//    VALU operations per word of D, is done once per workgroup and goes to
//    LDS, a plane per i, so four LDS words of a lane feed four operands.
//
// Both operands put the same bucket at the same (lane half, word, element),
// which is all the product needs.
//
// What bounds it. With 32 and 64 requests to a workgroup the reading of D: 24
// requests over 1 GiB 191 us (5.6 TB/s; 275 with paired Four-Russians tables),
// 64 requests 230 (313), where the reading meets products that would take 190
// by themselves: 5.1 VALU operations go with each of them. With 96 and 128 the
// products: the matrix cores make 4.9e15 of them a second in a loop of nothing
// else, and 2.9 - 3.3e15 here. 256 requests over 256 MiB: 165 - 170 us, read
// 178 (192 with tables), of which the launch that reduces two splits takes 4
// and the gap before it as much; the matrix cores are busy 64% of the cycles,
// with 3.0 VALU operations to a product (4 fit beside one), and the wave of a
// SIMD waits for the LDS, the barrier or memory in 15% of its cycles (a 16-byte
// LDS read holds the cores for about 10 clocks); the clock falls to 1.9 - 2.3
// GHz under the load. 1000 over 1 GiB 2.55 ms (2.26 with tables).
// Eight waves of 128 accumulators took 167 us, and with the requests' operands
// widened by every wave 172; 256 requests to a workgroup leave no registers
// for the staging.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "engine.h"

namespace talek {

uint64_t mfma_chunks(uint64_t n, const Plan &p);

namespace {

using u32x2 = uint32_t __attribute__((ext_vector_type(2)));
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
using i32x8 = int __attribute__((ext_vector_type(8)));
using f32x16 = float __attribute__((ext_vector_type(16)));

constexpr int THREADS = 256;  // 4 waves, one per SIMD
constexpr int FP4 = 4;        // element format code of the f8f6f4 product
constexpr uint32_t M1 = 0x11111111u;

// f(0), f(1) .. f(N - 1), the index a constant.
template <class F, int... I>
__device__ __forceinline__ void each(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void each(F &&f)
{
    each(f, std::make_integer_sequence<int, N>{});
}
#define INLINE __attribute__((always_inline))

struct MfmaArgs {
    const uint8_t *D;
    uint64_t row_bytes;    // stride
    uint32_t stride4, stride16;
    uint64_t nblk;         // 32-bucket blocks of D, ceil(n / 32)
    uint64_t chunks;       // ceil(n / buckets per chunk)
    const uint32_t *Q;
    uint64_t qpitch_w;
    uint32_t B;
    uint4 *out;
    uint64_t out_row16, out_split16;
    uint32_t n_rt, slices, tasks, tasks_per_xcd;
    uint64_t chunks_per_split;
};

// A workgroup's shape: each wave takes all its requests, MT tiles of 32, and
// NQ sets of 128 answer bits. One wave runs per SIMD, so that it may hold up
// to 256 accumulators: the widening of a database word then serves MT
// products, and every wave's other work fits between its own products. Two
// chunks of the bucket range are in LDS, one being multiplied, one staged.
template <int MT, int NQ>
struct Shape {
    static constexpr int M = 32 * MT;                 // requests
    static constexpr int U = 4 * NQ;                  // column sets of 128 bits
    static constexpr int CW = 4 * U;                  // 4-byte columns
    static constexpr int BLK = CW == 64 ? 8 : 16;     // 32-bucket blocks per chunk
    static constexpr int SB = BLK / 8;                // super-blocks of 256 buckets
    static constexpr int STEPS = 4 * SB;              // of 64 buckets
    static constexpr int SLOTS = 4 * MT * NQ;         // products per wave and step
    static constexpr int G = CW * BLK / THREADS;      // groups of 4 columns x 8 buckets per thread
    static constexpr int CG = CW / 4;                 // threads side by side
    static constexpr int A_ITEMS = M * BLK / 4;       // 16-byte pieces of request rows
    static constexpr int A_PER = (A_ITEMS + THREADS - 1) / THREADS;
    static constexpr int T_U4 = CW * BLK * 8;
    static constexpr int SET_U4 = T_U4 + M * BLK;
};

// Buffer descriptor over `bytes` bytes from p: loads take a lane offset and a
// scalar offset of 32 bits each, and read zero past the end.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}

// Chunk x of D: whole 32-bucket blocks of the database only.
template <class S>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chunk_of(const MfmaArgs &g, uint64_t x)
{
    const uint64_t cb = x * S::BLK, left = g.nblk - cb;
    const uint32_t blocks = left < (uint64_t)S::BLK ? (uint32_t)left : (uint32_t)S::BLK;
    return buffer_of(g.D + cb * 32 * g.row_bytes, blocks * 32u * (uint32_t)g.row_bytes);
}

// A thread's share of a chunk: four columns of a quarter of the buckets of one
// block, in G groups: row j of group e is bucket 4j + i, i = i0 + 2e (off: the
// place of bucket i0). Blocks past the database read zero, whatever request
// bits they meet. ONCE: no other workgroup reads these rows and no cache keeps
// them for the next read.
template <bool ONCE>
__device__ __forceinline__ u32x4 load_row(__amdgpu_buffer_rsrc_t rows, uint32_t off, uint32_t at)
{
    return __builtin_amdgcn_raw_buffer_load_b128(rows, off, at, ONCE ? 2 : 0);
}

// This thread's 16-byte pieces of the chunk's request words: item = (row m,
// 16 bytes p of the row's chunk), aoff their places in the tile's rows. Rows
// past B repeat the last one: their answers are not written. Words past a
// row's end are the next row's, or zero past the last row, and bits past n
// whatever the row holds: both meet zero rows of D only. Threads past the last
// piece take the first ones again.
template <class S>
__device__ __forceinline__ uint32_t request_offset(const MfmaArgs &g, uint32_t r0, uint32_t t, int k)
{
    constexpr uint32_t PP = S::BLK / 4;  // pieces per row and chunk
    const uint32_t item = (t + k * THREADS) % S::A_ITEMS;
    return (min(r0 + item / PP, g.B - 1) - r0) * (uint32_t)(g.qpitch_w * 4) + item % PP * 16;
}
template <class S>
__device__ __forceinline__ void load_a(u32x4 (&a)[S::A_PER], const MfmaArgs &g, uint32_t r0, uint64_t x,
                                       const uint32_t (&aoff)[S::A_PER])
{
    const uint64_t cb = x * S::BLK;
    const uint32_t last = min(r0 + S::M, g.B) - 1 - r0;
    const uint32_t words = (uint32_t)std::min<uint64_t>(g.nblk - cb, 1u << 24);
    const __amdgpu_buffer_rsrc_t q =
        buffer_of(g.Q + r0 * g.qpitch_w + cb, last * (uint32_t)(g.qpitch_w * 4) + words * 4);
    if (cb + S::BLK <= g.nblk) {
        each<S::A_PER>([&](auto k) INLINE { a[k()] = __builtin_amdgcn_raw_buffer_load_b128(q, aoff[k()], 0, 0); });
    } else {  // single words, each held to the buffer's end
        each<4 * S::A_PER>([&](auto e) INLINE {
            a[e() / 4][e() % 4] = __builtin_amdgcn_raw_buffer_load_b32(q, aoff[e() / 4] + e() % 4 * 4, 0, 0);
        });
    }
}

__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) { return (a & m) | (b & ~m); }

// Transposed words in LDS: [step][column set][plane i][64 places], block b of
// the chunk being step b & 3 of super-block b >> 3, lane half (b >> 2) & 1.
// Lane n of column set u is slot 32u + n = nibble * CW + column; its word is
// at place (32 half + n) ^ swizzle, which spreads what a wave stores together
// over the banks.
template <class S>
__device__ __forceinline__ constexpr uint32_t swizzle(uint32_t st, uint32_t u)
{
    return S::CW == 16 ? st * 16 : S::CW == 32 ? (st & 1u) * 32 : (u & 1u) * 32;
}
// Where nibble 0 of column c of block b goes, plane i.
template <class S>
__device__ __forceinline__ uint32_t word_base(uint32_t c, uint32_t b, uint32_t i)
{
    const uint32_t sb = b >> 3, half = (b >> 2) & 1u, st = b & 3u;
    return ((sb * 4 + st) * S::U + c / 32) * 256 + i * 64 + ((half * 32 + c % 32) ^ swizzle<S>(st, c / 32));
}
// Nibble q's column sets. With 16 columns odd nibbles take the upper half of
// a set's lanes, place bit 4 the other way round than their even neighbour.
template <class S>
constexpr uint32_t set_of_q(int q)
{
    return S::CW >= 32 ? q * (S::CW / 32) * 256 : q / 2 * 256;
}

__device__ __forceinline__ f32x16 product(const u32x4 &a, const u32x4 &b, const f32x16 &c)
{
    const i32x8 A = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], 0, 0, 0, 0};
    const i32x8 B = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A, B, c, FP4, FP4, 0, 0, 0, 0);
}

// A thread's staging state: its loads in flight, the columns transposed so far,
// a request word being widened, and its places in memory and LDS.
template <class S>
struct Stage {
    u32x4 raw[S::G][8], lo[4], hi[4], a[S::A_PER], wide;
    uint32_t off, aoff[S::A_PER], base;
};

// The words of one nibble: q = 2y + O of this thread's columns, group E.
template <class S, int E, int O, int y>
__device__ __forceinline__ void store_words(uint32_t *set, const u32x4 (&w)[4], uint32_t base)
{
    uint32_t *p = set + (S::CW == 16 && O ? base ^ 16u : base) + set_of_q<S>(2 * y + O) + E * 128;
    *reinterpret_cast<u32x4 *>(p) = u32x4{w[0][y], w[1][y], w[2][y], w[3][y]};
}

// A group's transposition in 68 small parts (ticks) of at most two VALU
// operations, one LDS store and one load each. The words of buckets 4j + i of
// each column become nibble pairs (ticks 0 - 31), which frees the registers
// of its loads for another chunk (LOAD); then the 4 x 4 bytes of the even (lo)
// and odd (hi) nibbles are transposed (32 - 47, 48 - 63): bucket 4j + i ends
// in nibble j of word q.
constexpr int TICKS = 68;

template <class S, bool ONCE, bool LOAD, int E, int T>
__device__ __forceinline__ void stage_tick(Stage<S> &z, uint32_t *set, __amdgpu_buffer_rsrc_t rows, uint32_t row_bytes)
{
    u32x4(&raw)[8] = z.raw[E];
    if constexpr (T < 32) {
        constexpr uint32_t LOW = 0x0f0f0f0fu;
        constexpr int C = T / 8, p = T / 2 % 4;
        const uint32_t x = raw[2 * p][C], y = raw[2 * p + 1][C];
        if constexpr (T % 2 == 0)
            z.lo[C][p] = bfi(LOW, x, y << 4);
        else
            z.hi[C][p] = bfi(LOW, x >> 4, y);
    } else if constexpr (T < 64) {
        u32x4 &b = T < 48 ? z.lo[T / 4 % 4] : z.hi[T / 4 % 4];
        // {b0 b1}, {b2 b3} byte by byte, then pair by pair
        if constexpr (T % 4 == 0) {
            const uint32_t x = b[0];
            b[0] = __builtin_amdgcn_perm(b[1], x, 0x05010400u);
            b[1] = __builtin_amdgcn_perm(b[1], x, 0x07030602u);
        } else if constexpr (T % 4 == 1) {
            const uint32_t x = b[2];
            b[2] = __builtin_amdgcn_perm(b[3], x, 0x05010400u);
            b[3] = __builtin_amdgcn_perm(b[3], x, 0x07030602u);
        } else if constexpr (T % 4 == 2) {
            const uint32_t x = b[0], y = b[2];
            b[0] = __builtin_amdgcn_perm(y, x, 0x05040100u);
            b[2] = __builtin_amdgcn_perm(y, x, 0x07060302u);
        } else {
            const uint32_t x = b[1], y = b[3], q1 = b[2];
            b[1] = q1;
            b[2] = __builtin_amdgcn_perm(y, x, 0x05040100u);
            b[3] = __builtin_amdgcn_perm(y, x, 0x07060302u);
        }
    }
    if constexpr (LOAD && T >= 32 && T < 64 && T % 4 == 0)
        raw[T / 4 - 8] = load_row<ONCE>(rows, z.off, (4 * (T / 4 - 8) + 2 * E) * row_bytes);
    if constexpr (T >= 50 && T < 64 && T % 4 == 2)
        store_words<S, E, 0, (T - 50) / 4>(set, z.lo, z.base);
    if constexpr (T >= 64)
        store_words<S, E, 1, T - 64>(set, z.hi, z.base);
}

// Word W of a thread's request pieces as four operand words, in four ticks, to
// LDS: [step][32-request tile][64 places], lane half g and row m of the tile
// at place (32 g + m) ^ 4 p, p = 2 * super-block + g being the row's piece
// (the rows and pieces that a wave stores together fall on different banks).
template <class S, int W, int T>
__device__ __forceinline__ void request_tick(Stage<S> &z, u32x4 *set, uint32_t t)
{
    constexpr uint32_t PP = S::BLK / 4;
    z.wide[T] = (z.a[W / 4][W % 4] >> T) & M1;
    if constexpr (T == 3) {
        const uint32_t item = (t + W / 4 * THREADS) % S::A_ITEMS;
        const uint32_t m = item / PP, p = item % PP;
        set[S::T_U4 + ((p >> 1) * 4 + W % 4) * (S::M * 2) + m / 32 * 64 + (((p & 1u) * 32 + m % 32) ^ (p << 2))] = z.wide;
    }
}

// A chunk's staging is G * TICKS ticks and 16 A_PER request ticks.
template <class S>
constexpr int STAGE_TICKS = S::G * TICKS + 16 * S::A_PER;

template <class S, bool ONCE, bool LOAD, int T>
__device__ __forceinline__ void any_tick(Stage<S> &z, u32x4 *set, __amdgpu_buffer_rsrc_t rows, uint32_t row_bytes,
                                         uint32_t t)
{
    if constexpr (T < S::G * TICKS)
        stage_tick<S, ONCE, LOAD, T / TICKS, T % TICKS>(z, reinterpret_cast<uint32_t *>(set), rows, row_bytes);
    else if constexpr (T < STAGE_TICKS<S>)
        request_tick<S, (T - S::G * TICKS) / 4, T % 4>(z, set, t);
}

// The share of slot SLOT of step K: the ticks are spread evenly over the slots
// up to a few before the last step.
template <class S, bool ONCE, int K, int SLOT>
__device__ __forceinline__ void stage_slot(Stage<S> &z, u32x4 *set, __amdgpu_buffer_rsrc_t rows, uint32_t row_bytes,
                                           uint32_t t)
{
    constexpr int AT = K * S::SLOTS + SLOT, END = (S::STEPS - 1) * S::SLOTS - 5;
    if constexpr (AT < END) {
        constexpr int T0 = AT * STAGE_TICKS<S> / END, T1 = (AT + 1) * STAGE_TICKS<S> / END;
        each<T1 - T0>([&](auto w) INLINE {
            any_tick<S, ONCE, true, T0 + decltype(w)::value>(z, set, rows, row_bytes, t);
        });
    }
}

// A step's operands: the requests' as they are, the database's as the
// transposed words, and the first mask of them.
template <int MT, int NQ>
struct Operands {
    u32x4 a[MT], w[NQ], fb;
};

// Read R of the 2 NQ + MT that step K's operands take.
template <class S, int MT, int NQ, int K, int R>
__device__ __forceinline__ void read_operand(Operands<MT, NQ> &op, const u32x4 *set4, uint32_t wn, uint32_t lane)
{
    constexpr int sb = K / 4, st = K % 4;
    if constexpr (R < 2 * NQ) {
        constexpr int j = R / 2, i = R % 2 * 2;
        const uint32_t *p = reinterpret_cast<const uint32_t *>(set4) + (K * S::U + wn * NQ + j) * 256 + i * 64 +
                            (lane ^ swizzle<S>(st, j));
        op.w[j][i] = p[0];
        op.w[j][i + 1] = p[64];
    } else if constexpr (R < 2 * NQ + MT) {
        constexpr int i = R - 2 * NQ;
        op.a[i] = set4[S::T_U4 + K * (S::M * 2) + i * 64 + ((lane ^ (lane >> 5 << 2)) ^ (sb << 3))];
    }
}

// Chunk x: its products, the next chunk's staging and the loads of the chunk
// after it, which have most of a chunk's time to arrive. Every product is
// followed by its share of the step's other work: the next operands and the
// staging; the order is kept as written, so that it runs while the matrix
// cores are busy, and spread so that the waves, which run in step, do not all
// wait for the LDS or the memory path at once. The barrier that ends the next
// chunk's staging comes before the last step, whose products hide the first
// operands of the next chunk.
template <int MT, int NQ, bool ONCE, class S = Shape<MT, NQ>>
__device__ __forceinline__ void chunk_steps(f32x16 (&acc)[MT][NQ][4], Operands<MT, NQ> &op, Stage<S> &z, u32x4 *lds,
                                            uint32_t cur, const MfmaArgs &g, uint32_t r0, uint64_t nx, uint32_t wn,
                                            uint32_t t)
{
    const uint32_t lane = t & 63u;
    const u32x4 *set = lds + cur;
    u32x4 *other = lds + (S::SET_U4 - cur);
    const __amdgpu_buffer_rsrc_t rows = chunk_of<S>(g, nx);
    const uint32_t row_bytes = (uint32_t)g.row_bytes;
    Operands<MT, NQ> next;
    each<S::STEPS>([&](auto kk) INLINE {
        constexpr int k = decltype(kk)::value;
        if (k == S::STEPS - 1) {
            __syncthreads();
            load_a<S>(z.a, g, r0, nx, z.aoff);
        }
        each<S::SLOTS>([&](auto ss) INLINE {
            constexpr int s = decltype(ss)::value, j = s / (4 * MT), b = s / MT % 4, i = s % MT;
            acc[i][j][b] = product(op.a[i], op.fb, acc[i][j][b]);
            read_operand<S, MT, NQ, (k + 1) % S::STEPS, s>(next, k + 1 < S::STEPS ? set : other, wn, lane);
            // the next database operand
            constexpr int nj = (s + MT) / (4 * MT), nb = (b + 1) % 4;
            const u32x4 &src = nj == NQ ? next.w[0] : op.w[nj % NQ];
            constexpr int e0 = i * 4 / MT, e1 = (i + 1) * 4 / MT;
            each<e1 - e0>([&](auto ee) INLINE {
                constexpr int e = e0 + decltype(ee)::value;
                next.fb[e] = nb < 3 ? src[e] & (M1 << nb) : (src[e] >> 3) & M1;
            });
            if (i == MT - 1)
                op.fb = next.fb;
            stage_slot<S, ONCE, k, s>(z, other, rows, row_bytes, t);
            __builtin_amdgcn_sched_barrier(0);
        });
        op = next;
    });
}

// Accumulators start at START<b>, where one count in them moves bit b of the
// float by one: products weigh 1/4, 1/2, 1 and 1/4 (request elements 1/2 times
// the mask's 1/2, 1, 2 and 1/2). Bit b then is the count's low bit, as long as
// a count stays below COUNT_LIMIT.
template <int b>
constexpr float START = b == 3 ? 0x1p18f : 0x1p21f;
constexpr uint64_t COUNT_LIMIT = 1ull << 20;

// The four answer bits of accumulator v.
template <int v>
__device__ __forceinline__ uint32_t answer_nibble(const f32x16 (&acc)[4])
{
    const float f0 = acc[0][v], f1 = acc[1][v], f2 = acc[2][v], f3 = acc[3][v];
    const uint32_t x0 = __builtin_bit_cast(uint32_t, f0), x1 = __builtin_bit_cast(uint32_t, f1);
    const uint32_t x2 = __builtin_bit_cast(uint32_t, f2), x3 = __builtin_bit_cast(uint32_t, f3);
    return bfi(1u, x0, bfi(2u, x1, bfi(4u, x2, x3))) & 15u;
}

template <int MT, int NQ, bool ONCE>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(1, 1)))
void xorpir_mfma_kernel(const MfmaArgs g)
{
    using S = Shape<MT, NQ>;
    __shared__ u32x4 lds[2 * S::SET_U4];
    const uint32_t L = blockIdx.x;
    const uint32_t task = (L & 7u) * g.tasks_per_xcd + (L >> 3);
    if (task >= g.tasks)
        return;
    const uint32_t rt = task % g.n_rt;
    const uint32_t rest = task / g.n_rt;
    const uint32_t slice = rest % g.slices;
    const uint32_t s = rest / g.slices;

    const uint32_t t = threadIdx.x;
    const uint32_t wn = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63u;
    const uint32_t r0 = rt * S::M;

    const uint64_t xb = (uint64_t)s * g.chunks_per_split;
    const uint64_t xe = std::min<uint64_t>(g.chunks, xb + g.chunks_per_split);

    f32x16 acc[MT][NQ][4];
    each<MT * NQ * 4>([&](auto ii) INLINE {
        constexpr int i = decltype(ii)::value;
        acc[i / (NQ * 4)][i / 4 % NQ][i % 4] = f32x16(START<i % 4>);
    });

    if (xb < xe) {
        const uint32_t c = t % S::CG * 4, blk = t / S::CG % S::BLK;
        const uint32_t i0 = __builtin_amdgcn_readfirstlane(t / (S::CG * S::BLK));
        const uint32_t row_bytes = (uint32_t)g.row_bytes;
        const uint64_t last = xe - 1;
        Stage<S> z, z0;
        // columns past the row repeat its last ones: their answers are not written
        z.off = (blk * 32 + i0) * row_bytes + min(slice * S::CW + c, g.stride4 - 4) * 4u;
        z.base = word_base<S>(c, blk, i0);
        each<S::A_PER>([&](auto k) INLINE { z.aoff[k()] = request_offset<S>(g, r0, t, k()); });
        z0.base = z.base;
        const __amdgpu_buffer_rsrc_t d0 = chunk_of<S>(g, xb);
        load_a<S>(z0.a, g, r0, xb, z.aoff);
        each<8 * S::G>([&](auto r) INLINE {
            z0.raw[r() / 8][r() % 8] = load_row<ONCE>(d0, z.off, (4 * (r() % 8) + r() / 8 * 2) * row_bytes);
        });
        load_a<S>(z.a, g, r0, std::min(xb + 1, last), z.aoff);
        const __amdgpu_buffer_rsrc_t d1 = chunk_of<S>(g, std::min(xb + 1, last));
        each<8 * S::G>([&](auto r) INLINE {
            z.raw[r() / 8][r() % 8] = load_row<ONCE>(d1, z.off, (4 * (r() % 8) + r() / 8 * 2) * row_bytes);
        });
        each<STAGE_TICKS<S>>([&](auto w) INLINE {
            any_tick<S, ONCE, false, decltype(w)::value>(z0, lds, d0, row_bytes, t);
        });
        __syncthreads();
        Operands<MT, NQ> op;
        each<2 * NQ + MT>([&](auto r) INLINE { read_operand<S, MT, NQ, 0, decltype(r)::value>(op, lds, wn, lane); });
        op.fb = op.w[0] & M1;
        uint32_t cur = 0;
        for (uint64_t x = xb; x < xe; ++x) {
            // past the split's end its last chunk is loaded again
            chunk_steps<MT, NQ, ONCE>(acc, op, z, lds, cur, g, r0, std::min(x + 2, last), wn, t);
            cur = S::SET_U4 - cur;
        }
        __syncthreads();  // the answers take over the LDS
    }

    // A wave holds nibbles 2 wn and 2 wn + 1 of every answer word: byte wn. For
    // 16 columns they are in neighbouring rows of 16 lanes, else in one lane.
    uint8_t *bytes = reinterpret_cast<uint8_t *>(lds) + wn;
    const uint32_t cl = S::CW == 16 ? lane & 15u : lane & 31u;
    each<MT * 16 * NQ / (NQ == 1 ? 2 : NQ)>([&](auto ee) INLINE {
        constexpr int e = decltype(ee)::value;
        if constexpr (NQ == 1) {
            constexpr int i = e / 8, v = e % 8 * 2;
            const auto sw = __builtin_amdgcn_permlane16_swap(answer_nibble<v>(acc[i][0]),
                                                             answer_nibble<v + 1>(acc[i][0]), false, false);
            const uint32_t m = i * 32 + 8 * (v / 4) + v % 4 + (lane >> 4 & 1u) + 4 * (lane >> 5);
            bytes[(m * S::CW + cl) * 4] = (uint8_t)(sw[0] | sw[1] << 4);
        } else {
            constexpr int i = e / 16, v = e % 16;
            const uint32_t m = i * 32 + 8 * (v / 4) + v % 4 + 4 * (lane >> 5);
            each<NQ / 2>([&](auto h) INLINE {
                bytes[(m * S::CW + h() * 32 + cl) * 4] =
                    (uint8_t)(answer_nibble<v>(acc[i][h()]) | answer_nibble<v>(acc[i][h() + NQ / 2]) << 4);
            });
        }
    });
    __syncthreads();
    constexpr uint32_t C16 = S::CW / 4;
    for (uint32_t i = t; i < S::M * C16; i += THREADS) {
        const uint32_t r = r0 + i / C16, c16 = slice * C16 + i % C16;
        if (r < g.B && c16 < g.stride16) {
            const u32x4 v = lds[i];
            g.out[(uint64_t)s * g.out_split16 + (uint64_t)r * g.out_row16 + c16] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    }
}

using MfmaFn = void (*)(const MfmaArgs);

// Shapes by requests per workgroup (the plan's tile).
struct MfmaShape {
    MfmaFn fn[2];      // D read by several request tiles or kept by the cache; read once
    uint32_t cw, blk;  // 4-byte columns, 32-bucket blocks per chunk
};

template <int MT, int NQ>
MfmaShape shape_of()
{
    using S = Shape<MT, NQ>;
    return {{xorpir_mfma_kernel<MT, NQ, false>, xorpir_mfma_kernel<MT, NQ, true>}, (uint32_t)S::CW,
            (uint32_t)S::BLK};
}

bool mfma_shape(uint32_t tile, MfmaShape *s)
{
    switch (tile) {
    case 32: *s = shape_of<1, 4>(); return true;
    case 64: *s = shape_of<2, 2>(); return true;
    case 96: *s = shape_of<3, 1>(); return true;
    case 128: *s = shape_of<4, 1>(); return true;
    default: return false;
    }
}

}  // namespace

// Offsets within a chunk of D, and within a tile's request rows, are 32 bits;
// one product a launch. (An unknown tile is refused as a plan, not here.)
bool mfma_geom_ok(const ReadGeom &g, const Plan &p)
{
    MfmaShape s;
    const uint32_t tile = p.tile ? p.tile : 128;
    if (!mfma_shape(tile, &s))
        return true;
    return g.leaves == 1 && 32ull * s.blk * g.stride < (1ull << 31) && tile * g.qpitch < (1ull << 31);
}

// A split's counts stay below the kernel's limit.
uint64_t mfma_min_splits(const ReadGeom &g, const Plan &p)
{
    MfmaShape s;
    if (!mfma_shape(p.tile, &s))
        return 1;
    const uint64_t most = (COUNT_LIMIT - 1) / (32 * s.blk), chunks = mfma_chunks(g.n, p);
    return (chunks + most - 1) / most;
}

bool mfma_plan_supported(const Plan &p)
{
    MfmaShape s;
    return mfma_shape(p.tile, &s) && p.unroll == 4 && p.flags == 0;
}

uint64_t mfma_chunks(uint64_t n, const Plan &p)
{
    MfmaShape s;
    const uint64_t per = mfma_shape(p.tile, &s) ? 32ull * s.blk : 1;
    return (n + per - 1) / per;
}

uint32_t mfma_units(const ReadGeom &g, const Plan &p)
{
    MfmaShape s;
    if (!mfma_shape(p.tile, &s))
        return 1;
    const uint64_t slices = (g.stride / 4 + s.cw - 1) / s.cw;
    return (uint32_t)(((g.B + p.tile - 1) / p.tile) * slices);
}

hipError_t launch_mfma_read(const ReadGeom &g, const Plan &p, void *partials, hipStream_t stream, hipEvent_t eb,
                            hipEvent_t ee)
{
    MfmaShape s;
    if (!mfma_plan_supported(p) || !mfma_shape(p.tile, &s) || !mfma_geom_ok(g, p) ||
        p.splits < mfma_min_splits(g, p))
        return hipErrorInvalidValue;
    MfmaArgs a{};
    a.D = static_cast<const uint8_t *>(g.D);
    a.row_bytes = g.stride;
    a.stride16 = (uint32_t)(g.stride / 16);
    a.stride4 = a.stride16 * 4;
    a.nblk = (g.n + 31) / 32;
    a.chunks = mfma_chunks(g.n, p);
    a.Q = static_cast<const uint32_t *>(g.Q);
    a.qpitch_w = g.qpitch / 4;
    a.B = g.B;
    a.n_rt = (g.B + p.tile - 1) / p.tile;
    a.slices = (a.stride4 + s.cw - 1) / s.cw;
    a.chunks_per_split = (a.chunks + p.splits - 1) / p.splits;
    if (p.splits > 1) {
        a.out = static_cast<uint4 *>(partials);
        a.out_row16 = a.stride16;
        a.out_split16 = (uint64_t)g.B * a.stride16;
    } else {
        a.out = static_cast<uint4 *>(g.out);
        a.out_row16 = g.out_pitch / 16;
        a.out_split16 = 0;
    }
    const uint64_t tasks = (uint64_t)a.n_rt * a.slices * p.splits;
    if ((tasks + 7) / 8 * 8 * THREADS > 0xffffffffull)  // a launch holds fewer than 2^32 work-items
        return hipErrorInvalidValue;
    a.tasks = (uint32_t)tasks;
    a.tasks_per_xcd = (uint32_t)((tasks + 7) / 8);
    const bool once = a.n_rt == 1 && g.n * g.stride > CACHED_BYTES;
    hipExtLaunchKernelGGL(s.fn[once], dim3(a.tasks_per_xcd * 8), dim3(THREADS), 0, stream, eb, ee, 0, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.splits <= 1)
        return e;
    return launch_split_reduce(partials, p.splits, g, stream);
}

}  // namespace talek
