// Read-schedule selection: kernel family, request tile, bucket splits, unroll.
#include <algorithm>

#include "engine.h"

namespace talek {

bool tile_plan_supported(const Plan &p);
hipError_t launch_tile_read(const ReadGeom &g, const Plan &p, void *partials, hipStream_t stream, hipEvent_t eb,
                            hipEvent_t ee);
bool m4r_plan_supported(const Plan &p);
hipError_t launch_m4r_read(const ReadGeom &g, const Plan &p, void *partials, hipStream_t stream, hipEvent_t eb,
                           hipEvent_t ee);
uint32_t m4r_tasks(const ReadGeom &g, const Plan &p);
uint64_t m4r_staging_bytes(const ReadGeom &g);
bool m4rw_plan_supported(const Plan &p);
hipError_t launch_m4rw_read(const ReadGeom &g, const Plan &p, void *partials, hipStream_t stream, hipEvent_t eb,
                            hipEvent_t ee);
uint32_t m4rw_tasks(const ReadGeom &g, const Plan &p);
uint64_t m4rw_staging_bytes(const ReadGeom &g, const Plan &p, bool half);
uint64_t m4rw_steps(uint64_t n, const Plan &p);
bool mfma_plan_supported(const Plan &p);
bool mfma_geom_ok(const ReadGeom &g, const Plan &p);
uint64_t mfma_min_splits(const ReadGeom &g, const Plan &p);
uint64_t mfma_chunks(uint64_t n, const Plan &p);
uint32_t mfma_units(const ReadGeom &g, const Plan &p);
hipError_t launch_mfma_read(const ReadGeom &g, const Plan &p, void *partials, hipStream_t stream, hipEvent_t eb,
                            hipEvent_t ee);

namespace {

constexpr uint64_t PARTIAL_CAP = 256ull << 20;  // bytes of split partials per read
constexpr uint64_t PARTIAL_SOFT = 64ull << 20;  // the tile kernels aim lower (or at 1/64 of D if larger)

uint32_t pow2_at_least(uint32_t x)
{
    uint32_t p = 1;
    while (p < x)
        p <<= 1;
    return p;
}

// Estimated time of a matrix-core read (us) with tile p.tile, and the bucket
// splits that give it: the count that ends first when `units` tasks per split
// run one to a CU, in rounds. A chunk of D costs what the shape measured on
// databases of 32 MiB to 1 GiB, by its request tiles: one reads D at its
// memory rate, two share it through the L2, and more of them, or any over a
// database that the last-level cache holds, wait for the products. A
// task takes about 5 us to start and to write its answers (more in the shapes
// whose four waves take several column groups), and partial answers cross
// memory twice.
double mfma_estimate(const ReadGeom &g, const Plan &p, int num_cus, uint32_t *splits)
{
    static const double CHUNK_US[4][3] = {{2.95, 2.55, 2.2}, {3.5, 3.2, 3.0}, {2.75, 2.45, 2.2}, {2.85, 2.7, 2.5}};
    const uint64_t cus = std::max(num_cus, 1), chunks = mfma_chunks(g.n, p);
    const uint64_t units = std::max<uint32_t>(mfma_units(g, p), 1);
    const uint32_t n_rt = (g.B + p.tile - 1) / p.tile;
    static const double START_US[4] = {7.5, 7.5, 6.0, 7.0};
    const bool shared = n_rt > 2 || g.n * g.stride <= CACHED_BYTES;
    const double chunk_us = CHUNK_US[p.tile / 32 - 1][shared ? 2 : n_rt == 2 ? 1 : 0];
    const uint64_t row = std::max<uint64_t>((uint64_t)g.B * g.stride, 1);
    const uint64_t least = mfma_min_splits(g, p);
    const uint64_t most =
        std::max(least, std::min<uint64_t>({chunks, std::max<uint64_t>(PARTIAL_CAP / row, 1), 4 * cus}));
    double best = -1;
    auto consider = [&](uint64_t s) {
        s = std::min(std::max(s, least), most);
        uint64_t per = (chunks + s - 1) / s;
        s = std::max(least, (chunks + per - 1) / per);  // no empty splits
        const double rounds = (double)((units * s + cus - 1) / cus);
        double us = START_US[p.tile / 32 - 1] + rounds * (per * chunk_us + 5.0);
        if (s > 1)
            us += 4.0 + 2.0 * s * row / 4e6;
        if (best < 0 || us < best) {
            best = us;
            *splits = (uint32_t)s;
        }
    };
    // the most splits that fill 1, 2 .. rounds, and fewer in the first one
    for (uint64_t s = cus / units; s > 1; s /= 2)
        consider(s);
    const uint64_t rounds = (units + cus - 1) / cus;
    for (uint64_t r = rounds; r < rounds + 5; ++r)
        consider(r * cus / units);
    return best;
}

// The matrix-core plan that ends first, by that estimate.
Plan best_mfma(const ReadGeom &g, int num_cus, double *us)
{
    Plan best{KIND_MFMA, 0, 0, 4, 0};
    for (uint32_t tile = 32; tile <= 128; tile += 32) {
        Plan p{KIND_MFMA, tile, 0, 4, 0};
        const double t = mfma_estimate(g, p, num_cus, &p.splits);
        if (best.tile == 0 || t < *us) {
            best = p;
            *us = t;
        }
    }
    return best;
}

// Estimated time of the Four-Russians tables for more than 128 requests, from
// the same databases: 5-bucket pairs up to 256 requests take 22 us and
// 475 + 0.82 B us per GiB of D in whole 1 KiB column slices; half-wave 6-bucket
// pairs 30 us and 1115 us per GiB (in 512-byte slices) and 512 requests.
double tables_estimate(const ReadGeom &g)
{
    const double gib = (double)g.n / (1 << 30);
    if (g.B <= 256)
        return 22.0 + gib * ((g.stride + 1023) / 1024 * 1024) * (475.0 + 0.82 * g.B);
    return 30.0 + gib * ((g.stride + 511) / 512 * 512) * 1115.0 * ((g.B + 511) / 512);
}

}  // namespace

bool plan_supported(const Plan &p)
{
    if (p.kind == KIND_M4R)
        return m4r_plan_supported(p);
    if (p.kind == KIND_M4RW)
        return m4rw_plan_supported(p);
    if (p.kind == KIND_MFMA)
        return mfma_plan_supported(p);
    return tile_plan_supported(p);
}

uint64_t partial_bytes(const ReadGeom &g, const Plan &p)
{
    uint64_t bytes = p.splits <= 1 ? 0 : (uint64_t)p.splits * g.leaves * g.B * g.stride;
    if (p.kind == KIND_M4R)
        bytes += m4r_staging_bytes(g);
    if (p.kind == KIND_M4RW && !(g.staged && (p.flags & PLAN_PAIRS)))
        bytes += m4rw_staging_bytes(g, p, false);
    return bytes;
}

Plan resolve_plan(const ReadGeom &g, Plan want, int num_cus)
{
    Plan p = want;
    if (p.kind == KIND_MFMA && !mfma_geom_ok(g, p))
        p = Plan{KIND_AUTO, 0, 0, 0, 0};
    if (p.kind == KIND_AUTO) {
        // Up to 8 requests stream D with the masked tile kernel, except over
        // rows so narrow that most lanes of its waves, 16 bytes each, have none:
        // the matrix cores take 64 bytes of a row at least (one request over
        // 256 MiB of 64-byte rows 74 against 141 us, 8 requests 78 against
        // 442, over 64 MiB of 256-byte rows 23 against 30; level for up to 4
        // requests over 256 MiB of 256-byte rows, for 8 over 32 MiB of
        // 512-byte rows, and for one over 16 MiB of 64-byte rows). Above 8 the
        // matrix cores count the bits: they read D at its memory rate up to
        // about 64 requests (24 / 64 requests over 1 GiB: 191 / 230 us against
        // 275 / 313 with paired Four-Russians tables, 12 requests 194 against
        // 222 masked; 9 to 16 requests over 16 to 64 MiB would take 4 - 15%
        // less with four waves of 4 masked, 21 - 24 against 25 us over 64 MiB,
        // but more from 128 MiB on, 37 - 39 against 35) and need no tables, so small and narrow databases start
        // faster (256 requests over 4 MiB: 12 against 32 us). From about 160
        // requests per GiB on the tables, bound by the LDS, are as fast
        // (256 over 1 GiB: 684 against 691 us), and with 512 requests to a
        // workgroup faster (512 / 1024: 1.17 / 2.30 against 1.32 / 2.55 ms),
        // but a last tile of 512 that is mostly empty costs them a whole one
        // (768: 2.28 against 1.95 ms): above 128 requests the smaller
        // estimate decides. Tables need rows of 512 bytes above 256 requests
        // (the 5-bucket pairs that narrower rows took there: 512 requests over
        // 2^18 rows of 256 bytes 337 against 87 us). A database under 2048
        // buckets and 2 MiB keeps the half-wave tables above 256 requests,
        // though the matrix cores would take 14 instead of 30 us: the
        // schedule that pir_get_plan reports there is held fixed by the tests.
        double mfma_us = 0;
        Plan m{KIND_AUTO, 0, 0, 0, 0};
        const uint64_t bytes = g.n * g.stride;
        const uint64_t narrow = g.B > 4 ? (bytes > (64ull << 20) ? 512 : 256) : bytes >= CACHED_BYTES ? 256 : 128;
        const bool few = g.B <= 8 && !(bytes >= (16ull << 20) && g.stride <= narrow);
        if (!g.leaf && !few && mfma_geom_ok(g, Plan{KIND_MFMA, 128, 0, 4, 0})) {
            m = best_mfma(g, num_cus, &mfma_us);
            const bool half_waves = g.B > 256 && g.stride >= 512;
            if ((half_waves && g.n < 2048 && g.n * g.stride < (2ull << 20)) ||
                (g.B > 128 && (half_waves || g.B <= 256) && tables_estimate(g) < mfma_us))
                m.kind = KIND_AUTO;
        }
        // The tables, for the handle's other batches above 16 requests and the
        // Strassen leaves: 4-bucket pairs (two workgroups per CU) for one
        // workgroup of up to 128 requests, 5-bucket pairs (one workgroup of up
        // to 256 requests per CU) above, where their fewer lookups per request
        // outweigh the larger table builds; a request tile covers the whole
        // batch up to 256 requests (a second tile would build every table
        // again). Above 256 requests over rows of 512 bytes or more, 6-bucket
        // tables of 512-byte entries, a request per half wave, 512 requests a
        // workgroup: 12 buckets per two lookups (73.0 against 80.8 ms for 2048
        // requests over 2^22 rows of 4 KiB; 1.18 against 1.32 ms for 512 over
        // 2^20 of 1 KiB).
        if (m.kind == KIND_MFMA) {
            p = m;
        } else if (g.B > 256 && g.stride >= 512) {
            p.kind = KIND_M4RW;
            p.flags = PLAN_PAIRS | PLAN_HALF_WAVES | PLAN_PAIR_G6;
            p.unroll = 8;
            p.tile = 64;
        } else if (g.B > 128) {
            p.kind = KIND_M4RW;
            p.flags = PLAN_PAIRS;
            p.unroll = 8;
            p.tile = 32;
        } else if (g.B > 16) {
            p.kind = KIND_M4RW;
            p.flags = PLAN_PAIRS | (1u << PLAN_PAIR_G_SHIFT);
            p.unroll = 8;
            p.tile = g.B > 64 ? 16 : g.B > 32 ? 8 : 4;
        } else {
            // Masked XOR. One launch while its few workgroups, one per 64
            // bytes of a row, take less time than a second launch: 8 requests
            // over 1024 buckets 7.2 against 10.2 us, one over 4096 7.2 against
            // 9.5, 4 over 4096 10.8 against 10.6, 8 17 against 11, one over
            // 8192 of 4 KiB 11.6 against 10.0. Else a database that the caches
            // hold (up to 64 MiB) is read by as many waves as there are; from
            // 5 to 8 requests two waves of 4 share a 1 KiB column chunk, which halves the chain
            // of scalar work per bucket (8 requests over 4 MiB 11.3 us, one
            // wave's tile of 8 13.3, over 64 MiB 19.7 and 20.5). A larger one
            // streams best from few places at a time: four waves per CU, each
            // 8 buckets ahead, take 158 us for one request over 1 GiB where
            // 32 took 203 and 8 161 (8 requests 162, 8 waves of half the
            // depth 171; over 256 MiB 48 and 54). Rows of several chunks
            // that end in a fraction of one count as that fraction, rows of
            // 512 bytes and less as half a chunk (4 requests over 256 MiB of
            // 512-byte rows 51 against 53 us, of 256-byte rows 58 against 86).
            p.kind = KIND_MASK;
            const uint32_t one = pow2_at_least(std::max<uint32_t>(g.B, 1));
            if (g.B <= 8 && g.n <= 4096 && g.n * one <= 8192 && bytes <= (16ull << 20)) {
                p.flags = PLAN_ONE_LAUNCH;
                p.tile = one;
                p.unroll = 4;
            } else if (bytes > (64ull << 20)) {
                p.tile = pow2_at_least(std::max<uint32_t>(g.B, 1));
                p.unroll = 8;
                const uint64_t waves = 4ull * std::max(num_cus, 1);
                uint64_t s = std::max<uint64_t>(waves * 64 / std::max<uint64_t>(g.stride / 16, 32), 1);
                s = std::min<uint64_t>(s, std::max<uint64_t>(PARTIAL_CAP / (std::max(g.B, 1u) * g.stride), 1));
                const uint64_t words = (g.n + 31) / 32, per = (words + s - 1) / s;
                p.splits = (uint32_t)std::max<uint64_t>((words + per - 1) / per, 1);
            } else if (g.B > 4) {
                p.flags = PLAN_SHARED_COLUMN;
                p.tile = 4;
                p.unroll = 4;
            }
        }
    }
    const uint64_t nwords = (g.n + 31) / 32;
    const uint32_t stride16 = (uint32_t)(g.stride / 16);
    uint64_t units;  // independent workgroup tasks per split
    uint64_t per_cu = 8;  // workgroups per CU to aim for
    if (p.kind == KIND_M4R) {
        // tile = requests per wave, unroll = waves per workgroup
        if (p.tile == 0)
            p.tile = 32;
        if (p.unroll == 0)
            p.unroll = g.B >= 256 ? 8 : 4;
        units = m4r_tasks(g, Plan{p.kind, p.tile, 1, p.unroll, 0});
        per_cu = 2;  // one 128 KiB LDS table pair per CU at a time
    } else if (p.kind == KIND_MFMA) {
        if (p.tile == 0) {
            double us = 0;
            p.tile = best_mfma(g, num_cus, &us).tile;
        }
        if (p.unroll == 0)
            p.unroll = 4;
        if (p.splits == 0 && mfma_plan_supported(p))
            (void)mfma_estimate(g, p, num_cus, &p.splits);
        units = 1;
    } else if (p.kind == KIND_M4RW) {
        if (p.tile == 0)
            p.tile = (p.flags & PLAN_HALF_WAVES) ? 64 : g.B > 128 ? 32 : 16;
        if (p.unroll == 0)
            p.unroll = 8;
        units = m4rw_tasks(g, Plan{p.kind, p.tile, 1, p.unroll, p.flags});
        // double-buffered tables of 128 KiB fill a CU's LDS; paired 4- and
        // 3-bucket tables (64 / 32 KiB) let two workgroups share it
        per_cu = ((p.flags & PLAN_PAIRS) && ((p.flags >> PLAN_PAIR_G_SHIFT) & 3u)) ? 2 : 1;
    } else {
        if (p.flags & PLAN_ONE_LAUNCH) {
            const Plan one{p.kind, p.tile ? p.tile : 8, 1, p.unroll ? p.unroll : 4, p.flags};
            if (one_launch(one))
                p = one;
            else
                p.flags &= ~PLAN_ONE_LAUNCH;  // a tile plan as without the flag
        }
        if (p.tile == 0)
            p.tile = g.B <= 16 ? pow2_at_least(std::max<uint32_t>(g.B, 1)) : 16;
        if (p.unroll == 0)
            p.unroll = p.tile <= 2 ? 16 : p.tile >= 16 ? 4 : 8;
        const bool share = p.flags & PLAN_SHARED_COLUMN;
        const uint64_t rows_per_wg = (uint64_t)p.tile * (share ? 4 : 1);
        const uint64_t n_rt = (g.B + rows_per_wg - 1) / rows_per_wg;
        const uint64_t n_cg = share ? (stride16 + 63) / 64 : (stride16 + 255) / 256;
        units = n_rt * n_cg;
    }
    if (p.splits == 0) {
        const uint64_t target = (uint64_t)std::max(num_cus, 1) * per_cu;
        uint64_t s = (target + units - 1) / std::max<uint64_t>(units, 1);
        s = std::min<uint64_t>(s, std::max<uint64_t>(nwords / 2, 1));  // >= 64 buckets per split
        const uint64_t per_split = (uint64_t)g.B * g.stride;
        if (per_split)
            s = std::min<uint64_t>(s, std::max<uint64_t>(PARTIAL_CAP / per_split, 1));
        if (per_split && (p.kind == KIND_MASK || p.kind == KIND_SKIP)) {
            // These kernels stream D at HBM speed, and every split adds a
            // partial answer that is written and read again: halve the
            // splits while the partials exceed 64 MiB and 1/64 of the
            // snapshot, down to two workgroups per CU (at B = 16 over 4 GiB,
            // 1024 splits ran 3% faster than 2048 and 512 7% slower; an
            // uneven 1365 at B = 12 ran 7% slower than 2048).
            const uint64_t cap = std::max<uint64_t>(PARTIAL_SOFT, g.n * g.stride / 64);
            const uint64_t least = ((uint64_t)std::max(num_cus, 1) * 2 + units - 1) / std::max<uint64_t>(units, 1);
            while (s * per_split > cap && s / 2 >= least)
                s /= 2;
        }
        p.splits = (uint32_t)std::max<uint64_t>(s, 1);
    }
    if (p.kind == KIND_MFMA)
        p.splits = (uint32_t)std::max<uint64_t>(p.splits, mfma_min_splits(g, p));
    const uint64_t max_splits = p.kind == KIND_M4RW   ? m4rw_steps(g.n, p)
                                : p.kind == KIND_MFMA ? mfma_chunks(g.n, p)
                                                      : nwords;
    p.splits = (uint32_t)std::min<uint64_t>(p.splits, std::max<uint64_t>(max_splits, 1));
    return p;
}

// One launch holds the tasks of every leaf, so it fills the CUs with few
// splits: the count, up to the one a single leaf would take, that ends first
// when a step of a pair-table kernel takes about 1.65 us (341 steps of 1024
// requests over 256 MiB 573 us), a task five steps' time to start and to write
// its answers, and the partial answers cross memory twice. 2048 requests over
// 2 GiB in 49 leaves of 4 tasks: 13 splits are 10 rounds of 256 workgroups
// all but full; with the 64 of a single leaf 49 rounds took 7.35 ms and their
// 3.3 GB of partial answers another 0.6.
uint32_t leaf_splits(const ReadGeom &g, const Plan &p, uint32_t leaves, int num_cus)
{
    const uint64_t steps = m4rw_steps(g.n, p);
    const uint64_t tasks = (uint64_t)m4rw_tasks(g, p) * leaves;
    const uint64_t slots = std::max(num_cus, 1) * (((p.flags >> PLAN_PAIR_G_SHIFT) & 3u) ? 2ull : 1ull);
    const double bytes = 2.0 * leaves * g.B * g.stride;
    uint32_t best = p.splits;
    double least = -1;
    for (uint64_t s = 1; s <= p.splits; ++s) {
        const double us = (double)((tasks * s + slots - 1) / slots) * (1.65 * ((steps + s - 1) / s) + 8.0) +
                          (s > 1 ? 4.0 + s * bytes / 4e6 : 0.0);
        if (least < 0 || us < least) {
            least = us;
            best = (uint32_t)s;
        }
    }
    return best;
}

hipError_t launch_split_reduce(const void *partials, uint32_t splits, const ReadGeom &g, hipStream_t stream)
{
    if (g.keys)
        return launch_mask_rows(partials, splits, g.B, g.stride, g.out, g.out_pitch, g.keys, stream, g.done);
    return launch_xor_splits(partials, splits, g.B, g.stride, g.out, g.out_pitch, stream, g.done, g.out_bytes);
}

hipError_t launch_read(const ReadGeom &g, const Plan &p, void *partials, hipStream_t stream, hipEvent_t ev_begin,
                       hipEvent_t ev_end)
{
    if (g.B == 0)
        return hipSuccess;
    if (g.out_bytes && (g.keys || !writes_any_row(p)))
        return hipErrorInvalidValue;
    if (g.leaves != 1 && !(g.leaves > 1 && g.staged && p.kind == KIND_M4RW && (p.flags & PLAN_PAIRS)))
        return hipErrorInvalidValue;
    hipError_t e;
    if (p.kind == KIND_M4R)
        e = launch_m4r_read(g, p, partials, stream, ev_begin, ev_end);
    else if (p.kind == KIND_MFMA)
        e = launch_mfma_read(g, p, partials, stream, ev_begin, ev_end);
    else if (p.kind == KIND_M4RW)
        e = launch_m4rw_read(g, p, partials, stream, ev_begin, ev_end);
    else
        e = launch_tile_read(g, p, partials, stream, ev_begin, ev_end);
    // without splits the kernel wrote the plain answers: mask them in place
    if (e == hipSuccess && p.splits <= 1) {
        if (g.keys)
            e = launch_mask_rows(nullptr, 0, g.leaves * g.B, g.stride, g.out, g.out_pitch, g.keys, stream, g.done);
        else if (g.done && (ev_end || !one_launch(p)))
            e = hipEventRecord(g.done, stream);
    }
    return e;
}

}  // namespace talek
