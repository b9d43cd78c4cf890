// Compressed interest vectors (section "Private Notifications": clients fetch
// compressed Bloom-filter deltas instead of the raw vector).
//
// Stream (little-endian): m (u64), c = set bits (u64), Rice parameter
// k = floor(log2(max(1, floor(m / (c + 1))))) (u32), 4 zero bytes, then for
// the set positions in increasing order the gaps g = p - p_prev - 1 (p_prev
// starts at -1), each as floor(g / 2^k) one-bits, a zero-bit and the k low
// bits of g least significant first; bits fill bytes LSB first.
//
// Device pipeline, over tiles of 1024 words, three launches: every tile's set
// bits and its last one, from which the launch's last workgroup has c, k and
// the position set just before each tile; every tile's code bits, from which
// it has their offsets; and the codes, ORed into the zeroed body, whose start
// it writes to mapped host memory. The host waits once, and a second time for
// what a body has past its first 64 KiB.
//
// What bounds it: launches and waits, not the vector (0.6 MB at the 100K
// messages' size). Library scans over single words and single codes took 11
// launches and three waits, 125 us an encoding; this takes about 25.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "db.h"

namespace talek {
namespace {

constexpr uint32_t WG = 256;
constexpr uint32_t PER = 4;           // words per thread
constexpr uint32_t TILE = WG * PER;   // words per workgroup
constexpr uint64_t DIRECT = 1 << 16;  // body bytes that come by mapped memory

// What the passes of one encoding share, in device memory.
struct CodecState {
    uint64_t c, bits;
    uint32_t k;
    uint32_t done;  // workgroups of the running pass that have finished
};

// The result, in mapped host memory (or, without it, on the device): the body's
// first DIRECT bytes follow.
struct CodecResult {
    uint64_t c, bits, k, pad;
};

struct CodecArgs {
    const uint32_t *words;
    uint64_t W, m;
    uint32_t tiles;
    CodecState *st;
    uint64_t *count;   // per tile: set bits, then the position (+ 1) set before it
    uint64_t *length;  // per tile: its last position (+ 1), then its code bits, then their offset
    uint32_t *body;
    uint64_t body_words;
    CodecResult *result;
};

// Inclusive scan of one value per thread; *total is the workgroup's.
template <class Op>
__device__ __forceinline__ uint64_t scan(uint64_t v, Op op, uint64_t *waves, uint64_t *total)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t u = __shfl_up(v, d);
        if (lane >= (uint32_t)d)
            v = op(u, v);
    }
    __syncthreads();  // the last scan's readers are done with `waves`
    if (lane == 63)
        waves[wave] = v;
    __syncthreads();
    uint64_t before = 0, all = 0;
    for (uint32_t w = 0; w < WG / 64; ++w) {
        if (w == wave)
            before = all;
        all = op(all, waves[w]);
    }
    *total = all;
    return op(before, v);
}

struct Sum {
    __device__ __forceinline__ uint64_t operator()(uint64_t a, uint64_t b) const { return a + b; }
};
struct Max {
    __device__ __forceinline__ uint64_t operator()(uint64_t a, uint64_t b) const { return a > b ? a : b; }
};

// The value of the thread before this one (v inclusive; 0 for the first).
__device__ __forceinline__ uint64_t before(uint64_t v, uint64_t *all)
{
    __syncthreads();
    all[threadIdx.x] = v;
    __syncthreads();
    return threadIdx.x ? all[threadIdx.x - 1] : 0;
}

// Whether this is the pass's last workgroup; it sees what the others' first
// threads stored, and every atomic: each wave waits for its own before the
// barrier, which by itself waits for no other wave's memory operations. (One
// release a workgroup: a fence by every thread, each a write-back of the L2,
// took 20 us a pass.)
__device__ __forceinline__ bool last_workgroup(CodecState *st, uint32_t tiles)
{
    __shared__ bool last;
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) {
        last = __hip_atomic_fetch_add(&st->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == tiles - 1;
        if (last)
            st->done = 0;
    }
    __syncthreads();
    if (last)
        __threadfence();
    return last;
}

// This thread's words, bits at and past m cleared.
__device__ __forceinline__ void load_words(const CodecArgs &a, uint64_t w0, uint32_t (&v)[PER])
{
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        const uint64_t w = w0 + j;
        v[j] = w < a.W ? a.words[w] : 0u;
        if (w < a.W && w * 32 + 32 > a.m)
            v[j] &= (1u << (a.m - w * 32)) - 1u;
    }
}

// The highest position (+ 1) set in them, 0 for none.
__device__ __forceinline__ uint64_t last_position(const uint32_t (&v)[PER], uint64_t w0)
{
    uint64_t last = 0;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
        if (v[j])
            last = (w0 + j) * 32 + 32 - __clz(v[j]);
    return last;
}

// f(gap) for every set bit, `prev` the position (+ 1) set before them.
template <class F>
__device__ __forceinline__ void each_gap(const uint32_t (&v)[PER], uint64_t w0, uint64_t prev, F f)
{
    for (uint32_t j = 0; j < PER; ++j) {
        uint32_t x = v[j];
        while (x) {
            const uint64_t p = (w0 + j) * 32 + (__ffs(x) - 1);
            x &= x - 1;
            f(p - prev);
            prev = p + 1;
        }
    }
}

__global__ __launch_bounds__(WG) void codec_count_kernel(const CodecArgs a)
{
    __shared__ uint64_t waves[WG / 64];
    const uint64_t w0 = (uint64_t)blockIdx.x * TILE + threadIdx.x * PER;
    uint32_t v[PER];
    load_words(a, w0, v);
    uint64_t n = 0, sum, last;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
        n += __popc(v[j]);
    scan(n, Sum(), waves, &sum);
    scan(last_position(v, w0), Max(), waves, &last);
    if (threadIdx.x == 0) {
        a.count[blockIdx.x] = sum;
        a.length[blockIdx.x] = last;
    }
    for (uint64_t i = (uint64_t)blockIdx.x * WG + threadIdx.x; i < a.body_words; i += (uint64_t)gridDim.x * WG)
        a.body[i] = 0u;
    if (!last_workgroup(a.st, a.tiles))
        return;
    __shared__ uint64_t all[WG];
    uint64_t c = 0, prev = 0;
    for (uint32_t t0 = 0; t0 < a.tiles; t0 += WG) {
        const uint32_t t = t0 + threadIdx.x;
        const bool in = t < a.tiles;
        scan(in ? a.count[t] : 0, Sum(), waves, &sum);
        const uint64_t upto = scan(in ? a.length[t] : 0, Max(), waves, &last);
        const uint64_t b = before(upto, all);
        if (in)
            a.count[t] = prev > b ? prev : b;
        c += sum;
        prev = prev > last ? prev : last;
    }
    if (threadIdx.x == 0) {
        const uint64_t mean = a.m / (c + 1);
        a.st->c = c;
        a.st->k = mean > 1 ? 63 - __clzll((long long)mean) : 0;
    }
}

__global__ __launch_bounds__(WG) void codec_length_kernel(const CodecArgs a)
{
    __shared__ uint64_t waves[WG / 64], all[WG];
    const uint64_t w0 = (uint64_t)blockIdx.x * TILE + threadIdx.x * PER;
    const uint32_t k = a.st->k;
    uint32_t v[PER];
    load_words(a, w0, v);
    uint64_t sum, bits = 0;
    const uint64_t prev = before(scan(last_position(v, w0), Max(), waves, &sum), all);
    each_gap(v, w0, std::max<uint64_t>(prev, a.count[blockIdx.x]), [&](uint64_t g) { bits += (g >> k) + 1 + k; });
    scan(bits, Sum(), waves, &sum);
    if (threadIdx.x == 0)
        a.length[blockIdx.x] = sum;
    if (!last_workgroup(a.st, a.tiles))
        return;
    uint64_t at = 0;
    for (uint32_t t0 = 0; t0 < a.tiles; t0 += WG) {
        const uint32_t t = t0 + threadIdx.x;
        const uint64_t own = t < a.tiles ? a.length[t] : 0;
        const uint64_t upto = scan(own, Sum(), waves, &sum);
        if (t < a.tiles)
            a.length[t] = at + upto - own;
        at += sum;
    }
    if (threadIdx.x == 0) {
        a.st->bits = at;
        a.result->c = a.st->c;
        a.result->bits = at;
        a.result->k = k;
    }
}

// ORs the nb low bits of x (x = ~0: ones) into the body at bit `at`.
__device__ __forceinline__ void put(uint32_t *body, uint64_t at, uint64_t nb, uint64_t x, bool ones)
{
    while (nb) {
        const uint32_t s = (uint32_t)(at & 31), here = (uint32_t)std::min<uint64_t>(32 - s, nb);
        const uint32_t part = (ones ? ~0u : (uint32_t)x) & (here == 32 ? ~0u : (1u << here) - 1u);
        if (part)
            atomicOr(body + (at >> 5), part << s);
        x >>= here;
        at += here;
        nb -= here;
    }
}

__global__ __launch_bounds__(WG) void codec_write_kernel(const CodecArgs a)
{
    __shared__ uint64_t waves[WG / 64], all[WG];
    const uint64_t w0 = (uint64_t)blockIdx.x * TILE + threadIdx.x * PER;
    const uint32_t k = a.st->k;
    uint32_t v[PER];
    load_words(a, w0, v);
    uint64_t sum, bits = 0;
    uint64_t prev = before(scan(last_position(v, w0), Max(), waves, &sum), all);
    prev = std::max<uint64_t>(prev, a.count[blockIdx.x]);
    each_gap(v, w0, prev, [&](uint64_t g) { bits += (g >> k) + 1 + k; });
    uint64_t at = a.length[blockIdx.x] + scan(bits, Sum(), waves, &sum) - bits;
    each_gap(v, w0, prev, [&](uint64_t g) {
        const uint64_t q = g >> k;
        put(a.body, at, q, 0, true);
        put(a.body, at + q + 1, k, g, false);
        at += q + 1 + k;
    });
    if (!last_workgroup(a.st, a.tiles))
        return;
    const uint64_t words = std::min<uint64_t>((a.st->bits + 31) / 32, DIRECT / 4);
    uint32_t *to = reinterpret_cast<uint32_t *>(a.result + 1);
    for (uint64_t i = threadIdx.x; i < words; i += WG)
        to[i] = a.body[i];
}

}  // namespace

// Encode the m-bit device vector `words` into host memory; see the stream
// format above. out may be NULL (size query). Ordered on `s`, synchronous.
int encode_interest(pir_db *db, const uint32_t *words, uint64_t m, uint8_t *out, uint64_t cap, uint64_t *out_bytes,
                    hipStream_t s)
{
    const uint64_t W = (m + 31) / 32;
    if (W == 0 || W > 0x7fffffffull)
        return PIR_EINVAL;
    CodecArgs a{};
    a.words = words;
    a.W = W;
    a.m = m;
    a.tiles = (uint32_t)((W + TILE - 1) / TILE);
    // The codes take at most 3 m / 2 bits: c (k + 1) + (m - c) / 2^k with
    // c < m / 2^k for k > 0, and m for k = 0.
    const uint64_t body_words = (m + m / 2 + 31) / 32 + 1;
    if (!db->codec) {
        (void)host_mapped(sizeof(CodecResult) + DIRECT, &db->codec_host, &db->codec_map);
        const uint64_t result = db->codec_host ? 0 : sizeof(CodecResult) + DIRECT;
        int rc = ensure_device(&db->codec, &db->codec_cap, sizeof(CodecState) + result);
        if (rc == PIR_OK && launch_fill_zero(db->codec, sizeof(CodecState), s) != hipSuccess)
            rc = PIR_EDEVICE;
        if (rc != PIR_OK) {
            hipFree(db->codec);
            db->codec = nullptr;
            db->codec_cap = 0;
            if (db->codec_host)
                hipHostFree(db->codec_host);
            db->codec_host = nullptr;
            return rc;
        }
    }
    int rc = ensure_device(&db->codec2, &db->codec2_cap, 2ull * a.tiles * 8);
    if (rc != PIR_OK)
        return rc;
    a.st = static_cast<CodecState *>(db->codec);
    a.count = static_cast<uint64_t *>(db->codec2);
    a.length = a.count + a.tiles;
    a.result = db->codec_host ? static_cast<CodecResult *>(db->codec_map) : reinterpret_cast<CodecResult *>(a.st + 1);
    if (out) {
        rc = ensure_device(&db->codec3, &db->codec3_cap, body_words * 4);
        if (rc != PIR_OK)
            return rc;
        a.body = static_cast<uint32_t *>(db->codec3);
        a.body_words = body_words;
    }
    hipLaunchKernelGGL(codec_count_kernel, dim3(a.tiles), dim3(WG), 0, s, a);
    hipLaunchKernelGGL(codec_length_kernel, dim3(a.tiles), dim3(WG), 0, s, a);
    if (out)
        hipLaunchKernelGGL(codec_write_kernel, dim3(a.tiles), dim3(WG), 0, s, a);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return PIR_EDEVICE;
    CodecResult res;
    if (db->codec_host)
        res = *static_cast<const CodecResult *>(db->codec_host);
    else if (hipMemcpyAsync(&res, a.result, sizeof res, hipMemcpyDeviceToHost, s) != hipSuccess ||
             hipStreamSynchronize(s) != hipSuccess)
        return PIR_EDEVICE;
    if (res.c > 0x7fffffffull)  // the stream's documented limit
        return PIR_EINVAL;
    const uint64_t bytes = (res.bits + 7) / 8, total = 24 + bytes;
    if (out_bytes)
        *out_bytes = total;
    if (!out)
        return PIR_OK;
    if (cap < total)
        return PIR_EINVAL;
    for (int i = 0; i < 8; ++i) {
        out[i] = (uint8_t)(m >> (8 * i));
        out[8 + i] = (uint8_t)(res.c >> (8 * i));
    }
    for (int i = 0; i < 4; ++i) {
        out[16 + i] = (uint8_t)(res.k >> (8 * i));
        out[20 + i] = 0;
    }
    const uint64_t direct = db->codec_host ? std::min(bytes, DIRECT) : 0;
    if (direct)
        std::memcpy(out + 24, static_cast<const CodecResult *>(db->codec_host) + 1, direct);
    if (bytes > direct &&
        (hipMemcpyAsync(out + 24 + direct, reinterpret_cast<const uint8_t *>(a.body) + direct, bytes - direct,
                        hipMemcpyDeviceToHost, s) != hipSuccess ||
         hipStreamSynchronize(s) != hipSuccess))
        return PIR_EDEVICE;
    return PIR_OK;
}

}  // namespace talek
