// A HIP runtime of this program's own, in host memory, under the built library:
// the functions below take the place of the runtime's, so that the library's
// host code runs on the CPU. Kernels do not run; their launches are recorded by
// name. Each scenario checks what the host code allocates, copies, captures and
// launches, or how it goes on when an allocation fails.
//
//   fake_hip SCENARIO      exit status 0 = every check passed
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "talek_pir.h"

namespace {

// Host stub -> device name; the library registers its kernels before this
// file's own objects exist.
std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> k;
    return k;
}
std::vector<std::string> launches;
uint64_t pinned = 0, device_bytes = 0, captures = 0, replays = 0, copies = 0;
uint64_t pinned_fail_from = UINT64_MAX;  // pinned allocations of this many bytes and more fail
int handle = 0;                          // what streams, events and graphs point to

template <class T>
hipError_t give(T *out)
{
    *out = reinterpret_cast<T>(&handle);
    return hipSuccess;
}

uint64_t launched(const char *part)
{
    uint64_t c = 0;
    for (const std::string &s : launches)
        c += s.find(part) != std::string::npos;
    return c;
}

int failures = 0;
void check(bool ok, const char *what)
{
    if (!ok) {
        fprintf(stderr, "FAILED: %s\n", what);
        ++failures;
    }
}
#define CHECK(x) check((x), #x)

}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *stub, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    kernels()[stub] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, hipStream_t *s)
{
    *g = *b = dim3(1);
    *shared = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t)
{
    launches.push_back(kernels()[f]);
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t, hipEvent_t, hipEvent_t, int)
{
    launches.push_back(kernels()[f]);
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    device_bytes += n;
    return (*p = calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = n >= pinned_fail_from ? nullptr : calloc(n, 1);
    pinned += *p != nullptr;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **dev, void *host, unsigned)
{
    *dev = host;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    ++copies;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t)
{
    ++copies;
    for (size_t i = 0; i < h; ++i)
        memcpy(static_cast<char *>(d) + i * dp, static_cast<const char *>(s) + i * sp, w);
    return hipSuccess;
}

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = const_cast<void *>(s); return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return give(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return give(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return give(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { ++captures; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return give(g); }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) { return give(e); }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { ++replays; return hipSuccess; }
}

namespace {

struct Db {
    pir_db *h = nullptr;
    Db(uint64_t n, uint32_t d, uint32_t z) { CHECK(pir_db_create(n, d, z, &h) == PIR_OK); }
    ~Db() { pir_db_destroy(h); }
    int read(uint32_t B)
    {
        uint64_t n = 0, row = 0;
        pir_db_shape(h, &n, nullptr, nullptr, &row);
        std::vector<uint8_t> q(B * ((n + 7) / 8)), r(B * row);
        return pir_read_batch(h, q.data(), B, r.data());
    }
    int encode()
    {
        std::vector<uint8_t> out(1 << 16);
        uint64_t size = 0;
        return pir_interest_vector_encoded(h, out.data(), out.size(), &size);
    }
};

// A handle's first small read allocates no pinned memory and copies nothing.
void first_read()
{
    Db db(2632, 4, 1024);
    const uint64_t before = pinned, copied = copies;
    CHECK(db.read(1) == PIR_OK);
    CHECK(pinned == before);
    CHECK(launched("fetch_kernel") == 1 && copies == copied);
}

// Without pinned memory for them, such reads still are answered: requests and
// answers are copied.
void read_without_pinned_memory()
{
    pinned_fail_from = 1ull << 20;
    Db db(256, 1, 64);  // 16 KiB of staged rows
    pinned_fail_from = 0;
    for (int i = 0; i < 2; ++i)
        CHECK(db.read(3) == PIR_OK);
    CHECK(launched("fetch_kernel") == 0 && copies >= 4);
}

// Without pinned memory for the result, a code still is answered.
void code_without_pinned_memory()
{
    Db db(256, 1, 64);
    pinned_fail_from = 0;
    const uint64_t copied = copies;
    CHECK(db.encode() == PIR_OK && copies == copied + 1);
    pinned_fail_from = UINT64_MAX;
    CHECK(db.encode() == PIR_OK && copies == copied + 2);
}

// A matrix-core plan tuned for a plain database of the leaves' shape leaves
// their read as it is: staged together, one launch for all of them.
void tuned_leaves()
{
    char path[] = "/tmp/fake_hip_plans_XXXXXX";
    const int fd = mkstemp(path);
    FILE *f = fdopen(fd, "w");
    fprintf(f, "[\n {\"n\": 2048, \"bclass\": 256, \"stride\": 256, \"kind\": 5, \"tile\": 64, \"splits\": 2, "
               "\"unroll\": 4, \"flags\": 0, \"us\": 20.0}\n]\n");
    fclose(f);
    CHECK(pir_tune_load(path) == PIR_OK);
    remove(path);
    Db db(8192, 1, 1024);  // 49 leaves of 2048 rows of 256 bytes, 256 requests each
    CHECK(pir_preprocess(db.h, 2, 1) == PIR_OK);
    launches.clear();
    CHECK(db.read(1024) == PIR_OK);
    CHECK(launched("xorpir_mfma_kernel") == 0 && launched("xorpir_m4r") == 1);
    Db plain(2048, 1, 256);  // where the plan was tuned it is taken
    launches.clear();
    CHECK(plain.read(256) == PIR_OK);
    CHECK(launched("xorpir_mfma_kernel") == 1);
}

// A stream captured under one plan is not replayed under another, whichever
// fields differ.
void stream_plans()
{
    const uint64_t n = 32 * 65600;
    const uint32_t sizes[] = {5, 3}, B = 8;
    Db db(n, 1, 16);
    std::vector<uint8_t> q(B * n / 8), out(B * 16 + 16);
    void *resp = reinterpret_cast<void *>((reinterpret_cast<uintptr_t>(out.data()) + 15) & ~15ull);
    const pir_plan plans[] = {
        {PIR_KERNEL_MASK, 8, 65537, 4, 0},
        {PIR_KERNEL_MASK, 8, 1, 4, PIR_PLAN_SHARED_COLUMN},
        {PIR_KERNEL_MASK, 8, 1, 4, 0},
        {PIR_KERNEL_MASK, 8, 1, 4, PIR_PLAN_ONE_LAUNCH},
        {PIR_KERNEL_MFMA, 32, 3, 4, 0},
    };
    for (const pir_plan &p : plans)
        for (int again = 0; again < 2; ++again) {
            CHECK(pir_set_plan(db.h, &p) == PIR_OK);
            const uint64_t c = captures, r = replays;
            CHECK(pir_read_stream_async(db.h, q.data(), n / 8, sizes, nullptr, 2, resp, 16, nullptr, nullptr) == PIR_OK);
            CHECK(captures == c + !again && replays == r + 1);
        }
}

// Answers that kernels write where they belong take no scratch: the calls
// allocate the restaged requests and the splits' partial answers.
void answer_scratch()
{
    const uint64_t n = 8200, row = 999, B = 40, restaged = B * 1040;
    std::vector<uint8_t> q(B * 1026 + 1), out(B * 1001);
    for (bool sync : {false, true}) {
        Db db(n, 3, 333);
        const pir_plan p = {PIR_KERNEL_MFMA, 64, 4, 4, 0};
        CHECK(pir_set_plan(db.h, &p) == PIR_OK);
        const uint64_t before = device_bytes;
        CHECK((sync ? pir_read_batch(db.h, q.data(), B, out.data())
                    : pir_read_batch_async(db.h, q.data() + 1, 1026, B, out.data() + 1, 1000, nullptr)) == PIR_OK);
        CHECK(device_bytes - before == restaged + 4 * B * 1008);
        CHECK(B * row <= out.size() && launched("xor_splits_kernel") >= 1);
    }
}

}  // namespace

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> all = {
        {"first_read", first_read},
        {"read_without_pinned_memory", read_without_pinned_memory},
        {"code_without_pinned_memory", code_without_pinned_memory},
        {"tuned_leaves", tuned_leaves},
        {"stream_plans", stream_plans},
        {"answer_scratch", answer_scratch},
    };
    const auto it = argc > 1 ? all.find(argv[1]) : all.end();
    if (it == all.end())
        return 2;
    it->second();
    return failures ? 1 : 0;
}
