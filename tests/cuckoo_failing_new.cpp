// Host-only driver: a blocked cuckoo table whose allocations fail at chosen
// points (operator new throws). After every insertion that is refused with
// PIR_ENOMEM, and at the end, each occupied slot has to hold its own message's
// bytes and each free one zeros. Exit status 0 = every check passed.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "talek_pir.h"

extern "C" {
int pir_db_write_range(pir_db *, uint64_t, uint64_t, const uint8_t *) { return PIR_EINVAL; }
int pir_db_write_bucket(pir_db *, uint64_t, const uint8_t *) { return PIR_EINVAL; }
}

static bool failing = false;
void *operator new(size_t n)
{
    void *p = failing ? nullptr : malloc(n ? n : 1);
    if (!p)
        throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

static const uint32_t Z = 16;
static void payload(uint64_t id, uint8_t *out)
{
    for (uint32_t k = 0; k < Z; ++k)
        out[k] = (uint8_t)((id * 0x9E3779B97F4A7C15ull) >> (8 * (k % 8))) ^ (uint8_t)k;
}

// `fill` writes into n buckets of d slots, then `more`, every second of these
// under failing allocations.
static int run(uint64_t n, uint32_t d, uint64_t fill, uint64_t more, uint64_t seed, uint64_t *refused)
{
    pir_cuckoo *c = nullptr;
    if (pir_cuckoo_create_detached(n, d, Z, 0, seed, 100, &c) != PIR_OK)
        return 1;
    std::vector<uint8_t> table(n * d * Z), occ(n * d);
    std::vector<uint64_t> ids(n * d);
    uint64_t x = seed;
    auto draw = [&] { return (x = x * 6364136223846793005ull + 1442695040888963407ull) >> 33; };
    int bad = 0;
    for (uint64_t i = 1; i <= fill + more && !bad; ++i) {
        uint8_t p[Z], want[Z];
        payload(i, p);
        const uint64_t b1 = draw() % n, b2 = draw() % n;
        failing = i > fill && i % 2;
        const int rc = pir_cuckoo_insert(c, i, b1, b2, p, nullptr);
        failing = false;
        *refused += rc == PIR_ENOMEM;
        if (i <= fill)
            continue;
        pir_cuckoo_table(c, table.data(), table.size());
        pir_cuckoo_slots(c, ids.data(), occ.data());
        for (uint64_t s = 0; s < n * d && !bad; ++s) {
            payload(ids[s], want);
            if (!occ[s])
                memset(want, 0, Z);
            if (memcmp(want, table.data() + s * Z, Z)) {
                fprintf(stderr, "insertion %llu (rc %d): slot %llu does not hold message %llu\n",
                        (unsigned long long)i, rc, (unsigned long long)s, (unsigned long long)ids[s]);
                bad = 1;
            }
        }
    }
    pir_cuckoo_destroy(c);
    return bad;
}

int main()
{
    // the list of changed buckets outgrows its storage (at 256 and 512 of them)
    // within walks, which touch buckets for the first time
    int bad = 0;
    uint64_t refused = 0;
    for (uint64_t seed = 1; seed <= 60 && !bad; ++seed)
        bad = run(300 + seed, 1, 200 + seed, 160, seed, &refused) || run(540 + seed, 2, 900, 300, seed, &refused);
    printf("%llu insertions refused\n", (unsigned long long)refused);
    return bad || refused == 0;
}
