// Driver for wg_api.cpp on the CPU (test infrastructure): the C ABI's host code under
// -fsanitize=address,undefined with device memory played by malloc and the kernel launchers by functions
// that look at every table they are given.  Instances are added to a live handle while one allocation, copy
// or launch after the other fails: whatever a call that failed left behind, the next fill has to find tables
// that are there, states within them, and, where the arena is addressed by key, a row for every key.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../paper_2507_16768_amd/csrc/wg_device.h"

static long until_failure = -1;          // calls of the runtime that may fail before one does; -1: none does
static int failures = 0;

#define EXPECT(cond, ...) do { if (!(cond)) { std::printf("FAILED "); std::printf(__VA_ARGS__); std::printf("\n"); failures++; } } while (0)

static long copies = 0;                  // copies between host and device so far

static bool fails() { return until_failure >= 0 && until_failure-- == 0; }

static long until_bad_alloc = -1;        // the same for the host's own allocations
void *operator new(size_t n) {
    if (until_bad_alloc >= 0 && until_bad_alloc-- == 0) throw std::bad_alloc();
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void *operator new(size_t n, const std::nothrow_t &) noexcept { return std::malloc(n ? n : 1); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (fails()) return hipErrorOutOfMemory;
    *p = std::malloc(n ? n : 1);
    std::memset(*p, 0xA5, n);
    return hipSuccess;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { copies++; if (fails()) return hipErrorUnknown; std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void *d, int v, size_t n) { if (fails()) return hipErrorUnknown; std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipDeviceSynchronize(void) { return fails() ? hipErrorUnknown : hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return fails() ? hipErrorUnknown : hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)1 << 30; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorInvalidHandle; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "made up"; }
}

namespace wg {

// What the kernels take for granted of their tables.
static void look_at(const DeviceTable &T, const DeviceVocab &Vc, const DeviceCache &Cc) {
    uint64_t sum = 0;
    for (uint32_t sid = 0; sid < T.n_states; sid++) {
        const StateDesc d = T.states[sid];
        const uint32_t kind = d.kind_byte & 0xFFu;
        const uint32_t keys = kind == WG_KIND_WAIT && d.max != WG_UNBOUNDED ? T.lmax + 1u : 1u;
        EXPECT((uint64_t)d.key_base + keys <= Cc.n_keys, "state %u: keys from %u on, %u of them, %u in the table", sid, d.key_base, keys, Cc.n_keys);
        if (Cc.direct) EXPECT((uint64_t)d.key_base + keys <= Cc.cap_rows, "state %u: key %u of an arena of %u rows", sid, d.key_base + keys - 1u, Cc.cap_rows);
        for (uint32_t nt : {d.next_a, d.next_b, d.eos_next}) EXPECT(nt < T.n_states || nt == WG_SID_ERROR, "state %u: successor %u of %u", sid, nt, T.n_states);
        if (kind == WG_KIND_WAIT || kind == WG_KIND_COND) {
            sum += T.classes[(size_t)d.cls * 256u + 255u] + T.plans[d.cls].ids[259] + Cc.class_tags[d.cls];
            sum += Cc.class_rows[(size_t)(2u * d.cls + 2u) * Vc.row_stride - 1u];
            for (uint32_t x = 0; x < 256u; x++)
                EXPECT((T.codes[sid].word[x / 16u] >> 2u * (x % 16u) & 3u) == T.classes[(size_t)d.cls * 256u + x], "state %u: the code of byte value %u", sid, x);
        }
        sum += T.lit[sid];
    }
    for (uint32_t i = 0; i < 16u; i++) sum += T.lit[T.n_states + i];
    for (uint32_t k = 0; k < Cc.n_keys; k++) {
        sum += Cc.tags[k];
        if (!Cc.direct) sum += Cc.slots[k];
    }
    sum += Cc.arena[(size_t)Cc.cap_rows * Vc.row_stride - 1u];
    if (!Cc.direct && Cc.free_rows) sum += Cc.free_rows[Cc.cap_rows - 1u];
    if (sum == 1u) std::printf(" ");                 // (the reads are not to be left out)
}

FillPlan plan_fill(const DeviceVocab &, const DeviceCache &, uint32_t, bool, int, uint32_t) { return FillPlan{8u, false, false}; }
hipError_t launch_fill(const FillPlan &, const DeviceTable &T, const DeviceVocab &Vc, const DeviceCache &Cc, wg_state_t *, const int32_t *, uint32_t,
                       uint32_t *, void *, int, int64_t, hipStream_t, hipEvent_t *, hipEvent_t *) {
    look_at(T, Vc, Cc);
    for (uint32_t k = 0; k < 3u; k++) Cc.tags[k] = (unsigned long long)Cc.epoch << kTagEpochShift | 1ull;      // three keys have their rows
    return hipSuccess;
}
hipError_t launch_append(const AppendSlices &a, uint32_t n, hipStream_t) {
    if (fails()) return hipErrorUnknown;
    for (uint32_t i = 0; i < n; i++) std::memcpy(a.slice[i].dst, a.slice[i].src, a.slice[i].bytes);
    return hipSuccess;
}
hipError_t launch_count_rows(const DeviceCache &Cc, hipStream_t) {
    if (fails()) return hipErrorUnknown;
    for (uint32_t k = 0; k < Cc.n_keys; k++) Cc.ctr->held += (uint32_t)(Cc.tags[k] >> kTagEpochShift) == Cc.epoch;
    return hipSuccess;
}
hipError_t launch_free_rows(const DeviceCache &Cc, uint32_t n_keys, uint32_t *free_rows, hipStream_t) {
    if (fails()) return hipErrorUnknown;
    for (uint32_t i = 0; i < n_keys; i++) Cc.slots[i] = i;
    for (uint32_t i = 0; i < Cc.cap_rows; i++) free_rows[i] = i;
    return hipSuccess;
}
uint32_t rows_lds_bytes(const DeviceVocab &) { return 1024u; }
hipError_t static_topk_scratch(unsigned long long **out) { *out = nullptr; return hipSuccess; }
hipError_t launch_apply(void *, int, uint32_t, uint32_t, int64_t, const uint32_t *, hipStream_t, hipEvent_t *) { return hipSuccess; }
hipError_t launch_masked_argmax(const void *, int, uint32_t, uint32_t, int64_t, const uint32_t *, int32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_masked_topk(const void *, int, uint32_t, uint32_t, int64_t, const uint32_t *, uint32_t, int32_t *, void *, unsigned long long *,
                              hipStream_t) { return hipSuccess; }
hipError_t launch_advance(const DeviceTable &, const DeviceVocab &, const DeviceCache &, wg_state_t *, const int32_t *, uint32_t, uint32_t, hipStream_t,
                          hipEvent_t *) { return hipSuccess; }
hipError_t launch_forced_bytes(const DeviceTable &, const wg_state_t *, uint32_t, uint32_t, uint8_t *, uint32_t *, wg_state_t *, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_select(const uint32_t *, uint32_t, uint32_t, const uint64_t *, int32_t *, hipStream_t) { return hipSuccess; }

}  // namespace wg

// One handle; the addition's k-th call of the runtime (or host allocation) fails, and another addition follows.
static bool one(wg_vocab_t vocab, long k, bool host, uint32_t rows, const std::vector<std::string> &texts, bool clear_between) {
    const char *base = "Sequence(Write(\"ab\"), Wait(allow={a, b}, wait={c}, max=4))";
    wg_handle_t h = nullptr;
    wg_state_t start, more[4], states[2] = {};
    uint32_t mask[64];
    EXPECT(wg_compile(&base, nullptr, 1, vocab, WG_EOS_RESTART | (host ? WG_SHARE_STATES : 0u), &h, &start) == WG_OK, "compile: %s", wg_last_error());
    if (rows) EXPECT(wg_cache_resize(h, rows) == WG_OK, "resize: %s", wg_last_error());
    EXPECT(wg_fill_masks(h, states, 2, mask, nullptr) == WG_OK, "fill: %s", wg_last_error());
    std::vector<const char *> c;
    for (const auto &t : texts) c.push_back(t.c_str());
    long &until = host ? until_bad_alloc : until_failure;
    until = k;
    const int rc = wg_add_instances(h, c.data(), nullptr, (uint32_t)c.size(), more, nullptr);
    const bool failed = until < 0;
    until = -1;
    EXPECT(failed == (rc != WG_OK), "call %ld: status %d", k, rc);
    if (failed && host) EXPECT(rc == WG_ERR_NOMEM, "allocation %ld: status %d", k, rc);
    const uint32_t n_before = wg_num_instances(h);
    EXPECT(wg_fill_masks(h, states, 2, mask, nullptr) == WG_OK, "fill after a failure: %s", wg_last_error());
    if (clear_between) EXPECT(wg_cache_clear(h, nullptr) == WG_OK, "clear: %s", wg_last_error());
    const char *last = "Sequence(Write(\"z\"))";
    EXPECT(wg_add_instances(h, &last, nullptr, 1, more, nullptr) == WG_OK, "addition after a failure: %s", wg_last_error());
    EXPECT(wg_fill_masks(h, states, 2, mask, nullptr) == WG_OK, "fill at the end: %s", wg_last_error());
    EXPECT(wg_num_instances(h) == n_before + 1u, "%u instances after %u", wg_num_instances(h), n_before);
    EXPECT(wg_num_states(h) > more[0].sid, "%u states, the last instance starts at %u", wg_num_states(h), more[0].sid);
    wg_destroy(h);
    return failed;
}

int main() {
    const uint8_t bytes[] = "abcz";
    const uint64_t offsets[] = {0, 1, 2, 3, 4};
    wg_vocab_t vocab = nullptr;
    EXPECT(wg_vocab_create(bytes, offsets, 4, -1, &vocab) == WG_OK, "vocabulary: %s", wg_last_error());
    // more states and keys than there is room for, as many class tables, and slices too large for the staging memory
    std::string many = "Sequence(", tables = "Sequence(";
    for (int i = 0; i < 9000; i++) many += std::string(i ? ", " : "") + "Write(\"" + std::string(1 + i % 3, (char)('a' + i % 23)) + "\")";
    for (int i = 0; i < 120; i++) {
        char t[64];
        std::snprintf(t, sizeof t, "%sWait(allow={\\x%02X}, wait={\\xFF}, max=3)", i ? ", " : "", 0x20 + i);
        tables += t;
    }
    many += ")"; tables += ")";
    const std::vector<std::vector<std::string>> additions = {{"Sequence(Write(\"c\"))"}, {many}, {tables}, {many, tables, many + " "}};
    long calls = 0;
    for (const auto &a : additions)
        for (uint32_t rows : {0u, 8u, 30000u})
            for (int clear = 0; clear < 2; clear++)
                for (long k = 0;; k++) {
                    calls++;
                    if (!one(vocab, k, false, rows, a, clear != 0)) break;
                }
    // host memory runs out: nothing is thrown through the C entries
    for (const auto &a : std::vector<std::vector<std::string>>{additions[0], additions[2]})
        for (long k = 0;; k++) {
            calls++;
            if (!one(vocab, k, true, 0, a, false)) break;
        }
    // what the statistics cost does not grow with the keys
    for (const auto &text : {additions[0][0], many}) {
        wg_handle_t h = nullptr;
        const char *t = text.c_str();
        std::vector<wg_state_t> start(1);
        wg_state_t state{};
        uint32_t mask[1];
        wg_cache_stats_t s{};
        EXPECT(wg_compile(&t, nullptr, 1, vocab, WG_EOS_RESTART, &h, start.data()) == WG_OK, "compile: %s", wg_last_error());
        EXPECT(wg_cache_stats(h, &s) == WG_OK && s.rows_in_use == 0, "rows of a new handle: %llu", (unsigned long long)s.rows_in_use);
        EXPECT(wg_fill_masks(h, &state, 1, mask, nullptr) == WG_OK, "fill: %s", wg_last_error());
        for (int i = 0; i < 2; i++) {
            const long before = copies;
            EXPECT(wg_cache_stats(h, &s) == WG_OK && s.rows_in_use == 3, "rows in use: %llu", (unsigned long long)s.rows_in_use);
            EXPECT(copies - before <= 2, "%ld copies for %llu keys", copies - before, (unsigned long long)s.keys);
        }
        EXPECT(wg_cache_clear(h, nullptr) == WG_OK && wg_cache_stats(h, &s) == WG_OK && s.rows_in_use == 0, "rows after a clear: %llu", (unsigned long long)s.rows_in_use);
        wg_destroy(h);
    }
    wg_vocab_destroy(vocab);
    for (int what = 0; what < 2; what++)
        for (long k = 0;; k++) {
            wg_vocab_t v = nullptr;
            wg_handle_t h = nullptr;
            wg_state_t start;
            const char *text = "Sequence(Write(\"ab\"), Wait(allow={a, b}, wait={c}, max=4))";
            if (what) EXPECT(wg_vocab_create(bytes, offsets, 4, -1, &v) == WG_OK, "vocabulary: %s", wg_last_error());
            until_bad_alloc = k;
            const int rc = what ? wg_compile(&text, nullptr, 1, v, 0, &h, &start) : wg_vocab_create(bytes, offsets, 4, -1, &v);
            const bool failed = until_bad_alloc < 0;
            until_bad_alloc = -1;
            EXPECT(rc == (failed ? WG_ERR_NOMEM : WG_OK), "call %d, allocation %ld: status %d", what, k, rc);
            wg_destroy(h);
            wg_vocab_destroy(v);
            calls++;
            if (!failed) break;
        }
    std::printf("%ld additions, failures %d\n", calls, failures);
    return failures != 0;
}
