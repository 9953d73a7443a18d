// C ABI: handles, device uploads, argument checks, kernel launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <new>
#include <stdexcept>
#include <string>
#include <vector>

#include "wg_device.h"

namespace wg {
static thread_local std::string g_last_error;
void set_last_error(const std::string &msg) { g_last_error = msg; }
}  // namespace wg

using namespace wg;

struct wg_table_s {
    Lowering low;
    wg_table_s(uint32_t flags, uint32_t lmax) : low(flags, lmax) {}
};

struct wg_vocab_s {
    DeviceVocab dv{};
    uint8_t *d_len8 = nullptr;
    uint64_t *d_chunks = nullptr;
    ExitEntry *d_index = nullptr;
    uint32_t *d_dirs = nullptr, *d_rows = nullptr;
    int device = 0;
    void release() {
        (void)hipFree(d_len8); (void)hipFree(d_chunks); (void)hipFree(d_index); (void)hipFree(d_dirs); (void)hipFree(d_rows);
    }
};

struct wg_handle_s {
    wg_vocab_s *vocab = nullptr;
    Lowering low;
    DeviceTable dt{};
    DeviceCache dc{};
    // device copies of the table, with room to append (capacities in elements)
    ClassCodes *d_codes = nullptr;                    // the tables by state lie in one allocation, which begins here
    StateDesc *d_states = nullptr;
    uint8_t *d_lit = nullptr;
    uint8_t *d_classes = nullptr;
    ClassPlan *d_plans = nullptr;
    std::vector<ClassPlan> plans;                     // by class table
    std::vector<ClassCodes> codes;                    // the same
    uint32_t cap_states = 0, cap_classes = 0, cap_keys = 0;
    uint32_t up_states = 0, up_classes = 0;           // how much of the host table is on the device
    uint32_t max_batch = 0;
    uint32_t n_cu = 256;
    uint8_t *stage = nullptr;                  // pinned host memory, kStageBytes
    uint32_t *d_free_rows = nullptr;
    // kernel timing: events recorded since the last wg_profile_read
    bool profiling = false;
    // (begin / end pairs; a fill that does its lookups in its one kernel has no pair in lookup_events)
    std::vector<hipEvent_t> lookup_events, rows_events, advance_events, apply_events;
    std::vector<hipEvent_t> spare_events;
    wg_handle_s(uint32_t flags, uint32_t lmax) : low(flags, lmax) {}
};

namespace {

int fail(int code, const std::string &msg) { set_last_error(msg); return code; }

// What a C entry does, f, with the exceptions of the host's allocations turned into its status: they must
// not leave the library.  who: the entry's name with what went wrong.
template <typename F> int no_throw(const char *who, F f) {
    try {
        return f();
    } catch (const std::bad_alloc &) {
        try { set_last_error(who); } catch (...) {}
        return WG_ERR_NOMEM;
    }
}

// Additions up to this size are uploaded by one launch.  (Each page of it costs 1.5 us when it is first written: 128 and 256 instances took 3.0 and 5.2 ms
// to compile with 3 MiB of it, 2.7 and 4.3 with 1; 1,024 take 3.2 and 3.4 to add.)
constexpr size_t kStageBytes = 1u << 20;
constexpr uint32_t kDefaultBatch = 1024;   // requests per call a handle has room for after wg_compile

#define WG_HIP(call)                                                                          \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return fail(e_ == hipErrorOutOfMemory ? WG_ERR_NOMEM : WG_ERR_HIP,                \
                        std::string(#call) + ": " + hipGetErrorString(e_));                   \
    } while (0)

template <class T> hipError_t upload(T **dst, const T *src, size_t n) {
    hipError_t e = hipMalloc(reinterpret_cast<void **>(dst), (n ? n : 1) * sizeof(T));
    if (e != hipSuccess) return e;
    return n ? hipMemcpy(*dst, src, n * sizeof(T), hipMemcpyHostToDevice) : hipSuccess;
}

// A kernel's pair of timing events: taken before the launch, entered into the record once the kernel is
// launched (an event that no launch has recorded has no time to read), given back otherwise.
class Timing {
  public:
    Timing(wg_handle_s *h, bool on, std::vector<hipEvent_t> *record) : h_(h), record_(on && h->profiling ? record : nullptr) {
        if (!record_) return;
        try {                                          // room for the pair here and where it is given back, so that nothing throws later
            for (auto *v : {record_, &h->spare_events})
                if (v->capacity() < v->size() + 2) v->reserve(2 * v->size() + 64);
        } catch (const std::bad_alloc &) {
            record_ = nullptr;                         // not timed
            return;
        }
        for (hipEvent_t &e : ev_) {
            e = nullptr;
            if (!h->spare_events.empty()) { e = h->spare_events.back(); h->spare_events.pop_back(); }
            else (void)hipEventCreate(&e);
        }
    }
    ~Timing() {
        if (record_) record_->insert(record_->end(), ev_, ev_ + 2);
    }
    Timing(const Timing &) = delete;
    Timing &operator=(const Timing &) = delete;
    hipEvent_t *events() { return record_ ? ev_ : nullptr; }
    hipError_t launched(hipError_t e) {
        if (e != hipSuccess && record_) record_ = &h_->spare_events;
        return e;
    }

  private:
    wg_handle_s *h_;
    std::vector<hipEvent_t> *record_;
    hipEvent_t ev_[2];
};

// Room for the per-call lists of a batch of B requests.  Never called from the step path: the
// device is synchronised and the lists are allocated anew.
int reserve_batch(wg_handle_s *h, uint32_t B) {
    if (B <= h->max_batch) return WG_OK;
    WG_HIP(hipDeviceSynchronize());
    (void)hipFree(h->dc.row_ref);
    (void)hipFree(h->dc.tasks);
    h->dc.row_ref = nullptr; h->dc.tasks = nullptr; h->max_batch = 0;
    WG_HIP(hipMalloc(reinterpret_cast<void **>(&h->dc.row_ref), B * sizeof(uint32_t)));
    WG_HIP(hipMalloc(reinterpret_cast<void **>(&h->dc.tasks), B * sizeof(RowTask)));
    h->max_batch = B;
    return WG_OK;
}

// Gives *p room for new_n elements, keeping the first keep_n and zero-filling the rest.
template <class T> int regrow(T **p, size_t keep_n, size_t new_n) {
    T *q = nullptr;
    WG_HIP(hipMalloc(reinterpret_cast<void **>(&q), new_n * sizeof(T)));
    hipError_t e = hipMemset(q, 0, new_n * sizeof(T));
    if (e == hipSuccess && keep_n && *p) e = hipMemcpy(q, *p, keep_n * sizeof(T), hipMemcpyDeviceToDevice);
    if (e != hipSuccess) {
        (void)hipFree(q);
        return fail(WG_ERR_HIP, std::string("growing a device table: ") + hipGetErrorString(e));
    }
    (void)hipFree(*p);
    *p = q;
    return WG_OK;
}

uint32_t grown(uint32_t need, uint32_t floor_n) {
    uint64_t n = need < floor_n ? floor_n : need;
    n += n / 2;                                        // headroom for instances added later
    return n > 0xFFFFFFF0ull ? 0xFFFFFFF0u : (uint32_t)n;
}

// The same for the three tables by state, in one allocation.  (In one each, 100 additions of 16 mixed instances to a handle of 256 took 7.0 to 7.7 ms
// and the longest of them 0.74 to 1.0, now 5.4 to 6.2 and 0.23 to 0.44.)
int regrow_states(wg_handle_s *h, uint32_t new_n) {
    const uint32_t keep = h->up_states;
    ClassCodes *codes = nullptr;
    // the literal bytes are read 8 at a time: keep 16 zero bytes behind the last state
    const size_t bytes = (size_t)new_n * (sizeof(ClassCodes) + sizeof(StateDesc) + 1u) + 16u;
    WG_HIP(hipMalloc(reinterpret_cast<void **>(&codes), bytes));
    StateDesc *states = reinterpret_cast<StateDesc *>(codes + new_n);
    uint8_t *lit = reinterpret_cast<uint8_t *>(states + new_n);
    hipError_t e = hipMemset(codes, 0, bytes);
    if (e == hipSuccess && keep) e = hipMemcpy(codes, h->d_codes, keep * sizeof(ClassCodes), hipMemcpyDeviceToDevice);
    if (e == hipSuccess && keep) e = hipMemcpy(states, h->d_states, keep * sizeof(StateDesc), hipMemcpyDeviceToDevice);
    if (e == hipSuccess && keep) e = hipMemcpy(lit, h->d_lit, keep, hipMemcpyDeviceToDevice);
    if (e != hipSuccess) {
        (void)hipFree(codes);
        return fail(WG_ERR_HIP, std::string("growing a device table: ") + hipGetErrorString(e));
    }
    (void)hipFree(h->d_codes);
    h->d_codes = codes;
    h->d_states = states;
    h->d_lit = lit;
    return WG_OK;
}

// Room in the device tables for what the host table holds.  Beyond the reserved capacities the device is
// synchronised once and the tables move.
int grow_table(wg_handle_s *h, uint32_t n_states, uint32_t n_classes) {
    const Table &t = h->low.table;
    const uint32_t row_stride = h->dc.row_stride;
    if (t.n_keys > kMaxKeys) return fail(WG_ERR_NOMEM, "more than 2^31 - 2 cache keys");
    if (n_states > h->cap_states || n_classes > h->cap_classes || t.n_keys > h->cap_keys)
        WG_HIP(hipDeviceSynchronize());
    if (n_states > h->cap_states) {
        const uint32_t nc = grown(n_states, 4096);
        const int rc = regrow_states(h, nc);
        if (rc != WG_OK) return rc;
        h->cap_states = nc;
    }
    if (t.n_keys > h->cap_keys) {
        const uint32_t nc = grown(t.n_keys, 4096);
        int rc = regrow(&h->dc.tags, h->cap_keys, nc);
        if (rc == WG_OK) rc = regrow(&h->dc.slots, h->cap_keys, nc);
        if (rc != WG_OK) return rc;
        h->cap_keys = nc;
    }
    if (n_classes > h->cap_classes) {
        const uint32_t nc = grown(n_classes, 64);
        int rc = regrow(&h->d_classes, (size_t)h->up_classes * 256, (size_t)nc * 256);
        if (rc == WG_OK) rc = regrow(&h->d_plans, h->up_classes, nc);
        if (rc == WG_OK) rc = regrow(&h->dc.class_tags, h->cap_classes, nc);
        if (rc == WG_OK) rc = regrow(&h->dc.class_rows, (size_t)h->cap_classes * 2 * row_stride, (size_t)nc * 2 * row_stride);
        if (rc != WG_OK) return rc;
        h->cap_classes = nc;
    }
    return WG_OK;
}

// Brings the device copy of the table up to date with the host table after instances were
// appended: the new slices are copied, ordered on `s` with the caller's other work.  Where a step
// fails, what the kernels are given is as before the call (the tables perhaps at new addresses): the
// new states become known to them last, when everything they refer to is in place.
int sync_table(wg_handle_s *h, hipStream_t s) {
    const Table &t = h->low.table;
    const uint32_t n_states = (uint32_t)t.states.size(), n_classes = (uint32_t)(t.classes.size() / 256);
    const int rc = grow_table(h, n_states, n_classes);
    h->dt = DeviceTable{h->d_states, h->d_classes, h->d_plans, h->d_lit, h->d_codes, h->dt.n_states, t.lmax};
    if (rc != WG_OK) return rc;
    if (n_states > h->up_states || n_classes > h->up_classes) {
        const uint32_t s0 = h->up_states, ns = n_states - s0, c0 = h->up_classes, nc = n_classes - c0;
        h->plans.resize(n_classes);
        h->codes.resize(n_classes);
        for (uint32_t c = c0; c < n_classes; c++) {
            h->plans[c] = wide_plan_of(t.classes.data() + (size_t)c * 256);
            h->codes[c] = class_codes_of(t.classes.data() + (size_t)c * 256);
        }
        auto put_codes = [&](uint8_t *to, size_t at, size_t bytes) {        // of the new states
            for (uint32_t s = s0 + (uint32_t)(at / sizeof(ClassCodes)); bytes; s++, to += sizeof(ClassCodes), bytes -= sizeof(ClassCodes)) {
                const uint32_t kind = t.states[s].kind_byte & 0xFFu;
                if (kind == WG_KIND_WAIT || kind == WG_KIND_COND) std::memcpy(to, &h->codes[t.states[s].cls], sizeof(ClassCodes));
                else std::memset(to, 0, sizeof(ClassCodes));
            }
        };
        const struct { void *dst; const void *src; size_t bytes; } part[5] = {
            {h->d_codes + s0, nullptr, ns * sizeof(ClassCodes)},
            {h->d_states + s0, t.states.data() + s0, ns * sizeof(StateDesc)},
            {h->d_lit + s0, t.lit.data() + s0, ns},
            {h->d_classes + (size_t)c0 * 256, t.classes.data() + (size_t)c0 * 256, (size_t)nc * 256},
            {h->d_plans + c0, h->plans.data() + c0, nc * sizeof(ClassPlan)}};
        size_t all = 0;
        for (const auto &p : part) all += p.bytes ? p.bytes + 32u : 0u;
        // What fits into the pinned memory goes in one launch, more in halves of it: one is filled while the kernel reads the other.
        // (As copies from pageable memory, behind codes in memory of their own, 4,096 mixed instances took 20.6 ms to add, now 16.4.)
        const size_t room = all <= kStageBytes ? kStageBytes : kStageBytes / 2u;
        uint8_t *half = h->stage;
        AppendSlices slices{};
        uint32_t n = 0;
        size_t at = 0;
        bool reads = false;
        auto send = [&]() -> int {
            if (reads) WG_HIP(hipStreamSynchronize(s));              // (the other half, before it is filled again)
            WG_HIP(launch_append(slices, n, s));
            reads = true;
            half = half == h->stage ? h->stage + kStageBytes / 2u : h->stage;
            n = 0; at = 0;
            return WG_OK;
        };
        for (const auto &p : part)
            for (size_t done = 0; done < p.bytes;) {
                uint8_t *dst = static_cast<uint8_t *>(p.dst) + done;
                const size_t to = ((at + 15u) & ~(size_t)15u) + (reinterpret_cast<uintptr_t>(dst) & 15u);
                size_t take = p.bytes - done;
                if (to + take > room) take = to < room ? (room - to) / sizeof(ClassCodes) * sizeof(ClassCodes) : 0u;
                if (!take) {
                    const int sent = send();
                    if (sent != WG_OK) return sent;
                    continue;
                }
                if (p.src) std::memcpy(half + to, static_cast<const uint8_t *>(p.src) + done, take);
                else put_codes(half + to, done, take);
                slices.slice[n++] = AppendSlice{dst, half + to, (uint32_t)take};
                at = to + take;
                done += take;
            }
        const int sent = send();
        if (sent != WG_OK) return sent;
        // (what is copied from is filled again by a later append)
        WG_HIP(hipStreamSynchronize(s));
        h->up_states = n_states;
        h->up_classes = n_classes;
    }
    if (h->dc.direct && t.n_keys > h->dc.cap_rows) {
        // more keys than rows from now on: the rows in use stay where they are, the others are handed out
        // in order of first use
        if (!h->d_free_rows) WG_HIP(hipMalloc(reinterpret_cast<void **>(&h->d_free_rows), (size_t)h->dc.cap_rows * sizeof(uint32_t)));
        WG_HIP(launch_free_rows(h->dc, h->dc.n_keys, h->d_free_rows, s));
        h->dc.direct = 0;
        h->dc.free_rows = h->d_free_rows;
    }
    h->dc.n_keys = t.n_keys;
    h->dt.n_states = n_states;
    return WG_OK;
}

int set_cache_rows(wg_handle_s *h, uint32_t rows) {
    const size_t row_bytes = (size_t)h->dc.row_stride * 4u;
    uint32_t *arena = nullptr;
    WG_HIP(hipMalloc(reinterpret_cast<void **>(&arena), (size_t)rows * row_bytes + 16));
    (void)hipFree(h->dc.arena);
    h->dc.arena = arena;
    h->dc.cap_rows = rows;
    (void)hipFree(h->d_free_rows);                     // (it has a place for every row)
    h->d_free_rows = nullptr;
    h->dc.free_rows = nullptr;
    return WG_OK;
}

// A new cache generation: every row and class index made so far is stale from the next call on.
int next_generation(wg_handle_s *h, hipStream_t s) {
    h->dc.direct = h->dc.n_keys <= h->dc.cap_rows;
    h->dc.free_rows = nullptr;
    if (++h->dc.epoch >= (1u << 30)) {                 // out of generation numbers: reset the tags for real
        WG_HIP(hipMemsetAsync(h->dc.tags, 0, (size_t)h->cap_keys * sizeof(unsigned long long), s));
        WG_HIP(hipMemsetAsync(h->dc.class_tags, 0, (size_t)h->cap_classes * sizeof(unsigned long long), s));
        WG_HIP(hipMemsetAsync(&h->dc.ctr->slot_ctr, 0, sizeof(unsigned long long), s));
        h->dc.epoch = 1;
    }
    return WG_OK;
}

}  // namespace

extern "C" {

const char *wg_last_error(void) { return g_last_error.c_str(); }

// ---- vocabulary ------------------------------------------------------------------------------

static int create_vocab(const uint8_t *host_bytes, const uint64_t *host_offsets, uint32_t V,
                        int32_t eos_id, wg_vocab_t *out) {
    if (!out) return fail(WG_ERR_INVALID, "wg_vocab_create: out is null");
    *out = nullptr;
    if (!host_offsets || V == 0) return fail(WG_ERR_INVALID, "wg_vocab_create: empty vocabulary");
    if (eos_id >= (int64_t)V) return fail(WG_ERR_INVALID, "wg_vocab_create: eos_id outside the vocabulary");
    VocabIndex ix;
    {
        std::string err;
        const int rc = build_vocab_index(host_bytes, host_offsets, V, eos_id, &ix, &err);
        if (rc != WG_OK) return fail(rc, err);
    }
    std::unique_ptr<wg_vocab_s, void (*)(wg_vocab_t)> v(new (std::nothrow) wg_vocab_s, wg_vocab_destroy);
    if (!v) return fail(WG_ERR_NOMEM, "wg_vocab_create: out of host memory");
    WG_HIP(hipGetDevice(&v->device));
    {
        // set-up time on this device: the address of the library's own top-k workspace is asked
        // for here, so that wg_masked_topk_static finds it known (it asks itself otherwise)
        unsigned long long *unused = nullptr;
        (void)static_topk_scratch(&unused);
    }
    std::vector<ExitEntry> index;
    std::vector<uint32_t> dirs;
    if (!candidates(ix, &index, &dirs)) return fail(WG_ERR_INVALID, "wg_vocab_create: the candidate indexes have more than 2^32 entries");
    const std::vector<uint32_t> rows = token_rows(ix);
    hipError_t e = upload(&v->d_len8, ix.len8.data(), ix.len8.size());
    if (e == hipSuccess) e = upload(&v->d_chunks, ix.chunks.data(), ix.chunks.size());
    if (e == hipSuccess) e = upload(&v->d_rows, rows.data(), rows.size());
    if (e == hipSuccess) e = upload(&v->d_index, index.data(), index.size());
    if (e == hipSuccess) e = upload(&v->d_dirs, dirs.data(), dirs.size());
    if (e != hipSuccess)
        return fail(e == hipErrorOutOfMemory ? WG_ERR_NOMEM : WG_ERR_HIP,
                    std::string("wg_vocab_create: ") + hipGetErrorString(e));
    v->dv = DeviceVocab{v->d_len8, v->d_chunks, v->d_rows, v->d_index, v->d_dirs, V, ix.W, eos_id, ix.lmax, ix.n_chunks, ix.row_stride};
    *out = v.release();
    return WG_OK;
}

int wg_vocab_create(const uint8_t *host_bytes, const uint64_t *host_offsets, uint32_t V,
                    int32_t eos_id, wg_vocab_t *out) {
    return no_throw("wg_vocab_create: out of host memory", [&] { return create_vocab(host_bytes, host_offsets, V, eos_id, out); });
}

void wg_vocab_destroy(wg_vocab_t v) {
    if (!v) return;
    v->release();
    delete v;
}

// ---- lowering (host only) ----------------------------------------------------------------------

int wg_lower(const char *const *templates, const wg_args_t *args, uint32_t n_templates,
             uint32_t flags, uint32_t lmax, wg_table_t *out) {
    if (!out) return fail(WG_ERR_INVALID, "wg_lower: out is null");
    *out = nullptr;
    if (!templates || n_templates == 0) return fail(WG_ERR_INVALID, "wg_lower: no templates");
    if (flags & ~(uint32_t)(WG_EOS_RESTART | WG_SHARE_STATES)) return fail(WG_ERR_INVALID, "wg_lower: unknown flag bits");
    try {
        std::unique_ptr<wg_table_s> t(new wg_table_s(flags, lmax));
        t->low.add(templates, args, n_templates);
        *out = t.release();
        return WG_OK;
    } catch (const std::bad_alloc &) {
        return fail(WG_ERR_NOMEM, "wg_lower: out of host memory");
    } catch (const std::exception &e) {
        return fail(WG_ERR_PARSE, e.what());
    }
}

int wg_table_add_instances(wg_table_t t, const char *const *templates, const wg_args_t *args,
                           uint32_t n_templates) {
    if (!t) return fail(WG_ERR_INVALID, "wg_table_add_instances: null table");
    if (!templates || n_templates == 0) return fail(WG_ERR_INVALID, "wg_table_add_instances: no templates");
    try {
        t->low.add(templates, args, n_templates);
        return WG_OK;
    } catch (const std::bad_alloc &) {
        return fail(WG_ERR_NOMEM, "wg_table_add_instances: out of host memory");
    } catch (const std::exception &e) {
        return fail(WG_ERR_PARSE, e.what());
    }
}

int wg_regex_to_template(const char *regex, char *out, uint64_t capacity, uint64_t *needed) {
    if (!regex) return fail(WG_ERR_INVALID, "wg_regex_to_template: regex is null");
    try {
        const std::string text = regex_to_template(regex);
        if (needed) *needed = text.size() + 1;
        if (!out || capacity < text.size() + 1)
            return fail(WG_ERR_INVALID, "wg_regex_to_template: the template needs " +
                                            std::to_string(text.size() + 1) + " bytes");
        std::memcpy(out, text.c_str(), text.size() + 1);
        return WG_OK;
    } catch (const std::bad_alloc &) {
        return fail(WG_ERR_NOMEM, "wg_regex_to_template: out of host memory");
    } catch (const std::exception &e) {
        return fail(WG_ERR_PARSE, e.what());
    }
}

uint32_t wg_table_num_instances(wg_table_t t) { return t ? (uint32_t)t->low.table.start.size() : 0; }

uint32_t wg_table_num_states(wg_table_t t) { return t ? (uint32_t)t->low.table.states.size() : 0; }

uint32_t wg_table_start_state(wg_table_t t, uint32_t i) {
    return (t && i < t->low.table.start.size()) ? t->low.table.start[i] : WG_SID_ERROR;
}

int wg_table_state(wg_table_t t, uint32_t sid, wg_state_info_t *out) {
    if (!t || !out || sid >= t->low.table.states.size()) return fail(WG_ERR_INVALID, "wg_table_state: bad argument");
    const Table &tb = t->low.table;
    const StateDesc &d = tb.states[sid];
    out->kind = d.kind_byte & 0xFFu; out->byte = (d.kind_byte >> 8) & 0xFFu;
    out->next_a = d.next_a; out->next_b = d.next_b; out->eos_next = d.eos_next; out->max = d.max;
    out->tmpl = tb.tmpl[sid]; out->n_keys = tb.key_count[sid]; out->key = d.key_base;
    return WG_OK;
}

int wg_table_symbol_class(wg_table_t t, uint32_t sid, uint32_t symbol) {
    if (!t || sid >= t->low.table.states.size() || symbol > kSymEos) return fail(WG_ERR_INVALID, "wg_table_symbol_class: bad argument");
    const StateDesc &d = t->low.table.states[sid];
    uint32_t kind = d.kind_byte & 0xFFu;
    if (symbol == kSymEos) return d.eos_next == WG_SID_ERROR ? CLS_REJECT : CLS_EXIT_A;
    if (kind == WG_KIND_LIT) return symbol == ((d.kind_byte >> 8) & 0xFFu) ? CLS_EXIT_A : CLS_REJECT;
    if (kind == WG_KIND_WAIT || kind == WG_KIND_COND) return t->low.table.classes[(size_t)d.cls * 256 + symbol];
    return CLS_REJECT;
}

void wg_table_destroy(wg_table_t t) { delete t; }

// ---- compile ------------------------------------------------------------------------------------

void wg_destroy(wg_handle_t h) {
    if (!h) return;
    (void)hipDeviceSynchronize();
    (void)hipFree(h->d_codes); (void)hipFree(h->d_classes); (void)hipFree(h->d_plans);
    (void)hipFree(h->dc.ctr); (void)hipFree(h->dc.tags); (void)hipFree(h->dc.slots);
    (void)hipFree(h->dc.arena); (void)hipFree(h->dc.row_ref); (void)hipFree(h->dc.tasks);
    if (h->stage) (void)hipHostFree(h->stage);
    (void)hipFree(h->d_free_rows);
    (void)hipFree(h->dc.class_tags); (void)hipFree(h->dc.class_rows);
    for (auto *v : {&h->lookup_events, &h->rows_events, &h->advance_events, &h->apply_events, &h->spare_events})
        for (hipEvent_t e : *v) if (e) (void)hipEventDestroy(e);
    delete h;
}

static int compile(const char *const *templates, const wg_args_t *args, uint32_t n_templates,
                   wg_vocab_t vocab, uint32_t flags, wg_handle_t *out, wg_state_t *start_states_out) {
    if (!out) return fail(WG_ERR_INVALID, "wg_compile: out is null");
    *out = nullptr;
    if (!vocab) return fail(WG_ERR_INVALID, "wg_compile: vocab is null");
    if (!templates || n_templates == 0) return fail(WG_ERR_INVALID, "wg_compile: no templates");
    if (flags & ~(uint32_t)(WG_EOS_RESTART | WG_SHARE_STATES)) return fail(WG_ERR_INVALID, "wg_compile: unknown flag bits");
    std::unique_ptr<wg_handle_s, void (*)(wg_handle_t)> h(
        new (std::nothrow) wg_handle_s(flags, vocab->dv.lmax), wg_destroy);
    if (!h) return fail(WG_ERR_NOMEM, "wg_compile: out of host memory");
    try {
        h->low.add(templates, args, n_templates);
    } catch (const std::bad_alloc &) {
        throw;
    } catch (const std::exception &e) {
        return fail(WG_ERR_PARSE, e.what());
    }
    h->vocab = vocab;
    const Table &t = h->low.table;
    WG_HIP(hipSetDevice(vocab->device));
    const uint32_t row_stride = vocab->dv.row_stride;
    const uint64_t row_bytes = (uint64_t)row_stride * 4ull;
    if (rows_lds_bytes(vocab->dv) > kRowsLdsMax)
        return fail(WG_ERR_INVALID, "wg_compile: a share of a mask row does not fit the LDS of the row builder (vocabulary too large)");
    h->dc.row_stride = row_stride;
    h->dc.epoch = 1;                                   // tags start at 0 = never built

    // The row cache: room for every key of the instances given here (at least 4096 rows), but
    // no more than a quarter of the free device memory; keys beyond it are served uncached.
    size_t free_b = 0, total_b = 0;
    WG_HIP(hipMemGetInfo(&free_b, &total_b));
    const uint64_t n_classes = t.classes.size() / 256;
    const uint64_t class_bytes = n_classes * 2ull * row_bytes;
    if (class_bytes > (uint64_t)free_b / 4)
        return fail(WG_ERR_NOMEM, "wg_compile: the class indexes (" + std::to_string(class_bytes >> 20) +
                                      " MiB for " + std::to_string(n_classes) +
                                      " allow / wait set tables) exceed a quarter of the free device memory");
    uint64_t rows = t.n_keys < 4096u ? 4096u : t.n_keys;
    const uint64_t fit = (uint64_t)free_b / 4 / row_bytes;
    if (rows > fit) rows = fit ? fit : 1;
    if (rows > kMaxRows) rows = kMaxRows;

    WG_HIP(hipMalloc(reinterpret_cast<void **>(&h->dc.ctr), sizeof(Control)));
    WG_HIP(hipMemset(h->dc.ctr, 0, sizeof(Control)));
    int cus = 0;
    WG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, vocab->device));
    if (cus > 0) h->n_cu = (uint32_t)cus;
    WG_HIP(hipHostMalloc(reinterpret_cast<void **>(&h->stage), kStageBytes, hipHostMallocDefault));
    int rc = set_cache_rows(h.get(), (uint32_t)rows);
    if (rc == WG_OK) rc = sync_table(h.get(), nullptr);
    h->dc.direct = t.n_keys <= h->dc.cap_rows;
    if (rc == WG_OK) rc = reserve_batch(h.get(), kDefaultBatch);
    if (rc != WG_OK) return rc;
    WG_HIP(hipDeviceSynchronize());
    if (start_states_out)
        for (uint32_t i = 0; i < n_templates; i++) start_states_out[i] = wg_state_t{t.start[i], 0u};
    *out = h.release();
    return WG_OK;
}

int wg_compile(const char *const *templates, const wg_args_t *args, uint32_t n_templates,
               wg_vocab_t vocab, uint32_t flags, wg_handle_t *out, wg_state_t *start_states_out) {
    return no_throw("wg_compile: out of host memory", [&] { return compile(templates, args, n_templates, vocab, flags, out, start_states_out); });
}

static int add_instances(wg_handle_t h, const char *const *templates, const wg_args_t *args,
                         uint32_t n_templates, wg_state_t *start_states_out, void *stream) {
    if (!h) return fail(WG_ERR_INVALID, "wg_add_instances: null handle");
    if (!templates || n_templates == 0) return fail(WG_ERR_INVALID, "wg_add_instances: no templates");
    const size_t first = h->low.table.start.size();
    try {
        h->low.add(templates, args, n_templates);
    } catch (const std::bad_alloc &) {
        throw;
    } catch (const std::exception &e) {
        return fail(WG_ERR_PARSE, e.what());
    }
    WG_HIP(hipSetDevice(h->vocab->device));
    int rc = sync_table(h, static_cast<hipStream_t>(stream));
    if (rc != WG_OK) return rc;
    if (start_states_out)
        for (uint32_t i = 0; i < n_templates; i++)
            start_states_out[i] = wg_state_t{h->low.table.start[first + i], 0u};
    return WG_OK;
}

int wg_add_instances(wg_handle_t h, const char *const *templates, const wg_args_t *args,
                     uint32_t n_templates, wg_state_t *start_states_out, void *stream) {
    return no_throw("wg_add_instances: out of host memory", [&] { return add_instances(h, templates, args, n_templates, start_states_out, stream); });
}

int wg_cache_resize(wg_handle_t h, uint32_t rows) {
    if (!h) return fail(WG_ERR_INVALID, "wg_cache_resize: null handle");
    if (rows == 0 || rows > kMaxRows) return fail(WG_ERR_INVALID, "wg_cache_resize: rows must be 1 .. 2^30");
    WG_HIP(hipSetDevice(h->vocab->device));
    WG_HIP(hipDeviceSynchronize());
    int rc = set_cache_rows(h, rows);
    if (rc != WG_OK) return rc;
    return next_generation(h, nullptr);
}

int wg_reserve_batch(wg_handle_t h, uint32_t max_batch) {
    if (!h) return fail(WG_ERR_INVALID, "wg_reserve_batch: null handle");
    if (max_batch == 0 || max_batch > kMaxBatch) return fail(WG_ERR_INVALID, "wg_reserve_batch: max_batch must be 1 .. 65535");
    WG_HIP(hipSetDevice(h->vocab->device));
    return reserve_batch(h, max_batch);
}

uint32_t wg_max_batch(wg_handle_t h) { return h ? h->max_batch : 0; }

int wg_set_scan_batch(wg_handle_t h, uint32_t tables) {
    if (!h) return fail(WG_ERR_INVALID, "wg_set_scan_batch: null handle");
    if (tables > 8u) return fail(WG_ERR_INVALID, "wg_set_scan_batch: tables must be 0 .. 8");
    return WG_OK;                                      // (masks are made without a scan of class tables)
}

uint32_t wg_num_instances(wg_handle_t h) { return h ? (uint32_t)h->low.table.start.size() : 0; }
uint32_t wg_num_states(wg_handle_t h) { return h ? h->dt.n_states : 0; }
uint32_t wg_mask_words(wg_handle_t h) { return h ? h->vocab->dv.W : 0; }

// ---- per-step calls -----------------------------------------------------------------------------

namespace {
int fill(wg_handle_t h, wg_state_t *d_states, const int32_t *d_tokens, uint32_t B, uint32_t *d_bitmask,
         void *stream, const char *who, void *d_logits = nullptr, int dtype = WG_F32, int64_t logits_stride = 0) {
    if (B == 0) return fail(WG_ERR_INVALID, std::string(who) + ": B is 0");
    if (B > kMaxBatch) return fail(WG_ERR_INVALID, std::string(who) + ": B above 65535");
    if (B > h->max_batch)
        return fail(WG_ERR_INVALID, std::string(who) + ": B = " + std::to_string(B) + " is above the " +
                                        std::to_string(h->max_batch) + " requests the handle has room for (wg_reserve_batch)");
    const FillPlan plan = plan_fill(h->vocab->dv, h->dc, B, d_logits != nullptr, dtype, h->n_cu);
    Timing lookup(h, !plan.one_kernel, &h->lookup_events), rows(h, true, &h->rows_events);
    const hipError_t e = launch_fill(plan, h->dt, h->vocab->dv, h->dc, d_states, d_tokens, B, d_bitmask, d_logits, dtype, logits_stride,
                                     static_cast<hipStream_t>(stream), lookup.events(), rows.events());
    (void)lookup.launched(e);
    WG_HIP(rows.launched(e));
    return WG_OK;
}
}  // namespace

int wg_fill_masks(wg_handle_t h, const wg_state_t *d_states, uint32_t B, uint32_t *d_bitmask,
                  void *stream) {
    if (!h || !d_states || !d_bitmask) return fail(WG_ERR_INVALID, "wg_fill_masks: null argument");
    // the states are only read when no tokens are given
    return fill(h, const_cast<wg_state_t *>(d_states), nullptr, B, d_bitmask, stream, "wg_fill_masks");
}

int wg_advance_fill_masks(wg_handle_t h, wg_state_t *d_states, const int32_t *d_tokens, uint32_t B,
                          uint32_t *d_bitmask, void *stream) {
    if (!h || !d_states || !d_tokens || !d_bitmask)
        return fail(WG_ERR_INVALID, "wg_advance_fill_masks: null argument");
    return fill(h, d_states, d_tokens, B, d_bitmask, stream, "wg_advance_fill_masks");
}

int wg_decode_step(wg_handle_t h, wg_state_t *d_states, const int32_t *d_tokens, uint32_t B,
                   uint32_t *d_bitmask, void *d_logits, wg_dtype_t dtype, int64_t row_stride_elems,
                   void *stream) {
    if (!h || !d_states || !d_bitmask || !d_logits) return fail(WG_ERR_INVALID, "wg_decode_step: null argument");
    if (dtype != WG_F32 && dtype != WG_BF16) return fail(WG_ERR_INVALID, "wg_decode_step: unknown dtype");
    if (row_stride_elems < (int64_t)h->vocab->dv.V) return fail(WG_ERR_INVALID, "wg_decode_step: row stride smaller than V");
    return fill(h, d_states, d_tokens, B, d_bitmask, stream, "wg_decode_step", d_logits, dtype, row_stride_elems);
}

int wg_apply_mask(void *d_logits, wg_dtype_t dtype, uint32_t B, uint32_t V, int64_t row_stride_elems,
                  const uint32_t *d_bitmask, void *stream) {
    if (!d_logits || !d_bitmask) return fail(WG_ERR_INVALID, "wg_apply_mask: null argument");
    if (B == 0 || V == 0) return fail(WG_ERR_INVALID, "wg_apply_mask: empty batch or vocabulary");
    if (dtype != WG_F32 && dtype != WG_BF16) return fail(WG_ERR_INVALID, "wg_apply_mask: unknown dtype");
    if (row_stride_elems < (int64_t)V) return fail(WG_ERR_INVALID, "wg_apply_mask: row stride smaller than V");
    if (B > kMaxBatch) return fail(WG_ERR_INVALID, "wg_apply_mask: B above 65535");
    WG_HIP(launch_apply(d_logits, dtype, B, V, row_stride_elems, d_bitmask, static_cast<hipStream_t>(stream), nullptr));
    return WG_OK;
}

int wg_profile_apply_mask(wg_handle_t h, void *d_logits, wg_dtype_t dtype, uint32_t B, uint32_t V,
                          int64_t row_stride_elems, const uint32_t *d_bitmask, void *stream) {
    if (!h) return fail(WG_ERR_INVALID, "wg_profile_apply_mask: null handle");
    if (!h->profiling) return wg_apply_mask(d_logits, dtype, B, V, row_stride_elems, d_bitmask, stream);
    if (!d_logits || !d_bitmask) return fail(WG_ERR_INVALID, "wg_profile_apply_mask: null argument");
    if (B == 0 || V == 0 || B > kMaxBatch) return fail(WG_ERR_INVALID, "wg_profile_apply_mask: bad batch or vocabulary size");
    if (dtype != WG_F32 && dtype != WG_BF16) return fail(WG_ERR_INVALID, "wg_profile_apply_mask: unknown dtype");
    if (row_stride_elems < (int64_t)V) return fail(WG_ERR_INVALID, "wg_profile_apply_mask: row stride smaller than V");
    Timing apply(h, true, &h->apply_events);
    WG_HIP(apply.launched(launch_apply(d_logits, dtype, B, V, row_stride_elems, d_bitmask, static_cast<hipStream_t>(stream), apply.events())));
    return WG_OK;
}

int wg_masked_argmax(const void *d_logits, wg_dtype_t dtype, uint32_t B, uint32_t V,
                     int64_t row_stride_elems, const uint32_t *d_bitmask, int32_t *d_tokens, void *stream) {
    if (!d_logits || !d_bitmask || !d_tokens) return fail(WG_ERR_INVALID, "wg_masked_argmax: null argument");
    if (B == 0 || V == 0) return fail(WG_ERR_INVALID, "wg_masked_argmax: empty batch or vocabulary");
    if (dtype != WG_F32 && dtype != WG_BF16) return fail(WG_ERR_INVALID, "wg_masked_argmax: unknown dtype");
    if (row_stride_elems < (int64_t)V) return fail(WG_ERR_INVALID, "wg_masked_argmax: row stride smaller than V");
    if (B > kMaxBatch) return fail(WG_ERR_INVALID, "wg_masked_argmax: B above 65535");
    WG_HIP(launch_masked_argmax(d_logits, dtype, B, V, row_stride_elems, d_bitmask, d_tokens,
                                static_cast<hipStream_t>(stream)));
    return WG_OK;
}

uint64_t wg_masked_topk_workspace(uint32_t B, uint32_t V, uint32_t k) {
    const uint64_t n_slices = ((uint64_t)V + kTopkSlice - 1u) / kTopkSlice;
    return (uint64_t)B * n_slices * k * sizeof(unsigned long long);
}

int wg_masked_topk(const void *d_logits, wg_dtype_t dtype, uint32_t B, uint32_t V, int64_t row_stride_elems,
                   const uint32_t *d_bitmask, uint32_t k, int32_t *d_ids, void *d_values,
                   void *d_workspace, uint64_t workspace_bytes, void *stream) {
    if (!d_logits || !d_bitmask || !d_ids || !d_values || !d_workspace)
        return fail(WG_ERR_INVALID, "wg_masked_topk: null argument");
    if (B == 0 || V == 0) return fail(WG_ERR_INVALID, "wg_masked_topk: empty batch or vocabulary");
    if (dtype != WG_F32 && dtype != WG_BF16) return fail(WG_ERR_INVALID, "wg_masked_topk: unknown dtype");
    if (row_stride_elems < (int64_t)V) return fail(WG_ERR_INVALID, "wg_masked_topk: row stride smaller than V");
    if (B > kMaxBatch) return fail(WG_ERR_INVALID, "wg_masked_topk: B above 65535");
    if (k == 0 || k > kTopkMax) return fail(WG_ERR_INVALID, "wg_masked_topk: k must be 1 .. 64");
    const uint64_t n_slices = ((uint64_t)V + kTopkSlice - 1u) / kTopkSlice;
    if (n_slices * k > kTopkMergeKeys)
        return fail(WG_ERR_INVALID, "wg_masked_topk: ceil(V / 8192) * k above 4096 (the lists of a row do not fit the merge)");
    if (workspace_bytes < wg_masked_topk_workspace(B, V, k))
        return fail(WG_ERR_INVALID, "wg_masked_topk: the workspace needs " +
                                        std::to_string(wg_masked_topk_workspace(B, V, k)) + " bytes");
    if (reinterpret_cast<uintptr_t>(d_workspace) % 8 != 0)
        return fail(WG_ERR_INVALID, "wg_masked_topk: the workspace must be 8-byte aligned");
    WG_HIP(launch_masked_topk(d_logits, dtype, B, V, row_stride_elems, d_bitmask, k, d_ids, d_values,
                              static_cast<unsigned long long *>(d_workspace), static_cast<hipStream_t>(stream)));
    return WG_OK;
}

uint64_t wg_masked_topk_static_capacity(void) { return kTopkStaticKeys * sizeof(unsigned long long); }

int wg_masked_topk_static(const void *d_logits, wg_dtype_t dtype, uint32_t B, uint32_t V, int64_t row_stride_elems,
                          const uint32_t *d_bitmask, uint32_t k, int32_t *d_ids, void *d_values, void *stream) {
    if (!d_logits || !d_bitmask || !d_ids || !d_values)
        return fail(WG_ERR_INVALID, "wg_masked_topk_static: null argument");
    if (B == 0 || V == 0) return fail(WG_ERR_INVALID, "wg_masked_topk_static: empty batch or vocabulary");
    if (dtype != WG_F32 && dtype != WG_BF16) return fail(WG_ERR_INVALID, "wg_masked_topk_static: unknown dtype");
    if (row_stride_elems < (int64_t)V) return fail(WG_ERR_INVALID, "wg_masked_topk_static: row stride smaller than V");
    if (B > kMaxBatch) return fail(WG_ERR_INVALID, "wg_masked_topk_static: B above 65535");
    if (k == 0 || k > kTopkMax) return fail(WG_ERR_INVALID, "wg_masked_topk_static: k must be 1 .. 64");
    const uint64_t n_slices = ((uint64_t)V + kTopkSlice - 1u) / kTopkSlice;
    if (n_slices * k > kTopkMergeKeys)
        return fail(WG_ERR_INVALID, "wg_masked_topk_static: ceil(V / 8192) * k above 4096 (the lists of a row do not fit the merge)");
    const uint64_t need = wg_masked_topk_workspace(B, V, k);
    if (need > wg_masked_topk_static_capacity())
        return fail(WG_ERR_INVALID, "wg_masked_topk_static: B * ceil(V / 8192) * k * 8 = " + std::to_string(need) +
                                        " bytes of lists, above the " + std::to_string(wg_masked_topk_static_capacity()) +
                                        " the library holds per GPU (use wg_masked_topk with a workspace)");
    unsigned long long *lists = nullptr;
    WG_HIP(static_topk_scratch(&lists));
    WG_HIP(launch_masked_topk(d_logits, dtype, B, V, row_stride_elems, d_bitmask, k, d_ids, d_values, lists,
                              static_cast<hipStream_t>(stream)));
    return WG_OK;
}

int wg_advance(wg_handle_t h, wg_state_t *d_states, const int32_t *d_tokens, uint32_t B, void *stream) {
    if (!h || !d_states || !d_tokens) return fail(WG_ERR_INVALID, "wg_advance: null argument");
    if (B == 0) return fail(WG_ERR_INVALID, "wg_advance: B is 0");
    Timing advance(h, true, &h->advance_events);
    WG_HIP(advance.launched(launch_advance(h->dt, h->vocab->dv, h->dc, d_states, d_tokens, B, h->n_cu, static_cast<hipStream_t>(stream), advance.events())));
    return WG_OK;
}

int wg_forced_bytes(wg_handle_t h, const wg_state_t *d_states, uint32_t B, uint32_t cap, uint8_t *d_bytes,
                    uint32_t *d_lens, wg_state_t *d_end_states, void *stream) {
    if (!h || !d_states || !d_bytes || !d_lens) return fail(WG_ERR_INVALID, "wg_forced_bytes: null argument");
    if (B == 0 || cap == 0) return fail(WG_ERR_INVALID, "wg_forced_bytes: B or cap is 0");
    WG_HIP(launch_forced_bytes(h->dt, d_states, B, cap, d_bytes, d_lens, d_end_states, h->n_cu, static_cast<hipStream_t>(stream)));
    return WG_OK;
}

int wg_cache_clear(wg_handle_t h, void *stream) {
    if (!h) return fail(WG_ERR_INVALID, "wg_cache_clear: null handle");
    // The generation number travels with every later launch as a kernel argument, so the
    // clear is ordered with the caller's other calls on this handle without touching the GPU.
    return next_generation(h, static_cast<hipStream_t>(stream));
}

int wg_cache_stats(wg_handle_t h, wg_cache_stats_t *host_out) {
    if (!h || !host_out) return fail(WG_ERR_INVALID, "wg_cache_stats: null argument");
    Counters c;
    WG_HIP(hipDeviceSynchronize());
    if (h->dc.direct) {                                // nothing counts the rows there: a key of this generation holds its own
        WG_HIP(hipMemsetAsync(&h->dc.ctr->held, 0, sizeof c.held, nullptr));
        WG_HIP(launch_count_rows(h->dc, nullptr));
    }
    WG_HIP(hipMemcpy(&c, h->dc.ctr, sizeof c, hipMemcpyDeviceToHost));
    host_out->lookups = c.lookups; host_out->builds = c.builds;
    host_out->uncached_builds = c.uncached_builds;
    host_out->class_scans = c.class_scans;
    unsigned long long spread[kSpread * kSpreadStride];
    WG_HIP(hipMemcpy(spread, h->dc.ctr->spread, sizeof spread, hipMemcpyDeviceToHost));
    host_out->entries_walked = host_out->hits = 0;
    for (uint32_t i = 0; i < kSpread; i++) {
        host_out->entries_walked += spread[i * kSpreadStride + kSpreadWalked];
        host_out->hits += spread[i * kSpreadStride + kSpreadHits];
        host_out->builds += spread[i * kSpreadStride + kSpreadBuilds];
        host_out->class_scans += spread[i * kSpreadStride + kSpreadClasses];
    }
    host_out->keys = h->dc.n_keys;
    host_out->cache_rows = h->dc.cap_rows;
    const uint64_t taken = h->dc.direct ? c.held : (uint32_t)(c.slot_ctr >> 32) == h->dc.epoch ? (uint32_t)c.slot_ctr : 0u;
    host_out->rows_in_use = taken < h->dc.cap_rows ? taken : h->dc.cap_rows;
    const uint64_t row_bytes = (uint64_t)h->dc.row_stride * 4ull;
    host_out->arena_bytes = ((uint64_t)h->dc.cap_rows + h->cap_classes * 2ull) * row_bytes;
    return WG_OK;
}

int wg_error_count(wg_handle_t h, uint64_t *host_out) {
    if (!h || !host_out) return fail(WG_ERR_INVALID, "wg_error_count: null argument");
    unsigned long long spread[kSpread * kSpreadStride];
    WG_HIP(hipDeviceSynchronize());
    WG_HIP(hipMemcpy(spread, h->dc.ctr->spread, sizeof spread, hipMemcpyDeviceToHost));
    uint64_t n = 0;
    for (uint32_t i = 0; i < kSpread; i++) n += spread[i * kSpreadStride + kSpreadErrors];
    *host_out = n;
    return WG_OK;
}

int wg_profile_enable(wg_handle_t h, int on) {
    if (!h) return fail(WG_ERR_INVALID, "wg_profile_enable: null handle");
    h->profiling = on != 0;
    return WG_OK;
}

static int read_profile(wg_handle_t h, wg_profile_t *host_out) {
    if (!h || !host_out) return fail(WG_ERR_INVALID, "wg_profile_read: null argument");
    WG_HIP(hipDeviceSynchronize());
    wg_profile_t p{};
    // milliseconds of a record's pairs; its events are free for use again
    auto total = [&](std::vector<hipEvent_t> &v, uint64_t *calls) {
        double sum = 0.0;
        for (size_t i = 0; i + 1 < v.size(); i += 2) {
            float ms = 0.f;
            if (v[i] && v[i + 1] && hipEventElapsedTime(&ms, v[i], v[i + 1]) == hipSuccess) sum += (double)ms;
            else (void)hipGetLastError();              // (nobody else's error)
        }
        if (calls) *calls = v.size() / 2;
        h->spare_events.insert(h->spare_events.end(), v.begin(), v.end());
        v.clear();
        return sum;
    };
    p.lookup_ms = total(h->lookup_events, nullptr);
    p.build_ms = total(h->rows_events, &p.fill_calls);
    p.advance_ms = total(h->advance_events, &p.advance_calls);
    p.apply_ms = total(h->apply_events, &p.apply_calls);
    *host_out = p;
    return WG_OK;
}

int wg_profile_read(wg_handle_t h, wg_profile_t *host_out) {
    return no_throw("wg_profile_read: out of host memory", [&] { return read_profile(h, host_out); });
}

int wg_select_tokens(const uint32_t *d_bitmask, uint32_t B, uint32_t V, const uint64_t *d_draws,
                     int32_t *d_tokens, void *stream) {
    if (!d_bitmask || !d_draws || !d_tokens) return fail(WG_ERR_INVALID, "wg_select_tokens: null argument");
    if (B == 0 || V == 0) return fail(WG_ERR_INVALID, "wg_select_tokens: empty batch or vocabulary");
    WG_HIP(launch_select(d_bitmask, B, V, d_draws, d_tokens, static_cast<hipStream_t>(stream)));
    return WG_OK;
}

}  // extern "C"
