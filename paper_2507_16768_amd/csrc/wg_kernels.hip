// HIP kernels of the structured-decoding hot path for gfx950 (wave64).
//
//   rows         : the mask row of every request, a workgroup per (request, token range): copied from
//                  the cache, or made in LDS from the vocabulary's static indexes; to the caller's
//                  bitmask, to the cache, and (wg_decode_step) as -inf into the logits.  In front of
//                  it, in the same kernel for batches of up to a request per compute unit and some larger ones (plan_fill), the state is advanced
//                  by the sampled token (wg_advance_fill_masks, wg_decode_step) and looked up
//   lookup       : the same by itself: request state -> cache key; claims a missing key and leaves the
//                  task of making its row
//   apply        : logits <- -inf where the mask bit is 0
//   advance      : per-request walk of the sampled token
//   forced_bytes : per request, the rest of the Write run its state lies in
//   select       : harness sampler stand-in (k-th set bit of a row)
//
// No MFMA anywhere: the path is byte matching and memory traffic.
#include <hip/hip_runtime.h>

#include "wg_buffer.h"
#include "wg_device.h"
#include "wg_launch.h"

namespace wg {

// ---------------------------------------------------------------------------------------------
// Arguments of the kernels that a step launches.  What their first loads need comes first, each by itself: it is in
// scalar registers when a wavefront begins (kernarg preload, 14 dwords: build.py).  The rest lies behind it in the
// kernel's argument memory and is read from there where it is needed, through references: structures passed by value were
// loaded as a whole at the kernel's beginning, 60 registers in four to seven rounds of waiting, and put away in lanes of
// vector registers.  A pass of 8 cached steps, us, by value / by reference: 1 request, V = 32000 49.5 / 38.8; 64, V = 128256 70.3 / 60.5;
// 256, V = 151936 181 / 170; a cached fill of 1,024 rows behind a lookup 10.9 / 8.6.
struct LateArgs {
    DeviceTable T;
    DeviceVocab Vc;
    DeviceCache Cc;
    uint32_t *bitmask;
    void *logits;
    int64_t logits_stride;
    uint32_t span, shares, rows; // token ranges of a workgroup, workgroups of a row, rows of the call
};
#define WG_EARLY_ARGS wg_state_t *__restrict__ states, const int32_t *__restrict__ tokens, Control *ctr, const StateDesc *descs, \
                      const uint64_t *chunks, const uint8_t *len8, uint32_t n_states, uint32_t V, LateArgs
// Where the last of a kernel's arguments lies in its argument memory.
template <typename... P>
constexpr uint32_t last_argument(void (*)(P...))
{
    size_t at = 0, last = 0;
    ((last = (at + alignof(P) - 1) / alignof(P) * alignof(P), at = last + sizeof(P)), ...);
    return (uint32_t)last;
}
typedef void StepKernel(WG_EARLY_ARGS);
constexpr uint32_t kEarlyBytes = last_argument(static_cast<StepKernel *>(nullptr));
static_assert(kEarlyBytes == 4u * WG_PRELOADED_DWORDS, "the early arguments are those that are preloaded (build.py), the late ones lie right behind them");
typedef const __attribute__((address_space(4))) LateArgs Late;
template <typename M> using LateRef = const __attribute__((address_space(4))) M &;
__device__ __forceinline__ Late &late_args()
{
    return *(Late *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + kEarlyBytes);
}
struct TableView {
    const StateDesc *states;
    uint32_t n_states;
    LateRef<const uint8_t *> classes, lit;
    LateRef<const ClassPlan *> plans;
    LateRef<uint32_t> lmax;
};
struct VocabView {
    const uint8_t *len8;
    const uint64_t *chunks;
    uint32_t V;
    LateRef<const uint32_t *> rows, dirs;
    LateRef<const ExitEntry *> index;
    LateRef<uint32_t> W, lmax, n_chunks;
    LateRef<int32_t> eos_id;
};
struct CacheView {
    Control *ctr;
    LateRef<unsigned long long *> tags, class_tags;
    LateRef<uint32_t *> slots, arena, class_rows, row_ref;
    LateRef<const uint32_t *> free_rows;
    LateRef<RowTask *> tasks;
    LateRef<uint32_t> cap_rows, direct, row_stride, epoch;
};
#define WG_VIEWS \
    Late &late = late_args(); \
    const TableView T{descs, n_states, late.T.classes, late.T.lit, late.T.plans, late.T.lmax}; \
    const VocabView Vc{len8, chunks, V, late.Vc.rows, late.Vc.dirs, late.Vc.index, late.Vc.W, late.Vc.lmax, late.Vc.n_chunks, late.Vc.eos_id}; \
    const CacheView Cc{ctr, late.Cc.tags, late.Cc.class_tags, late.Cc.slots, late.Cc.arena, late.Cc.class_rows, late.Cc.row_ref, late.Cc.free_rows, \
                   late.Cc.tasks, late.Cc.cap_rows, late.Cc.direct, late.Cc.row_stride, late.Cc.epoch}

// ---------------------------------------------------------------------------------------------
// Walking a token through the state table.

// A token's bytes as 8-byte chunks of the vocabulary, two of them in registers at a time; the
// chunk array is strided by token, so the walk of a token of any length loads what it reaches.
struct TokenBytes {
    const uint64_t *chunks;      // chunk 0 of the token
    size_t stride;               // elements from one chunk of a token to the next (V)
    uint64_t w0, w1;             // chunks q and q + 1
    uint32_t q, n;               // n: chunks of the token
};

__device__ __forceinline__ TokenBytes token_bytes(const VocabView &Vc, uint32_t tok, uint32_t L)
{
    TokenBytes t;
    t.chunks = Vc.chunks + tok; t.stride = Vc.V;
    t.n = (L + 7u) >> 3; t.q = 0;
    t.w0 = t.chunks[0];
    t.w1 = t.n > 1u ? t.chunks[t.stride] : 0ull;
    return t;
}

// The eight bytes from byte i on (zeros behind the token's end); i never decreases.
__device__ __forceinline__ uint64_t window(TokenBytes &t, uint32_t i)
{
    const uint32_t q = i >> 3, sh = (i & 7u) * 8u;
    if (q != t.q) {
        t.w0 = q == t.q + 1u ? t.w1 : t.chunks[q * t.stride];
        t.w1 = q + 1u < t.n ? t.chunks[(q + 1u) * t.stride] : 0ull;
        t.q = q;
    }
    return sh ? (t.w0 >> sh) | (t.w1 << (64u - sh)) : t.w0;
}

// The classes of eight bytes, two bits each, and from them the first of the n bytes that does not
// stay: its place, or n.
__device__ __forceinline__ uint32_t class_code(const uint8_t *lut, uint64_t bytes)
{
    const uint32_t lo = (uint32_t)bytes, hi = (uint32_t)(bytes >> 32);
    uint32_t code = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        code |= (uint32_t)lut[(lo >> (8 * i)) & 0xFFu] << (2 * i);
        code |= (uint32_t)lut[(hi >> (8 * i)) & 0xFFu] << (2 * i + 8);
    }
    return code;
}
__device__ __forceinline__ uint32_t first_leaving(uint32_t code, uint32_t n)
{
    const uint32_t x = code ^ 0x5555u;               // a 2-bit field is 0 iff its byte stays
    const uint32_t mm = (x | (x >> 1)) & 0x5555u & ((1u << (2u * n)) - 1u);
    return mm ? (uint32_t)__builtin_ctz(mm) >> 1 : n;
}

// One visit of a literal state by a walk whose next eight bytes are tb, n of them the token's; l0, l1:
// the literal bytes around the state's.  False: a byte differs.
__device__ __forceinline__ bool literal_step(const StateDesc &d, uint64_t l0, uint64_t l1, uint64_t tb, uint32_t n,
                                             uint32_t &sid, uint32_t &aux, uint32_t &i)
{
    const uint32_t sh = (sid & 7u) * 8u;
    const uint64_t lv = sh ? (l0 >> sh) | (l1 << (64u - sh)) : l0;
    const uint32_t m = n < d.run ? n : d.run;                // literal bytes compared now
    const uint64_t mask = m == 8u ? ~0ull : (1ull << (8u * m)) - 1ull;
    if ((tb ^ lv) & mask) return false;
    sid = m == d.run ? d.cls : sid + m;                      // d.cls: state after the Write
    aux = 0; i += m;
    return true;
}
// The same of a checkpoint, code: the classes of the eight bytes.  left: the exit that was taken, or
// CLS_STAY.
__device__ __forceinline__ bool class_step(const StateDesc &d, uint32_t code, uint32_t n, uint32_t &aux, uint32_t &i, uint32_t &left)
{
    const uint32_t stays = first_leaving(code, n);
    if (d.max != WG_UNBOUNDED && stays) {                    // each stay needs budget left
        if (aux >= d.max || stays > d.max - aux) return false;
        aux += stays;
    }
    i += stays;
    left = CLS_STAY;
    if (stays == n) return true;
    left = (code >> (2u * stays)) & 3u;
    aux = 0; i += 1u;
    return left != CLS_REJECT;
}

__device__ __forceinline__ bool is_checkpoint(uint32_t kind) { return kind == WG_KIND_WAIT || kind == WG_KIND_COND; }

// Walks bytes [i, L) of a token from (sid, aux), up to eight bytes per state visit: a run of
// literal states is one masked 8-byte compare against the state table's literal bytes, a stay-run
// inside a checkpoint is eight independent class look-ups.  Every state entered on the way starts
// with aux = 0; only a bounded Wait counts.  False on the first rejected byte.
__device__ __forceinline__ bool walk(const TableView &T, uint32_t &sid, uint32_t &aux, TokenBytes &t, uint32_t i, uint32_t L)
{
    const uint64_t *lit64 = reinterpret_cast<const uint64_t *>(T.lit);
    while (i < L) {
        if (sid >= T.n_states) return false;                 // ERROR or corrupt state
        const StateDesc d = T.states[sid];
        const uint32_t kind = d.kind_byte & 0xFFu;
        const uint32_t n = L - i < 8u ? L - i : 8u;
        const uint64_t tb = window(t, i);
        if (kind == WG_KIND_LIT) {
            if (!literal_step(d, lit64[sid >> 3], lit64[(sid >> 3) + 1u], tb, n, sid, aux, i)) return false;
        } else if (kind == WG_KIND_WAIT || kind == WG_KIND_COND) {
            uint32_t left;
            if (!class_step(d, class_code(T.classes + (size_t)d.cls * 256u, tb), n, aux, i, left)) return false;
            if (left != CLS_STAY) sid = left == CLS_EXIT_A ? d.next_a : d.next_b;
        } else return false;                                 // FINAL / END accept no byte
    }
    return true;
}

__device__ __forceinline__ bool walk_from(const TableView &T, uint32_t sid, TokenBytes &t, uint32_t i, uint32_t L)
{
    uint32_t aux = 0;
    return walk(T, sid, aux, t, i, L);
}

// ---------------------------------------------------------------------------------------------
// advance: a wavefront per request, lane p the p-th byte of the token (EOS is the one-symbol string [EOS]; any other
// byte-less token is rejected).  What the request is at is the same for all lanes, in scalar registers.
__device__ __forceinline__ uint32_t of_first(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint32_t of_lane(uint32_t x, uint32_t lane) { return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)lane); }

// The descriptors of two states in one load: lane k (modulo 16) has dword k % 8 of a's, from 8 on of b's (of state 0 where
// there is no such state).
__device__ __forceinline__ uint32_t two_states(const TableView &T, uint32_t a, uint32_t b)
{
    const uint32_t s = threadIdx.x & 8u ? b : a;
    return reinterpret_cast<const uint32_t *>(T.states + (s < T.n_states ? s : 0u))[threadIdx.x & 7u];
}
__device__ __forceinline__ StateDesc state_of(uint32_t words, uint32_t at)      // at: 0 the first of the two, 8 the second
{
    return StateDesc{of_lane(words, at), of_lane(words, at + 1u), of_lane(words, at + 2u), of_lane(words, at + 3u),
                     of_lane(words, at + 4u), of_lane(words, at + 5u), of_lane(words, at + 6u), of_lane(words, at + 7u)};
}

// (0 where the vocabulary has no chunk for it)
__device__ __forceinline__ uint32_t token_byte(const VocabView &Vc, uint32_t n_chunks, uint32_t t, uint32_t p)
{
    if (p >= n_chunks * 8u) return 0u;
    return reinterpret_cast<const uint8_t *>(Vc.chunks + (size_t)(p >> 3) * Vc.V + t)[p & 7u];
}

// What a walk takes from memory for a state, in one trip: the descriptors of eight states from it on (lane k: dword k % 8 of
// the k / 8-th), 64 literal bytes from its own on (a lane each) and, of a checkpoint, the classes of all byte values
// (lane k: word k % 16 of its codes).
struct Ahead { uint32_t sid, words, lits, codes; };
constexpr uint32_t kAheadStates = 8u;
// The late arguments that it needs, kept in registers: read from the arguments' memory where they were needed, each was a wait of
// 100 cycles on the way of the one wavefront that everything waits for.
struct WalkArgs {
    const uint8_t *lit;
    const ClassCodes *codes;
    uint32_t n_chunks;
    int32_t eos_id;
    WalkArgs() = default;
    __device__ __forceinline__ explicit WalkArgs(Late &late) : lit(late.T.lit), codes(late.T.codes), n_chunks(late.Vc.n_chunks), eos_id(late.Vc.eos_id) {}
};
// Values that the compiler must not read again from memory.
template <typename X> __device__ __forceinline__ void hold_one(X &x) { asm volatile("" : "+s"(x)); }
template <typename X> __device__ __forceinline__ void hold_one(X *&x)               // (they stay pointers to device memory for the compiler)
{
    auto g = (__attribute__((address_space(1))) X *)x;
    asm volatile("" : "+s"(g));
    x = (X *)g;
}
template <typename... X> __device__ __forceinline__ void hold(X &...x) { (hold_one(x), ...); }
__device__ __forceinline__ Ahead look_ahead(const TableView &T, const WalkArgs &w, uint32_t sid)
{
    // (what is no state, ERROR among them, is state 0 here; who asks looks at the number first)
    const uint32_t lane = threadIdx.x & 63u, s = sid + lane / 8u, c = sid + lane;
    Ahead a;
    a.sid = sid;
    a.words = reinterpret_cast<const uint32_t *>(T.states + (s < T.n_states ? s : 0u))[lane & 7u];
    a.codes = w.codes[sid < T.n_states ? sid : 0u].word[lane & 15u];
    a.lits = w.lit[c < T.n_states ? c : 0u];
    return a;
}
// walk() for one token by a wavefront, where every trip to memory is one that nothing else hides: none for the state that the
// request is in (its surroundings come with its descriptor), nor for the literal states and the last state within reach of them; one
// for any other.  All bytes that a state might consume are compared or looked up together, a byte per lane.  (A thread
// per request, eight bytes at a time, took two trips for every eight bytes of free text, and the longest walk of a
// batch decides: of 256 mixed requests, V = 151936, the last had its state 8.9 us after the kernel's beginning.  With a trip for
// each state's bytes and the descriptors behind it 4.2.  Times with that / now, us: wg_advance in a decode loop, mixed, V = 151936, B = 256 4.88 / 3.84, outlines,
// V = 128256, B = 64 3.84 / 2.68 (20 calls in a row, which hide most of it, 3.06 / 2.98 and 2.93 / 2.85); eight cached steps of them 171.2 / 165.8 and 54.5 / 53.7.  The codes cost 64 bytes a state; asked for
// by the number of the class table they would be a trip behind the descriptor.)
// a: what lies ahead of sid, at the call; d: the descriptor of sid, at the call and after it.  byte: the lane's.
__device__ __forceinline__ bool walk_wide(const TableView &T, const VocabView &Vc, const WalkArgs &w, uint32_t &sid, uint32_t &aux, Ahead a, StateDesc &d,
                                          uint32_t t, uint32_t byte, uint32_t L)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t i = 0, base = 0;                                // bytes consumed; the byte that lane 0 has
    auto renew = [&]() {
        a = look_ahead(T, w, sid);
        asm volatile("" : "+v"(a.words), "+v"(a.codes), "+v"(a.lits));
    };
    auto arrived = [&]() {                                   // in sid: its descriptor
        if (sid - a.sid >= kAheadStates) renew();
        d = state_of(a.words, (sid - a.sid) * 8u);
    };
    while (i < L) {
        const uint32_t kind = d.kind_byte & 0xFFu;
        const bool lit = kind == WG_KIND_LIT;
        if (sid >= T.n_states || !(lit || is_checkpoint(kind))) return false;          // ERROR; FINAL and END accept no byte
        if (i == base + 64u) { base = i; byte = token_byte(Vc, w.n_chunks, t, base + lane); }      // a token longer than the wavefront
        uint32_t n = (L - base < 64u ? L - base : 64u) - (i - base);
        const uint32_t k = base + lane - i;                  // the lane's byte is the k-th from here, if k < n
        if (lit) {
            if (d.run < n) n = d.run;
            if (sid - a.sid + n > 64u) renew();
            uint32_t x = a.lits;                             // literal byte a.sid + lane; wanted: sid + k
            const uint32_t shift = sid - a.sid + base - i;
            if (shift) x = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane + shift) * 4u), (int)x);
            if (__ballot(k < n && x != byte)) return false;
            sid = n == d.run ? d.cls : sid + n;              // d.cls: state after the Write
            aux = 0; i += n;
            arrived();
            continue;
        }
        if (sid != a.sid) renew();
        const uint32_t codes = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(byte >> 4 << 2), (int)a.codes), c = codes >> (byte & 15u) * 2u & 3u;
        const unsigned long long off = __ballot(k < n && c != CLS_STAY);
        const uint32_t stays = off ? (uint32_t)__builtin_ctzll(off) - (i - base) : n;
        if (d.max != WG_UNBOUNDED && stays) {                // each stay needs budget left
            if (aux >= d.max || stays > d.max - aux) return false;
            aux += stays;
        }
        i += stays;
        if (!off) continue;
        const uint32_t left = of_lane(c, (uint32_t)__builtin_ctzll(off));
        if (left == CLS_REJECT) return false;
        sid = left == CLS_EXIT_A ? d.next_a : d.next_b;
        aux = 0; i++;
        arrived();
    }
    return true;
}
// What an advance takes from memory at first, in one trip: the state's surroundings, the token's length and bytes.
struct Sampled {
    uint32_t len, byte;
    Ahead ahead;
};
__device__ __forceinline__ bool is_token(const VocabView &Vc, int32_t t) { return t >= 0 && (uint32_t)t < Vc.V; }
__device__ __forceinline__ Sampled ask_sampled(const TableView &T, const VocabView &Vc, const WalkArgs &w, uint32_t sid, int32_t t)
{
    const uint32_t tok = is_token(Vc, t) ? (uint32_t)t : 0u;
    Sampled s;
    s.len = Vc.len8[tok];
    s.byte = token_byte(Vc, w.n_chunks, tok, threadIdx.x & 63u);
    s.ahead = look_ahead(T, w, sid);
    return s;
}
// d: the descriptor of sid after it.
__device__ __forceinline__ void advance_one(const TableView &T, const VocabView &Vc, const CacheView &Cc, const WalkArgs &w, Sampled s,
                                            uint32_t &sid, uint32_t &aux, StateDesc &d, int32_t t, bool count_error, uint32_t b)
{
    // (here: all of it has to have been requested; the compiler would move a load to where it is used)
    asm volatile("" : "+v"(s.len), "+v"(s.byte), "+v"(s.ahead.words), "+v"(s.ahead.codes), "+v"(s.ahead.lits));
    d = state_of(s.ahead.words, 0u);
    bool ok = is_token(Vc, t) && sid < T.n_states;
    if (ok) {
        if (w.eos_id == t) {
            sid = d.eos_next; aux = 0;
            ok = sid != WG_SID_ERROR;
            d = state_of(two_states(T, sid, sid), 0u);
        } else {
            const uint32_t L = of_first(s.len);
            ok = L != 0u && walk_wide(T, Vc, w, sid, aux, s.ahead, d, (uint32_t)t, s.byte, L);
        }
    }
    if (!ok) {
        sid = WG_SID_ERROR; aux = 0;
        // (spread as the statistics are: on one address a batch of rejected tokens took 12 ns a request, wg_advance, B = 256, 1,024 and 60,000
        // 4.5, 13.8 and 722 us, now 1.8, 2.2 and 15)
        if (count_error && (threadIdx.x & 63u) == 0u) atomicAdd(&Cc.ctr->spread[(b % kSpread) * kSpreadStride + kSpreadErrors], 1ull);
    }
}

// One request to a workgroup up to two on a compute unit, four above: with one / with four, V = 151936, us of 20 calls in a row, B = 64 mixed 2.89 / 2.98,
// random trees 2.86 / 3.00, 256 2.98 / 3.18, 2.97 / 3.08, 512 3.06 / 3.15, 3.02 / 3.08, 1024 3.21 / 3.33, 3.10 / 3.17, 2048 3.53 / 3.47, 3.47 / 3.32, 4096 4.30 / 3.89, 4.25 / 3.69,
// 8192 5.84 / 4.90, 5.87 / 4.85, 60,000 18.2 / 18.4, 18.0 / 19.4: the sides change between 1,024 and 2,048 and differ by 2 to 4 % from 513 on to there.  The first request's
// state and token come in one wait with the arguments that follow the early ones (one after the other, B = 1 4.2 us with a copy of the states, in one 4.0, 64 4.4, 4.3).
// Before look_ahead 256 took 3.06, 8192 5.28, 16,384 7.8 (now 7.2), 60,000 21.0; a thread each with eight bytes at a time took 6.1 to 8.6 us at 16,384 and 13 to 19 at
// 60,000.
constexpr uint32_t kAdvanceBlocks = 1u << 20;
template <uint32_t kWaves>
__global__ void __launch_bounds__(64 * kWaves)
advance_kernel(WG_EARLY_ARGS)
{
    WG_VIEWS;
    uint64_t b = (uint64_t)blockIdx.x * kWaves + (kWaves > 1u ? of_first(threadIdx.x >> 6) : 0u);
    if (kWaves > 1u && b >= late.rows) return;
    wg_state_t st = states[b];
    uint32_t t = of_first((uint32_t)tokens[b]);
    // (in one wait with them a word of each line of the arguments)
    WalkArgs walk(late);
    uint32_t rows = late.rows;
    asm volatile("" :: "s"(of_first(st.sid)), "s"(t), "s"(walk.lit), "s"(walk.codes), "s"(walk.n_chunks), "s"(walk.eos_id), "s"(rows));
    hold(walk.lit, walk.codes, walk.n_chunks, walk.eos_id, rows);
    for (;;) {
        uint32_t sid = of_first(st.sid), aux = of_first(st.aux);
        StateDesc d;
        advance_one(T, Vc, Cc, walk, ask_sampled(T, Vc, walk, sid, (int32_t)t), sid, aux, d, (int32_t)t, true, (uint32_t)b);
        if ((threadIdx.x & 63u) == 0u) states[b] = wg_state_t{sid, aux};
        // (wg_advance takes any number of requests: more than the grid holds come in turn)
        b += (uint64_t)gridDim.x * kWaves;
        if (b >= rows) return;
        st = states[b];
        t = of_first((uint32_t)tokens[b]);
    }
}

// ---------------------------------------------------------------------------------------------
// lookup: state -> cache key.  A missing key is claimed by exactly one request (CAS on the key's
// tag), which keeps the row it makes: in the arena row of the key's own number (Cc.direct: the arena
// has a row for every key), or else the i-th claim of a call takes the i-th free row, and a claim
// that finds none left keeps nothing: its row is made again by every call that needs it.  The count
// of rows in use is brought up to date once per call, when all its lookups are done.  Any other
// request of the call with that key makes the row for itself: no request waits for another.
struct Found {
    uint32_t key, ref;           // ref: as left in row_ref
    bool hit, claimed, class_claimed, keep;   // keep: this request claimed the key (here or in another workgroup of its row)
    RowTask me;                  // when ref is kRefBuild
};

// In a fill of one kernel no workgroup waits to learn whether it owns the key or the class table that it makes: all
// workgroups of every row that needs one, up to 32 of each, would swap on one tag, 10 ns each (a cold call of 256
// requests 42 us, now 18).  All workgroups of a row make their shares and keep them; the row's first one then enters the tags,
// behind what it has to do, and the first of a call to do so counts.  A workgroup that finds the tag entered by
// another row of the call keeps nothing: that row's workgroups all find it old or their own, and keep theirs.
struct Claim { unsigned long long key_tag, class_tag; uint32_t key, cls; };      // tags as the lookup found them

// What a call writes into the tags it claims, but for the request; `launch` is ctr->launch.
__device__ __forceinline__ unsigned long long tag_now(uint32_t epoch, unsigned long long launch)
{
    return (unsigned long long)epoch << kTagEpochShift | (launch & kTagLaunchMask) << kTagRequestBits;
}

// The key of the state (sid, aux), d its descriptor; kNoKey: no such state.
__device__ __forceinline__ uint32_t key_of(const TableView &T, uint32_t lmax, uint32_t sid, uint32_t aux, const StateDesc &d, uint32_t &variant)
{
    variant = 0;
    if ((d.kind_byte & 0xFFu) == WG_KIND_WAIT && d.max != WG_UNBOUNDED) {
        const uint32_t left = d.max > aux ? d.max - aux : 0u;
        variant = lmax - (left < lmax ? left : lmax);
    }
    return sid < T.n_states ? d.key_base + variant : kNoKey;
}

// What a lookup reads of the state with the descriptor d: the key's tag and, although only a missing key needs them, the two
// successors' descriptors and the tag of the class table, requested together so that nothing waits for them before the
// tag has decided.
struct Asked {
    uint32_t key, variant, slot;
    unsigned long long tag, class_tag;
    uint32_t next;               // as two_states leaves them
};
// slots: null where the arena is addressed by key.
template <bool kDirect>
__device__ __forceinline__ Asked ask(const TableView &T, uint32_t lmax, const unsigned long long *tags, const unsigned long long *class_tags, const uint32_t *slots,
                                     uint32_t sid, uint32_t aux, const StateDesc &d)
{
    Asked q{};
    q.key = key_of(T, lmax, sid, aux, d, q.variant);
    if (q.key == kNoKey) return q;
    q.tag = __hip_atomic_load(&tags[q.key], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    q.class_tag = __hip_atomic_load(&class_tags[is_checkpoint(d.kind_byte & 0xFFu) ? d.cls : 0u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    q.next = two_states(T, d.next_a, d.next_b);
    q.slot = q.key;
    if (!kDirect && slots) q.slot = slots[q.key];
    return q;
}
__device__ __forceinline__ unsigned long long of_first(unsigned long long x) { return (unsigned long long)of_first((uint32_t)(x >> 32)) << 32 | of_first((uint32_t)x); }

// The tag t was entered in this generation, by an earlier call than the one that enters `now`.
__device__ __forceinline__ bool made_before(unsigned long long t, unsigned long long now)
{
    return t >> kTagEpochShift == now >> kTagEpochShift && (t >> kTagRequestBits) != (now >> kTagRequestBits);
}

// The lookup of request b in state sid, d its descriptor.  kShares: by every workgroup of its row, with the
// arena addressed by key, and claimed by nobody: see Claim.
template <bool kShares>
__device__ __forceinline__ Found look_up(const TableView &T, const CacheView &Cc, unsigned long long now, uint32_t b,
                                         uint32_t sid, const StateDesc &d, const Asked &q, Claim *claim)
{
    Found f{};
    f.ref = kNoKey;
    f.key = q.key;
    if (f.key == kNoKey) return f;
    const unsigned long long mine = now | b, t = of_first(q.tag), ct = of_first(q.class_tag);
    const uint32_t kind = d.kind_byte & 0xFFu, cls = is_checkpoint(kind) ? d.cls : 0u, slot = of_first(q.slot);
    const bool leads = (threadIdx.x & 63u) == 0u;
    const bool ckpt = is_checkpoint(kind);
    // (a slot is only read where the tag is of this generation and an earlier call: it does not
    // change after that call, so the two loads need no order)
    const bool this_call = (t >> kTagRequestBits) == (now >> kTagRequestBits);
    f.hit = made_before(t, now) && slot != kNoSlot;
    f.ref = f.hit ? slot : kRefBuild;
    if (f.hit) return f;
    const bool class_this_call = (ct >> kTagRequestBits) == (now >> kTagRequestBits);
    uint32_t class_state = made_before(ct, now) ? CLASS_READY : CLASS_SELF;
    if (kShares) {
        f.keep = !this_call || t == mine;
        if (ckpt && class_state != CLASS_READY && (!class_this_call || ct == mine)) class_state = CLASS_OWN;
        claim->key = f.key; claim->key_tag = t;
        claim->cls = class_state == CLASS_OWN ? cls : kNoKey; claim->class_tag = ct;
    } else {
        unsigned long long is = t;
        if (!this_call) {
            if (leads) is = atomicCAS(&Cc.tags[f.key], t, mine);
            is = of_first(is);
            f.claimed = is == t;
        }
        f.keep = f.claimed || is == mine;
        if (f.keep && ckpt && class_state != CLASS_READY) {
            unsigned long long cis = ct;
            if (!class_this_call) {
                if (leads) cis = atomicCAS(&Cc.class_tags[cls], ct, mine);
                cis = of_first(cis);
                f.class_claimed = cis == ct;
            }
            if (f.class_claimed || cis == mine) class_state = CLASS_OWN;
        }
    }
    auto hop = [&](uint32_t nt, const StateDesc &n) {
        if (nt >= T.n_states) return HopState{0xFFu, 0u, WG_SID_ERROR, WG_SID_ERROR, WG_UNBOUNDED, 0u};
        const bool lit = (n.kind_byte & 0xFFu) == WG_KIND_LIT;
        return HopState{n.kind_byte & 0xFFu, (n.kind_byte >> 8) & 0xFFu, lit ? nt : n.next_a, n.next_b, lit ? n.run : n.max, n.cls};
    };
    f.me = RowTask{sid, kind, (d.kind_byte >> 8) & 0xFFu, d.cls, d.run, T.lmax - q.variant, class_state, d.eos_next,
                   f.keep && Cc.direct ? f.key : kNoSlot, {hop(d.next_a, state_of(q.next, 0u)), hop(d.next_b, state_of(q.next, 8u))}};
    return f;
}

// A wavefront per request, four of them to a workgroup (with 1 / 4 / 16, mixed, us, found and claimed: B = 300 4.1 / 4.2 / 5.1 and 7.3 /
// 7.4 / 9.1, B = 1024 5.2 / 5.2 / 5.8 and 13.8 / 13.2 / 15.4; with a thread per request and four to a wavefront 5.4 and 7.7,
// 6.6 and 16.5).  With tokens the states are advanced first.
constexpr uint32_t kLookupWaves = 4;
__global__ void __launch_bounds__(64 * kLookupWaves)
lookup_kernel(WG_EARLY_ARGS)
{
    WG_VIEWS;
    const uint32_t B = late.rows;
    __shared__ uint32_t claims[kLookupWaves], first_claim;
    const uint32_t wave = of_first(threadIdx.x >> 6), b = blockIdx.x * kLookupWaves + wave;
    const bool leads = (threadIdx.x & 63u) == 0u;
    const unsigned long long sc = Cc.ctr->slot_ctr, launch = Cc.ctr->launch;
    Found f{};
    f.ref = kNoKey;
    if (b < B) {
        uint32_t sid = of_first(states[b].sid), aux = of_first(states[b].aux);
        StateDesc d;
        if (tokens) {
            const WalkArgs walk(late);
            const int32_t t = (int32_t)of_first((uint32_t)tokens[b]);
            advance_one(T, Vc, Cc, walk, ask_sampled(T, Vc, walk, sid, t), sid, aux, d, t, true, b);
            if (leads) states[b] = wg_state_t{sid, aux};
        } else d = state_of(two_states(T, sid, sid), 0u);
        f = look_up<false>(T, Cc, tag_now(Cc.epoch, of_first(launch)), b, sid, d, ask<false>(T, T.lmax, Cc.tags, Cc.class_tags, Cc.direct ? nullptr : Cc.slots, sid, aux, d), nullptr);
    }
    // (an atomic on one address costs 10 ns per wavefront of the launch: statistics are spread, and the claims too
    // where nothing is handed out by their number)
    unsigned long long *count = &Cc.ctr->spread[(b % kSpread) * kSpreadStride];
    if (leads && f.hit) atomicAdd(&count[kSpreadHits], 1ull);
    if (Cc.direct) {
        if (leads && f.claimed) atomicAdd(&count[kSpreadBuilds], 1ull);
        if (leads && f.class_claimed) atomicAdd(&count[kSpreadClasses], 1ull);
    } else {
        // the claimers of a workgroup take their arena rows together
        if (leads) claims[wave] = (uint32_t)f.claimed | (uint32_t)f.class_claimed << 16;
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (uint32_t w = 0; w < kLookupWaves; w++) { if (w < wave) before += claims[w]; all += claims[w]; }
        if (threadIdx.x == 0) {
            if (all & 0xFFFFu) first_claim = atomicAdd(&Cc.ctr->n_claims, all & 0xFFFFu);
            if (all >> 16) atomicAdd(&Cc.ctr->n_class_claims, all >> 16);
        }
        __syncthreads();
        if (f.claimed) {
            const uint32_t rows0 = (uint32_t)(sc >> 32) == Cc.epoch ? (uint32_t)sc : 0u;      // rows in use before this call
            const uint32_t idx = rows0 + first_claim + (before & 0xFFFFu);
            f.me.slot = idx < Cc.cap_rows ? (Cc.free_rows ? Cc.free_rows[idx] : idx) : kNoSlot;
            if (leads) Cc.slots[f.key] = f.me.slot;
        }
    }
    if (b < B && leads) {
        Cc.row_ref[b] = f.ref;
        if (f.ref == kRefBuild) Cc.tasks[b] = f.me;
    }
}

// ---------------------------------------------------------------------------------------------
// Masking: -inf over the tokens whose bit is 0.  Nothing is read from the logits where it can be helped.
//
// A wavefront takes 64 tokens at a time, a lane each, and their mask bits are the lanes that store: one instruction
// and two to four 64-byte requests per 64 tokens, whatever the pattern and wherever the row starts.  With a 16-byte
// piece to a lane, and a store per disallowed token of a mixed piece, each of the stores was a request for every 64
// bytes that the wavefront spans.  Before -> now, html outlines / JSON / mixed / random trees, us: wg_apply_mask, bf16,
// V = 151936, B = 256 11.7 / 11.9 / 14.7 / 20.4 -> 11.2 / 11.2 / 13.4 / 15.6; V = 128256, B = 64 4.5 / 5.5 / 5.8 / 7.8 -> 4.3 / 4.4
// / 4.6 / 5.0; fp32 6.2 / 6.4 / 7.0 / 9.4 -> 4.7 / 5.2 / 5.9 / 6.9; a cached wg_decode_step, V = 151936, B = 256, mixed 22.9 ->
// 18.8, V = 128256, B = 64 8.8 / 9.3 / 9.8 / 11.9 -> 8.9 / 8.9 / 9.2 / 9.8.  (Wavefronts that take pieces where these are fewer
// instructions were 5 to 15 % slower; so were stores without the compiler's branch around them, which skips words that
// are allowed as a whole.)
// What is left is the memory's: a store that covers part of a 64-byte block costs it 2.3 times a whole block.  The
// last-level cache (256 MB) merges such stores as long as the logits fit it; beyond that the memory reads and writes
// the block, and whole lines are written instead (mask_lines).
//
// Lanes first ... first + kChunk - 1 hold the mask bits of 64 tokens each in lo and hi, the first of them at p.
constexpr uint32_t kChunk = 8u;
// kThrough: the stores go through the die's L2 (masks_through).
template <typename Elem, bool kThrough>
__device__ __forceinline__ void mask_chunk(Elem *p, uint32_t lo, uint32_t hi, uint32_t first)
{
    constexpr Elem kNinf = sizeof(Elem) == 4 ? (Elem)0xFF800000u : (Elem)0xFF80u;
    const uint32_t lane = threadIdx.x & 63u;
    // (all into scalar registers before the first store: one by one between the stores each was waited for; a cached
    // step, html, V = 151936, B = 256, 16.9 -> 16.6 us)
    lo = ~lo; hi = ~hi;
    unsigned long long m[kChunk];
#pragma unroll
    for (uint32_t u = 0; u < kChunk; u++)
        m[u] = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)hi, (int)(first + u)) << 32 |
               (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)(first + u));
#pragma unroll
    for (uint32_t u = 0; u < kChunk; u++)
        if (__builtin_amdgcn_inverse_ballot_w64(m[u])) {
            if (kThrough) __hip_atomic_store(&p[u * 64u + lane], kNinf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else p[u * 64u + lane] = kNinf;
        }
}
// Word w of the `words` that hold a row's V tokens; what lies behind the last token counts as allowed.
__device__ __forceinline__ uint32_t word_or_ones(const uint32_t *row, uint32_t w, uint32_t words, uint32_t V)
{
    uint32_t x = w < words ? row[w] : 0xFFFFFFFFu;
    if (w + 1u == words && (V & 31u)) x |= ~0u << (V & 31u);
    return x;
}
// Tokens that the first of a row lies behind a 128-byte line's beginning (0 where elements do not lie at multiples of their size).
// Chunks are cut at the lines, so that a store covers one line and not parts of two, of which stores that go through the L2
// (masks_through) would each cost a whole one: cut at the row's beginning / at lines, outlines, mixed, random trees, V = 100003,
// bf16, B = 96, us, wg_apply_mask 4.4 4.8 6.3 / 4.0 4.3 5.1 (4.8 5.1 6.1 cut at the beginning and not through the L2).
template <typename Elem>
__device__ __forceinline__ uint32_t skew_of(const Elem *first)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(first);
    return at % sizeof(Elem) ? 0u : (uint32_t)(at % 128u / sizeof(Elem));
}
// The mask bits of the 64 tokens from 64 * i - skew on; what lies in front of the first token counts as allowed too.
__device__ __forceinline__ void bits_of_chunk(const uint32_t *row, uint32_t i, uint32_t words, uint32_t V, uint32_t skew, uint32_t &a, uint32_t &b)
{
    const uint32_t w = 2u * i - (skew >> 5), r = skew & 31u;         // (below 0: beyond the words)
    a = word_or_ones(row, w, words, V);
    b = word_or_ones(row, w + 1u, words, V);
    if (r) {
        b = __builtin_amdgcn_alignbit(b, a, 32u - r);
        a = __builtin_amdgcn_alignbit(a, word_or_ones(row, w - 1u, words, V), 32u - r);
    }
}
// The whole workgroup masks the tokens [lo, hi) of a row; `row` is in LDS, its bit 0 is token lo.  The wavefronts
// take chunks in turn, so that all of them write close together (a quarter of the share each was 3 to 8 % slower).
template <typename Elem, bool kThrough>
__device__ __forceinline__ void mask_span(Elem *logits, uint32_t lo, uint32_t hi, const uint32_t *row)
{
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t V = hi - lo, words = (V + 31u) >> 5, skew = skew_of(logits + lo), pairs = (V + skew + 63u) >> 6, step = (blockDim.x >> 6) * kChunk;
    Elem *p = logits + lo - skew;
    for (uint32_t i0 = wave * kChunk; i0 < pairs; i0 += step * (64u / kChunk)) {
        uint32_t a, b;                                              // a lane per chunk of 64 tokens, eight stretches of kChunk at a time
        bits_of_chunk(row, i0 + lane / kChunk * step + lane % kChunk, words, V, skew, a, b);
        if (!__ballot((a & b) != 0xFFFFFFFFu)) continue;            // a step in text without an end: 12.4 -> 9.0 us
        for (uint32_t c = 0; c < 64u / kChunk && i0 + c * step < pairs; c++)
            mask_chunk<Elem, kThrough>(p + (size_t)(i0 + c * step) * 64u, a, b, c * kChunk);
    }
}

// The same by whole lines: every 128-byte line with a disallowed token is read where it has to be and written
// whole, 8 lanes x 16 bytes.  The pieces are cut where the addresses allow it, the tokens before and behind them
// are stored one by one.  Without a branch around a piece's load or store, and as streams: behind branches each store was
// waited for before the next one (loads and stores count together), and logits that the last-level cache does not hold
// only take its place.  us, V = 151936, bf16, B = 1000, outlines, mixed, random trees, branches / none / none and streams:
// wg_apply_mask 101 108 103 / 98 105 101 / 78 84 81 (streamed loads alone 96 101 96, stores alone 97 106 94), a cold step 124 139 139 / 121
// 136 137 / 108 119 124; fp32, V = 128256, B = 700, the cold step 108 127 149 / 103 123 147 / 97 112 136.
// kBatch: pieces of a thread in flight together.  In the rows' kernel 5 (fp32: 8); by itself 4, a workgroup's share of bf16 (fp32: 8).  us a cold
// step, V = 151936, B = 1000, mixed, random trees, with 4 / 5 / 8 121.3 127.6 / 118.8 123.8 / 121.9 129.2; fp32, V = 128256, B = 700, with 4 / 6 / 8
// 111.9 136.4 / 112.5 136.0 / 110.0 133.9; by itself fp32 with 4 / 8 88.1 107.2 / 85.5 103.7.
template <typename Elem, uint32_t kBatch>
__device__ __forceinline__ void mask_lines(Elem *logits, uint32_t lo, uint32_t hi, const uint32_t *row)
{
    constexpr uint32_t kPer = 16u / sizeof(Elem);                  // tokens of a piece
    constexpr uint32_t kAlign = 128u;
    constexpr uint32_t kAll = (1u << kPer) - 1u;
    constexpr Elem kNinf = sizeof(Elem) == 4 ? (Elem)0xFF800000u : (Elem)0xFF80u;
    constexpr uint32_t kFill = sizeof(Elem) == 4 ? 0xFF800000u : 0xFF80FF80u;
    const uint32_t tid = threadIdx.x, nt = blockDim.x;
    const uintptr_t at = reinterpret_cast<uintptr_t>(logits + lo);
    uint32_t head = at % sizeof(Elem) ? hi - lo : (uint32_t)((kAlign - at % kAlign) % kAlign / sizeof(Elem));
    if (head > hi - lo) head = hi - lo;
    const uint32_t t0 = lo + head, pieces = (hi - t0) / kPer, t1 = t0 + pieces * kPer;
    auto disallowed = [&](uint32_t t) { return !((row[(t - lo) >> 5] >> ((t - lo) & 31u)) & 1u); };
    for (uint32_t i = tid; i < head; i += nt) if (disallowed(lo + i)) logits[lo + i] = kNinf;
    for (uint32_t t = t1 + tid; t < hi; t += nt) if (disallowed(t)) logits[t] = kNinf;
    const Window win = window_of(logits + t0, pieces * 16u);
    for (uint32_t p0 = 0; p0 < pieces; p0 += nt * kBatch) {
        uint32_t z[kBatch], at_piece[kBatch];                      // disallowed tokens of the pieces
        uint4 v[kBatch];
        const unsigned long long line = 0xFFull << (tid & 56u);
#pragma unroll
        for (uint32_t i = 0; i < kBatch; i++) {
            const uint32_t p = p0 + i * nt + tid, bit = head + (p < pieces ? p : pieces - 1u) * kPer;
            // (the word behind the row's last one is there to be read)
            z[i] = ~__builtin_amdgcn_alignbit(row[(bit >> 5) + 1u], row[bit >> 5], bit & 31u) & kAll;
            if (p >= pieces) z[i] = 0u;
        }
#pragma unroll
        for (uint32_t i = 0; i < kBatch; i++) {
            const uint32_t p = p0 + i * nt + tid;
            at_piece[i] = p < pieces && (__ballot(z[i] != 0u) & line) ? p * 16u : kNowhere;
            v[i] = block_at<kStream>(win, z[i] != kAll ? at_piece[i] : kNowhere);
        }
#pragma unroll
        for (uint32_t i = 0; i < kBatch; i++) {
            uint32_t d[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (uint32_t k = 0; k < 4u; k++) {
                uint32_t m;
                if (sizeof(Elem) == 4) m = (uint32_t)__builtin_amdgcn_sbfe(z[i], k, 1);
                else m = ((uint32_t)__builtin_amdgcn_sbfe(z[i], 2 * k, 1) & 0xFFFFu) | ((uint32_t)__builtin_amdgcn_sbfe(z[i], 2 * k + 1, 1) << 16);
                d[k] = (d[k] & ~m) | (kFill & m);
            }
            put_block<kStream>(win, at_piece[i], uint4{d[0], d[1], d[2], d[3]});
        }
    }
}

// ---------------------------------------------------------------------------------------------
// rows: a workgroup per (request, share of the token ranges).  A row made in an earlier call is
// copied; a missing one is made in LDS from the request's task and the vocabulary's static
// indexes, each workgroup making the words of its own tokens:
//   a literal state admits the tokens that begin with its byte and go on with what follows it:
//     candidates by the first two bytes (or by the first byte, where a checkpoint follows);
//   a checkpoint admits tokens whose bytes all stay, tokens that leave it with their last byte
//     (these two depend on its class table only, and are kept per table), and tokens that leave it
//     earlier and go on in the successor.  A table that few byte values enter (kFewLive) takes every
//     token that begins with one of them as a candidate and decides it from its bytes.  Any other
//     table gets its all-stay tokens 32 at a time, as the complement of the OR of the rows of the
//     byte values that do not stay; the tokens that leave with their last byte are found by that
//     byte, those that leave earlier by the exit byte and the literal byte behind it (or, where a
//     checkpoint follows, by the exit byte).
// The first wavefront sees to the candidates (and to all that it needs for them itself: the successors' class
// tables and literal bytes come with the directories), the others to the rest.  What the walks need of the
// successors lies in LDS and not in scalar registers, of which this kernel has too few: what they do not hold is kept in
// lanes of vector registers, 61 or 62 values with the lookup in a kernel before it and 77 to 80 with it in front.
// Every candidate is then decided by its bytes, so an index may offer any superset of the tokens
// that count.  The candidates of all ranges are one sequence, handed out to the wavefronts in
// stretches of kRowBatch * 64; a wavefront filters its entries by their neighbouring byte, queues
// what is left in LDS and decides them 64 at a time, so that the walks run on full wavefronts.
//
// What bounds it (V = 151936, masks only).  B = 256, one kernel: copied rows 6.9 us, the launch and the
// chain state -> descriptor -> tag -> row of four trips to memory; made rows 14.8 us for 19 MB, the same chain and
// then plan -> directory -> entries -> chunks -> walk, with 2.9 M instructions of wavefronts (5 us of the chip's
// vector units) in it.  The first wavefront is what the others wait for: stamps of a cold fill, cycles from a workgroup's beginning, median: the state and
// its key 3,700, looked up 6,800, directories 10,800, entries 13,100, filtered 15,200, walked and at the barrier 19,300, row out 21,100; the other three are at the barrier
// at 11,200 (128 JSON requests on 128,256 tokens 18,200 and 8,400 to 9,900, 96 mixed ones on 100,003 18,200 and 9,300 to 10,600; the first share of a row, whose last wavefront
// claims, 21,100 and 11,200 to 13,300).  B = 1024 and 141 class tables a call, two kernels: copied rows 5 + 9.8 us, made rows 5 + 57,
// with 15 M vector instructions of wavefronts (25 us).
constexpr uint32_t kRowThreads = 256;
constexpr uint32_t kRowWaves = kRowThreads / 64u;
constexpr uint32_t kRowBatch = 4;          // index entries of a lane in flight together
constexpr uint32_t kRanges = 256;          // index ranges of a key: at most one per byte value
constexpr uint32_t kAlone = 128;           // candidates that one wavefront sees to, while the others do the rows
// token rows in flight together, 16 bytes of each a thread: a table of thirty rows is four trips to memory (with four
// rows of four single words, where a share of 500 words also left lanes to load twice, it was eight: a
// checkpoint of digits, V = 128256, 5.6 us of the row's 15)
constexpr uint32_t kOrBatch = 8;

enum : uint32_t {
    FROM_PREFIX = 1,    // sorted, by two bytes
    FROM_STAY = 2,      // by first byte, which stays
    FROM_A = 3,         // by first byte, which leaves through A (or is the literal state's own)
    FROM_B = 4,
    FROM_PAIR = 5,      // by exit byte and the literal byte behind it
    FROM_DEEP_A = 6,    // by exit byte (and range), a checkpoint behind it
    FROM_DEEP_B = 7,
};

typedef __attribute__((address_space(1))) uint2 global_u2;   // a load known to go to device memory

struct RowShared {
    uint8_t own[256], hop[2][256];             // class tables of the state and of its successors
    uint64_t run[2][3];                        // 24 literal bytes from the state itself, or behind its exits
    ClassPlan plan;                            // of the state's class table
    uint32_t start[kRanges], upto[kRanges];    // first entry of a range, candidates up to its end
    uint16_t code[kRanges];                    // byte value | FROM_* << 8
    uint32_t queue[kRowWaves][64u * (kRowBatch + 1u)];   // tokens to decide: id | length << 24
    uint32_t n_ranges, total;
    RowTask task;                              // what the row's lookup left; two kernels: its successors only
    uint32_t key, ref;                         // the row's key, and what its lookup found
    wg_state_t state;                          // the request's, advanced
    StateDesc desc;                            // of its state
    Claim claim;
    unsigned long long launch;
};

// Inclusive prefix sum over the wavefront, in registers (every lane calls it).
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);    // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);    // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);    // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);    // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // last lane of row 0 / 2 into row 1 / 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // lane 31 into the upper half
    return x;
}

// Walks bytes [i, L), i < L, of a token from a literal state with `run` bytes to go, its first 24 in
// `lit` (LDS), then the state table from the state `after` them.
__device__ __forceinline__ bool walk_run(const TableView &T, const uint64_t *lit, uint32_t sid, uint32_t run, uint32_t after,
                                         TokenBytes &t, uint32_t i, uint32_t L)
{
    const uint32_t n = L - i < run ? L - i : run;
#pragma unroll
    for (uint32_t k = 0; k < 3u; k++) {
        if (8u * k >= n) break;
        const uint32_t m = n - 8u * k;
        const uint64_t mask = m >= 8u ? ~0ull : (1ull << (8u * m)) - 1ull;
        if ((window(t, i + 8u * k) ^ lit[k]) & mask) return false;
    }
    if (n <= 24u) { sid = n == run ? after : sid + n; i += n; }
    else { sid += 24u; i += 24u; }
    return walk_from(T, sid, t, i, L);
}

// Walks bytes [i, L), i < L, of a token from the staged successor; goes on through the state table
// when the token moves on to a third state.
__device__ __forceinline__ bool walk_hop(const TableView &T, const HopState &h, const uint8_t *lut, const uint64_t *lit,
                                         TokenBytes &t, uint32_t i, uint32_t L)
{
    uint32_t sid = WG_SID_ERROR, aux = 0;
    if (h.kind == WG_KIND_LIT) return walk_run(T, lit, h.next_a, h.max, h.cls, t, i, L);
    if (is_checkpoint(h.kind)) {
        for (;;) {
            const uint32_t n = L - i < 8u ? L - i : 8u;
            const uint32_t code = class_code(lut, window(t, i)), stays = first_leaving(code, n);
            if (h.max != WG_UNBOUNDED) { if (stays > h.max - aux) return false; aux += stays; }
            i += stays;
            if (stays < n) {
                const uint32_t c = (code >> (2u * stays)) & 3u;
                if (c == CLS_REJECT) return false;
                sid = c == CLS_EXIT_A ? h.next_a : h.next_b;
                i++;
                break;
            }
            if (i >= L) return true;
        }
    } else return false;
    return walk_from(T, sid, t, i, L);
}

// First token of range p (as the vocabulary's index is made; computed, because an array in a kernel
// argument is not indexed in registers).
__host__ __device__ __forceinline__ uint32_t range_token(uint32_t V, uint32_t p)
{
    const uint32_t groups = (V + kPartGroup - 1u) / kPartGroup, t = p * groups / kParts * kPartGroup;
    return p >= kParts || t > V ? V : t;
}

__device__ __forceinline__ uint4 operator|(const uint4 &a, const uint4 &b) { return uint4{a.x | b.x, a.y | b.y, a.z | b.z, a.w | b.w}; }
__device__ __forceinline__ uint4 operator&(const uint4 &a, const uint4 &b) { return uint4{a.x & b.x, a.y & b.y, a.z & b.z, a.w & b.w}; }
__device__ __forceinline__ uint4 operator~(const uint4 &a) { return uint4{~a.x, ~a.y, ~a.z, ~a.w}; }

// A class table and its plan, asked for and brought to LDS; one wavefront, a piece per lane.
struct StagedClass { uint32_t table; uint4 plan; };
__device__ __forceinline__ StagedClass ask_class(const TableView &T, uint32_t cls, uint32_t lane)
{
    static_assert(sizeof(ClassPlan) % 16 == 0 && sizeof(ClassPlan) / 16 <= 64, "a piece per lane");
    StagedClass s{};
    s.table = reinterpret_cast<const uint32_t *>(T.classes + (size_t)cls * 256u)[lane];
    if (lane < sizeof(ClassPlan) / 16u) s.plan = reinterpret_cast<const uint4 *>(T.plans + cls)[lane];
    return s;
}
__device__ __forceinline__ void put_class(RowShared &sh, const StagedClass &s, uint32_t lane)
{
    reinterpret_cast<uint32_t *>(sh.own)[lane] = s.table;
    if (lane < sizeof(ClassPlan) / 16u) reinterpret_cast<uint4 *>(&sh.plan)[lane] = s.plan;
}

// Enters a row's claims (see Claim).
__device__ __forceinline__ void claim_tags(const CacheView &Cc, const RowShared &sh, uint32_t b)
{
    const unsigned long long now = tag_now(Cc.epoch, sh.launch), mine = now | b;
    const Claim c = sh.claim;
    unsigned long long key_was = ~c.key_tag, class_was = ~c.class_tag;
    if ((c.key_tag >> kTagRequestBits) != (now >> kTagRequestBits)) key_was = atomicCAS(&Cc.tags[c.key], c.key_tag, mine);
    if (c.cls != kNoKey && (c.class_tag >> kTagRequestBits) != (now >> kTagRequestBits)) class_was = atomicCAS(&Cc.class_tags[c.cls], c.class_tag, mine);
    unsigned long long *count = Cc.ctr->spread + (b % kSpread) * kSpreadStride;
    if (key_was == c.key_tag) atomicAdd(&count[kSpreadBuilds], 1ull);
    if (class_was == c.class_tag) atomicAdd(&count[kSpreadClasses], 1ull);
}

// A row's workgroups that have read its state are counted, the last of a row counts in its group of rows, the last of a
// group in the call: who closes a row or the call is known by the ticket it took.  (With 256 rows on one address the die
// whose workgroups took them, one of the eight, had its loads up to 2.5 us later than the others: the last row of a
// cached fill, V = 151936, was out 8.6 us after the kernel's beginning, of a made one 15.7, in groups 7.0 and 14.0.)
struct Tickets {
    uint32_t group, call;        // as taken (of rows and of groups before), or kNoTicket
    bool row_last;
};
constexpr uint32_t kNoTicket = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t *group_counter(const CacheView &Cc, uint32_t b) { return &Cc.ctr->group_tickets[b / kTicketGroup * kTicketStride]; }
__device__ __forceinline__ bool group_last(const Tickets &t, uint32_t b, uint32_t rows)
{
    const uint32_t first = b / kTicketGroup * kTicketGroup;
    return t.group + 1u == (rows - first < kTicketGroup ? rows - first : kTicketGroup);
}

// What the last of a row and the last of the call do, once all of them have read the row's state and the call's number: on the
// way, since the kernel's end would wait for these stores (a pass of 8 cached steps, 1 request 39.7 -> 37.8 us, 64
// requests 61.0 -> 59.4).
__device__ __forceinline__ void close_row(const CacheView &Cc, const Tickets &t, uint32_t b, wg_state_t *states, const int32_t *tokens, const RowShared &sh)
{
    if (!t.row_last) return;
    Cc.ctr->tickets[b * kTicketStride] = 0u;
    if (tokens) states[b] = sh.state;
}
__device__ __forceinline__ void close_call(const CacheView &Cc, const Tickets &t, uint32_t b, uint32_t rows, const RowShared &sh)
{
    if (!t.row_last) return;
    const bool last = group_last(t, b, rows);
    if (last) *group_counter(Cc, b) = 0u;
    if (rows > kTicketGroup ? t.call + 1u == (rows + kTicketGroup - 1u) / kTicketGroup : last) {
        Cc.ctr->call_ticket = 0u;
        atomicAdd(&Cc.ctr->lookups, (unsigned long long)rows);       // (nobody waits for it)
        Cc.ctr->launch = sh.launch + 1ull;
    }
}

// The words [w_lo, w_hi) of a missing row are row[] | early[] (LDS, word 0 = w_lo): early holds what
// the candidates add, row the rest, so that the two are made side by side.
__device__ __forceinline__ void make_row(const TableView &T, const VocabView &Vc, const CacheView &Cc, RowShared &sh,
                                         const RowTask &me, const HopState &ha, const HopState &hb, uint32_t p0, uint32_t span,
                                         uint32_t w_lo, uint32_t w_hi, uint32_t *row, uint32_t *early, uint32_t b, bool claims)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t n_words = w_hi - w_lo, rs = Cc.row_stride;
    const uint32_t tok_lo = range_token(Vc.V, p0), tok_hi = range_token(Vc.V, p0 + span);
    const bool literal = me.kind == WG_KIND_LIT, ckpt = is_checkpoint(me.kind);
    const bool ckpt_a = is_checkpoint(ha.kind), ckpt_b = is_checkpoint(hb.kind);
    // the literal byte behind an exit, or a value no byte has
    const uint32_t lit_a = ha.kind == WG_KIND_LIT ? ha.lit : 0x100u, lit_b = hb.kind == WG_KIND_LIT ? hb.lit : 0x100u;
    auto before = [](unsigned long long bal) {
        return (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
    };
    const bool few_budget = ckpt && me.r < Vc.lmax;            // the byte budget binds inside a token
    const uint32_t n_exits = sh.plan.n_exits, n_ids = sh.plan.n_ids;
    const bool by_first = ckpt && sh.plan.by_first;
    uint32_t total = 0;
    if (wave == 0u) {
        // the index ranges with the key's candidates; rest: what a lane's ranges hold for the row's other workgroups, counted
        // by the first
        uint32_t n = 0, sure = 0, rest = 0;
        // with them the class tables of the successors and the literal bytes, for this wavefront's own candidates
        uint32_t table[2] = {0u, 0u}, byte = 0;
        if (ckpt_a) table[0] = reinterpret_cast<const uint32_t *>(T.classes + (size_t)ha.cls * 256u)[lane];
        if (ckpt_b) table[1] = reinterpret_cast<const uint32_t *>(T.classes + (size_t)hb.cls * 256u)[lane];
        const uint32_t side = lane >= 24u, at = side ? lane - 24u : lane;
        const uint32_t of = at + (literal ? me.sid : side ? (hb.kind == WG_KIND_LIT ? hb.next_a : 0u) : ha.kind == WG_KIND_LIT ? ha.next_a : 0u);
        if (lane < 48u && of < T.n_states) byte = T.lit[of];
        if (literal) {
            // (the one-byte tokens are taken as rows below: examined, but not one by one)
            if (lane == 0) {
                if (!ckpt_a) sure = Vc.dirs[kDirSorted + me.lit * 257u + 1u] - Vc.dirs[kDirSorted + me.lit * 257u];
            }
            n = ckpt_a || lit_a < 0x100u ? 1u : 0u;
        } else if (ckpt) n = n_exits;
        for (uint32_t r0 = 0; r0 < n; r0 += 64u) {
            const uint32_t i = r0 + lane;
            uint32_t lo = 0, len = 0;
            if (i < n) {
                const uint32_t id = literal ? me.lit : sh.plan.ids[i], x = id & 0xFFu, c = id >> 8;
                const bool side = c == CLS_EXIT_B;
                const uint32_t lit = side ? lit_b : lit_a;
                uint32_t from = literal ? (ckpt_a ? FROM_A : FROM_PREFIX)
                                        : by_first ? (c == CLS_STAY ? FROM_STAY : side ? FROM_B : FROM_A)
                                                   : lit < 0x100u ? FROM_PAIR : (side ? ckpt_b : ckpt_a) ? (side ? FROM_DEEP_B : FROM_DEEP_A) : 0u;
                uint32_t a = x * kParts + p0, n_at = span;
                if (from == FROM_PREFIX) { a = kDirSorted + x * 257u + 1u + lit; n_at = 1u; }
                else if (from == FROM_PAIR) { a = kDirPairs + (x << 8 | lit); n_at = 1u; }
                else if (from && from <= FROM_B) a += kDirFirst;
                else a += kDirPlaces;
                const bool by_range = from && from != FROM_PREFIX && from != FROM_PAIR;
                if (!from) n_at = 0u;                          // nothing goes on behind this exit
                lo = Vc.dirs[a];
                len = Vc.dirs[a + n_at] - lo;
                if (p0 == 0u && by_range) rest += Vc.dirs[a + kParts] - Vc.dirs[a + span];
                sh.code[i] = (uint16_t)(x | from << 8);
            }
            const uint32_t inc = wave_prefix_sum(len);
            if (i < n) { sh.start[i] = lo; sh.upto[i] = total + inc; }
            total += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
        if (ckpt_a) reinterpret_cast<uint32_t *>(sh.hop[0])[lane] = table[0];
        if (ckpt_b) reinterpret_cast<uint32_t *>(sh.hop[1])[lane] = table[1];
        if (lane < 48u) reinterpret_cast<uint8_t *>(sh.run[side])[at] = (uint8_t)byte;
        if (p0 == 0u) sure += of_lane(wave_prefix_sum(rest), 63u) + total;
        if (lane == 0) {
            sh.n_ranges = n; sh.total = total;
            if (p0 == 0u && sure) atomicAdd(&Cc.ctr->spread[(b % kSpread) * kSpreadStride + kSpreadWalked], (unsigned long long)sure);
            if (Vc.eos_id >= 0 && me.eos_next != WG_SID_ERROR) {
                const uint32_t ew = (uint32_t)Vc.eos_id >> 5;
                if (ew >= w_lo && ew < w_hi) early[ew - w_lo] |= 1u << ((uint32_t)Vc.eos_id & 31u);
            }
        }
        __builtin_amdgcn_wave_barrier();
    } else {
        // meanwhile the other wavefronts fill in what does not depend on a token's neighbours, four words
        // of a thread at a time (rows are padded to whole 16 bytes with zeros); the last one comes after what it
        // has claimed, if it has
        const uint32_t n4 = (n_words + 3u) / 4u, n3 = kRowThreads - (claims ? 128u : 64u), w4 = w_lo / 4u;
        const uint32_t q0 = claims && wave == kRowWaves - 1u ? n4 : tid - 64u;
        const uint4 *rows = reinterpret_cast<const uint4 *>(Vc.rows) + w4;
        const uint32_t rs4 = rs / 4u;
        auto token_row = [&](uint32_t id) { return rows + (size_t)id * rs4; };
        uint4 *row4 = reinterpret_cast<uint4 *>(row), *keep = reinterpret_cast<uint4 *>(Cc.class_rows) + (size_t)(2u * me.cls) * rs4 + w4;
        if (literal && !ckpt_a) {
            const uint4 *has = token_row(me.lit), *one = token_row(kLenRow + 1u);
            for (uint32_t q = q0; q < n4; q += n3) row4[q] = has[q] & one[q];
        } else if (!ckpt || by_first) {
            for (uint32_t q = q0; q < n4; q += n3) row4[q] = uint4{0u, 0u, 0u, 0u};
        } else {
            const uint4 *len_stay = token_row(kLenRow + me.r), *len_end = len_stay + rs4;
            if (me.class_state == CLASS_READY) {
                for (uint32_t q = q0; q < n4; q += n3) {
                    uint4 stay = keep[q], end = keep[rs4 + q];
                    if (few_budget) { stay = stay & len_stay[q]; end = end & len_end[q]; }
                    row4[q] = stay | end;
                }
            } else {
                const uint4 *has = token_row(kLenRow + Vc.lmax + 1u);
                for (uint32_t q = q0; q < n4; q += n3) {
                    // one: tokens with a byte value that does not stay, two: with several; tail: tokens with
                    // an exit byte once, at their end.  A token leaves with its last byte iff it is in tail and
                    // not in two, its bytes all stay iff it is not in one.
                    uint4 one{0u, 0u, 0u, 0u}, two = one, tail = one;
                    for (uint32_t i = 0; i < n_exits; i++) {
                        const uint32_t id = sh.plan.ids[i] & 0xFFu;
                        const uint4 x = token_row(id)[q], y = token_row(kTailRow + id)[q];
                        two = two | (one & x); one = one | x; tail = tail | y;
                    }
                    for (uint32_t i = n_exits; i < n_ids; i += kOrBatch) {
                        uint4 x[kOrBatch];
#pragma unroll
                        for (uint32_t u = 0; u < kOrBatch; u++) x[u] = token_row(sh.plan.ids[i + u < n_ids ? i + u : i])[q];
#pragma unroll
                        for (uint32_t u = 0; u < kOrBatch; u++) if (i + u < n_ids) { two = two | (one & x[u]); one = one | x[u]; }
                    }
                    uint4 s = ~one & has[q], x = tail & ~two;
                    if (me.class_state == CLASS_OWN) { keep[q] = s; keep[rs4 + q] = x; }
                    if (few_budget) { s = s & len_stay[q]; x = x & len_end[q]; }
                    row4[q] = s | x;
                }
            }
        }
        if (claims && tid == kRowThreads - 64u) claim_tags(Cc, sh, b);
    }
    // The candidates: a few are the first wavefront's, right away; many are everybody's, once all
    // know the ranges.
    auto set_bit = [&](uint32_t tok) { atomicOr(&early[(tok >> 5) - w_lo], 1u << (tok & 31u)); };
    auto decide = [&](uint32_t e) {
        const uint32_t tok = e & 0xFFFFFFu, L = e >> 24;
        TokenBytes t = token_bytes(Vc, tok, L);
        if (!ckpt) {
            if (walk_run(T, sh.run[0], me.sid, me.run, me.cls, t, 0u, L)) set_bit(tok);
            return;
        }
        uint32_t j = 0, c = CLS_STAY;
        while (j < L) {
            const uint32_t n = L - j < 8u ? L - j : 8u;
            const uint32_t code = class_code(sh.own, window(t, j)), s = first_leaving(code, n);
            j += s;
            if (s < n) { c = (code >> (2u * s)) & 3u; break; }
        }
        if (c == CLS_REJECT || j > me.r) return;               // j bytes that stay
        bool ok = c == CLS_STAY || j + 1u == L;
        if (!ok) {
            const bool side_b = c == CLS_EXIT_B;
            ok = walk_hop(T, sh.task.hop[side_b], sh.hop[side_b], sh.run[side_b], t, j + 1u, L);
        }
        if (ok) set_bit(tok);
    };
    const global_u2 *index = (const global_u2 *)Vc.index;
#pragma nounroll
    for (uint32_t pass = 0; pass < 2u; pass++) {
        if (pass) total = sh.total;
        if (pass ? total > kAlone : wave == 0u && total <= kAlone) {
            const uint32_t first_at = pass ? wave * 64u : 0u, step = pass ? kRowThreads : 64u;
            const uint32_t n_ranges = sh.n_ranges;
            uint32_t n_q = 0, widest = 1u;                             // first step of the search for a candidate's range
            while (widest * 2u < n_ranges) widest *= 2u;
            for (uint32_t base = first_at;; base += step * kRowBatch) {
                const bool more = base < total;
                if (more) {
                    uint2 e[kRowBatch];
                    uint32_t from[kRowBatch];
#pragma unroll
                    for (uint32_t u = 0; u < kRowBatch; u++) {
                        const uint32_t i = base + u * step + lane, ii = i < total ? i : total - 1u;
                        uint32_t k = 0;                                // the range that holds candidate ii
                        if (n_ranges > 1u)
                            for (uint32_t s = widest; s; s >>= 1)
                                if (k + s < n_ranges && sh.upto[k + s - 1u] <= ii) k += s;
                        const global_u2 *src = index + sh.start[k] + (ii - (k ? sh.upto[k - 1u] : 0u));
                        e[u] = uint2{src->x, src->y};
                        from[u] = i < total ? sh.code[k] >> 8 : 0u;
                    }
#pragma unroll
                    for (uint32_t u = 0; u < kRowBatch; u++) {
                        const uint32_t tok = e[u].x, first = (e[u].y >> 16) & 0xFFu, L = (e[u].y & 0xFFu) + (e[u].y >> 24);
                        const uint32_t f = from[u];
                        bool decide_it = false;
                        if (f != 0u && tok >= tok_lo && tok < tok_hi) {
                            const bool side_b = f == FROM_B || f == FROM_DEEP_B;
                            if (f == FROM_PREFIX || f == FROM_PAIR) decide_it = true;
                            // a one-byte token is settled by the byte's class
                            else if (L == 1u) { if (f != FROM_STAY || me.r != 0u) set_bit(tok); }
                            else if (f == FROM_STAY) decide_it = sh.own[first] != CLS_REJECT;
                            else if (side_b ? ckpt_b : ckpt_a) decide_it = sh.hop[side_b][first] != CLS_REJECT;
                            else decide_it = (side_b ? lit_b : lit_a) == first;
                        }
                        const unsigned long long m = __ballot(decide_it);
                        if (decide_it) sh.queue[wave][n_q + before(m)] = tok | L << 24;
                        n_q += (uint32_t)__popcll(m);
                    }
                }
                while (n_q >= 64u || (!more && n_q)) {
                    const uint32_t take = n_q < 64u ? n_q : 64u;
                    n_q -= take;
                    if (lane < take) decide(sh.queue[wave][n_q + lane]);
                }
                if (!more) break;
            }
        }
        __syncthreads();
        if (sh.total <= kAlone) break;
    }
}

// The call is over for the cache once its lookups are: one thread then counts the claimed rows as used
// and opens the next call.
__device__ __forceinline__ void close_fill(const CacheView &Cc, uint32_t B, uint32_t n, uint32_t n_classes)
{
    const unsigned long long sc = Cc.ctr->slot_ctr;
    const uint32_t used = (uint32_t)(sc >> 32) == Cc.epoch ? (uint32_t)sc : 0u;
    const uint32_t room = Cc.cap_rows - used;
    if (n > room) Cc.ctr->uncached_builds += n - room;
    Cc.ctr->slot_ctr = ((unsigned long long)Cc.epoch << 32) | (used + (n < room ? n : room));
    Cc.ctr->lookups += B;
    Cc.ctr->builds += n;
    Cc.ctr->class_scans += n_classes;
    Cc.ctr->launch++;
}

// The late arguments that the way of a cached row needs, asked for before it needs them: behind the advance's first loads, or while
// the other wavefronts wait for the first.  Read where they were needed they were eight waits of 100 cycles in turn.  Held in registers from there to the
// end (kHeld) where the logits are masked through the L2: eight cached steps, outlines, V = 128256, B = 64, us, so / not, 51.4 / 51.5, cold ones of 96 mixed
// requests on V = 100003 111.7 / 112.3.  Else asked for again behind the lookup, when their lines are near: the kernel has too few scalar registers to hold
// what its end needs through the lookup, and puts other values into lanes of vector registers on the way of every wavefront.  Held / asked for again,
// V = 151936, B = 256, eight steps, mixed, cached 169.7 / 167.5, cold 216.9 / 216.4, random trees 183.6 / 182.4, outlines 135.2 / 134.7, cold 174.5 / 173.1; masks
// alone behind a sampled token, outlines and mixed, copied 7.21 / 7.13, 7.28 / 7.10, made 15.7 / 14.5, 16.9 / 15.8; up to 16 requests, masks alone 0.99 to 1.01 of it, logits of
// up to 1 MiB 1.00 to 1.01.  (Neither held nor asked for again, by which the compiler has them in lanes, eight cached steps took 166.0, 179 and 135.8, but
// cold ones 218.2 and 175.2, and those of 600 requests, V = 128256, 440.5, not 437.8.)  (Every wavefront deciding for itself by the tag, without the barrier
// behind the lookup, and lanes that take the bits they mask from memory instead of LDS: 1 to 10 % slower with logits of 20 MB and more.)
struct RowArgs {
    unsigned long long *tags, *class_tags;
    uint32_t *arena, *bitmask;
    void *logits;
    int64_t logits_stride;
    uint32_t cap_rows, row_stride, epoch, lmax, W, rows;
    RowArgs() = default;
    __device__ __forceinline__ explicit RowArgs(Late &late)
        : tags(late.Cc.tags), class_tags(late.Cc.class_tags), arena(late.Cc.arena), bitmask(late.bitmask), logits(late.logits), logits_stride(late.logits_stride),
          cap_rows(late.Cc.cap_rows), row_stride(late.Cc.row_stride), epoch(late.Cc.epoch), lmax(late.T.lmax), W(late.Vc.W), rows(late.rows) {}
};
// (which the compiler does not see to be the same: it would keep them in registers meanwhile)
__device__ __forceinline__ RowArgs read_again(Late &late)
{
    Late *l = &late;
    asm volatile("" : "+s"(l));
    return RowArgs(*l);
}

// kMode 0: masks only; 1: -inf into the logits as well; 2: the same, whole lines (see mask_lines); 3: as 1, the stores
// through the L2.
// kWhole: the lookups have not been done: each workgroup of a row does its row's, with the advance
// before it (tokens may be null).  One launch instead of two, and a row waits for its own lookup only, not for
// the longest walk of the batch.  While the first wavefront walks, the last one takes the row's ticket.  The last
// workgroup of a row to have read its state writes the new one as soon as it has it (close_row), before it looks it up; the last such row of all opens the next call (close_call).  (A ticket on one address for every workgroup of the call, taken by the wavefront that walks, cost
// 10 ns a workgroup: this fill took 28 us for 2,048 workgroups, 18 as it is now.)  Within 64 vector registers, so
// that 8 workgroups of a unit are resident: with 7 the last 256 of 2,048 began 7 to 11 us after the others.
template <typename Elem, int kMode, bool kWhole>
__global__ void __launch_bounds__(kRowThreads, 8)
rows_kernel(WG_EARLY_ARGS)
{
    WG_VIEWS;
    extern __shared__ __attribute__((aligned(16))) uint32_t row[];
    __shared__ __attribute__((aligned(16))) RowShared sh;
    const uint32_t b = blockIdx.y, tid = threadIdx.x, span = late.span, p0 = blockIdx.x * span;
    const uint32_t tok_lo = range_token(Vc.V, p0), tok_hi = range_token(Vc.V, p0 + span);
    const uint32_t w_lo = tok_lo >> 5, w_hi = (tok_hi + 31u) >> 5, n_words = w_hi - w_lo;
    const uint32_t n4 = (n_words + 3u) / 4u;      // (rows are padded to whole 16 bytes)
    uint4 *row4 = reinterpret_cast<uint4 *>(row), *early4 = row4 + n4 + 1u;
    Tickets ticket{kNoTicket, kNoTicket, false};
    uint4 ahead{0u, 0u, 0u, 0u};                      // the cached row's piece of this thread, should there be one
    constexpr bool kSpan = kMode == 1 || kMode == 3;
    constexpr bool kHeld = kMode == 3;
    RowArgs args;
    if (kWhole) {
        const uint32_t wave = of_first(tid >> 6);
        uint32_t sid = 0, aux = 0, t = 0;
        unsigned long long launch = 0;
        StateDesc d{};
        Asked asked{};
        WalkArgs walk;
        if (wave == 0u) {
            launch = Cc.ctr->launch;
            const wg_state_t st = states[b];
            if (tokens) t = of_first((uint32_t)tokens[b]);
            sid = of_first(st.sid); aux = of_first(st.aux);
            // The state and the call's number have to be here before the row's ticket counts this workgroup: the last one of the row
            // replaces the state, the last one of the call the number (close_row, close_call).  In one wait with them what the advance
            // needs of the late arguments and a word of each of their lines, so that whoever reads them later does not wait for memory.
            walk = WalkArgs(late);
            asm volatile("" :: "s"(launch), "s"(sid), "s"(aux), "s"(walk.lit), "s"(walk.codes), "s"(walk.n_chunks), "s"(walk.eos_id), "s"(late.Vc.rows), "s"(late.Cc.tags), "s"(late.Cc.tasks), "s"(late.rows));
            hold(walk.lit, walk.codes, walk.n_chunks, walk.eos_id);
            if (tid == 0) sh.launch = launch;
        }
        __syncthreads();
        if (tid == kRowThreads - 64u) {
            ticket.row_last = atomicAdd(&Cc.ctr->tickets[b * kTicketStride], 1u) == late.shares - 1u;
            if (ticket.row_last) ticket.group = atomicAdd(group_counter(Cc, b), 1u);       // (waited for behind the walk)
        }
        // (behind the advance's first loads, or while the first wavefront is busy)
        auto read_args = [&]() {
            args = RowArgs(late);
            if (kHeld) hold(args.tags, args.class_tags, args.arena, args.cap_rows, args.row_stride, args.epoch, args.lmax, args.bitmask, args.W, args.rows, args.logits, args.logits_stride);
            else asm volatile("" :: "s"(args.tags), "s"(args.arena), "s"(args.bitmask), "s"(args.lmax));
        };
        if (wave == 0u) {
            if (tokens) {
                const Sampled s = ask_sampled(T, Vc, walk, sid, (int32_t)t);
                read_args();
                advance_one(T, Vc, Cc, walk, s, sid, aux, d, (int32_t)t, p0 == 0u, b);
            } else {
                const uint32_t words = two_states(T, sid, sid);
                read_args();
                d = state_of(words, 0u);
            }
            asked = ask<true>(T, args.lmax, args.tags, args.class_tags, nullptr, sid, aux, d);
            if (tid == 0) {
                sh.state = wg_state_t{sid, aux};
                sh.key = asked.key;
                sh.desc = d;
            }
        } else {
            read_args();
            if (wave >= 2u) for (uint32_t q = tid - 128u; q < n4; q += kRowThreads - 128u) early4[q] = uint4{0u, 0u, 0u, 0u};
        }
        __syncthreads();
        // (key k has arena row k: the row is requested while its tag is looked at, and what a missing row takes from the
        // state's own class table)
        const uint32_t key = of_first(sh.key);
        bool ckpt = false;
        StagedClass staged{};
        if (wave == 1u) {
            ckpt = is_checkpoint(of_first(sh.desc.kind_byte) & 0xFFu);
            if (ckpt) staged = ask_class(T, of_first(sh.desc.cls), tid & 63u);
        }
        if (key < args.cap_rows && tid < n4) ahead = reinterpret_cast<const uint4 *>(args.arena + (size_t)key * args.row_stride + w_lo)[tid];
        if (args.rows > kTicketGroup && group_last(ticket, b, args.rows)) ticket.call = atomicAdd(&Cc.ctr->call_ticket, 1u);
        close_row(Cc, ticket, b, states, tokens, sh);
        if (ckpt) put_class(sh, staged, tid & 63u);
        if (wave == 0u) {
            const Found f = look_up<true>(T, Cc, tag_now(args.epoch, launch), b, sid, d, asked, &sh.claim);
            if (tid == 0) {
                sh.ref = f.ref;
                if (f.ref == kRefBuild) sh.task = f.me;
                if (f.hit && p0 == 0u) atomicAdd(&Cc.ctr->spread[(b % kSpread) * kSpreadStride + kSpreadHits], 1ull);
            }
        }
        __syncthreads();
    }
    const RowTask in = kWhole ? sh.task : Cc.tasks[b];   // (requested with the reference; only used where that asks for it)
    const uint32_t ref = (uint32_t)__builtin_amdgcn_readfirstlane((int)(kWhole ? sh.ref : Cc.row_ref[b]));
    uint32_t slot = kNoSlot;
    if (ref == kRefBuild) {
        // (the same for every lane: to scalar registers)
        auto one = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
        auto hop = [&](const HopState &h) { return HopState{one(h.kind), one(h.lit), one(h.next_a), one(h.next_b), one(h.max), one(h.cls)}; };
        const HopState ha = hop(in.hop[0]), hb = hop(in.hop[1]);
        const RowTask me{one(in.sid), one(in.kind), one(in.lit), one(in.cls), one(in.run), one(in.r), one(in.class_state), one(in.eos_next), one(in.slot), {}};
        slot = me.slot;
        if (!kWhole) {
            if (tid == kRowThreads - 1u) { sh.task.hop[0] = ha; sh.task.hop[1] = hb; }
            for (uint32_t q = tid; q < n4; q += kRowThreads) early4[q] = uint4{0u, 0u, 0u, 0u};
            if (tid >> 6 == 1u && is_checkpoint(me.kind)) put_class(sh, ask_class(T, me.cls, tid & 63u), tid & 63u);
            __syncthreads();
        }
        make_row(T, Vc, Cc, sh, me, ha, hb, p0, span, w_lo, w_hi, row, reinterpret_cast<uint32_t *>(early4), b, kWhole && p0 == 0u);
        if (kWhole) args = read_again(late);
        ahead = uint4{0u, 0u, 0u, 0u};
    }
    if (!kWhole) {
        // (each where it is needed: asked for together, the cached rows of 257 to 1,024 requests took 0.3 % longer)
        args.arena = Cc.arena; args.cap_rows = Cc.cap_rows; args.row_stride = Cc.row_stride;
        args.bitmask = late.bitmask; args.W = Vc.W;
    } else if (!kHeld) args = read_again(late);
    // out: to the cache, the caller's bitmask, and LDS for the masking
    const bool copied = ref < args.cap_rows;
    const uint32_t *row_in = args.arena + (size_t)(copied ? ref : 0u) * args.row_stride + w_lo;
    const uint4 *src = reinterpret_cast<const uint4 *>(row_in);
    uint4 *kept = reinterpret_cast<uint4 *>(args.arena + (size_t)slot * args.row_stride + w_lo);
    uint32_t *dst = args.bitmask + (size_t)b * args.W + w_lo;
    Elem *logits = kWhole ? static_cast<Elem *>(args.logits) + (int64_t)b * args.logits_stride : nullptr;
    const bool aligned = reinterpret_cast<uintptr_t>(dst) % 16u == 0u;
    for (uint32_t q = tid; q < n4; q += kRowThreads) {
        uint4 x{0u, 0u, 0u, 0u};
        if (ref == kRefBuild) x = row4[q] | early4[q];
        else if (copied) x = kWhole && q == tid ? ahead : src[q];
        if (slot != kNoSlot) kept[q] = x;
        if (aligned) {
            if (4u * q + 4u <= n_words) reinterpret_cast<uint4 *>(dst)[q] = x;
            else {
                dst[4u * q] = x.x;
                if (4u * q + 1u < n_words) dst[4u * q + 1u] = x.y;
                if (4u * q + 2u < n_words) dst[4u * q + 2u] = x.z;
            }
        }
        if (kMode || !aligned) row4[q] = x;
    }
    if (kWhole) close_call(Cc, ticket, b, args.rows, sh);
    if (kMode || !aligned) __syncthreads();
    if (!aligned) for (uint32_t w = tid; w < n_words; w += kRowThreads) dst[w] = row[w];
    if (!kWhole) logits = static_cast<Elem *>(late.logits) + (int64_t)b * late.logits_stride;
    if (kSpan) mask_span<Elem, kMode == 3>(logits, tok_lo, tok_hi, row);
    if (kMode == 2) mask_lines<Elem, sizeof(Elem) == 4 ? 8u : 5u>(logits, tok_lo, tok_hi, row);
    if (!kWhole && blockIdx.x == 0 && b == 0 && tid == 0) {
        close_fill(Cc, late.rows, Cc.ctr->n_claims, Cc.ctr->n_class_claims);
        Cc.ctr->n_claims = 0; Cc.ctr->n_class_claims = 0;
    }
}

// The arena stops being addressed by key (more keys than rows): the rows that no key of this
// generation holds, behind as many places as rows are in use; the held keys get their slots.
__global__ void __launch_bounds__(1024)
free_rows_kernel(DeviceCache Cc, uint32_t n_keys, uint32_t *__restrict__ free_rows)
{
    __shared__ uint32_t wave_n[16], base;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    if (tid == 0) base = 0u;
    __syncthreads();
    uint32_t held = 0;
    for (uint32_t i = tid; i < n_keys; i += 1024u) {
        Cc.slots[i] = i;
        held += (uint32_t)(Cc.tags[i] >> kTagEpochShift) == Cc.epoch;
    }
    atomicAdd(&base, held);
    __syncthreads();
    if (tid == 0) Cc.ctr->slot_ctr = (unsigned long long)Cc.epoch << 32 | base;
    for (uint32_t r0 = 0; r0 < Cc.cap_rows; r0 += 1024u) {
        const uint32_t r = r0 + tid;
        const bool is_free = r < Cc.cap_rows && !(r < n_keys && (uint32_t)(Cc.tags[r] >> kTagEpochShift) == Cc.epoch);
        const unsigned long long m = __ballot(is_free);
        __syncthreads();
        if (lane == 0) wave_n[wave] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t at = base, all = 0;
        for (uint32_t w = 0; w < 16u; w++) { if (w < wave) at += wave_n[w]; all += wave_n[w]; }
        at += (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (is_free && at < Cc.cap_rows) free_rows[at] = r;
        __syncthreads();
        if (tid == 0) base += all;
    }
}

// wg_cache_stats: the keys that hold a row (brought to the host a page at a time they took 460 us for 64,000 keys, now 38).
__global__ void __launch_bounds__(256) count_rows_kernel(DeviceCache Cc)
{
    uint32_t held = 0;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < Cc.n_keys; i += gridDim.x * 256u) held += (uint32_t)(Cc.tags[i] >> kTagEpochShift) == Cc.epoch;
    held = wave_prefix_sum(held);
    if ((threadIdx.x & 63u) == 63u && held) atomicAdd(&Cc.ctr->held, (unsigned long long)held);
}

// apply: a wavefront takes kPairs times 64 tokens of a row, its mask straight from memory: 32 (with 8, 16, 32 and 64, V =
// 151936, B = 256, bf16, mixed 14.8, 13.3, 13.4 and 13.1 us; V = 32000, B = 256 5.1, 4.9, 4.6 and 5.2), and 24 of bf16 logits of
// more than kApplyLarge bytes, where 32 were up to 5 % slower than a store per disallowed token of each piece on scattered
// tokens (by pieces / 32 / 24, V = 151936, B = 600, 182 MB: 4 % at random 27.7 / 28.1 / 27.3, 8 % 34.4 / 35.3 / 33.1, html 24.7 / 25.3 /
// 24.3, mixed 29.0 / 28.0 / 28.0; B = 400, 122 MB, 4 % 19.4 / 20.0 / 19.1).  Why is not shown; 3 KB of logits to a wavefront instead
// of 4 may keep neighbours from storing to one channel at a time, but 40 (5 KB) are 3 % slower and 16 cost more launches.
// Below: 78 MB html, JSON, mixed, random trees 0.98 0.98 1.01 1.01 of the time with 32, 33 MB 1.04 1.05 1.03 1.01; fp32, V =
// 128256, B = 600, random trees 1.05.
// A wavefront with at most 1.5 tokens of 64 to mask lists them in LDS and stores them all at once: reading lanes and
// storing for every 64 tokens it was slower than a store per disallowed token of each piece had been (that / always 64 at
// a time / now, V = 151936, bf16, tokens disallowed at random: 0.2 % B = 256 5.4 / 6.7 / 4.3, 600 11.6 / 12.7 / 9.3; 1.2 % B = 64
// 3.7 / 4.0 / 3.5, 256 8.2 / 8.4 / 7.1, 600 15.4 / 15.0 / 14.0; 1.8 % B = 128 5.8 / 6.3 / 5.5, 256 9.2 / 9.3 / 8.8).  With 1 of 64
// the gain ends at 1.5 %; with 2 the free text of html and JSON (V = 128256, 3 %) is listed too, in 9.9 instead of 9.7 and 10.5
// instead of 10.2 us, B = 256.
constexpr uint64_t kApplyLarge = 96ull << 20;
template <typename Elem, uint32_t kPairs, bool kThrough>
__global__ void __launch_bounds__(256)
apply_kernel(Elem *__restrict__ logits, int64_t row_stride, uint32_t V, uint32_t W, const uint32_t *__restrict__ bitmask)
{
    constexpr Elem kNinf = sizeof(Elem) == 4 ? (Elem)0xFF800000u : (Elem)0xFF80u;
    constexpr uint32_t kFew = kPairs * 3u / 2u;
    static_assert(kPairs % kChunk == 0u && kPairs <= 64u && kFew <= 64u, "a lane each");
    __shared__ uint16_t few[4][kFew];
    const uint32_t b = blockIdx.y, lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t first = (blockIdx.x * 4u + wave) * kPairs;
    const uint32_t *row = bitmask + (size_t)b * W;
    Elem *p = logits + (int64_t)b * row_stride;
    const uint32_t skew = skew_of(p);
    uint32_t lo = 0xFFFFFFFFu, hi = 0xFFFFFFFFu;
    if (lane < kPairs) bits_of_chunk(row, first + lane, W, V, skew, lo, hi);
    p += (int64_t)first * 64 - skew;
    const uint32_t off = (uint32_t)(__popc(~lo) + __popc(~hi)), upto = wave_prefix_sum(off);
    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    if (n <= kFew) {
        uint32_t at = upto - off;
        for (unsigned long long z = ~((unsigned long long)hi << 32 | lo); z; z &= z - 1ull)
            few[wave][at++] = (uint16_t)(lane * 64u + (uint32_t)__builtin_ctzll(z));
        __builtin_amdgcn_wave_barrier();
        if (lane < n) p[few[wave][lane]] = kNinf;
        return;
    }
#pragma unroll
    for (uint32_t c = 0; c < kPairs; c += kChunk) mask_chunk<Elem, kThrough>(p + (size_t)c * 64u, lo, hi, c);
}

// The same by whole lines: a workgroup takes kLineTokens tokens of a row.
constexpr uint32_t kLineTokens = 8192;
template <typename Elem>
__global__ void __launch_bounds__(256)
apply_lines_kernel(Elem *__restrict__ logits, int64_t row_stride, uint32_t V, uint32_t W, const uint32_t *__restrict__ bitmask)
{
    __shared__ uint32_t row[kLineTokens / 32u + 1u];
    const uint32_t b = blockIdx.y, lo = blockIdx.x * kLineTokens, hi = lo + kLineTokens < V ? lo + kLineTokens : V;
    static_assert(kLineTokens == 32u * 256u, "a mask word per thread");
    const uint32_t w = (lo >> 5) + threadIdx.x;
    row[threadIdx.x] = w < W ? bitmask[(size_t)b * W + w] : 0u;
    __syncthreads();
    mask_lines<Elem, sizeof(Elem) == 4 ? 8u : 4u>(logits + (int64_t)b * row_stride, lo, hi, row);
}

// The bytes a request is forced to produce next: from a state inside a Write, the rest of that
// Write and of the Writes that follow it directly, up to the next state that is not a literal
// byte.  A wavefront per request, a byte per lane: a Write costs one trip to memory, for its bytes and its descriptor
// together, and the stores of one overlap the next one's trip.  (With a thread per request, a byte at a
// time, a jump-forward step of 64 outlines took 17.9 us, now 17.3.)
__global__ void __launch_bounds__(256)
forced_bytes_kernel(const wg_state_t *__restrict__ states, const StateDesc *__restrict__ descs, const uint8_t *__restrict__ lit,
                    uint8_t *__restrict__ bytes, uint32_t *__restrict__ lens, wg_state_t *__restrict__ end_states,
                    uint32_t n_states, uint32_t cap, uint32_t B)
{
    const uint32_t lane = threadIdx.x & 63u, waves = blockDim.x >> 6;
    // (any number of requests: more than the grid holds come in turn)
    for (uint64_t b = (uint64_t)blockIdx.x * waves + of_first(threadIdx.x >> 6); b < B; b += (uint64_t)gridDim.x * waves) {
        uint32_t sid = of_first(states[b].sid), n = 0;
        const uint32_t aux = of_first(states[b].aux);
        uint8_t *out = bytes + b * cap;
        uint32_t words = 0, byte = 0;                        // dword lane % 8 of the state's descriptor; literal byte sid + lane
        auto request = [&]() {
            if (sid >= n_states) return;
            words = reinterpret_cast<const uint32_t *>(descs + sid)[lane & 7u];
            if (lane < n_states - sid) byte = lit[sid + lane];
        };
        request();
        while (n < cap && sid < n_states) {
            const StateDesc d = state_of(words, 0u);
            if ((d.kind_byte & 0xFFu) != WG_KIND_LIT) break;
            const uint32_t m = d.run < cap - n ? d.run : cap - n, from = sid, first = byte;
            sid = m == d.run ? d.cls : sid + m;              // d.cls: state after the Write
            request();
            if (lane < m) out[n + lane] = (uint8_t)first;
            for (uint32_t i = lane + 64u; i < m; i += 64u) out[n + i] = lit[from + i];
            n += m;
        }
        if (lane) continue;
        lens[b] = n;
        if (end_states) end_states[b] = wg_state_t{sid, n ? 0u : aux};
    }
}

// The same by a thread per request, for batches whose wavefronts would have to take turns (launch_forced_bytes).
__global__ void __launch_bounds__(64)
forced_bytes_of_many_kernel(const wg_state_t *__restrict__ states, const StateDesc *__restrict__ descs, const uint8_t *__restrict__ lit,
                            uint8_t *__restrict__ bytes, uint32_t *__restrict__ lens, wg_state_t *__restrict__ end_states,
                            uint32_t n_states, uint32_t cap, uint32_t B)
{
    for (uint64_t b = (uint64_t)blockIdx.x * 64u + threadIdx.x; b < B; b += (uint64_t)gridDim.x * 64u) {
        const wg_state_t st = states[b];
        uint32_t sid = st.sid, n = 0;
        while (n < cap && sid < n_states) {
            const StateDesc d = descs[sid];
            if ((d.kind_byte & 0xFFu) != WG_KIND_LIT) break;
            const uint32_t m = d.run < cap - n ? d.run : cap - n;
            for (uint32_t i = 0; i < m; i++) bytes[b * cap + n + i] = lit[sid + i];
            n += m;
            sid = m == d.run ? d.cls : sid + m;              // d.cls: state after the Write
        }
        lens[b] = n;
        if (end_states) end_states[b] = wg_state_t{sid, n ? 0u : st.aux};
    }
}

// One block per row: d_tokens[b] = index of the (draw mod popcount)-th set bit.
__global__ void __launch_bounds__(256)
select_kernel(const uint32_t *__restrict__ bitmask, uint32_t W, const uint64_t *__restrict__ draws,
              int32_t *__restrict__ tokens)
{
    __shared__ uint32_t cnt[256];
    __shared__ uint32_t total;
    uint32_t b = blockIdx.x, tid = threadIdx.x;
    const uint32_t *row = bitmask + (size_t)b * W;
    uint32_t per = (W + 255u) / 256u, lo = tid * per, hi = lo + per < W ? lo + per : W;
    uint32_t c = 0;
    for (uint32_t w = lo; w < hi; w++) c += __popc(row[w]);
    cnt[tid] = c;
    __syncthreads();
    if (tid == 0) {
        uint32_t s = 0;
        for (int i = 0; i < 256; i++) { uint32_t x = cnt[i]; cnt[i] = s; s += x; }   // exclusive scan
        total = s;
        if (s == 0) tokens[b] = -1;
    }
    __syncthreads();
    if (total == 0) return;
    uint32_t k = (uint32_t)(draws[b] % (uint64_t)total);
    if (k >= cnt[tid] && k < cnt[tid] + c) {
        k -= cnt[tid];
        for (uint32_t w = lo; w < hi; w++) {
            uint32_t x = row[w], pc = __popc(x);
            if (k >= pc) { k -= pc; continue; }
            for (int bit = 0; bit < 32; bit++)
                if ((x >> bit) & 1u) { if (k == 0) { tokens[b] = (int32_t)(w * 32u + bit); return; } k--; }
        }
    }
}
// ---------------------------------------------------------------------------------------------
// launchers (host)

static inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// Logits of more bytes than these are masked by whole lines (see mask_lines): 128 bytes are read where a
// line is mixed, but no store leaves the memory to read and write the block around it.  What it gains
// depends on how many tokens of a line are disallowed, which the host does not know; the limits lie near where
// the geometric mean over four kinds of masks is the same for both: 215 MB of bf16 and 345 MB of fp32 by these
// figures.  By elements / by lines, us, a cached step on the masks of html outlines, of JSON objects, of
// both mixed, and of random trees (16, 25, 45 and 63 % of the tokens disallowed), two buffers in turn:
//   bf16, V = 151936: 182 MB 29 / 60, 31 / 59, 54 / 64, 80 / 64; 213 MB 50 / 69, 61 / 68, 84 / 74, 89 / 72; 243 MB 81 / 78,
//   87 / 76, 105 / 83, 107 / 83
//   fp32, V = 128256: 257 MB 26 / 64, 31 / 67, 44 / 73, 113 / 87; 308 MB 42 / 75, 73 / 78, 85 / 86, 124 / 96; 359 MB 64 / 87, 95 / 89,
//   111 / 99, 160 / 121
// (a block holds twice as many bf16 tokens, so fewer of them stay untouched.)  So html outlines lose up to a
// third right above the limit and random trees a quarter right below it.  Deciding by the density of each
// row or line was slower than the better of the two for all.
constexpr uint64_t kLineBytes16 = 208ull << 20, kLineBytes32 = 320ull << 20;

static bool by_lines(int dtype, uint32_t B, uint32_t V)
{
    const uint64_t n = (uint64_t)B * V;
    return dtype == WG_F32 ? n * 4u > kLineBytes32 : n * 2u > kLineBytes16;
}

// Where the logits are not masked by whole lines, a store goes through the die's L2 (sc1) as long as the buffers that an engine
// has in turn stay in the last-level cache: the end of the kernel then does not wait for the L2 to write back what it
// holds.  40 MiB: six such buffers fit the 256 MB.  us, into the L2 / through it, outlines, mixed, random trees, bf16, V =
// 151936: B = 64, two buffers in turn, wg_apply_mask 4.7 5.0 5.6 / 3.9 4.4 5.0, a cached wg_decode_step 7.4 7.8 8.1 / 6.8 7.0
// 7.4; six in turn, the step with B = 128 (39 MB) 9.2 9.8 11.4 / 8.7 9.2 10.7, 160 (49 MB) 10.5 11.5 15.5 / 11.0 12.0 15.5, 256
// (78 MB) 23.1 32.3 34.2 / 24.0 32.4 35.1.  (Two in turn gain up to 120 MB: 256 13.7 15.0 17.8 / 13.1 14.4 17.2.)
// Up to 1 MiB the L2s have next to nothing to write back, and what goes through takes longer to be stored: geometric means over 24 to 54 batches each of bf16 and
// fp32, into / through, wg_apply_mask up to 0.25 MiB 0.99, 0.5 0.99, 1 1.00, 2 1.01, a cached wg_decode_step 0.98, 0.98, 0.99, 1.00 (one
// request, V = 32,000, fp32 4.41 / 4.47 us, 151,936, bf16 4.82 / 4.93).  With the greedy choice over all logits behind the step, which reads what
// was stored, four buffers in turn, through / into, 207 batches: up to 4 MiB 1.00, 8 0.98, 12 to 25 0.95 to 0.96, 40 0.98, 50 0.99, 60 1.01, 80 1.03.
constexpr uint64_t kThroughLeast = 1ull << 20, kThroughBytes = 40ull << 20;
static bool masks_through(const void *logits, int dtype, uint32_t B, uint32_t V)
{
    const uint32_t e = dtype == WG_F32 ? 4u : 2u;
    const uint64_t bytes = (uint64_t)B * V * e;
    return logits && reinterpret_cast<uintptr_t>(logits) % e == 0u && bytes > kThroughLeast && bytes <= kThroughBytes;
}

// Workgroups per row (it is cut at its token ranges).  8, which with long rows of 256 requests is as many as are
// resident together (8 to a unit); more where that leaves compute units idle, as long as a workgroup keeps enough
// tokens to be worth what it starts with: 4,096 up to 4 workgroups on a unit, 6,144 up to 7.  Geometric means over the
// masks of four kinds of templates, wg_decode_step, time with 16 / with 8, rows made and rows copied:
//   V = 151936 B = 64 0.90 0.94, 96 0.95 0.98, 112 0.93 0.98, 128 0.96 1.01; 100003 B = 64 0.93 0.96, 96 0.94 1.00, 112 1.00
//   1.00, 128 1.03 1.02; 65536 B = 24 0.93 0.96, 64 0.95 0.99, 96 1.01 1.01; with 32 / with 16, 151936 B = 16 0.96 0.97, 32 0.96
//   0.99, 48 1.03 1.02; mixed, us with 8 / 16 / 32, 151936 B = 1 11.3 / 9.7 / 8.8 and 8.3 / 6.8 / 6.0
// Up to a workgroup per unit as many as a row has groups (kPartGroup): with 16 or 32 / with 8, made rows, 8000 (4 / 2) B = 64 0.93, 20000
// B = 8 0.97, 32000 B = 1 0.95, 50257 B = 6 0.94, 90000 B = 4 0.97; copied ones are a launch either way
// (but for the masks alone of up to 8 requests, 32 / 16 shares, V = 50257 to 128256: 4.25 / 4.12 us copied, 0.91 to 1.02 of it made).
// Fewer where a short row would be cut into scraps: with 4 / 2, V = 12000 B = 64 11.1 / 11.5 and 6.9 / 7.1.  Above a request per unit a share
// pays for what it starts with the more, the more workgroups wait for a place; but what takes longest to make (states of random trees with
// thousands of candidates) takes longer still in longer shares, while the units that are done wait for it.  So a share has 1.25 tokens per workgroup of
// the call (of 256 units), 3,072 at least, 12,288 at most.  Cold wg_fill_masks on outlines, JSON, mixed, random trees, 4 shares / 8: B = 400 V =
// 24576 (24 us with 8) 0.78 0.79 0.82 0.80; 512 32000 0.81 0.77 0.84 0.83, 40000 0.80 0.79 0.77 0.88; 1024 50257 0.78 0.80 0.77 0.97, 65536 0.77 0.75
// 0.77 1.06; 2 / 8, 2048 32000 (68 us with 8) 0.51 0.57 0.58 0.60; copied rows 0.5 to 0.9.  Random trees, 4 / 8, mean and worst of six sets, on this
// side of the line: B = 512 V = 40000 0.92 0.99, 700 50257 0.91 0.99, 1000 65536 0.91 0.99; beyond it: 257 50257 1.10 1.22, 65536 1.20 1.37, 90000 1.32
// 1.43; 400 65536 1.12 1.29, 90000 1.18 1.36; 700 65536 1.04 1.15 (outlines there 0.75 to 1.0).
// Fewer too where the lookup that each repeats is most of a short share's work: up to a request per unit and more than
// seven workgroups on one (above, rows are looked up once).  With 8 / 4, B = 256, us of a wg_decode_step on outlines, JSON,
// mixed, random trees: copied V = 24576 7.4 7.4 7.4 7.4 / 6.4 6.4 6.4 6.5, 32768 7.6 7.6 7.6 7.7 / 6.7 6.7 6.8 7.1; made 24576 12.9 13.7
// 14.5 20.4 / 12.4 13.1 13.1 18.1, 32768 14.9 15.0 14.4 22.0 / 14.3 13.9 13.3 22.6.  Longer rows gain less and random trees
// take up to a fifth longer to make (wg_fill_masks, 4 over 8, B = 225, V = 36800 1.01 1.01 0.93 1.14, 65536 0.89 1.00 1.00 1.21; copied 0.88).
constexpr uint32_t kLeastParts = 8;
static uint32_t row_parts(uint32_t V, uint32_t B, uint32_t n_cu)
{
    uint32_t parts = kLeastParts;
    while (parts < kParts) {
        const uint64_t n = (uint64_t)B * parts * 2u;
        if (n > 7ull * n_cu || parts * 2u * (n <= n_cu ? kPartGroup / 2u : n <= 4ull * n_cu ? 4096u : 6144u) > V) break;
        parts *= 2u;
    }
    if (parts == kLeastParts && B <= n_cu && B * parts > 7u * n_cu && V <= parts * 4096u) parts >>= 1;
    for (; parts > 1u; parts >>= 1) {
        const uint64_t n = (uint64_t)B * parts, busy = n * 320u / n_cu;
        if (parts * (B > n_cu ? (busy < 3072u ? 3072u : busy > 12288u ? 12288u : (uint32_t)busy) : n > n_cu ? 2560u : kPartGroup / 2u) <= V) break;
    }
    return parts;
}

static uint32_t rows_lds(const DeviceVocab &Vc, uint32_t parts)
{
    const uint32_t span = kParts / parts;
    uint32_t most = 0;
    for (uint32_t p = 0; p < kParts; p += span) {
        const uint32_t n = ((range_token(Vc.V, p + span) + 31u) >> 5) - (range_token(Vc.V, p) >> 5);
        most = n > most ? n : most;
    }
    return 2u * (((most + 3u) & ~3u) + 4u) * 4u;
}
// (the most for any batch: a row in fewer parts than kLeastParts is short)
uint32_t rows_lds_bytes(const DeviceVocab &Vc) { return rows_lds(Vc, row_parts(Vc.V, kMaxBatch, 1u)); }

// Workgroups of the rows kernel that a unit holds: 8 by their registers, as many by its 160 KB of LDS.
static uint32_t resident_rows(const DeviceVocab &Vc, uint32_t parts)
{
    const uint32_t fit = 160u * 1024u / (rows_lds(Vc, parts) + (uint32_t)sizeof(RowShared));
    return fit < 8u ? fit : 8u;
}

FillPlan plan_fill(const DeviceVocab &Vc, const DeviceCache &Cc, uint32_t B, bool masks_logits, int dtype, uint32_t n_cu)
{
    FillPlan p;
    p.lines = masks_logits && by_lines(dtype, B, Vc.V);
    p.parts = row_parts(Vc.V, B, n_cu);
    // One kernel while its workgroups are resident together: what every workgroup of a row repeats of the lookup
    // is then paid once, and a launch with its lookup is saved.  us a call with two kernels / with one, outlines, mixed, random
    // trees, wg_fill_masks copied and made, then wg_decode_step: V = 151936, B = 16 4.7 4.9 4.9 / 4.3 4.3 4.3, 9.9 10.8 13.6 / 7.9 8.5
    // 10.7, 6.0 6.1 6.1 / 5.2 5.1 5.1, 11.4 12.4 15.0 / 9.2 10.1 12.3; B = 256 6.9 6.9 6.8 / 6.6 6.7 6.7, 17.9 17.8 37.9 / 13.8 14.1 35.0, 17.1
    // 18.3 20.7 / 14.7 16.1 18.1, 27.2 27.6 45.5 / 21.8 22.0 41.7; V = 65536, B = 256 9.7 10.4 11.9 / 8.5 8.8 10.6 and 18.3 19.6 32.3 /
    // 14.3 15.4 29.3 a step.  Above, workgroups that start late repeat it when the others are done: copied rows, masks alone,
    // V = 151936, B = 288 7.1 / 7.8, V = 65536, B = 512 7.5 / 9.2, while made ones and steps
    // gain, up to a fifth.  So it is with
    // fewer rows whose shares take so much LDS that fewer workgroups are resident, from V = 350,000 on (masks only, outlines /
    // mixed / random trees, one over two kernels, made and copied: V = 340001, B = 256, 8 to a unit, 0.80 0.85 0.95 and 0.93
    // 0.94 0.97; 350000, B = 256, 7 to a unit, 0.88 1.00 1.00 and 1.04 1.06 1.10; 500000, B = 224, 6 to a unit, 0.94 0.99 0.98
    // and 1.03 1.01 1.09).  With logits to mask behind them the workgroups
    // that are late find memory less busy, and one kernel gains up to where lines begin (V = 400000, B = 256 copied 0.94 0.97
    // 0.97, made 0.89 0.93 0.96); whole lines are masked behind a lookup of its own.
    //
    // Above a request per unit one kernel gains where all of its workgroups are resident with a few places left (rows are in four shares or
    // fewer there), and where rows are so long, and so many, that masking them outlasts what late workgroups repeat.  Time with one kernel over two,
    // outlines, JSON, mixed, random trees, cached and then made, bf16, a step of a decode loop (profiles/dispatch_rules.txt: single steps without a sampled token): V = 9000 B = 264 0.69 0.72 0.71 0.75, 0.84 0.79 0.74 0.81, 700 0.78 0.81
    // 0.81 0.79, 0.97 0.87 0.79 0.87; 14000 350 0.81 0.81 0.82 0.77, 0.82 0.75 0.73 0.86, 440 0.82 0.82 0.82 0.80, 0.88 0.80 0.73 0.87; 101000 560 0.99 0.99
    // 0.96 0.94, 0.94 0.98 0.94 0.99; 128256 512 0.95 0.95 0.93 0.94, 0.92 0.90 0.91 0.95, 800 0.95 0.96 0.96 0.97, 0.90 0.86 0.91 0.96; 151936 640 0.95 0.95 0.96
    // 0.97, 0.90 0.88 0.92 0.96; fp32, 101000 650 0.94 0.95 0.96 0.97, 0.91 0.87 0.92 0.97.  Masks alone, with the two calls behind them: 12000 272 0.67
    // 0.64 0.67 0.68, 0.88 0.83 0.82 0.86, 512 0.74 0.76 0.75 0.76, 0.91 0.87 0.83 0.87; long rows only gain where they are made (65536 272 1.02 1.02 1.02
    // 1.02, 0.98 1.03 0.94 0.94).  On the other sides of the lines, steps: 9000 880 (more than 7 workgroups to a unit) made outlines 1.08; 14000 500 1.03;
    // 65536 384 made outlines and JSON 1.05; 80000 500 cached outlines 1.06, made JSON 1.09; 96000 350 made JSON 1.02, 101000 300 1.14; whole lines, 151936 1000 0.93 to
    // 0.98, but made random trees 1.02.  Masks alone that are not resident together: 14000 600 copied 1.12 to 1.14, 16384 768 1.19 to 1.20.
    // The lower line of V is not where the gain ends: rows of 16,385 to 24,575 tokens are resident together up to the same batches and gain as much (steps, 20011 350 0.89 0.89
    // 0.87 0.82, 0.74 0.74 0.77 0.86, 24000 448 0.87 0.87 0.85 0.86, 0.77 0.79 0.80 0.94; masks alone 0.93 to 0.96, 0.71 to 0.91).  They have been two kernels, each
    // timed by itself (wg_profile_read), and still are.
    const bool together = B * p.parts <= resident_rows(Vc, p.parts) * n_cu, few = B <= n_cu, short_rows = B <= 3u * n_cu && Vc.V <= 16384u,
               long_rows = 2u * B >= 3u * n_cu && Vc.V >= 100000u;
    p.one_kernel = Cc.direct && B <= kOneKernelRows &&
                   (masks_logits ? !p.lines && (few || (short_rows && B * p.parts <= 7u * n_cu) || long_rows) : (few || short_rows) && together);
    return p;
}

#define WG_EARLY_VALUES states, tokens, Cc.ctr, T.states, Vc.chunks, Vc.len8, T.n_states, Vc.V

hipError_t launch_fill(const FillPlan &plan, const DeviceTable &T, const DeviceVocab &Vc, const DeviceCache &Cc,
                       wg_state_t *states, const int32_t *tokens, uint32_t B, uint32_t *bitmask,
                       void *logits, int dtype, int64_t logits_stride,
                       hipStream_t s, hipEvent_t *lookup_ev, hipEvent_t *rows_ev)
{
    const dim3 g(plan.parts, B);
    const uint32_t lds = rows_lds(Vc, plan.parts);
    const bool whole = plan.one_kernel;
    const LateArgs late{T, Vc, Cc, bitmask, logits, logits_stride, kParts / plan.parts, plan.parts, B};
    if (!whole) {
        const hipError_t e = launch(lookup_kernel, dim3(cdiv(B, kLookupWaves)), dim3(64 * kLookupWaves), 0, s, lookup_ev, WG_EARLY_VALUES, late);
        if (e != hipSuccess) return e;
    }
    auto rows = [&](auto kernel) { return launch(kernel, g, dim3(kRowThreads), lds, s, rows_ev, WG_EARLY_VALUES, late); };
    auto of_type = [&](auto elem) {
        using E = decltype(elem);
        if (plan.lines) return rows(rows_kernel<E, 2, false>);
        if (masks_through(logits, dtype, B, Vc.V)) return whole ? rows(rows_kernel<E, 3, true>) : rows(rows_kernel<E, 3, false>);
        return whole ? rows(rows_kernel<E, 1, true>) : rows(rows_kernel<E, 1, false>);
    };
    if (!logits) return whole ? rows(rows_kernel<uint16_t, 0, true>) : rows(rows_kernel<uint16_t, 0, false>);
    return dtype == WG_F32 ? of_type(uint32_t{}) : of_type(uint16_t{});
}

// New states and classes from pinned host memory to the ends of the device tables, all slices by one
// launch (the copies of two to four slices from pageable memory took 25 us to enqueue and wait for).  A
// slice lies in the staging memory as it does in the device's, modulo 16 bytes.
__global__ void __launch_bounds__(256) append_kernel(AppendSlices a)
{
    const AppendSlice s = a.slice[blockIdx.y];
    const uint32_t skew = (uint32_t)(reinterpret_cast<uintptr_t>(s.dst) & 15u), blocks = (skew + s.bytes + 15u) / 16u;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < blocks; q += gridDim.x * 256u) {
        const uint32_t lo = q ? q * 16u - skew : 0u, hi = q * 16u + 16u - skew < s.bytes ? q * 16u + 16u - skew : s.bytes;
        if (hi - lo == 16u) *reinterpret_cast<uint4 *>(s.dst + lo) = *reinterpret_cast<const uint4 *>(s.src + lo);
        else for (uint32_t i = lo; i < hi; i++) s.dst[i] = s.src[i];
    }
}

hipError_t launch_append(const AppendSlices &a, uint32_t n, hipStream_t s)
{
    uint32_t most = 0;
    for (uint32_t i = 0; i < n; i++) most = a.slice[i].bytes > most ? a.slice[i].bytes : most;
    const uint32_t blocks = cdiv(most / 16u + 2u, 256u);
    return launch(append_kernel, dim3(blocks < 256u ? blocks : 256u, n), dim3(256), 0, s, nullptr, a);
}

hipError_t launch_count_rows(const DeviceCache &Cc, hipStream_t s)
{
    const uint32_t blocks = cdiv(Cc.n_keys, 256u);
    return launch(count_rows_kernel, dim3(blocks < 256u ? blocks : 256u), dim3(256), 0, s, nullptr, Cc);
}

hipError_t launch_free_rows(const DeviceCache &Cc, uint32_t n_keys, uint32_t *free_rows, hipStream_t s)
{
    return launch(free_rows_kernel, dim3(1), dim3(1024), 0, s, nullptr, Cc, n_keys, free_rows);
}

hipError_t launch_apply(void *logits, int dtype, uint32_t B, uint32_t V, int64_t row_stride,
                        const uint32_t *bitmask, hipStream_t s, hipEvent_t *ev)
{
    const uint32_t W = (V + 31u) / 32u;
    if (by_lines(dtype, B, V)) {
        const dim3 g(cdiv(V, kLineTokens), B);
        if (dtype == WG_F32) return launch(apply_lines_kernel<uint32_t>, g, dim3(256), 0, s, ev, static_cast<uint32_t *>(logits), row_stride, V, W, bitmask);
        return launch(apply_lines_kernel<uint16_t>, g, dim3(256), 0, s, ev, static_cast<uint16_t *>(logits), row_stride, V, W, bitmask);
    }
    // (a row that begins inside a line has up to 63 tokens more to its chunks)
    const uint32_t e = dtype == WG_F32 ? 4u : 2u;
    const bool at_lines = reinterpret_cast<uintptr_t>(logits) % 128u == 0u && (B == 1u || (uint64_t)row_stride * e % 128u == 0u);
    auto apply = [&](auto kernel, auto *x, uint32_t tokens) {
        return launch(kernel, dim3(cdiv((uint64_t)V + (at_lines ? 0u : 63u), tokens), B), dim3(256), 0, s, ev, x, row_stride, V, W, bitmask);
    };
    const bool through = masks_through(logits, dtype, B, V);
    constexpr uint32_t kMany = 4u * 64u * 32u, kFewer = 4u * 64u * 24u;
    if (dtype == WG_F32) {
        uint32_t *x = static_cast<uint32_t *>(logits);
        return through ? apply(apply_kernel<uint32_t, 32u, true>, x, kMany) : apply(apply_kernel<uint32_t, 32u, false>, x, kMany);
    }
    uint16_t *x = static_cast<uint16_t *>(logits);
    if (through) return apply(apply_kernel<uint16_t, 32u, true>, x, kMany);
    return (uint64_t)B * V * 2u > kApplyLarge ? apply(apply_kernel<uint16_t, 24u, false>, x, kFewer) : apply(apply_kernel<uint16_t, 32u, false>, x, kMany);
}

hipError_t launch_advance(const DeviceTable &T, const DeviceVocab &Vc, const DeviceCache &Cc,
                          wg_state_t *states, const int32_t *tokens, uint32_t B, uint32_t n_cu, hipStream_t s,
                          hipEvent_t *ev)
{
    const uint32_t waves = B <= 2u * n_cu ? 1u : 4u, blocks = cdiv(B, waves);
    return launch(waves == 1u ? advance_kernel<1> : advance_kernel<4>, dim3(blocks < kAdvanceBlocks ? blocks : kAdvanceBlocks), dim3(64u * waves), 0, s, ev, WG_EARLY_VALUES,
                  LateArgs{T, Vc, Cc, nullptr, nullptr, 0, 0u, 1u, B});
}

// A wavefront per request up to 32 requests to a unit, which are resident together.  A wavefront / a thread each, us, outlines, JSON, mixed,
// random trees: B = 4,096 2.8 2.8 2.9 3.4 / 2.9 2.7 3.3 7.0; 8,192 3.3 3.3 3.4 4.1 / 2.9 2.7 3.3 7.1; 16,384 4.2 4.2 4.6 5.3 / 3.1 2.7 3.3 5.8; 60,000 9.4 9.3
// 10.9 12.9 / 3.1 2.9 3.6 6.4.
hipError_t launch_forced_bytes(const DeviceTable &T, const wg_state_t *states, uint32_t B, uint32_t cap,
                               uint8_t *bytes, uint32_t *lens, wg_state_t *end_states, uint32_t n_cu, hipStream_t s)
{
    auto run = [&](auto kernel, uint32_t requests, uint32_t threads) {
        const uint32_t blocks = cdiv(B, requests);
        return launch(kernel, dim3(blocks < kAdvanceBlocks ? blocks : kAdvanceBlocks), dim3(threads), 0, s, nullptr, states, T.states, T.lit, bytes, lens, end_states, T.n_states, cap, B);
    };
    if (B > 32u * n_cu) return run(forced_bytes_of_many_kernel, 64u, 64u);
    return B <= 2u * n_cu ? run(forced_bytes_kernel, 1u, 64u) : run(forced_bytes_kernel, 4u, 256u);
}

hipError_t launch_select(const uint32_t *bitmask, uint32_t B, uint32_t V, const uint64_t *draws,
                         int32_t *tokens, hipStream_t s)
{
    return launch(select_kernel, dim3(B), dim3(256), 0, s, nullptr, bitmask, (V + 31u) / 32u, draws, tokens);
}

}  // namespace wg
