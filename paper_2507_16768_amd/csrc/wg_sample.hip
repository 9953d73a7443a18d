// Sampling under the mask for gfx950 (wave64): the greedy choice and the k best allowed tokens of every
// row, logits read once and never written.
//
// A workgroup of 1,024 threads takes a row.  The row's mask goes to LDS; every thread then keeps the
// largest allowed logit of its 16-byte pieces and where it was.  From 256 rows on that is HBM bound,
// and nothing has to be merged.  Smaller batches cut their rows: the greedy choice into as
// many workgroups as there are compute units, merged in pairs; the k best of
// long rows into slices of 8,192 tokens, merged by a second kernel.  The greedy choice from long fp32 rows is
// made from such slices too (argmax_slice_kernel): a row of 600 KB per workgroup left compute units
// idle whenever the rows did not come out even.
//
// The loads of logits and mask go through buffer descriptors: what is not wanted lies behind the buffer's end and costs no
// branch, and the loads count by themselves.  (As flat loads behind a branch for rows at odd addresses each was waited for before
// the next was issued, and the mask came in five trips, one after the other.)  Times of the greedy choice and of k = 50, us, so / now, bf16, every
// token allowed: V = 128,256 B = 64 8.7 16.5 / 7.6 13.3; 151,936 B = 128 11.6 19.8 / 10.4 15.5, B = 256 18.5 26.1 / 15.9 (5.0 TB/s,
// near a copy's rate) 19.8, B = 1,000 61.9 86.1 / 53.7 59.6; under the masks of 256 requests, half outlines and half JSON, 16.3 21.5 / 13.6 17.2.
//
// The k best need no sorting of the row: in each of n wavefronts the ceil(k / n)-th largest of the 64
// thread maxima is found by bisection on ballots, and the least of these is a lower bound for the k-th
// best token.  Two to three times k tokens reach it; they are ranked by counting.
//
// Rows may start at any byte.  Where elements lie at multiples of their size, pieces are aligned 16-byte blocks, the first of them may begin
// before the row and the last may end behind it, and the staged mask has those tokens as disallowed.
#include <hip/hip_runtime.h>

#include <mutex>

#include "wg_buffer.h"
#include "wg_device.h"
#include "wg_launch.h"
#include "wg_order.h"

namespace wg {

constexpr uint32_t kThreads = 1024;
constexpr uint32_t kWaves = kThreads / 64u;
constexpr uint32_t kSegWords = 8192;                 // mask words staged at a time (32 KB: 262,144 tokens)
constexpr uint32_t kCand = 1024;                     // candidates ranked in LDS
constexpr uint32_t kNoPiece = 0xFFFFFFFFu;

// One row of logits as 16-byte pieces.  kWhole: elements lie at multiples of their size, and pieces are aligned.  Else pieces are
// cut at the row's beginning, each out of the five aligned words that it lies in.  (Element by element, behind branches, a piece was up
// to eight trips to memory one after the other; a kernel for both spent 1 % of the whole rows' time on the choice.)  us at an odd byte,
// mixed masks, so / now, the greedy choice and k = 50: bf16, V = 151,936, B = 40 15.2 41.0 / 7.4 15.3, 256 39.7 56.4 / 12.3 16.5; fp32, V =
// 128,256, B = 64 12.6 34.9 / 8.1 18.4.
template <typename Elem, bool kWhole>
struct Row {
    static constexpr uint32_t kPer = 16u / sizeof(Elem);          // tokens of a piece: 8 bf16, 4 fp32
    static constexpr uint32_t kAll = (1u << kPer) - 1u;
    const Elem *tokens;
    const char *first;                               // the aligned block, or word, that the row's first byte lies in
    uint32_t skew, pieces, V;                        // piece p holds the tokens p * kPer - skew ...
    uint32_t odd;                                    // not whole: bytes of the first word in front of the row

    __device__ __forceinline__ Row(const Elem *row, uint32_t V_) : tokens(row), V(V_)
    {
        const uintptr_t at = reinterpret_cast<uintptr_t>(row);
        odd = (uint32_t)(at % 4u);
        skew = kWhole ? (uint32_t)(at % 16u / sizeof(Elem)) : 0u;
        first = reinterpret_cast<const char *>(row) - (kWhole ? at % 16u : at % 4u);
        pieces = (V + skew + kPer - 1u) / kPer;
    }
    // n pieces from p on.  An aligned block, or word, that holds a byte of the row lies in the row's own memory page, also
    // where it begins before the row or ends behind it.
    __device__ __forceinline__ Window window(uint32_t p, uint32_t n) const
    {
        if (kWhole) return window_of(first + (size_t)p * 16u, n * 16u);
        const uint64_t left = ((odd + (uint64_t)V * sizeof(Elem) + 3u) & ~3ull) - (uint64_t)p * 16u, most = n * 16u + 4u;
        return window_of(first + (size_t)p * 16u, (uint32_t)(left < most ? left : most));
    }
    // The piece at an offset of a window (kNowhere: one without anything to look at).
    __device__ __forceinline__ uint4 piece(const Window &win, uint32_t at) const
    {
        if (kWhole) return block_at(win, at);
        uint32_t w[5];
#pragma unroll
        for (uint32_t k = 0; k < 5u; k++) w[k] = word_at(win, at + 4u * k);
        return uint4{__builtin_amdgcn_alignbyte(w[1], w[0], odd), __builtin_amdgcn_alignbyte(w[2], w[1], odd),
                     __builtin_amdgcn_alignbyte(w[3], w[2], odd), __builtin_amdgcn_alignbyte(w[4], w[3], odd)};
    }
    __device__ __forceinline__ uint32_t token(uint32_t p, uint32_t i) const { return p * kPer + i - skew; }
};

// Word i of the row's mask moved up by the skew: bit s of the result is the token s - skew.
__device__ __forceinline__ uint32_t mask_word(const uint32_t *mask, uint32_t W, uint32_t V, uint32_t skew, uint32_t i)
{
    auto word = [&](uint32_t w) {
        uint32_t x = w < W ? mask[w] : 0u;
        if (w == W - 1u && (V & 31u)) x &= (1u << (V & 31u)) - 1u;
        return x;
    };
    const uint32_t hi = word(i);
    return skew ? (hi << skew) | ((i ? word(i - 1u) : 0u) >> (32u - skew)) : hi;
}

// The words [w0, w0 + nw) of the same, nw up to kSegWords, to LDS, and a zero behind them; all of a thread's in flight together.
// The whole workgroup calls it.
__device__ __forceinline__ void stage_mask(const uint32_t *mask, uint32_t W, uint32_t V, uint32_t skew, uint32_t w0, uint32_t nw, uint32_t *words)
{
    constexpr uint32_t kMost = kSegWords / kThreads;
    const Window win = window_of(mask + w0, (W > w0 ? W - w0 < nw ? W - w0 : nw : 0u) * 4u);
    const uint32_t tid = threadIdx.x, last = W - 1u - w0, tail = V & 31u ? (1u << (V & 31u)) - 1u : 0xFFFFFFFFu;
    uint32_t x[kMost], y[kMost];
#pragma unroll
    for (uint32_t j = 0; j < kMost; j++) {
        x[j] = 0u; y[j] = 0u;
        if (j * kThreads >= nw) continue;
        x[j] = word_at(win, (tid + j * kThreads) * 4u);
        if (skew) y[j] = tid + j * kThreads ? word_at(win, (tid + j * kThreads - 1u) * 4u) : w0 ? mask[w0 - 1u] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < kMost; j++) {
        const uint32_t i = tid + j * kThreads;
        if (j * kThreads >= nw) break;
        if (i == last) x[j] &= tail;
        if (skew) x[j] = x[j] << skew | (i == last + 1u ? y[j] & tail : y[j]) >> (32u - skew);
        if (i < nw) words[i] = x[j];
    }
    if (tid == 0) words[nw] = 0u;
}

// The allowed tokens of piece p, from the mask as it lies in memory.
template <typename Elem, bool kWhole>
__device__ __forceinline__ uint32_t piece_mask(const Row<Elem, kWhole> &r, const uint32_t *mask, uint32_t W, uint32_t p)
{
    const uint32_t bit = p * r.kPer;
    return (mask_word(mask, W, r.V, r.skew, bit >> 5) >> (bit & 31u)) & r.kAll;
}

// The largest allowed number of a piece (NaN when there is none): a disallowed token's bits are
// forced to all ones, which is a NaN in both formats, and the hardware maximum ignores NaNs, so
// NaN logits drop out the same way.
__device__ __forceinline__ float piece_max(const uint4 &v, uint32_t m, uint16_t)
{
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    const uint32_t nm = ~m;
    float a = __builtin_nanf(""), b = a;
#pragma unroll
    for (int k = 0; k < 4; k++) {                     // dword k holds tokens 2k (low half) and 2k+1
        const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe(nm, 2 * k, 1), hi = (uint32_t)__builtin_amdgcn_sbfe(nm, 2 * k + 1, 1);
        const uint32_t x = d[k] | (lo & 0xFFFFu) | (hi << 16);
        a = __builtin_fmaxf(a, __uint_as_float(x << 16));
        b = __builtin_fmaxf(b, __uint_as_float(x & 0xFFFF0000u));
    }
    return __builtin_fmaxf(a, b);
}
__device__ __forceinline__ float piece_max(const uint4 &v, uint32_t m, uint32_t)
{
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    const uint32_t nm = ~m;
    float a = __builtin_nanf("");
#pragma unroll
    for (int k = 0; k < 4; k++) a = __builtin_fmaxf(a, __uint_as_float(d[k] | (uint32_t)__builtin_amdgcn_sbfe(nm, k, 1)));
    return a;
}

// Streams the pieces [lo, hi) of the row, lo a multiple of 32: what(p, piece, allowed tokens) for every
// piece of the thread that has an allowed token, in ascending order.  `words` is kSegWords + 1
// words of LDS.  The whole workgroup calls it.
template <typename Elem, bool kWhole, typename F>
__device__ __forceinline__ void stream_row(const Row<Elem, kWhole> &r, const uint32_t *mask, uint32_t W, uint32_t *words,
                                           uint32_t lo, uint32_t hi, F what)
{
    constexpr uint32_t kPer = Row<Elem, kWhole>::kPer, kSegPieces = kSegWords * 32u / kPer;
    const uint32_t tid = threadIdx.x;
    for (uint32_t s0 = lo; s0 < hi; s0 += kSegPieces) {
        const uint32_t n = hi - s0 < kSegPieces ? hi - s0 : kSegPieces;
        const uint32_t w0 = s0 / (32u / kPer), nw = (n * kPer + 31u) / 32u;
        if (s0 != lo) __syncthreads();                     // the segment before is done with the LDS
        stage_mask(mask, W, r.V, r.skew, w0, nw, words);
        __syncthreads();
        const uint32_t none = nw * (32u / kPer);           // a piece of the zero behind the words
        auto allowed = [&](uint32_t q) {
            if (q > none) q = none;
            if (kPer == 8u) return (uint32_t)reinterpret_cast<const uint8_t *>(words)[q];
            return words[q / (32u / kPer)] >> (q * kPer & 31u) & r.kAll;
        };
        // Up to three pieces of a thread are one round: the loop below takes two more for nothing (the greedy choice, mixed, us, before there was
        // the loop / with it alone / so: V = 8,000, B = 1 3.9 / 4.3 / 3.7, 256 4.5 / 5.1 / 4.3; a row of 151,936 tokens in eight shares 5.6 / 6.3 / 5.8).
        constexpr uint32_t kRound = 3u;
        if (n <= kThreads * kRound) {
            const Window win = r.window(s0, n);
            uint32_t mm[kRound];
            uint4 vv[kRound];
#pragma unroll
            for (uint32_t j = 0; j < kRound; j++) mm[j] = allowed(tid + j * kThreads);
#pragma unroll
            for (uint32_t j = 0; j < kRound; j++) vv[j] = r.piece(win, mm[j] ? (tid + j * kThreads) * 16u : kNowhere);
#pragma unroll
            for (uint32_t j = 0; j < kRound; j++) if (mm[j]) what(s0 + tid + j * kThreads, vv[j], mm[j]);
            continue;
        }
        constexpr uint32_t kHalf = kWhole ? 3u : 2u;       // (of five words each, three are 3 % slower)
        const Window win = r.window(s0, n);
        uint32_t m[2][kHalf];
        uint4 v[2][kHalf];
        auto request = [&](uint32_t (&mm)[kHalf], uint4 (&vv)[kHalf], uint32_t q0) {
#pragma unroll
            for (uint32_t j = 0; j < kHalf; j++) mm[j] = allowed(q0 + j * kThreads);
#pragma unroll
            for (uint32_t j = 0; j < kHalf; j++) vv[j] = r.piece(win, mm[j] ? (q0 + j * kThreads) * 16u : kNowhere);
        };
        auto look = [&](const uint32_t (&mm)[kHalf], const uint4 (&vv)[kHalf], uint32_t q0) {
#pragma unroll
            for (uint32_t j = 0; j < kHalf; j++)
                if (mm[j]) what(s0 + q0 + j * kThreads, vv[j], mm[j]);
        };
        request(m[0], v[0], tid);
#pragma nounroll
        for (uint32_t q0 = tid; q0 < n; q0 += kThreads * kHalf * 2u) {
            request(m[1], v[1], q0 + kThreads * kHalf);
            look(m[0], v[0], q0);
            request(m[0], v[0], q0 + kThreads * kHalf * 2u);
            look(m[1], v[1], q0 + kThreads * kHalf);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// masked argmax.  The workgroups of a row that is cut into 2^n are merged in pairs, by keys (the order key of a logit
// << 32 | ~id): each swaps its key into its pair's node; the first to come finds zero there and is done, the
// second finds the other's key, leaves zero for the next call and goes on with the larger one.  (Rows in slices,
// below, raise one key per row, which a second kernel takes.)  One copy per GPU: calls that cut their rows must not overlap on one GPU.
constexpr uint32_t kCutRows = 256;                   // most workgroups of a call that cuts its rows
__device__ unsigned long long g_argmax_key[kMaxBatch];
__device__ unsigned long long g_argmax_node[kCutRows];

template <typename Elem, bool kWhole>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8)))
masked_argmax_kernel(const Elem *__restrict__ logits, int64_t row_stride, uint32_t V, uint32_t W,
                     const uint32_t *__restrict__ bitmask, int32_t *__restrict__ tokens)
{
    __shared__ uint32_t words[kSegWords + 1u];
    __shared__ float part[kWaves];
    __shared__ uint32_t best_token;
    const uint32_t b = blockIdx.y, tid = threadIdx.x;
    const uint32_t *mask = bitmask + (size_t)b * W;
    const Row<Elem, kWhole> r(logits + (int64_t)b * row_stride, V);
    const uint32_t share = ((r.pieces + gridDim.x - 1u) / gridDim.x + 31u) & ~31u;
    const uint32_t lo = blockIdx.x * share < r.pieces ? blockIdx.x * share : r.pieces;
    const uint32_t hi = r.pieces - lo < share ? r.pieces : lo + share;
    float best = __builtin_nanf("");
    // the thread's first piece with `best`, and its elements (looked up again at the end they were a trip to memory: V =
    // 151936, bf16, B = 256 19.6 -> 18.8 us, B = 128 12.4 -> 11.9, B = 1 5.6 -> 5.5)
    uint32_t where = kNoPiece;
    union { uint4 v; Elem e[16u / sizeof(Elem)]; } held;
    held.v = uint4{0u, 0u, 0u, 0u};
    uint32_t held_mask = 0;
    auto see = [&](uint32_t p, const uint4 &v, uint32_t m) {
        const float x = __builtin_fmaxf(best, piece_max(v, m, Elem(0)));
        if (!(x == best)) { best = x; where = p; held.v = v; held_mask = m; }      // (also while there is no number)
    };
    stream_row(r, mask, W, words, lo, hi, see);
    float top = best;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = __builtin_fmaxf(top, __shfl_xor(top, o));
    if ((tid & 63u) == 0u) part[tid >> 6] = top;
    if (tid == 0) best_token = 0xFFFFFFFFu;
    __syncthreads();
    top = part[0];
#pragma unroll
    for (uint32_t w = 1; w < kWaves; w++) top = __builtin_fmaxf(top, part[w]);
    const bool number = top == top;
    if (number) {
        // The lowest token whose logit equals the maximum (as numbers, so -0.0 and +0.0 tie), from the
        // threads that hold it, in the first such piece of each.
        if (where != kNoPiece && best == top) {
            uint32_t eq = 0;
#pragma unroll
            for (uint32_t i = 0; i < r.kPer; i++) eq |= (uint32_t)(elem_float(held.e[i]) == top) << i;
            atomicMin(&best_token, r.token(where, (uint32_t)__builtin_ctz(eq & held_mask)));
        }
    } else {
        // no number among the allowed tokens: the lowest of them (all NaN), if there is one
        for (uint32_t p = lo + tid; where != kNoPiece && p < hi; p += kThreads) {
            const uint32_t m = piece_mask(r, mask, W, p);
            if (m) { atomicMin(&best_token, r.token(p, (uint32_t)__builtin_ctz(m))); break; }
        }
    }
    __syncthreads();
    if (tid) return;
    uint32_t token = best_token;                      // all ones is -1: nothing allowed
    if (gridDim.x > 1u) {
        unsigned long long key = token == 0xFFFFFFFFu ? 0ull :
            (unsigned long long)(number ? order_key(__float_as_uint(top)) : 0u) << 32 | (0xFFFFFFFFu - token);
        key += key == 0ull;                           // (0: nobody has been here)
        unsigned long long *node = g_argmax_node + (size_t)b * (gridDim.x - 1u);
        for (uint32_t n = gridDim.x >> 1, i = blockIdx.x >> 1; n; node += n, n >>= 1, i >>= 1) {
            const unsigned long long other = atomicExch(&node[i], key);
            if (!other) return;                       // the pair's other one goes on
            __hip_atomic_store(&node[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            key = other > key ? other : key;
        }
        token = key == 1ull ? 0xFFFFFFFFu : 0xFFFFFFFFu - (uint32_t)key;
    }
    tokens[b] = (int32_t)token;
}

// fp32 rows of larger batches: a workgroup of 256 threads takes 8,192 tokens, all of its loads in flight
// together, raises the row's key and is done; a second kernel turns the keys into tokens.  Bound by HBM.
// Against a workgroup of 1,024 threads per row (two of which fit a compute unit, so that every count of
// rows but a multiple of 512 leaves units without work) it costs a launch and evens out rows of any number
// and of any number of allowed tokens.  V = 151,936, everything allowed / a few tokens in every other row, by row
// -> in slices, us: B = 40 8.7 -> 8.9 / 8.3 -> 6.7, B = 64 10.4 -> 11.0 / 10.0 -> 7.8, B = 128 15.9 -> 16.6 / 12.0 -> 10.7, B = 256
// 29.9 -> 31.2 / 20.2 -> 17.0; a ticket in place of the second kernel kept each workgroup for two more trips to memory
// (B = 1,024 110 -> 167).  bf16 rows are not taken so (B = 256 20.1 -> 25.1, B = 1,024 63 -> 74 when by row was slower than now).
constexpr uint32_t kChoiceThreads = 256, kChoicePieces = 8;
constexpr uint32_t kChoiceTokens = kChoiceThreads * kChoicePieces * Row<uint32_t, true>::kPer;
__global__ void __launch_bounds__(kChoiceThreads)
argmax_slice_kernel(const uint32_t *__restrict__ logits, int64_t row_stride, uint32_t V, uint32_t W,
                    const uint32_t *__restrict__ bitmask)
{
    constexpr uint32_t kPer = Row<uint32_t, true>::kPer, kWords = kChoiceTokens / 32u;
    __shared__ uint32_t words[kWords];
    __shared__ float part[kChoiceThreads / 64u];
    __shared__ uint32_t best_token;
    const uint32_t b = blockIdx.y, tid = threadIdx.x, base = blockIdx.x * (kChoicePieces * kChoiceThreads) + tid;
    const Row<uint32_t, true> r(logits + (int64_t)b * row_stride, V);
    static_assert(kWords == kChoiceThreads, "a mask word per thread");
    words[tid] = mask_word(bitmask + (size_t)b * W, W, V, r.skew, blockIdx.x * kWords + tid);
    if (tid == 0) best_token = 0xFFFFFFFFu;
    __syncthreads();
    const Window win = r.window(blockIdx.x * (kChoicePieces * kChoiceThreads), kChoicePieces * kChoiceThreads);
    uint32_t m[kChoicePieces];
    union { uint4 v; uint32_t e[kPer]; } u[kChoicePieces];
#pragma unroll
    for (uint32_t j = 0; j < kChoicePieces; j++) {
        const uint32_t bit = (j * kChoiceThreads + tid) * kPer;
        m[j] = (words[bit >> 5] >> (bit & 31u)) & Row<uint32_t, true>::kAll;
    }
#pragma unroll
    for (uint32_t j = 0; j < kChoicePieces; j++)               // (elements lie at multiples of their size: launch_masked_argmax)
        u[j].v = block_at(win, m[j] ? (j * kChoiceThreads + tid) * 16u : kNowhere);
    float best = __builtin_nanf("");
#pragma unroll
    for (uint32_t j = 0; j < kChoicePieces; j++) best = __builtin_fmaxf(best, piece_max(u[j].v, m[j], 0u));
    float top = best;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = __builtin_fmaxf(top, __shfl_xor(top, o));
    if ((tid & 63u) == 0u) part[tid >> 6] = top;
    __syncthreads();
    top = part[0];
#pragma unroll
    for (uint32_t w = 1; w < kChoiceThreads / 64u; w++) top = __builtin_fmaxf(top, part[w]);
    const bool number = top == top;
    if (!number || best == top) {
        // the thread's lowest token whose logit equals the maximum (as numbers, so -0.0 and +0.0 tie), or
        // where no allowed token has a number its lowest allowed one
        uint32_t token = 0xFFFFFFFFu;
#pragma unroll
        for (int j = (int)kChoicePieces - 1; j >= 0; j--) {
            uint32_t eq = 0;
#pragma unroll
            for (uint32_t i = 0; i < kPer; i++) eq |= (uint32_t)(__uint_as_float(u[j].e[i]) == top) << i;
            eq = number ? eq & m[j] : m[j];
            if (eq) token = r.token(base + (uint32_t)j * kChoiceThreads, (uint32_t)__builtin_ctz(eq));
        }
        if (token != 0xFFFFFFFFu) atomicMin(&best_token, token);
    }
    __syncthreads();
    if (tid == 0 && best_token != 0xFFFFFFFFu)
        atomicMax(&g_argmax_key[b], (unsigned long long)(number ? order_key(__float_as_uint(top)) : 0u) << 32 | (0xFFFFFFFFu - best_token));
}
// The choices of a batch from its rows' keys, which are left zero for the next call.
__global__ void __launch_bounds__(64)
argmax_finish_kernel(int32_t *__restrict__ tokens, uint32_t B)
{
    const uint32_t b = blockIdx.x * 64u + threadIdx.x;
    if (b >= B) return;
    const unsigned long long row = g_argmax_key[b];
    tokens[b] = row ? (int32_t)(0xFFFFFFFFu - (uint32_t)row) : -1;
    g_argmax_key[b] = 0ull;
}

// ---------------------------------------------------------------------------------------------
// masked top-k.  The rank of a token is its order key plus one (0: not allowed, 1: a NaN), then the
// lower id.
template <typename Elem>
__device__ __forceinline__ uint32_t rank_of(Elem e) { return order_key(__float_as_uint(elem_float(e))) + 1u; }

// The n-th largest of the wavefront's 64 values with its low 12 bits cleared (0 when fewer than n are
// above 0), by bisection: a ballot and a count per bit.
__device__ __forceinline__ uint32_t nth_of_wave(uint32_t v, uint32_t n)
{
    uint32_t bound = 0;
#pragma unroll
    for (uint32_t bit = 31u; bit >= 12u; bit--) {
        const uint32_t test = bound | 1u << bit;
        if ((uint32_t)__popcll(__ballot(v >= test)) >= n) bound = test;
    }
    return bound;
}

// A value that at least k of the workgroup's values reach (0 when there are none such): the least of
// the wavefronts' ceil(k / n)-th largest.  `least` is a word of LDS per wavefront.
template <uint32_t kN>
__device__ __forceinline__ uint32_t bound_of(uint32_t own, uint32_t k, uint32_t *least)
{
    const uint32_t mine = nth_of_wave(own, (k + kN - 1u) / kN);
    if ((threadIdx.x & 63u) == 0u) least[threadIdx.x >> 6] = mine;
    __syncthreads();
    uint32_t bound = least[0];
#pragma unroll
    for (uint32_t w = 1; w < kN; w++) bound = least[w] < bound ? least[w] : bound;
    return bound;
}

// The number from which on tokens reach a bound above 0 (ranks are order keys plus one).
__device__ __forceinline__ float bound_value(uint32_t bound)
{
    const uint32_t key = bound - 1u;
    uint32_t u = (key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key;
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) u = 0xFF800000u;       // below every number: from -inf on
    return __uint_as_float(u);
}
// Which of the allowed tokens of a piece reach the bound (all of them a bound of 0, NaNs too).
__device__ __forceinline__ uint32_t reaching(const uint4 &v, uint32_t m, uint32_t bound, float value, uint16_t)
{
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t take = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        take |= (uint32_t)(__uint_as_float(d[k] << 16) >= value) << (2 * k);
        take |= (uint32_t)(__uint_as_float(d[k] & 0xFFFF0000u) >= value) << (2 * k + 1);
    }
    return bound ? take & m : m;
}
__device__ __forceinline__ uint32_t reaching(const uint4 &v, uint32_t m, uint32_t bound, float value, uint32_t)
{
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t take = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) take |= (uint32_t)(__uint_as_float(d[k]) >= value) << k;
    return bound ? take & m : m;
}

// Element i of a piece, and the key of its token.
__device__ __forceinline__ uint32_t element(const uint4 &v, uint32_t i, uint32_t)
{
    // (values: a choice between members is one between their addresses, which puts the piece into memory)
    const uint32_t x = v.x, y = v.y, z = v.z, w = v.w, odd = 0u - (i & 1u), high = 0u - (i >> 1 & 1u);
    const uint32_t lo = (x & ~odd) | (y & odd), hi = (z & ~odd) | (w & odd);
    return (lo & ~high) | (hi & high);
}
__device__ __forceinline__ uint16_t element(const uint4 &v, uint32_t i, uint16_t)
{
    return (uint16_t)(element(v, i >> 1, 0u) >> (16u * (i & 1u)));
}
template <typename Elem, bool kWhole>
__device__ __forceinline__ unsigned long long key_of(const Row<Elem, kWhole> &r, const uint4 &v, uint32_t p, uint32_t i)
{
    return (unsigned long long)rank_of(element(v, i, Elem(0))) << 32 | (0xFFFFFFFFu - r.token(p, i));
}

// The keys of n candidate tokens, from their logits read again (which register of which thread holds a
// candidate's is not known at compile time; they are in the L2).
template <uint32_t kT, typename Elem, bool kWhole>
__device__ __forceinline__ void make_keys(unsigned long long *cand, const uint32_t *ids, uint32_t n, const Row<Elem, kWhole> &r)
{
    for (uint32_t i = threadIdx.x; i < n; i += kT) {
        const uint32_t id = ids[i];
        cand[i] = (unsigned long long)rank_of(r.tokens[id]) << 32 | (0xFFFFFFFFu - id);
    }
}

// Ranks n keys by counting, eight lanes to a key; calls emit(rank, key) for the best k.
template <uint32_t kT, typename F>
__device__ __forceinline__ void rank_keys(const unsigned long long *cand, uint32_t n, uint32_t k, F emit)
{
    const uint32_t sub = threadIdx.x & 7u;
    for (uint32_t i = threadIdx.x >> 3; i < n; i += kT / 8u) {
        const unsigned long long x = cand[i];
        uint32_t better = 0;
#pragma unroll 4
        for (uint32_t q = sub; q < n; q += 8u) better += cand[q] > x;
        better += __shfl_xor(better, 1); better += __shfl_xor(better, 2); better += __shfl_xor(better, 4);
        if (sub == 0u && better < k) emit(better, x);
    }
}

// The logit behind a key: its bits follow from the rank, except that a zero's sign and a NaN's payload
// are lost in it, so those are read again.
template <typename Elem>
__device__ __forceinline__ Elem logit_of(unsigned long long key, const Elem *row)
{
    const uint32_t order = (uint32_t)(key >> 32) - 1u;
    const uint32_t u = (order & 0x80000000u) ? order & 0x7FFFFFFFu : ~order;
    if (u == 0u || order == 0u) return row[0xFFFFFFFFu - (uint32_t)key];
    return (Elem)(sizeof(Elem) == 4 ? u : u >> 16);
}

struct TopkShared {
    uint32_t words[kSegWords + 1u];                  // the staged mask
    union {
        unsigned long long cand[kCand];              // the candidates: rank << 32 | ~id
        uint32_t bins[256];
    };
    uint32_t threads[kThreads];                      // threads that hold candidates
    uint32_t count[kWaves];
    uint32_t n, n_threads, digit, above;
};

template <typename Elem, bool kWhole>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8)))
masked_topk_kernel(const Elem *__restrict__ logits, int64_t row_stride, uint32_t V, uint32_t W,
                   const uint32_t *__restrict__ bitmask, uint32_t k, int32_t *__restrict__ ids,
                   Elem *__restrict__ values, Elem ninf)
{
    constexpr uint32_t kPer = Row<Elem, kWhole>::kPer;
    __shared__ TopkShared sh;
    const uint32_t b = blockIdx.x, tid = threadIdx.x;
    const uint32_t *mask = bitmask + (size_t)b * W;
    const Row<Elem, kWhole> r(logits + (int64_t)b * row_stride, V);
    int32_t *id_out = ids + (size_t)b * k;
    Elem *value_out = values + (size_t)b * k;
    // the thread's first piece with `best`, and the most of its other pieces
    float best = __builtin_nanf(""), second = best;
    uint32_t any = 0, where = 0, held_mask = 0;       // any: the thread has an allowed token
    uint4 held{0u, 0u, 0u, 0u};
    stream_row(r, mask, W, sh.words, 0u, r.pieces, [&](uint32_t p, const uint4 &v, uint32_t m) {
        const float x = piece_max(v, m, Elem(0)), most = __builtin_fmaxf(best, x);
        second = __builtin_fmaxf(second, most == best ? x : best);
        if (!(most == best)) { best = most; where = p; held = v; held_mask = m; }
        any = 1u;
    });
    const uint32_t own = best == best ? order_key(__float_as_uint(best)) + 1u : any;
    if (tid == 0) { sh.n = 0u; sh.n_threads = 0u; }
    const uint32_t bound = bound_of<kWaves>(own, k, sh.count);
    const float value = bound_value(bound);
    auto put = [&](const uint4 &v, uint32_t p, uint32_t m) {
        uint32_t take = reaching(v, m, bound, value, Elem(0));
        while (take) {
            const uint32_t i = (uint32_t)__builtin_ctz(take);
            take &= take - 1u;
            const uint32_t at = atomicAdd(&sh.n, 1u);
            if (at < kCand) sh.cand[at] = key_of(r, v, p, i);
        }
    };
    // Candidates: the allowed tokens at or above the bound.  Those of most threads lie in the one piece that the
    // thread holds; the pieces of the others are looked at again, by all threads (V = 151,936, bf16, k = 50, with those of all
    // threads looked at again / now: B = 256 20.0 / 17.2 us, B = 1,000 62.3 / 48.9).  Of up to four pieces of a thread so are all: two ways one
    // after the other are 4 % slower there (V = 20,011, B = 700 16.5 / 17.2).  The candidates fit their list unless hundreds
    // of tokens tie at the bound or are NaN.
    if (any && own >= bound) {
        if (bound == 0u || r.pieces <= 4u * kThreads || second >= value) sh.threads[atomicAdd(&sh.n_threads, 1u)] = tid;
        else put(held, where, held_mask);
    }
    __syncthreads();
    const uint32_t per = (r.pieces + kThreads - 1u) / kThreads, items = sh.n_threads * per;
    const bool staged = r.pieces * kPer <= kSegWords * 32u;        // the row's mask is in LDS as a whole
    constexpr uint32_t kItems = sizeof(Elem) == 4u ? 1u : 2u;      // in flight together, within 64 registers
    for (uint32_t i0 = tid; i0 < items; i0 += kThreads * kItems) {
        uint4 v[kItems];
        uint32_t m[kItems], p[kItems];
#pragma unroll
        for (uint32_t j = 0; j < kItems; j++) {
            const uint32_t i = i0 + j * kThreads, of = i / per;
            m[j] = 0u; p[j] = 0u;
            v[j] = uint4{0u, 0u, 0u, 0u};
            if (i < items) p[j] = sh.threads[of] + (i - of * per) * kThreads;
            if (i < items && p[j] < r.pieces) {
                const uint32_t bit = p[j] * kPer;
                m[j] = staged ? (sh.words[bit >> 5] >> (bit & 31u)) & r.kAll : piece_mask(r, mask, W, p[j]);
                if (kWhole && m[j]) v[j] = reinterpret_cast<const uint4 *>(r.first)[p[j]];
            }
            if (!kWhole) v[j] = r.piece(r.window(0u, r.pieces), m[j] ? p[j] * 16u : kNowhere);
        }
#pragma unroll
        for (uint32_t j = 0; j < kItems; j++) put(v[j], p[j], m[j]);
    }
    __syncthreads();
    uint32_t n = sh.n;
    if (n > kCand) {
        __syncthreads();                              // every thread has read the count
        // Too many tie.  The rank of the k-th best exactly, a byte at a time from the counts of the
        // tokens that agree in the bytes before; then the tokens above it, and of those at it the
        // lowest ids.
        uint32_t rank = 0, above = 0;                 // tokens above the bytes fixed so far
#pragma nounroll
        for (uint32_t shift = 32u; shift;) {
            shift -= 8u;
            for (uint32_t i = tid; i < 256u; i += kThreads) sh.bins[i] = 0u;
            __syncthreads();
            for (uint32_t t = tid; t < V; t += kThreads)
                if ((mask[t >> 5] >> (t & 31u)) & 1u) {
                    const uint32_t x = rank_of(r.tokens[t]);
                    if (shift == 24u || (x >> (shift + 8u)) == (rank >> (shift + 8u))) atomicAdd(&sh.bins[(x >> shift) & 255u], 1u);
                }
            __syncthreads();
            if (tid == 0) {
                uint32_t d = 255u, c = above;
                while (d && c + sh.bins[d] < k) c += sh.bins[d--];
                sh.digit = d; sh.above = c;
            }
            __syncthreads();
            rank |= sh.digit << shift; above = sh.above;
            __syncthreads();
        }
        // the tokens above it leave their keys at the list's front, the ties behind them in order of id
        if (tid == 0) { sh.n = 0u; sh.digit = above; }
        __syncthreads();
        for (uint32_t t0 = 0; t0 < V; t0 += kThreads) {
            const uint32_t t = t0 + tid;
            const bool in = t < V && ((mask[t >> 5] >> (t & 31u)) & 1u);
            const uint32_t x = in ? rank_of(r.tokens[t]) : 0u;
            if (x > rank) sh.cand[atomicAdd(&sh.n, 1u)] = (unsigned long long)x << 32 | (0xFFFFFFFFu - t);
            const unsigned long long tie = __ballot(in && x == rank);
            if ((tid & 63u) == 0u) sh.count[tid >> 6] = (uint32_t)__popcll(tie);
            __syncthreads();
            uint32_t at = sh.digit, all = 0;
#pragma nounroll
            for (uint32_t w = 0; w < kWaves; w++) { if (w < (tid >> 6)) at += sh.count[w]; all += sh.count[w]; }
            at += (uint32_t)__popcll(tie & ((1ull << (tid & 63u)) - 1ull));
            if (in && x == rank && at < k) sh.cand[at] = (unsigned long long)x << 32 | (0xFFFFFFFFu - t);
            __syncthreads();
            if (tid == 0) sh.digit += all;
            __syncthreads();
        }
        n = k;                                        // (more than kCand tokens are allowed)
    }
    // ranked by counting, the best k leave
    rank_keys<kThreads>(sh.cand, n, k, [&](uint32_t at, unsigned long long key) {
        const uint32_t id = 0xFFFFFFFFu - (uint32_t)key;
        id_out[at] = (int32_t)id;
        value_out[at] = logit_of(key, r.tokens);
    });
    // fewer than k allowed tokens in the row: the rest says so
    for (uint32_t i = n + tid; i < k; i += kThreads) { id_out[i] = -1; value_out[i] = ninf; }
}

// Small batches: a slice of kTopkSlice tokens of a row per workgroup of 256 threads, a thread's 32
// tokens in registers.  The best k of the slice leave for the workspace, best first.  What it takes is the
// trips to memory one after the other: mask, logits, the candidates' logits again for their keys (a call, slices and merge, V = 128,256
// fp32, B = 8, everything allowed: 9.5 us with k = 20, 12.2 with k = 50).  7 registers of a thread (fp32; bf16 13) have no room and
// go to memory.
constexpr uint32_t kSliceThreads = 256;
constexpr uint32_t kSliceWaves = kSliceThreads / 64u;
constexpr uint32_t kSlicePer = kTopkSlice / kSliceThreads;       // tokens of a thread
constexpr uint32_t kSliceCand = kTopkMax * kSlicePer;            // k threads reach the exact bound, with 32 tokens each
static_assert(kSlicePer == 32u, "a bit per token of a thread");

struct SliceShared {
    unsigned long long cand[kSliceCand];
    uint32_t id[kSliceCand];
    uint32_t words[kTopkSlice / 32u + 1u];           // the staged mask
    uint32_t count[kSliceWaves];
    uint32_t n;
};

template <typename Elem, bool kWhole>
__global__ void __launch_bounds__(kSliceThreads) __attribute__((amdgpu_waves_per_eu(5)))
topk_slice_kernel(const Elem *__restrict__ logits, int64_t row_stride, uint32_t V, uint32_t W,
                  const uint32_t *__restrict__ bitmask, uint32_t k, unsigned long long *__restrict__ lists)
{
    constexpr uint32_t kPer = Row<Elem, kWhole>::kPer, kPieces = kSlicePer / kPer;
    __shared__ SliceShared sh;
    const uint32_t b = blockIdx.y, tid = threadIdx.x;
    const uint32_t *mask = bitmask + (size_t)b * W;
    const Row<Elem, kWhole> r(logits + (int64_t)b * row_stride, V);
    unsigned long long *out = lists + ((size_t)b * gridDim.x + blockIdx.x) * k;
    // Equal shares of whole mask words: a last slice of a few hundred tokens fills a wavefront or two, the
    // others then give no bound, and all of its tokens are ranked (V = 115,001: 10 us more).  Where the
    // row is a whole number of slices the last one also takes the piece that a skewed row has behind them.
    constexpr uint32_t kStep = 32u / kPer;
    const uint32_t even = ((r.pieces + gridDim.x - 1u) / gridDim.x + kStep - 1u) / kStep * kStep;
    const uint32_t share = even < kTopkSlice / kPer ? even : kTopkSlice / kPer;
    const uint32_t base = blockIdx.x * share < r.pieces ? blockIdx.x * share : r.pieces;      // first piece of the slice
    const uint32_t own_pieces = blockIdx.x == gridDim.x - 1u || r.pieces - base < share ? r.pieces - base : share;
    // the slice's mask words, and the one behind them (from memory, piece by piece, they were eight loads one
    // after the other in front of the logits')
    constexpr uint32_t kWords = kTopkSlice / 32u;
    static_assert(kWords == kSliceThreads, "a mask word per thread");
    const uint32_t first_word = base / kStep;
    sh.words[tid] = mask_word(mask, W, V, r.skew, first_word + tid);
    if (tid == 0) { sh.words[kWords] = mask_word(mask, W, V, r.skew, first_word + kWords); sh.n = 0u; }
    __syncthreads();
    uint32_t m[kPieces];
    union { uint4 v; Elem e[kPer]; } u[kPieces];
#pragma unroll
    for (uint32_t j = 0; j < kPieces; j++) {
        const uint32_t q = j * kSliceThreads + tid, bit = q * kPer;
        m[j] = q < own_pieces ? (sh.words[bit >> 5] >> (bit & 31u)) & r.kAll : 0u;
    }
    const uint32_t extra = base + kTopkSlice / kPer + tid;        // at most one such piece
    const uint32_t m_extra = kTopkSlice / kPer + tid < own_pieces ? sh.words[kWords] & r.kAll : 0u;
    float best = __builtin_nanf("");
    uint32_t any = m_extra;
#pragma unroll
    for (uint32_t j = 0; j < kPieces; j++) any |= m[j];
    uint4 v_extra;
    const Window win = r.window(base, own_pieces);
#pragma unroll
    for (uint32_t j = 0; j < kPieces; j++) u[j].v = r.piece(win, m[j] ? (j * kSliceThreads + tid) * 16u : kNowhere);
    v_extra = r.piece(win, m_extra ? (kTopkSlice / kPer + tid) * 16u : kNowhere);
#pragma unroll
    for (uint32_t j = 0; j < kPieces; j++) best = __builtin_fmaxf(best, piece_max(u[j].v, m[j], Elem(0)));
    if (m_extra) best = __builtin_fmaxf(best, piece_max(v_extra, m_extra, Elem(0)));
    const uint32_t own = best == best ? order_key(__float_as_uint(best)) + 1u : any ? 1u : 0u;
    const uint32_t bound = bound_of<kSliceWaves>(own, k, sh.count);
    const float value = bound_value(bound);
    auto put = [&](uint32_t p, uint32_t take) {
        while (take) {
            const uint32_t i = (uint32_t)__builtin_ctz(take);
            take &= take - 1u;
            const uint32_t at = atomicAdd(&sh.n, 1u);
            if (at < kSliceCand) sh.id[at] = r.token(p, i);
        }
    };
    if (own >= bound) {
#pragma unroll
        for (uint32_t j = 0; j < kPieces; j++) put(base + j * kSliceThreads + tid, reaching(u[j].v, m[j], bound, value, Elem(0)));
        put(extra, reaching(v_extra, m_extra, bound, value, Elem(0)));
    }
    __syncthreads();
    uint32_t n = sh.n;
    if (n > kSliceCand) {
        // Thousands tie at the bound or are NaN.  k rounds, the best key below the last one each time.
        unsigned long long last = ~0ull;
        for (uint32_t q = 0; q < k; q++) {
            unsigned long long top = 0ull;
            auto see = [&](uint32_t p, const Elem *e, uint32_t allowed) {
#pragma unroll
                for (uint32_t i = 0; i < kPer; i++) {
                    const unsigned long long key = (allowed >> i) & 1u ? (unsigned long long)rank_of(e[i]) << 32 | (0xFFFFFFFFu - r.token(p, i)) : 0ull;
                    if (key < last && key > top) top = key;
                }
            };
#pragma unroll
            for (uint32_t j = 0; j < kPieces; j++) see(base + j * kSliceThreads + tid, u[j].e, m[j]);
            union { uint4 v; Elem e[kPer]; } ux;
            ux.v = v_extra;
            see(extra, ux.e, m_extra);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) { const unsigned long long other = __shfl_xor(top, o); top = other > top ? other : top; }
            __syncthreads();
            if ((tid & 63u) == 0u) sh.cand[tid >> 6] = top;
            __syncthreads();
            last = sh.cand[0];
            for (uint32_t w = 1; w < kSliceWaves; w++) last = sh.cand[w] > last ? sh.cand[w] : last;
            if (tid == 0) out[q] = last;
        }
        return;
    }
    make_keys<kSliceThreads>(sh.cand, sh.id, n, r);
    __syncthreads();
    rank_keys<kSliceThreads>(sh.cand, n, k, [&](uint32_t at, unsigned long long x) { out[at] = x; });
    for (uint32_t i = n + tid; i < k; i += kSliceThreads) out[i] = 0ull;
}

// A row's slices merged: the same bound and count on the keys that they left, kHeld of a thread at most.  Its
// time is code fetched and a few trips to LDS and memory: unrolled for 16 keys of a thread always, it was 8.8
// us for V = 128,256, k = 50 (3.1 to 4 keys of a thread), now 4.4.
template <typename Elem, uint32_t kHeld>
__global__ void __launch_bounds__(kSliceThreads)
topk_merge_kernel(const Elem *__restrict__ logits, int64_t row_stride, uint32_t n_slices, uint32_t k,
                  const unsigned long long *__restrict__ lists, int32_t *__restrict__ ids, Elem *__restrict__ values, Elem ninf)
{
    __shared__ unsigned long long cand[kHeld * kSliceThreads];
    __shared__ uint32_t count[kSliceWaves], n_cand;
    const uint32_t b = blockIdx.x, tid = threadIdx.x, n = n_slices * k;
    // In order of rank, the slices' best first, and in turn to the wavefronts: then the thread maxima are about
    // the 256 best, every wavefront has as many good ones as another, and hardly more than k keys reach the
    // bound.  (In the order of the lists a lane held one rank, where k is 64, and hundreds of keys reached it:
    // 15.2 us instead of 8.5 for B = 8, V = 151,936 fp32, before the kernel was cut to size.)
    unsigned long long x[kHeld];
    uint32_t own = 0;
    const uint32_t place = (tid & 63u) * kSliceWaves + (tid >> 6);
#pragma unroll
    for (uint32_t j = 0; j < kHeld; j++) {
        const uint32_t i = place + j * kSliceThreads;
        x[j] = 0ull;
        if (j * kSliceThreads >= n) continue;
        const uint32_t rank = i / n_slices;
        if (i < n) x[j] = lists[(size_t)b * n + (i - rank * n_slices) * k + rank];
    }
#pragma unroll
    for (uint32_t j = 0; j < kHeld; j++) { const uint32_t h = (uint32_t)(x[j] >> 32); own = h > own ? h : own; }
    if (tid == 0) n_cand = 0u;
    const uint32_t bound = bound_of<kSliceWaves>(own, k, count);
#pragma unroll
    for (uint32_t j = 0; j < kHeld; j++) {
        if (j * kSliceThreads >= n) break;
        if (x[j] && (uint32_t)(x[j] >> 32) >= bound) cand[atomicAdd(&n_cand, 1u)] = x[j];
    }
    __syncthreads();
    const uint32_t c = n_cand;
    rank_keys<kSliceThreads>(cand, c, k, [&](uint32_t at, unsigned long long key) {
        const uint32_t id = 0xFFFFFFFFu - (uint32_t)key;
        ids[(size_t)b * k + at] = (int32_t)id;
        values[(size_t)b * k + at] = logit_of(key, logits + (int64_t)b * row_stride);
    });
    for (uint32_t i = c + tid; i < k; i += kSliceThreads) { ids[(size_t)b * k + i] = -1; values[(size_t)b * k + i] = ninf; }
}

// The lists of wg_masked_topk_static: what wg_masked_topk takes from its caller, one copy per GPU for
// the life of the process.  topk_slice writes every key that topk_merge reads.
static __device__ __align__(256) unsigned long long scratch[kTopkStaticKeys];

hipError_t static_topk_scratch(unsigned long long **out)
{
    constexpr int kDevices = 64;
    static std::mutex mu;
    static unsigned long long *ptr[kDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr[dev] = static_cast<unsigned long long *>(p);
    }
    *out = ptr[dev];
    return hipSuccess;
}

// All rows of a call are whole or none is: they lie a number of elements apart.
template <typename Elem> static bool rows_are_whole(const Elem *logits) { return reinterpret_cast<uintptr_t>(logits) % sizeof(Elem) == 0u; }

// Workgroups of the greedy choice per row: as many as the compute units hold one of each, at least
// 16,384 tokens in each.  (Two of each, bf16, V = 151,936, mixed masks, us: B = 64 7.5 -> 8.6, B = 128 9.2 -> 10.3, B = 256 13.7 -> 14.2; four:
// B = 256 18.2.)
static uint32_t argmax_parts(uint32_t B, uint32_t V)
{
    uint32_t parts = 1u;
    while (parts < 16u && parts * 2u * B <= kCutRows && parts * 2u * 16384u <= V) parts *= 2u;
    return parts;
}

// fp32 rows are taken in slices (argmax_slice_kernel) from 33 rows of eight slices on.  In slices / by row, everything allowed, nothing and a
// few tokens in every other row: V = 50,021 B = 40 1.09 1.10 1.16, 128 1.07 1.02 0.98, 256 1.11 0.95 0.96; 64,000 B = 40 0.99 1.05 0.94,
// 128 1.00 0.89 0.94, 256 1.06 0.90 0.91; 100,003 B = 24 0.93 1.02 0.91, 32 1.01 0.91 0.90, 40 0.99 0.90 0.93, 256 1.04 0.88 0.88;
// 151,936 B = 16 0.99 0.96 1.03, 32 1.11 0.92 0.94, 64 1.06 0.77 0.78, 256 1.04 0.85 0.84.
static bool argmax_in_slices(int dtype, uint32_t B, uint32_t V, const void *logits)
{
    return dtype == WG_F32 && B > 32u && V > 7u * kChoiceTokens && rows_are_whole(static_cast<const uint32_t *>(logits));
}

// The k best are taken by a workgroup per row where the row is short, or where there are rows enough to keep
// the chip busy; what a slice costs besides its bytes grows with k.  Slices / by row, k = 20, 50, 64, everything allowed (nothing in
// every other row up to 0.2 less from 64 rows on):
//   bf16, V = 50021 B = 8 1.05 1.24 1.37; 64000 B = 8 0.94 1.12 1.24, 48 1.01 1.19 1.30; 84000 B = 48 0.93 1.12 1.27, 96 1.07 1.28
//   1.41; 100003 B = 8 0.81 1.01 1.16, 64 0.99 1.21 1.34, 96 1.09 1.29 1.45; 128256 B = 24 0.79 1.00 1.10, 64 0.95 1.17 1.28, 96 1.16
//   1.40 1.54; 151936 B = 8 0.69 0.85 1.01, 48 0.85 1.03 1.17, 64 0.92 1.06 1.24, 96 1.12 1.27 1.42
//   fp32, V = 32000 1.09 to 1.43; 50021 B = 24 0.96 1.12 1.21, 64 1.05 1.21 1.33; 64000 B = 8 0.92 1.06 1.19, 64 1.04 1.24 1.35;
//   84000 B = 33 0.86 1.01 1.12, 64 1.00 1.12 1.22, 96 1.07 1.21 1.30; 100003 B = 8 0.76 0.89 0.98, 64 0.96 1.10 1.18, 96 1.04 1.12 1.24,
//   128 1.18 1.32 1.42; 128256 B = 48 0.84 1.00 1.08, 64 0.89 1.04 1.12, 96 1.09 1.27 1.36; 151936 B = 64 0.82 0.95 1.08, 96 1.03 1.17 1.31
static bool topk_by_row(uint32_t B, uint32_t V, uint32_t k, uint32_t elem_bytes)
{
    const uint32_t slices = V / kTopkSlice, kind = k <= 32u ? 0u : k <= 56u ? 1u : 2u;
    if (elem_bytes == 2u) {
        const uint32_t few[3] = {7u, 14u, 20u}, rows[3] = {slices < 10u ? 48u : 80u, 40u, 32u};
        return slices < few[kind] || B >= rows[kind];
    }
    const uint32_t few[3] = {6u, 9u, 14u}, rows[3] = {slices < 9u ? 56u : 96u, slices < 16u ? 64u : 96u, 56u};
    return slices < few[kind] || B >= rows[kind];
}

hipError_t launch_masked_argmax(const void *logits, int dtype, uint32_t B, uint32_t V, int64_t row_stride,
                                const uint32_t *bitmask, int32_t *tokens, hipStream_t s)
{
    const uint32_t W = (V + 31u) / 32u;
    if (argmax_in_slices(dtype, B, V, logits)) {
        const uint32_t slices = (V + 3u + kChoiceTokens - 1u) / kChoiceTokens;         // a row may begin 3 tokens into its first piece
        const hipError_t e = launch(argmax_slice_kernel, dim3(slices, B), dim3(kChoiceThreads), 0, s, nullptr, static_cast<const uint32_t *>(logits), row_stride, V, W, bitmask);
        if (e != hipSuccess) return e;
        return launch(argmax_finish_kernel, dim3((B + 63u) / 64u), dim3(64), 0, s, nullptr, tokens, B);
    }
    auto choose = [&](auto kernel, auto *x) { return launch(kernel, dim3(argmax_parts(B, V), B), dim3(kThreads), 0, s, nullptr, x, row_stride, V, W, bitmask, tokens); };
    if (dtype == WG_F32) {
        const uint32_t *x = static_cast<const uint32_t *>(logits);
        return rows_are_whole(x) ? choose(masked_argmax_kernel<uint32_t, true>, x) : choose(masked_argmax_kernel<uint32_t, false>, x);
    }
    const uint16_t *x = static_cast<const uint16_t *>(logits);
    return rows_are_whole(x) ? choose(masked_argmax_kernel<uint16_t, true>, x) : choose(masked_argmax_kernel<uint16_t, false>, x);
}

template <typename Elem>
static hipError_t topk(const Elem *logits, uint32_t B, uint32_t V, int64_t row_stride, const uint32_t *bitmask, uint32_t k,
                       int32_t *ids, Elem *values, Elem ninf, unsigned long long *lists, hipStream_t s)
{
    const uint32_t W = (V + 31u) / 32u;
    if (topk_by_row(B, V, k, sizeof(Elem)))
        return launch(rows_are_whole(logits) ? masked_topk_kernel<Elem, true> : masked_topk_kernel<Elem, false>, dim3(B), dim3(kThreads), 0, s, nullptr, logits, row_stride, V, W, bitmask, k, ids, values, ninf);
    const uint32_t n_slices = (V + kTopkSlice - 1u) / kTopkSlice;
    const hipError_t e = launch(rows_are_whole(logits) ? topk_slice_kernel<Elem, true> : topk_slice_kernel<Elem, false>, dim3(n_slices, B), dim3(kSliceThreads), 0, s, nullptr, logits, row_stride, V, W, bitmask, k, lists);
    if (e != hipSuccess) return e;
    constexpr uint32_t kMost = kTopkMergeKeys / kSliceThreads;
    const uint32_t held = (n_slices * k + kSliceThreads - 1u) / kSliceThreads;
    return launch(held <= 4u ? topk_merge_kernel<Elem, 4> : held <= 8u ? topk_merge_kernel<Elem, 8> : topk_merge_kernel<Elem, kMost>, dim3(B), dim3(kSliceThreads), 0, s,
                  nullptr, logits, row_stride, n_slices, k, lists, ids, values, ninf);
}

hipError_t launch_masked_topk(const void *logits, int dtype, uint32_t B, uint32_t V, int64_t row_stride,
                              const uint32_t *bitmask, uint32_t k, int32_t *ids, void *values, unsigned long long *lists, hipStream_t s)
{
    if (dtype == WG_F32)
        return topk<uint32_t>(static_cast<const uint32_t *>(logits), B, V, row_stride, bitmask, k, ids, static_cast<uint32_t *>(values), 0xFF800000u, lists, s);
    return topk<uint16_t>(static_cast<const uint16_t *>(logits), B, V, row_stride, bitmask, k, ids, static_cast<uint16_t *>(values), (uint16_t)0xFF80u, lists, s);
}

}  // namespace wg
