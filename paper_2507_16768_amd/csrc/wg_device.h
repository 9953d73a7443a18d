// Device-side views passed to the kernels by value, and the launcher prototypes.
#pragma once
#include <hip/hip_runtime.h>

#include "wg_internal.h"

namespace wg {

constexpr uint32_t kNoKey = 0xFFFFFFFFu;

struct DeviceTable {
    const StateDesc *states;
    const uint8_t *classes;      // 256-byte class tables
    const ClassPlan *plans;      // one per class table
    const uint8_t *lit;          // literal byte per state
    const ClassCodes *codes;     // per state: a checkpoint's class table once more (see look_ahead); else zeros
    uint32_t n_states;
    uint32_t lmax;
};

// The arrays of a vocabulary that the row builder reads lie one behind the other, rows with rows and
// directories with directories: a pointer costs it two of its scalar registers.
struct DeviceVocab {
    const uint8_t *len8;         // token length in bytes (0 for EOS and byte-less tokens)
    const uint64_t *chunks;      // chunks[k * V + t] = bytes 8k .. 8k+7 of token t, zero padded
    // token rows: row x (0 .. 255) the tokens that contain the byte x, row kBlockRow + k those that
    // contain a byte 4k .. 4k+3, row kBigBlockRow + k a byte 16k .. 16k+15; row kTailRow + x the tokens in
    // which x occurs once, as the last byte; kWideRow: see wide_plan_of; row kLenRow + r (r = 0 .. lmax+1) those with 1 <= length <= r
    const uint32_t *rows;
    const ExitEntry *index;      // the four candidate indexes, entries {tok, off, cls, first, rem}; off + rem is the token's length
    // the entry numbers at which the ranges of the indexes begin, four directories:
    //   kDirSorted: by byte order; range y0 * 257 is the token that is the single byte y0, range
    //     y0 * 257 + 1 + y1 the tokens of two or more bytes that start with y0 y1; first = second byte
    //   kDirFirst: by (first byte, token range); off = 1, first = second byte (rem = 0: a one-byte token)
    //   kDirPairs: every place where a byte y follows a byte e: range e * 256 + y; off = index of y, first = y
    //   kDirPlaces: the same by (e, token range)
    const uint32_t *dirs;
    uint32_t V, W;
    int32_t eos_id;
    uint32_t lmax;
    uint32_t n_chunks;           // ceil(lmax / 8)
    uint32_t row_stride;         // words per mask row in device arenas (multiple of 4)
};

// A successor state as the row builder needs it for the first hop of a walk.
struct HopState {
    uint32_t kind, lit;
    uint32_t next_a, next_b, max, cls;   // checkpoint: as in its descriptor
                                         // literal: the state itself, -, the bytes of its run, the state after the run
};

// What the lookup leaves for a request whose mask row has to be made in this call.
struct RowTask {
    uint32_t sid, kind, lit;
    uint32_t cls;                // checkpoint: class table; literal: the state after its run
    uint32_t run;                // literal: bytes of its run
    uint32_t r;                  // allow-bytes that may still be consumed, capped at lmax
    uint32_t class_state;        // CLASS_*: where the context-free rows of the class table come from
    uint32_t eos_next;
    uint32_t slot;               // arena row that keeps the result, or kNoSlot
    HopState hop[2];             // successors reached through exit A / exit B
};
static_assert(sizeof(RowTask) == 84, "row task layout");
//   CLASS_SELF  claimed in this call by another request: this one makes them for itself
//   CLASS_READY made in an earlier call
//   CLASS_OWN   made here, and kept
enum : uint32_t { CLASS_SELF = 0, CLASS_READY = 1, CLASS_OWN = 2 };

struct Counters {
    uint32_t n_claims;           // keys claimed in the call in flight
    uint32_t n_class_claims;     // class tables claimed in the call in flight
    unsigned long long slot_ctr; // generation << 32 | arena rows in use in that generation (<= cap_rows); not kept up while
                                 // the arena is addressed by key
    unsigned long long launch;   // number of the fill call in flight (its last kernel counts it up)
    unsigned long long lookups, builds, uncached_builds, class_scans;
    unsigned long long held;     // keys that hold a row, when last counted (launch_count_rows)
};

// The tag of a key or of a class table: the cache generation (30 bits) in which, the fill call (its
// number's low 18 bits) by which and the request for which it was claimed; 0 means never.  A key's
// row, or a table's two rows, are in place once that call is over: for every later call of the
// generation the tag says "made", for the claiming call itself "being made" -- a request of the same
// call that needs the same key makes its own copy of the row and waits for nobody.  (A call whose
// number agrees with an old claim's in all 18 bits takes that row for one being made and makes a
// copy too: the same row, one hit fewer.)
constexpr uint32_t kTagRequestBits = 16, kTagEpochShift = 34;
constexpr unsigned long long kTagLaunchMask = (1ull << (kTagEpochShift - kTagRequestBits)) - 1ull;
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;
// What the lookup leaves per request: the arena row of a mask made before the call, kRefBuild (its
// task says how to make it), or kNoKey (no such state: a row of zeros).  Rows stay below 2^30.
constexpr uint32_t kRefBuild = 0xFFFFFFFEu;
constexpr uint32_t kMaxRows = 1u << 30, kMaxKeys = 0x7FFFFFFEu;
constexpr uint32_t kMaxBatch = 65535u;     // requests of a call (grid.y)
// Statistics that many workgroups add to are spread over 64 cache lines, a counter of each in every one.
constexpr uint32_t kSpread = 64, kSpreadStride = 16, kSpreadWalked = 0, kSpreadHits = 1,
                   kSpreadBuilds = 2, kSpreadClasses = 3,       // of fills with the arena addressed by key
                   kSpreadErrors = 4;                           // rejected tokens
constexpr uint32_t kTicketStride = 32, kTicketGroup = 16;       // a 128-byte line for the tickets of a row; rows of a group
constexpr uint32_t kOneKernelRows = 1024;                       // most rows of a fill in one kernel

// All that calls count in, one piece of memory: a pointer costs the kernels two of their scalar registers.
struct Control : Counters {
    alignas(128) unsigned long long spread[kSpread * kSpreadStride];     // kSpread groups of counters, kSpreadStride apart
    // one-kernel fill, zero between calls: groups all of whose rows have, rows of a group all of whose workgroups have,
    // workgroups of a row that have read its state (the latter two kTicketStride apart)
    alignas(128) uint32_t call_ticket;
    alignas(128) uint32_t group_tickets[kOneKernelRows / kTicketGroup * kTicketStride];
    alignas(128) uint32_t tickets[kOneKernelRows * kTicketStride];
};

struct DeviceCache {
    Control *ctr;
    // per state key
    unsigned long long *tags;
    uint32_t *slots;             // not direct: arena row of a claimed key, or kNoSlot: the arena was full (and stays so)
    uint32_t *arena;             // cap_rows rows of row_stride words
    uint32_t cap_rows;
    uint32_t direct;             // the arena has a row for every key: key k keeps row k; else rows are handed out in order of first use,
    const uint32_t *free_rows;   // in this order (null: by number)
    // per class table (the context-free part of every mask of a state using that table)
    unsigned long long *class_tags;
    uint32_t *class_rows;        // 2 rows per class: [stay] all bytes stay, [end] exits on its last byte
    // per call
    uint32_t *row_ref;           // [B] arena row, kRefBuild or kNoKey
    RowTask *tasks;              // [B]
    uint32_t row_stride;         // words, multiple of 4
    uint32_t n_keys;
    uint32_t epoch;              // cache generation of this call
};

// How a fill of B requests is launched: workgroups per row, whether they do the lookups themselves
// (one kernel) or find them done by a kernel before theirs, and whether they mask logits by whole lines.
struct FillPlan { uint32_t parts; bool one_kernel, lines; };
// dtype: of the logits, where the fill masks any.
FillPlan plan_fill(const DeviceVocab &Vc, const DeviceCache &Cc, uint32_t B, bool masks_logits, int dtype, uint32_t n_cu);
// lookup_ev, rows_ev: a begin / end pair of events for each kernel that the plan has, or null.
// With tokens != nullptr the states are first advanced by them (in place, with the lookup); with
// logits != nullptr the mask is also applied to them (in the rows kernel).
hipError_t launch_fill(const FillPlan &plan, const DeviceTable &T, const DeviceVocab &Vc, const DeviceCache &Cc,
                       wg_state_t *states, const int32_t *tokens, uint32_t B, uint32_t *bitmask,
                       void *logits, int dtype, int64_t logits_stride,
                       hipStream_t s, hipEvent_t *lookup_ev, hipEvent_t *rows_ev);
struct AppendSlice { uint8_t *dst; const uint8_t *src; uint32_t bytes; };
struct AppendSlices { AppendSlice slice[5]; };
hipError_t launch_append(const AppendSlices &a, uint32_t n, hipStream_t s);
// While the arena is addressed by key: adds the keys that hold a row in this generation to Cc.ctr->held.
hipError_t launch_count_rows(const DeviceCache &Cc, hipStream_t s);
hipError_t launch_free_rows(const DeviceCache &Cc, uint32_t n_keys, uint32_t *free_rows, hipStream_t s);
// Dynamic LDS of the rows kernel for this vocabulary; with its static part it stays within the 64 KB
// a kernel gets without asking.
uint32_t rows_lds_bytes(const DeviceVocab &Vc);
constexpr uint32_t kRowsLdsMax = 52u * 1024u;
hipError_t launch_apply(void *logits, int dtype, uint32_t B, uint32_t V, int64_t row_stride,
                        const uint32_t *bitmask, hipStream_t s, hipEvent_t *ev);
hipError_t launch_masked_argmax(const void *logits, int dtype, uint32_t B, uint32_t V, int64_t row_stride,
                                const uint32_t *bitmask, int32_t *tokens, hipStream_t s);
// masked top-k: small batches rank kTopkSlice tokens of a row per workgroup; `lists` is room for
// B * ceil(V / kTopkSlice) * k 64-bit keys
constexpr uint32_t kTopkMax = 64;
constexpr uint32_t kTopkSlice = 8192;
constexpr uint32_t kTopkMergeKeys = 4096;    // most keys (slices * k) of a row
hipError_t launch_masked_topk(const void *logits, int dtype, uint32_t B, uint32_t V, int64_t row_stride,
                              const uint32_t *bitmask, uint32_t k, int32_t *ids, void *values, unsigned long long *lists, hipStream_t s);
// wg_masked_topk_static keeps its lists in a file-scope device array of this many 64-bit keys
// (4 MiB per GPU); static_topk_scratch gives the array's address on the current device.
constexpr uint64_t kTopkStaticKeys = 1ull << 19;
hipError_t static_topk_scratch(unsigned long long **out);
hipError_t launch_advance(const DeviceTable &T, const DeviceVocab &Vc, const DeviceCache &Cc,
                          wg_state_t *states, const int32_t *tokens, uint32_t B, uint32_t n_cu, hipStream_t s,
                          hipEvent_t *ev);
hipError_t launch_forced_bytes(const DeviceTable &T, const wg_state_t *states, uint32_t B, uint32_t cap,
                               uint8_t *bytes, uint32_t *lens, wg_state_t *end_states, uint32_t n_cu, hipStream_t s);
hipError_t launch_select(const uint32_t *bitmask, uint32_t B, uint32_t V, const uint64_t *draws,
                         int32_t *tokens, hipStream_t s);

}  // namespace wg
