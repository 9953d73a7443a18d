// Internal layouts shared by the host lowering code and the HIP kernels.
#pragma once
#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "../../include/wg.h"

namespace wg {

constexpr uint32_t kSymEos = 256;

// Byte classes of a WAIT / COND state (one 256-entry table per distinct set triple).
enum : uint8_t { CLS_REJECT = 0, CLS_STAY = 1, CLS_EXIT_A = 2, CLS_EXIT_B = 3 };

// One leaf state as the kernels read it: 32 bytes, so a wave fetches a descriptor
// with one scalar 8-dword load.
struct StateDesc {
    uint32_t kind_byte;   // bits 0..7 WG_KIND_*, bits 8..15 the literal byte of a LIT state
    uint32_t next_a;      // LIT / WAIT successor, COND true target
    uint32_t next_b;      // COND false target
    uint32_t eos_next;    // state after EOS, WG_SID_ERROR if rejected
    uint32_t cls;         // WAIT / COND: index of the 256-byte class table; LIT: state after its Write
    uint32_t max;         // WAIT bound, WG_UNBOUNDED if none
    uint32_t key_base;    // first mask-cache key of this state
    uint32_t run;         // LIT: literal bytes from this state to the end of its Write
};
static_assert(sizeof(StateDesc) == 32, "descriptor layout");

// Result of lowering a set of template instances (host memory).
struct Table {
    std::vector<StateDesc> states;        // index = sid; [0] is FINAL
    std::vector<uint8_t> classes;         // n_class_tables * 256
    std::vector<uint8_t> lit;             // lit[sid] = byte of a LIT state (else 0)
    std::vector<uint32_t> tmpl;           // template instance of each state
    std::vector<uint32_t> start;          // start state of each instance
    std::vector<uint32_t> key_count;      // masks per state (1, or lmax+1 for a bounded Wait)
    uint32_t n_keys = 0;
    uint32_t lmax = 0;
    uint32_t flags = 0;
};

// The token ids are cut into kParts contiguous ranges, on boundaries of kPartGroup tokens, so on
// 256-byte boundaries of a mask row.  Every list of candidate tokens is kept per range, so that a row
// can be made by several workgroups, each owning the words of some neighbouring ranges, without any
// merging.
constexpr uint32_t kParts = 32;
constexpr uint32_t kPartGroup = 2048;

// How the rows of a class table's states are made, worked out once per table.  A table that at most
// kFewLive byte values enter is taken by first byte: ids[0 .. n_exits) are those values, value |
// class << 8.  Any other table is taken by token rows: ids[0 .. n_exits) are its exit bytes (value
// | class << 8), ids[n_exits .. n_ids) the token rows that together hold every token with a
// rejected byte (kBlockRow + k: byte values 4k .. 4k+3, kBigBlockRow + k: 16k .. 16k+15).
constexpr uint32_t kFewLive = 8;
constexpr uint32_t kBlockRow = 256, kBigBlockRow = 320, kTailRow = 336, kWideRow = 592, kLenRow = 606;
struct ClassPlan {
    uint16_t n_exits, n_ids, by_first, pad;
    uint16_t ids[260];
};
static_assert(sizeof(ClassPlan) % 16 == 0, "class plan layout");
ClassPlan class_plan_of(const uint8_t *table);
// A class table as the walk of a sampled token reads it: two bits a byte value, sixteen values to a word.
struct ClassCodes { uint32_t word[16]; };
ClassCodes class_codes_of(const uint8_t *table);
// The same for the device, with the rows of 16 byte values put together where 32, 64 or 128 are rejected as a
// whole: kWideRow + k stands for the k-th of the blocks of 32 (k = 0 .. 7), of 64 (8 .. 11) and of 128 (12, 13).
// Most tables reject all that is not ASCII: a row for it instead of eight (kWideRows rows of 19 KB for 152k tokens).
constexpr uint32_t kWideRows = 14;
ClassPlan wide_plan_of(const uint8_t *table);
inline uint32_t wide_row(uint32_t first_value, uint32_t values) {
    return kWideRow + (values == 32 ? 0u : values == 64 ? 8u : 12u) + first_value / values;
}

// A token that leaves a checkpoint state before its last byte: the part of a mask that
// depends on what follows the state.  `off` bytes are consumed up to and including the
// exit byte, `rem` bytes remain, the first of which is `first`.
struct ExitEntry {
    uint32_t tok;
    uint8_t off, cls, first, rem;
};
static_assert(sizeof(ExitEntry) == 8, "entry layout");

// The static indexes of a vocabulary (they depend on the token bytes only), as host arrays in
// the layouts the kernels read.  Built once per vocabulary; wg_vocab_create copies them to the
// device as they are.
struct VocabIndex {
    uint32_t V = 0, W = 0, row_stride = 0, lmax = 0, n_chunks = 0;
    uint32_t part_tok[kParts + 1] = {};    // first token of each range; part_tok[kParts] == V
    std::vector<uint8_t> len8;             // per token
    std::vector<uint64_t> chunks;          // max(n_chunks, 1) * V
    std::vector<ExitEntry> lit_entries;    // never empty (one unused entry when no token has bytes)
    std::vector<uint32_t> lit_start;       // 256 * kParts + 1
    std::vector<uint32_t> len_rows;        // (lmax + 2) * row_stride
    std::vector<ExitEntry> sorted;         // never empty
    std::vector<uint32_t> dir0;            // 256 * 257 + 1
    std::vector<ExitEntry> bigram;         // never empty
    std::vector<uint32_t> dirN;            // 65536 + 1
    std::vector<uint32_t> byte_rows;       // 256 rows of row_stride words: tokens that contain the byte
    std::vector<uint32_t> block_rows;      // 64 + 16 rows: by any byte of a block of 4, of 16 byte values
    std::vector<uint32_t> tail_rows;       // 256 rows: tokens in which the byte occurs once, as the last one
    std::vector<ExitEntry> places;         // the byte pairs again, by (first byte of the pair, range); never empty
    std::vector<uint32_t> place_start;     // 256 * kParts + 1
};

// What the device is given of an index.  token_rows: all rows one behind the other, in the order of their numbers (byte
// values, blocks of 4 and 16, tails, wide blocks, lengths).  candidates: the four lists of entries one behind the other,
// and their directories with the places among all of them, at kDirSorted (dir0), kDirFirst (lit_start), kDirPairs (dirN) and
// kDirPlaces (place_start); false: more than 2^32 entries.
constexpr uint32_t kDirSorted = 0, kDirFirst = kDirSorted + 256 * 257 + 1, kDirPairs = kDirFirst + 256 * kParts + 1,
                   kDirPlaces = kDirPairs + 65536 + 1, kDirWords = kDirPlaces + 256 * kParts + 1;
std::vector<uint32_t> token_rows(const VocabIndex &ix);
bool candidates(const VocabIndex &ix, std::vector<ExitEntry> *index, std::vector<uint32_t> *dirs);

// Checks the vocabulary arguments of wg_vocab_create and builds the indexes.  Returns WG_OK, or
// an error code with the message in *err; `out` is then unspecified.
int build_vocab_index(const uint8_t *host_bytes, const uint64_t *host_offsets, uint32_t V, int32_t eos_id,
                      VocabIndex *out, std::string *err);

// The host operator compiler with its memory: parsed template texts (the static structures)
// and the class tables seen so far, so that instances can be added to a live table.
struct LoweringState;
class Lowering {
  public:
    Lowering(uint32_t flags, uint32_t lmax);
    ~Lowering();
    Lowering(const Lowering &) = delete;
    Lowering &operator=(const Lowering &) = delete;
    // Appends n template instances.  Throws std::runtime_error with a message naming the
    // template and the offset; the table is then as it was before the call.
    void add(const char *const *templates, const wg_args_t *args, uint32_t n);
    Table table;

  private:
    std::unique_ptr<LoweringState> st_;
};

// Translates a regular expression into template text in the operator syntax; throws
// std::runtime_error when the expression has no translation.
std::string regex_to_template(const char *regex);

void set_last_error(const std::string &msg);

}  // namespace wg
