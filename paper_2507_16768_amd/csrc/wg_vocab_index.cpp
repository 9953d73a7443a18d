// The static indexes of a vocabulary and the plans of class tables: host code without any
// device call, so that it can also be built and checked on its own.
#include <algorithm>
#include <cstring>
#include <new>

#include "wg_internal.h"

namespace wg {

ClassPlan class_plan_of(const uint8_t *table) {
    ClassPlan p{};
    uint32_t live = 0, n = 0;
    for (uint32_t x = 0; x < 256; x++) live += table[x] != CLS_REJECT;
    p.by_first = live <= kFewLive;
    auto rejects = [&](uint32_t from, uint32_t count) {
        for (uint32_t x = from; x < from + count; x++) if (table[x] != CLS_REJECT) return false;
        return true;
    };
    for (uint32_t x = 0; x < 256; x++)
        if (p.by_first ? table[x] != CLS_REJECT : table[x] >= CLS_EXIT_A) p.ids[n++] = (uint16_t)(x | table[x] << 8);
    p.n_exits = (uint16_t)n;
    if (!p.by_first)
        for (uint32_t k = 0; k < 16; k++) {
            if (rejects(16u * k, 16u)) { p.ids[n++] = (uint16_t)(kBigBlockRow + k); continue; }
            for (uint32_t q = 4u * k; q < 4u * k + 4u; q++) {
                if (rejects(4u * q, 4u)) { p.ids[n++] = (uint16_t)(kBlockRow + q); continue; }
                for (uint32_t x = 4u * q; x < 4u * q + 4u; x++) if (table[x] == CLS_REJECT) p.ids[n++] = (uint16_t)x;
            }
        }
    p.n_ids = (uint16_t)n;                                 // at most 256: a row stands for at least one value
    return p;
}

ClassCodes class_codes_of(const uint8_t *table) {
    ClassCodes c{};
    for (uint32_t x = 0; x < 256u; x++) c.word[x >> 4] |= (uint32_t)table[x] << (2u * (x & 15u));
    return c;
}

ClassPlan wide_plan_of(const uint8_t *table) {
    const ClassPlan p = class_plan_of(table);
    ClassPlan out = p;
    bool big[16] = {};
    uint32_t n = p.n_exits;
    for (uint32_t i = p.n_exits; i < p.n_ids; i++) {
        if (p.ids[i] >= kBigBlockRow) big[p.ids[i] - kBigBlockRow] = true;
        else out.ids[n++] = p.ids[i];
    }
    for (uint32_t k = 0; k < 16; k++) {
        uint32_t size = 8;                                 // the largest aligned block of 16-value rows from k on
        while (size && (!big[k] || k % size || !std::all_of(big + k, big + k + size, [](bool x) { return x; }))) size /= 2;
        if (!size) continue;
        out.ids[n++] = (uint16_t)(size == 1 ? kBigBlockRow + k : wide_row(16u * k, 16u * size));
        k += size - 1;
    }
    out.n_ids = (uint16_t)n;
    for (uint32_t i = n; i < p.n_ids; i++) out.ids[i] = 0;
    return out;
}

namespace {

int build(const uint8_t *host_bytes, const uint64_t *host_offsets, uint32_t V, int32_t eos_id,
          VocabIndex *out, std::string *err) {
    if (!host_offsets || V == 0) { *err = "wg_vocab_create: empty vocabulary"; return WG_ERR_INVALID; }
    if (eos_id >= (int64_t)V) { *err = "wg_vocab_create: eos_id outside the vocabulary"; return WG_ERR_INVALID; }
    uint64_t total = host_offsets[V];
    if (total && !host_bytes) { *err = "wg_vocab_create: host_bytes is null"; return WG_ERR_INVALID; }
    if (total >= 0xFFFFFFFFull) { *err = "wg_vocab_create: more than 4 GiB of token bytes"; return WG_ERR_INVALID; }
    std::vector<uint32_t> off(V + 1);
    uint32_t lmax = 0;
    for (uint32_t t = 0; t <= V; t++) {
        if (t && host_offsets[t] < host_offsets[t - 1])
            { *err = "wg_vocab_create: offsets are not non-decreasing"; return WG_ERR_INVALID; }
        off[t] = (uint32_t)host_offsets[t];
        if (t && off[t] - off[t - 1] > lmax) lmax = off[t] - off[t - 1];
    }
    if (host_offsets[0] != 0) { *err = "wg_vocab_create: offsets must start at 0"; return WG_ERR_INVALID; }
    if (lmax > 248) { *err = "wg_vocab_create: tokens longer than 248 bytes are not supported"; return WG_ERR_INVALID; }
    const uint32_t W = (V + 31u) / 32u, rs = (W + 3u) & ~3u;
    const uint32_t n_chunks = (lmax + 7u) / 8u;
    // Static indexes of the vocabulary (they depend on the token bytes only):
    //  - len8 / chunks: fixed-stride view, 8 bytes per load, for the walks
    //  - first-byte buckets (per token range): the only tokens a literal state can admit
    //  - per-length rows: tokens with 1 <= length <= r, for Waits with a byte budget
    std::vector<uint8_t> len8(V, 0), part(V, 0);
    const uint8_t *const bytes = host_bytes;
    std::vector<uint64_t> chunks((size_t)(n_chunks ? n_chunks : 1) * V, 0);
    std::vector<uint32_t> lit_start(256 * kParts + 1, 0), len_rows((size_t)(lmax + 2) * rs, 0);
    // the token ranges that can split the work of one mask row
    uint32_t part_tok[kParts + 1];
    const uint32_t n_groups = (V + kPartGroup - 1u) / kPartGroup;
    for (uint32_t p = 0; p <= kParts; p++) {
        const uint64_t t0 = ((uint64_t)p * n_groups / kParts) * kPartGroup;
        part_tok[p] = (p == kParts || t0 > V) ? V : (uint32_t)t0;
    }
    for (uint32_t t = 0, p = 0; t < V; t++) {
        while (p + 1 < kParts && t >= part_tok[p + 1]) p++;
        part[t] = (uint8_t)p;
    }
    for (uint32_t t = 0; t < V; t++) {
        uint32_t L = ((int64_t)t == eos_id) ? 0u : off[t + 1] - off[t];
        len8[t] = (uint8_t)L;
        for (uint32_t i = 0; i < L; i++)
            chunks[(size_t)(i / 8u) * V + t] |= (uint64_t)bytes[off[t] + i] << (8u * (i % 8u));
        if (L) {
            lit_start[bytes[off[t]] * kParts + part[t] + 1u]++;
            for (uint32_t r = L; r <= lmax + 1u; r++) len_rows[(size_t)r * rs + (t >> 5)] |= 1u << (t & 31u);
        }
    }
    for (uint32_t y = 0; y < 256 * kParts; y++) lit_start[y + 1] += lit_start[y];
    // Within a bucket the entries are ordered by remaining length, so that the lanes of a
    // wavefront walk remainders of similar length.
    std::vector<ExitEntry> lit_entries(lit_start[256 * kParts] ? lit_start[256 * kParts] : 1);
    {
        // (counting sorts, by length and then by bucket)
        std::vector<uint32_t> by_len(lmax + 2u, 0), order(lit_start[256 * kParts]), at(lit_start.begin(), lit_start.end() - 1);
        for (uint32_t t = 0; t < V; t++) if (len8[t]) by_len[len8[t] + 1u]++;
        for (uint32_t r = 0; r <= lmax; r++) by_len[r + 1u] += by_len[r];
        for (uint32_t t = 0; t < V; t++) if (len8[t]) order[by_len[len8[t]]++] = t;
        for (const uint32_t t : order) {
            const uint32_t L = len8[t];
            ExitEntry e;
            e.tok = t; e.off = 1; e.cls = CLS_EXIT_A;
            e.first = L > 1 ? bytes[off[t] + 1] : 0; e.rem = (uint8_t)(L - 1);
            lit_entries[at[bytes[off[t]] * kParts + part[t]]++] = e;
        }
    }
    // The vocabulary in byte order (the prefix-indexed view of it): a literal state admits the
    // tokens that are prefixes of the bytes still to be written and the tokens that go on
    // after them, and both lie in the range of tokens sharing the literal's first two bytes.
    std::vector<ExitEntry> sorted;
    std::vector<uint32_t> dir0(256 * 257 + 1, 0);
    {
        std::vector<uint32_t> order;
        order.reserve(V);
        for (uint32_t t = 0; t < V; t++) if (len8[t]) order.push_back(t);
        std::sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
            const uint32_t la = len8[a], lb = len8[b];
            const int c = std::memcmp(bytes + off[a], bytes + off[b], la < lb ? la : lb);
            return c != 0 ? c < 0 : la != lb ? la < lb : a < b;
        });
        sorted.resize(order.size() ? order.size() : 1);
        auto range_of = [&](uint32_t t) {
            return (uint32_t)bytes[off[t]] * 257u + (len8[t] > 1 ? 1u + bytes[off[t] + 1] : 0u);
        };
        for (size_t i = 0; i < order.size(); i++) {
            const uint32_t t = order[i];
            ExitEntry e;
            e.tok = t; e.off = 0; e.cls = 0; e.first = len8[t] > 1 ? bytes[off[t] + 1] : 0; e.rem = len8[t];
            sorted[i] = e;
            dir0[range_of(t) + 1u]++;
        }
        for (uint32_t y = 0; y < 256 * 257; y++) dir0[y + 1] += dir0[y];
    }
    // Every byte pair inside a token, grouped by the pair: a checkpoint whose exit byte e leads to
    // a literal byte y can only be left early by tokens in which y follows e.
    std::vector<uint32_t> dirN(65536 + 1, 0);
    for (uint32_t t = 0; t < V; t++)
        for (uint32_t i = 1; i < len8[t]; i++) dirN[((uint32_t)bytes[off[t] + i - 1] << 8 | bytes[off[t] + i]) + 1u]++;
    for (uint32_t y = 0; y < 65536; y++) dirN[y + 1] += dirN[y];
    std::vector<ExitEntry> bigram(dirN[65536] ? dirN[65536] : 1);
    {
        std::vector<uint32_t> at(dirN.begin(), dirN.end() - 1);
        for (uint32_t t = 0; t < V; t++)
            for (uint32_t i = 1; i < len8[t]; i++) {
                ExitEntry e;
                e.tok = t; e.off = (uint8_t)i; e.cls = 0; e.first = bytes[off[t] + i]; e.rem = (uint8_t)(len8[t] - i);
                bigram[at[(uint32_t)bytes[off[t] + i - 1] << 8 | bytes[off[t] + i]]++] = e;
            }
    }
    // The vocabulary by byte value, as rows of the tokens that contain it: what a class table does with 32
    // tokens is then the OR of a few words.
    std::vector<uint32_t> byte_rows((size_t)256 * rs, 0);
    for (uint32_t t = 0; t < V; t++)
        for (uint32_t i = 0; i < len8[t]; i++) byte_rows[(size_t)bytes[off[t] + i] * rs + (t >> 5)] |= 1u << (t & 31u);
    // Blocks of 4 and of 16 byte values: a set of byte values is the OR of the blocks it holds whole
    // and of the single rows of the rest, so that an allow list's complement is a few dozen rows.
    std::vector<uint32_t> block_rows((size_t)80 * rs, 0);
    for (uint32_t x = 0; x < 256; x++)
        for (uint32_t w = 0; w < rs; w++) {
            block_rows[(size_t)(x / 4u) * rs + w] |= byte_rows[(size_t)x * rs + w];
            block_rows[(size_t)(64u + x / 16u) * rs + w] |= byte_rows[(size_t)x * rs + w];
        }
    // The tokens in which a byte value occurs once, as the last byte: the ones that leave a checkpoint
    // with their last byte, when it is an exit byte and none of the others fails to stay.
    std::vector<uint32_t> tail_rows((size_t)256 * rs, 0);
    for (uint32_t t = 0; t < V; t++) {
        const uint32_t L = len8[t];
        if (!L) continue;
        const uint8_t last = bytes[off[t] + L - 1u];
        if (!std::memchr(bytes + off[t], last, L - 1u)) tail_rows[(size_t)last * rs + (t >> 5)] |= 1u << (t & 31u);
    }
    // The pairs again by their first byte and token range: what a checkpoint whose exit byte leads
    // to another checkpoint has to look at, each range's share apart.
    std::vector<uint32_t> place_start(256 * kParts + 1, 0);
    for (uint32_t t = 0; t < V; t++)
        for (uint32_t i = 1; i < len8[t]; i++) place_start[(uint32_t)bytes[off[t] + i - 1] * kParts + part[t] + 1u]++;
    for (uint32_t y = 0; y < 256 * kParts; y++) place_start[y + 1] += place_start[y];
    std::vector<ExitEntry> places(bigram.size());
    {
        std::vector<uint32_t> at(place_start.begin(), place_start.end() - 1);
        for (uint32_t t = 0; t < V; t++) {
            const uint32_t p = part[t];
            for (uint32_t i = 1; i < len8[t]; i++) {
                ExitEntry e;
                e.tok = t; e.off = (uint8_t)i; e.cls = 0; e.first = bytes[off[t] + i]; e.rem = (uint8_t)(len8[t] - i);
                places[at[(uint32_t)bytes[off[t] + i - 1] * kParts + p]++] = e;
            }
        }
    }
    VocabIndex &ix = *out;
    ix.V = V; ix.W = W; ix.row_stride = rs; ix.lmax = lmax; ix.n_chunks = n_chunks;
    for (uint32_t p = 0; p <= kParts; p++) ix.part_tok[p] = part_tok[p];
    ix.len8.swap(len8); ix.chunks.swap(chunks); ix.lit_entries.swap(lit_entries); ix.lit_start.swap(lit_start);
    ix.len_rows.swap(len_rows); ix.sorted.swap(sorted); ix.dir0.swap(dir0); ix.bigram.swap(bigram);
    ix.dirN.swap(dirN); ix.byte_rows.swap(byte_rows);
    ix.block_rows.swap(block_rows); ix.tail_rows.swap(tail_rows); ix.places.swap(places); ix.place_start.swap(place_start);
    return WG_OK;
}

}  // namespace

std::vector<uint32_t> token_rows(const VocabIndex &ix) {
    const size_t rs = ix.row_stride;
    std::vector<uint32_t> rows;
    rows.reserve(kLenRow * rs + ix.len_rows.size());
    for (const auto *r : {&ix.byte_rows, &ix.block_rows, &ix.tail_rows}) rows.insert(rows.end(), r->begin(), r->end());
    rows.resize((size_t)(kWideRow + kWideRows) * rs, 0u);
    for (uint32_t values = 32; values <= 128; values *= 2)
        for (uint32_t k = 0; k < 16; k++) {                // from the rows of 16 byte values
            uint32_t *to = rows.data() + wide_row(16u * k, values) * rs;
            const uint32_t *from = rows.data() + (kBigBlockRow + k) * rs;
            for (size_t w = 0; w < rs; w++) to[w] |= from[w];
        }
    rows.insert(rows.end(), ix.len_rows.begin(), ix.len_rows.end());
    return rows;
}

bool candidates(const VocabIndex &ix, std::vector<ExitEntry> *index, std::vector<uint32_t> *dirs) {
    const std::vector<ExitEntry> *parts[4] = {&ix.sorted, &ix.lit_entries, &ix.bigram, &ix.places};
    const std::vector<uint32_t> *dir[4] = {&ix.dir0, &ix.lit_start, &ix.dirN, &ix.place_start};
    uint64_t n = 0;
    for (const auto *p : parts) n += p->size();
    if (n > 0xFFFFFFFFull) return false;
    index->reserve(n);
    dirs->reserve(kDirWords);
    for (int i = 0; i < 4; i++) {
        const uint32_t at = (uint32_t)index->size();
        for (uint32_t x : *dir[i]) dirs->push_back(at + x);
        index->insert(index->end(), parts[i]->begin(), parts[i]->end());
    }
    return true;
}

int build_vocab_index(const uint8_t *host_bytes, const uint64_t *host_offsets, uint32_t V, int32_t eos_id,
                      VocabIndex *out, std::string *err) {
    try {
        return build(host_bytes, host_offsets, V, eos_id, out, err);
    } catch (const std::bad_alloc &) {
        *err = "wg_vocab_create: out of host memory";
        return WG_ERR_NOMEM;
    }
}

}  // namespace wg
