// cp_context_dedup: multi-turn context de-duplication behind the C ABI of cp_context_dedup.h
// (paper, Section 6 and the appendix algorithm "Context De-duplication").  Plain C++; no GPU call.
//
// Bound by FNV-1a, whose every byte waits for the product of the byte before (an exclusive or and a
// multiplication, 4 cycles).  So the lines of all blocks of a turn are hashed side by side, kLanes at a time, then
// their sub-blocks: a byte takes little more than the cycle its multiplication does.  One after the other, line by
// line and with a copy of the ownership table for every turn, 40 turns of 12 blocks of 200 lines took 8.1 ms on the
// host of an MI355X, with the binding's copies, its count of lines and an object per sub-block; now 2.3.
#include <stdint.h>
#include <string.h>

#include <new>
#include <unordered_set>
#include <vector>

#include "cp_context_dedup.h"

namespace {

constexpr uint64_t kBasis = 0xcbf29ce484222325ull, kPrime = 0x100000001b3ull;

inline uint64_t fnv1a(const uint8_t *p, int64_t len, uint64_t h = kBasis)
{
    for (int64_t i = 0; i < len; ++i) {
        h ^= p[i];
        h *= kPrime;
    }
    return h;
}

struct Piece {
    const uint8_t *text;
    int64_t len;
};

// Hashes of many pieces.  Six chains and their pointers fit the registers, and hide the multiplication.
constexpr int kLanes = 6;
void fnv1a_many(const std::vector<Piece> &pieces, std::vector<uint64_t> &hashes)
{
    const size_t n = pieces.size();
    hashes.resize(n);
    const uint8_t *p[kLanes];
    int64_t left[kLanes];
    uint64_t h[kLanes];
    size_t piece[kLanes], next = 0;
    auto take = [&](int k) { // the next piece that is not empty, false: none is left
        while (next < n && pieces[next].len == 0) hashes[next++] = kBasis;
        if (next == n) return false;
        p[k] = pieces[next].text;
        left[k] = pieces[next].len;
        h[k] = kBasis;
        piece[k] = next++;
        return true;
    };
    int lanes = 0;
    while (lanes < kLanes && take(lanes)) ++lanes;
    while (lanes == kLanes) {
        int64_t m = left[0];
        for (int k = 1; k < kLanes; ++k) m = left[k] < m ? left[k] : m;
        {
            const uint8_t *const p0 = p[0], *const p1 = p[1], *const p2 = p[2], *const p3 = p[3], *const p4 = p[4], *const p5 = p[5];
            uint64_t h0 = h[0], h1 = h[1], h2 = h[2], h3 = h[3], h4 = h[4], h5 = h[5];
            for (int64_t i = 0; i < m; ++i) {
                h0 = (h0 ^ p0[i]) * kPrime;
                h1 = (h1 ^ p1[i]) * kPrime;
                h2 = (h2 ^ p2[i]) * kPrime;
                h3 = (h3 ^ p3[i]) * kPrime;
                h4 = (h4 ^ p4[i]) * kPrime;
                h5 = (h5 ^ p5[i]) * kPrime;
            }
            h[0] = h0;
            h[1] = h1;
            h[2] = h2;
            h[3] = h3;
            h[4] = h4;
            h[5] = h5;
        }
        bool out = false;
        for (int k = 0; k < kLanes; ++k) {
            p[k] += m;
            left[k] -= m;
            if (left[k] > 0) continue;
            hashes[piece[k]] = h[k];
            out = !take(k) || out;
        }
        if (out) break;
    }
    for (int k = 0; k < lanes; ++k) // the last ones, one by one
        if (left[k] > 0) hashes[piece[k]] = fnv1a(p[k], left[k], h[k]);
}
static_assert(kLanes == 6, "the loop above is written out");

// The lines of bytes[0, len), without their newlines.
void add_lines(const uint8_t *bytes, int64_t len, std::vector<Piece> &lines)
{
    for (int64_t at = 0; at < len;) {
        const void *newline = memchr(bytes + at, '\n', (size_t)(len - at));
        const int64_t stop = newline ? static_cast<const uint8_t *>(newline) - bytes : len;
        lines.push_back(Piece{bytes + at, stop - at});
        at = stop + 1;
    }
}

// End offsets of the sub-blocks of bytes[0, len): after every line whose hash is 0 modulo
// `modulus`, and at the end.  `lines` and `hashes` from `line` on are the block's; returns the line behind them.
size_t add_ends(int64_t len, uint64_t modulus, const std::vector<Piece> &lines, const std::vector<uint64_t> &hashes,
                size_t line, std::vector<int64_t> &ends)
{
    const bool power = (modulus & (modulus - 1)) == 0;
    int64_t sub_start = 0;
    for (int64_t at = 0; at < len; ++line) {
        at += lines[line].len + 1; // a last line without a newline is tested like any other
        if ((power ? hashes[line] & (modulus - 1) : hashes[line] % modulus) != 0) continue;
        sub_start = at < len ? at : len;
        ends.push_back(sub_start);
    }
    if (sub_start < len) ends.push_back(len); // what is left over ends the block
    return line;
}

// Which block brought a sub-block's content first, by its hash: open addressing, never more than half full.
class Owners {
public:
    // Room for `more` further hashes, so that claim() cannot fail.
    void reserve(size_t more)
    {
        size_t size = slots_.empty() ? 64 : slots_.size();
        while (size < 2 * (used_ + more)) size *= 2;
        if (size == slots_.size()) return;
        std::vector<Slot> old(size);
        old.swap(slots_);
        for (const Slot &s : old)
            if (s.taken) slots_[find(s.hash)] = s;
    }
    int32_t claim(uint64_t hash, int32_t block)
    {
        Slot &s = slots_[find(hash)];
        if (!s.taken) {
            s = Slot{hash, block, true};
            ++used_;
        }
        return s.block;
    }

private:
    struct Slot {
        uint64_t hash = 0;
        int32_t block = 0;
        bool taken = false;
    };
    size_t find(uint64_t hash) const
    {
        const size_t mask = slots_.size() - 1;
        size_t at = (size_t)(hash ^ (hash >> 32)) & mask;
        while (slots_[at].taken && slots_[at].hash != hash) at = (at + 1) & mask;
        return at;
    }
    std::vector<Slot> slots_;
    size_t used_ = 0;
};

} // namespace

// State of one conversation: which blocks earlier turns brought, and for every sub-block content
// (by hash) the block that brought it first.
struct cp_dedup {
    uint64_t modulus = 1;
    std::unordered_set<int32_t> earlier_turn_blocks;
    Owners owners;
};

extern "C" uint64_t cp_dedup_hash(const uint8_t *bytes, int64_t len)
{
    return (bytes && len > 0) ? fnv1a(bytes, len) : kBasis;
}

extern "C" int cp_dedup_chunks(const uint8_t *bytes, int64_t len, uint64_t modulus, int64_t *ends, int32_t cap,
                               int32_t *count)
{
    if (!count || (len > 0 && !bytes)) return -1;
    if (len < 0 || modulus < 1 || cap < 0) return -2;
    std::vector<Piece> lines;
    std::vector<uint64_t> hashes;
    std::vector<int64_t> e;
    add_lines(bytes, len, lines);
    fnv1a_many(lines, hashes);
    add_ends(len, modulus, lines, hashes, 0, e);
    *count = (int32_t)e.size();
    if ((int32_t)e.size() > cap) return -2;
    if (!e.empty() && !ends) return -1;
    for (size_t i = 0; i < e.size(); ++i) ends[i] = e[i];
    return 0;
}

extern "C" int cp_dedup_create(uint64_t modulus, cp_dedup **out)
{
    if (!out) return -1;
    *out = nullptr;
    if (modulus < 1) return -2;
    cp_dedup *c = new (std::nothrow) cp_dedup();
    if (!c) return -2;
    c->modulus = modulus;
    *out = c;
    return 0;
}

extern "C" void cp_dedup_free(cp_dedup *conv) { delete conv; }

extern "C" int cp_dedup_turn(cp_dedup *conv, const int32_t *ids, const uint8_t *bytes, const int64_t *offsets,
                             int32_t n, int32_t *block_ref, cp_dedup_sub *subs, int32_t subs_cap,
                             int32_t *subs_count, int64_t *kept_bytes)
{
    if (!conv || !subs_count) return -1;
    if (n < 0 || subs_cap < 0) return -2;
    if (n > 0 && (!ids || !offsets || !block_ref)) return -1;
    for (int32_t i = 0; i < n; ++i)
        if (offsets[i] < 0 || offsets[i + 1] < offsets[i]) return -2;
    if (n > 0 && offsets[n] > 0 && !bytes) return -1;

    // Pass over whole blocks: a block that an earlier turn of the conversation brought is
    // answered by a reference and not looked into.
    std::vector<int32_t> to_cut;
    std::vector<Piece> lines;
    for (int32_t i = 0; i < n; ++i) {
        block_ref[i] = conv->earlier_turn_blocks.count(ids[i]) ? 1 : 0;
        if (block_ref[i]) continue;
        to_cut.push_back(i);
        add_lines(bytes + offsets[i], offsets[i + 1] - offsets[i], lines);
    }
    // The sub-blocks of the others, in order.
    std::vector<uint64_t> hashes;
    fnv1a_many(lines, hashes);
    std::vector<Piece> pieces;
    std::vector<cp_dedup_sub> out;
    std::vector<int64_t> ends;
    size_t line = 0;
    for (int32_t i : to_cut) {
        const uint8_t *text = bytes + offsets[i];
        ends.clear();
        line = add_ends(offsets[i + 1] - offsets[i], conv->modulus, lines, hashes, line, ends);
        int64_t begin = 0;
        for (int64_t end : ends) {
            out.push_back(cp_dedup_sub{i, -1, begin, end});
            pieces.push_back(Piece{text + begin, end - begin});
            begin = end;
        }
    }
    // Nothing is recorded before it is known that the output fits.
    *subs_count = (int32_t)out.size();
    if ((int32_t)out.size() > subs_cap) return -2;
    if (!out.empty() && !subs) return -1;
    fnv1a_many(pieces, hashes);
    conv->owners.reserve(out.size());
    // Content that a different block owns becomes a reference to that block, anything else is kept and owned from
    // now on.
    int64_t kept = 0;
    for (size_t k = 0; k < out.size(); ++k) {
        const int32_t id = ids[out[k].block];
        const int32_t owner = conv->owners.claim(hashes[k], id); // this block itself when the content is new
        subs[k] = out[k];
        if (owner == id) kept += out[k].end - out[k].begin;
        else subs[k].ref = owner;
    }
    conv->earlier_turn_blocks.insert(ids, ids + n);
    if (kept_bytes) *kept_bytes = kept;
    return 0;
}
