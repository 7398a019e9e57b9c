// Tables of the q-gram filter (host only).
//
// Wu-Manber's SHIFT and HASH (Section 3.2) look at one block per window and
// move on by a data-dependent shift; each lane's windows form a serial chain.
// Here the blocks that are looked at are the same for every text: the q-grams
// at multiples of t. A gram that occurs in no string at an offset below t
// rules out the t starting positions that end at it, so most text is read
// once and answered by one bit of an LDS table per t bytes, all of them
// independent. The grams that remain carry their (string, offset) pairs with
// the codes of the string's first 16 characters, as Wu-Manber's HASH and
// PREFIX do, and whatever passes those is compared byte by byte.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "mpm_internal.h"

namespace mpm {

namespace {

const uint32_t Q_MAX = 10;        // 4^10 bits = 128 KiB of the 160 KiB LDS
const uint32_t CHAIN_MAX = 64;    // entries of one gram
const uint32_t NONE = 0xffffffffu;

uint32_t gram_of(const uint8_t *p, uint32_t k, uint32_t sh)
{
    uint32_t h = 0;
    for (uint32_t j = 0; j < k; j++)
        h |= ((p[j] >> sh) & 3u) << (2 * j);
    return h;
}

template <typename T>
uint64_t append(std::vector<uint8_t> &img, const T *src, uint64_t count)
{
    const uint64_t off = (img.size() + 255) / 256 * 256;
    img.resize((off + count * sizeof(T) + 15) / 16 * 16, 0);
    if (count)
        memcpy(img.data() + off, src, count * sizeof(T));
    return off;
}

// The shift whose codes (b >> shift) & 3 two random pattern characters share
// least often (frequent bytes get codes of their own); freq receives the byte
// counts, share the codes' shares.
uint32_t code_shift_of(const std::vector<uint8_t> &bytes, double *freq, double *share)
{
    uint32_t n[4][256];  // four counters of a byte: neighbours do not wait for each other
    memset(n, 0, sizeof n);
    size_t i = 0;
    for (; i + 4 <= bytes.size(); i += 4)
        for (int k = 0; k < 4; k++)
            n[k][bytes[i + k]]++;
    for (; i < bytes.size(); i++)
        n[0][bytes[i]]++;
    for (uint32_t b = 0; b < 256; b++)
        freq[b] = (double)n[0][b] + n[1][b] + n[2][b] + n[3][b];
    uint32_t sh = 0;
    double best = 1e300;
    for (uint32_t s = 0; s < 7; s++) {
        double mass[4] = {0, 0, 0, 0}, c = 0;
        for (uint32_t b = 0; b < 256; b++)
            mass[(b >> s) & 3u] += freq[b];
        for (double x : mass)
            c += x * x;
        if (c < best * (1 - 1e-12)) {
            best = c;
            sh = s;
            for (int k = 0; share && k < 4; k++)
                share[k] = mass[k] / (double)bytes.size();
        }
    }
    return sh;
}

// The most frequent byte of each code (a byte of another code where none has
// it), and whether a byte is one of them.
void main_bytes(const double *freq, uint32_t sh, uint8_t *main4, bool *is_main)
{
    std::fill(is_main, is_main + 256, false);
    for (uint32_t k = 0; k < 4; k++) {
        int best = -1;
        for (uint32_t b = 0; b < 256; b++)
            if (((b >> sh) & 3u) == k && freq[b] > 0 && (best < 0 || freq[b] > freq[best]))
                best = (int)b;
        main4[k] = best < 0 ? (uint8_t)(((k + 1) & 3u) << sh) : (uint8_t)best;
        if (best >= 0)
            is_main[best] = true;
    }
}

struct Strings {
    const mpm_index *ix;
    const uint8_t *at(uint32_t u) const
    {
        return ix->upats.data() + (ix->var ? ix->upoff[u] : (uint64_t)u * ix->m);
    }
    uint32_t len(uint32_t u) const { return ix->var ? ix->upoff[u + 1] - ix->upoff[u] : ix->m; }
};

// Codes of the first t + q - 1 <= 25 characters of every string.
std::vector<uint64_t> head_codes(const mpm_index *ix, const Strings &S, uint32_t sh)
{
    std::vector<uint64_t> h(ix->du);
    for (uint32_t u = 0; u < ix->du; u++) {
        const uint8_t *p = S.at(u);
        const uint32_t k = std::min<uint32_t>(S.len(u), 25);
        uint64_t x = 0;
        for (uint32_t j = 0; j < k; j++)
            x |= (uint64_t)((p[j] >> sh) & 3u) << (2 * j);
        h[u] = x;
    }
    return h;
}

// Expected candidates and chain steps per text byte when text characters
// follow the code shares of the strings' characters.
struct Rate {
    double cand, steps;
    uint32_t longest;
};

Rate rate_of(const std::vector<uint64_t> &head, uint32_t q, uint32_t t, const double *share,
             std::vector<uint8_t> &count)
{
    // the share of a gram: a product of two table entries
    const uint32_t q1 = std::min<uint32_t>(q, 5), q2 = q - q1;
    std::vector<double> lo(1u << (2 * q1)), hi(1u << (2 * q2));
    for (size_t k = 0; k < 2; k++) {
        std::vector<double> &v = k ? hi : lo;
        const uint32_t len = k ? q2 : q1;
        for (uint32_t g = 0; g < v.size(); g++) {
            v[g] = 1;
            for (uint32_t j = 0; j < len; j++)
                v[g] *= share[(g >> (2 * j)) & 3u];
        }
    }
    count.assign(1ull << (2 * q), 0);
    Rate r = {0, 0, 0};
    const uint32_t mask = (1u << (2 * q)) - 1u, m1 = (uint32_t)lo.size() - 1;
    for (uint64_t h : head)
        for (uint32_t off = 0; off < t; off++) {
            const uint32_t g = (uint32_t)(h >> (2 * off)) & mask;
            const double pr = lo[g & m1] * hi[g >> (2 * q1)];
            r.steps += pr;
            if (count[g] == 0)
                r.cand += pr;
            if (count[g] < 255)
                count[g]++;
            r.longest = std::max<uint32_t>(r.longest, count[g]);
        }
    r.cand /= t;
    r.steps /= t;
    return r;
}

// Cost per text byte in vector instructions of a lane: packing, lookups
// (about six each) and batches of 64 candidates (about 120 each, plus their
// chain steps); a 128 KiB table halves the waves of a CU.
double cost_of(uint32_t q, uint32_t t, double cand, double steps)
{
    return (1.2 + 6.0 / t + 120.0 * cand + 20.0 * steps) * (q == Q_MAX ? 1.25 : 1.0);
}

// What a candidate costs more when the entries (16 bytes for each string and
// offset) outgrow the 4 MB L2 of an XCD, which they share with the text:
// 64 MiB, d = 100k, m = 32, q = 10, entries of 1.6, 3.2, 6.4, 12.8, 25.6 MB
// (t = 1 to 16): 97, 95, 105, 120, 132 us, for 0.091 to 0.049 candidates per
// byte.
double spread_of(uint32_t t, uint32_t du) { return pow(std::max(1.0, 16.0 * t * du / 3.4e6), 0.63); }

}  // namespace

// Choose q and t, and append the tables to the index's device image; leaves
// gram.ok = 0 when the set has no useful filter.
void build_gram(mpm_index *ix)
{
    mpm_index::Gram &G = ix->gram;
    const uint32_t m = ix->m;
    if (m < 4 || ix->du == 0 || ix->du >= (1u << 27))
        return;
    const Strings S = {ix};
    double freq[256], share[4];
    const uint32_t sh = code_shift_of(ix->upats, freq, share);
    // The cheapest (t, q), by the cost if grams were spread evenly; the first
    // few are then counted. (The spread of the entries decides between them
    // alone: the limits on the cost stand for what a candidate costs in L2.)
    struct Choice {
        double cost, plain;  // with and without the spread
        uint32_t tl, q;
    };
    std::vector<Choice> all;
    for (uint32_t tl = 0; tl <= 4; tl++) {
        const uint32_t t = 1u << tl;
        for (uint32_t q = 4; q <= Q_MAX && q + t - 1 <= m; q++) {
            const double even = (double)ix->du / (double)(1ull << (2 * q));
            const double cand = (1.0 - exp(-even * t)) / t;
            all.push_back({cost_of(q, t, cand * spread_of(t, ix->du), even), cost_of(q, t, cand, even), tl, q});
        }
    }
    std::stable_sort(all.begin(), all.end(), [](const Choice &x, const Choice &y) { return x.cost < y.cost; });
    const std::vector<uint64_t> head = head_codes(ix, S, sh);
    std::vector<uint8_t> count;
    double best = 1e300, chosen = 1e300;
    Rate rate = {0, 0, 0};
    uint32_t bq = 0, bt = 0;
    for (size_t k = 0; k < all.size() && k < 4 && (all[k].cost < 0.9 * chosen || best > 25.0); k++) {
        if (all[k].plain >= 25.0)
            continue;
        const uint32_t tk = 1u << all[k].tl;
        const Rate r = rate_of(head, all[k].q, tk, share, count);
        if (r.longest > CHAIN_MAX)
            continue;
        best = std::min(best, cost_of(all[k].q, tk, r.cand, r.steps));
        const double c = cost_of(all[k].q, tk, r.cand * spread_of(tk, ix->du), r.steps);
        if (c < chosen) {
            chosen = c;
            rate = r;
            bq = all[k].q;
            bt = all[k].tl;
        }
    }
    // Past about 25 the candidates' batches cost more than the walkers' chains:
    // 64 MiB of text, m = 10, d = 100k (cost 24.9) 436 us against 593 us for
    // the better walker; m = 8, d = 10k (27.0) 900 us against 397 us.
    if (best > 25.0)
        return;
    const uint32_t q = bq, t = 1u << bt;
    // Entries: the first one of each gram at the gram's number (grams in
    // order of word, then bit), the others behind them. Offsets descend so
    // that a chain's starting positions ascend; longer strings first.
    const uint32_t wb = 2 * q - 5, nw = 1u << wb, gmask = (1u << (2 * q)) - 1u;
    std::vector<uint32_t> order(ix->du);
    for (uint32_t u = 0; u < ix->du; u++)
        order[u] = u;
    if (ix->var)
        std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return S.len(a) > S.len(b); });
    std::vector<uint32_t> bits(nw, 0);
    for (uint32_t u = 0; u < ix->du; u++) {
        uint64_t h = head[u];
        for (uint32_t off = 0; off < t; off++, h >>= 2)
            bits[h & (nw - 1)] |= 1u << ((uint32_t)(h >> wb) & 31u);
    }
    std::vector<uint2> words(nw);
    uint32_t ngrams = 0;
    for (uint32_t w = 0; w < nw; w++) {
        words[w] = make_uint2(bits[w], ngrams);
        ngrams += (uint32_t)__builtin_popcount(bits[w]);
    }
    uint8_t main4[4];
    bool is_main[256];
    main_bytes(freq, sh, main4, is_main);
    std::vector<uint8_t> plain(ix->du);
    for (uint32_t u = 0; u < ix->du; u++)
        plain[u] = !ix->var && m <= 16 && std::all_of(S.at(u), S.at(u) + m, [&](uint8_t c) { return is_main[c]; });
    std::vector<GramEnt> ents;
    ents.reserve((uint64_t)ix->du * t);
    ents.resize(ngrams, GramEnt{0, 0, 0, NONE});
    std::vector<uint32_t> tail(ngrams, NONE);
    for (uint32_t k = 0; k < t; k++) {
        const uint32_t off = t - 1 - k;
        for (uint32_t u : order) {
            const uint64_t h = head[u] >> (2 * off);
            const uint2 w = words[h & (nw - 1)];
            const uint32_t g = w.y + (uint32_t)__builtin_popcount(w.x & ((1u << ((h >> wb) & 31u)) - 1u));
            const uint32_t kl = std::min<uint32_t>(16, S.len(u));
            GramEnt e;
            e.key = (uint32_t)head[u];
            e.mask = kl == 16 ? NONE : (1u << (2 * kl)) - 1u;
            e.meta = u << 5 | (uint32_t)plain[u] << 4 | off;
            e.next = NONE;
            if (tail[g] == NONE) {
                ents[g] = e;
                tail[g] = g;
            } else {
                ents[tail[g]].next = (uint32_t)ents.size();
                tail[g] = (uint32_t)ents.size();
                ents.push_back(e);
            }
        }
    }
    std::vector<uint2> strs(ix->du);
    uint64_t nrows = 0;
    for (uint32_t u = 0; u < ix->du; u++) {
        strs[u] = make_uint2((uint32_t)nrows, S.len(u));
        nrows += (S.len(u) + 15) / 16;
    }
    std::vector<uint8_t> rows(16 * nrows, 0);
    for (uint32_t u = 0; u < ix->du; u++)
        memcpy(rows.data() + 16ull * strs[u].x, S.at(u), S.len(u));
    ix->image.reserve(ix->image.size() + 4ull * (2 * bits.size() + 4 * ents.size() + 2 * strs.size()) +
                      rows.size() + 2048);
    G.q = q;
    G.cost = best;
    G.hit = 1e-9;
    double share5[1024];  // of five codes
    for (uint32_t g = 0; g < 1024; g++) {
        share5[g] = 1;
        for (uint32_t j = 0; j < 5; j++)
            share5[g] *= share[(g >> (2 * j)) & 3u];
    }
    for (uint32_t u = 0; u < ix->du; u++) {
        const uint32_t k = std::min<uint32_t>(S.len(u), 25);
        double pr = 1;
        uint32_t j = 0;
        for (; j + 5 <= k; j += 5)
            pr *= share5[(head[u] >> (2 * j)) & 1023u];
        for (; j < k; j++)
            pr *= share[(head[u] >> (2 * j)) & 3u];
        G.hit += pr;
    }
    G.t_log = bt;
    G.code_shift = sh;
    memcpy(&G.main4, main4, 4);
    G.bit_bytes = nw * 4;
    // Behind the bits the grams before each word. Where they fit beside the bits
    // in LDS they are copied too: a candidate then finds its entry without a load
    // (256 MiB, d = 1000, m = 16: 68.3 -> 63.2 us; 128 MiB, lengths 8-32:
    // 69.8 -> 67.0).
    G.ranked = q <= 9;
    for (uint32_t w = 0; w < nw; w++)
        bits.push_back(words[w].y);
    // With every position a sample (t = 1) the answers for two positions are
    // read at once, two bits at the code of the q + 1 characters that both
    // span (128 MiB, lengths 8-32: 66.2 -> 62.9 us; 64 MiB, d = 1000, m = 8 with
    // counts 75.0 -> 72.5): 64 KiB at q = 8, which leaves the occurrence lists
    // enough where occurrences are few.
    if (G.ranked && bt == 0 && q <= 8 && G.hit <= 0.02) {
        const uint32_t pw = 2 * q - 2;
        std::vector<uint32_t> pairs(1u << pw, 0);
        auto set = [&](uint32_t z, uint32_t k) { pairs[z & ((1u << pw) - 1u)] |= 1u << (2 * (z >> pw) + k); };
        for (uint32_t u = 0; u < ix->du; u++)
            for (uint32_t c = 0; c < 4; c++) {
                const uint32_t g = (uint32_t)head[u] & gmask;
                set(g | c << (2 * q), 0);
                set(g << 2 | c, 1);
            }
        bits.insert(bits.end(), pairs.begin(), pairs.end());
        G.pair_bytes = (uint32_t)(4 * pairs.size());
    }
    G.off_bits = append(ix->image, bits.data(), bits.size());
    G.off_ents = append(ix->image, ents.data(), ents.size());
    G.off_strs = append(ix->image, strs.data(), strs.size());
    G.off_rows = append(ix->image, rows.data(), rows.size());
    if (ix->algo == MPM_ALGO_AC && std::max(m, ix->m_max) < (1u << 20)) {  // (32-bit places in a lane's walk)
        GramWalk w;
        memset(&w, 0, sizeof w);
        w.self = (ix->image.size() + 255) / 256 * 256;
        w.dfa = ix->off_a;
        w.cls = ix->off_b;
        w.term = ix->var ? ix->off_e : 0;
        w.rowb = (ix->n_classes + 1) * ix->state_bytes;
        w.first_term = (uint32_t)(ix->var ? ix->first_term : ix->n_states - ix->du);
        w.wide = ix->state_bytes == 4;
        w.past = (ix->var ? ix->m_max : m) - 1;
        G.off_walk = append(ix->image, &w, 1);
        // Where runs and repeats fill a block, nearly all its samples are
        // candidates. Below three in five the candidates stay cheaper (32 MiB,
        // us by the candidates, by the walk of a block, by the walkers: records
        // with poly-A tails, m = 12, A^12 in the set 115, 255, 424; one string
        // of the set over and over 38, 125, 149), unless many strings share the
        // gram (lengths 8-32, 50 strings of one head of nine A, such records:
        // 220, 152, 108): then past twice the candidates that a block should
        // have, and one batch. Wu-Manber indexes have no automaton, and their
        // own walk takes as long on such texts.
        G.crowd = (uint32_t)(64 + 2 * 4096 * rate.cand);
        if (rate.longest <= 4 * t)
            G.crowd = std::max(G.crowd, 2457 / t);
    }
    ix->image.resize((ix->image.size() + 255) / 256 * 256, 0);
    G.ok = 1;
}

// The direct-address tables of a set with 2 <= m <= 8 (after build_gram);
// leaves direct.ok = 0 when the set does not fit them or its filter is the
// better scan.
void build_direct(mpm_index *ix)
{
    mpm_index::Direct &D = ix->direct;
    const uint32_t m = ix->m;
    if (ix->var || m < 2 || m > 8 || ix->du == 0 || ix->uids.size() >= (1u << 24))
        return;
    // The scan costs the same whatever the candidates; past a filter cost of
    // about 18 it is the faster one (64 MiB, m = 8: d = 5000, cost 16.7, filter
    // 155 us, direct 186; d = 6000, 18.4, 201 and 189). Below it no scan would
    // read the table (d = 100, m = 8: 130 us of the build and 66 KB of the
    // image).
    if (ix->gram.ok && ix->gram.cost <= 18.0)
        return;
    const uint32_t H = 1u << (2 * m);
    double freq[256];
    const uint32_t sh = code_shift_of(ix->upats, freq, nullptr);
    uint8_t main4[4];
    bool is_main[256];
    main_bytes(freq, sh, main4, is_main);
    std::vector<uint32_t> string_of(H, NONE), odd;
    for (uint32_t u = 0; u < ix->du; u++) {
        const uint8_t *p = ix->upats.data() + (uint64_t)u * m;
        bool all = true;
        for (uint32_t j = 0; j < m; j++)
            all &= is_main[p[j]];
        if (!all)
            odd.push_back(u);
        else if (ix->uoff[u + 1] - ix->uoff[u] > 15)  // counts have four bits
            return;
        else
            string_of[gram_of(p, m, sh)] = u;
    }
    if (odd.size() * 10 > ix->du)  // most windows would be compared byte by byte
        return;
    const uint32_t nw = std::max<uint32_t>(4, H / 8);
    std::vector<uint32_t> table(2 * nw, 0), ids;
    ids.reserve(ix->uids.size());
    auto take = [&](uint32_t u) {
        ids.insert(ids.end(), ix->uids.begin() + ix->uoff[u], ix->uids.begin() + ix->uoff[u + 1]);
        return ix->uoff[u + 1] - ix->uoff[u];
    };
    for (uint32_t c = 0; c < H; c++) {
        if ((c & 7) == 0)
            table[nw + (c >> 3)] = (uint32_t)ids.size();
        if (string_of[c] != NONE)
            table[c >> 3] |= take(string_of[c]) << (4 * (c & 7));
    }
    D.code_shift = sh;
    memcpy(&D.main4, main4, 4);
    D.table_bytes = nw * 4;
    if (!odd.empty()) {
        std::vector<uint32_t> bits(std::max<uint32_t>(4, H / 32), 0);
        for (uint32_t u : odd) {
            const uint32_t c = gram_of(ix->upats.data() + (uint64_t)u * m, m, sh);
            bits[c >> 5] |= 1u << (c & 31);
        }
        std::vector<uint2> words(bits.size());
        uint32_t n = 0;
        for (size_t w = 0; w < bits.size(); w++) {
            words[w] = make_uint2(bits[w], n);
            n += (uint32_t)__builtin_popcount(bits[w]);
        }
        std::vector<OddEnt> ents(n, OddEnt{0, 0, 0, NONE, 0});
        std::vector<uint32_t> tail(n, NONE);
        for (uint32_t u : odd) {
            const uint8_t *p = ix->upats.data() + (uint64_t)u * m;
            const uint32_t c = gram_of(p, m, sh);
            const uint32_t k = words[c >> 5].y + (uint32_t)__builtin_popcount(bits[c >> 5] & ((1u << (c & 31)) - 1u));
            OddEnt e = {0, (uint32_t)ids.size(), 0, NONE, 0};
            e.count = take(u);
            memcpy(&e.bytes, p, m);
            if (tail[k] == NONE) {
                ents[k] = e;
                tail[k] = k;
            } else {
                ents[tail[k]].next = (uint32_t)ents.size();
                tail[k] = (uint32_t)ents.size();
                ents.push_back(e);
            }
        }
        D.odd_bytes = (uint32_t)bits.size() * 4;
        D.off_bits = append(ix->image, bits.data(), bits.size());
        D.off_words = append(ix->image, words.data(), words.size());
        D.off_ents = append(ix->image, ents.data(), ents.size());
    }
    D.off_table = append(ix->image, table.data(), table.size());
    D.off_ids = append(ix->image, ids.data(), ids.size());
    ix->image.resize((ix->image.size() + 255) / 256 * 256, 0);
    D.ok = 1;
}

}  // namespace mpm
