// q-gram filter scan: the kernel behind automatic placement for sets whose
// strings rule out most of a text by a few characters.
//
// The walkers of mpm_scan_impl.h advance one dependent table lookup per byte
// (Aho-Corasick) or per window (Wu-Manber), and a wave waits for its slowest
// lane. Here every lookup is at a position known beforehand (mpm_gram.cpp),
// so a lane's lookups are independent of each other:
//
//   1. A wave takes 4 KiB of text, 64 contiguous bytes per lane (four 16-byte
//      loads back to back, the next block's in flight), and packs them to
//      2-bit codes: four registers per lane. (128 bytes per lane measured 10 %
//      slower, 24 waves per CU instead of 16 as well.)
//   2. One LDS bit per sample (every t-th position) tells whether the q-gram
//      there occurs in a string at an offset below t: a shift, a mask, a
//      ds_read, two shifts, one v_alignbit to collect the bit. (t = 1: two
//      bits for two samples, where their table fits.)
//   3. The block's candidates, in text order, are dealt to the lanes 128 at a
//      time; each walks its gram's chain of (string, offset) entries and
//      compares the codes of the string's first 16 characters.
//   4. What remains is compared byte by byte, with bytes made from the codes
//      where those tell them, else with the string's row; occurrences go to a
//      list in LDS in text order (ballots keep the order).
//   5. Per chunk: wave counts -> workgroup offsets -> decoupled look-back, as
//      the walkers do, then the wave writes its pairs 64 at a time. A wave
//      whose list overflows runs its part again and writes as it goes.
//
// Steps 1 and 2 cost about 1 + 6 / t vector instructions per byte of a lane,
// step 3 about 120 per 64 candidates: for 1,000 strings of 16 characters
// (t = 8, q = 9, one candidate per 260 bytes) that is below what HBM asks for.
//
// Measured (EST-shaped text, walkers before, filter after, us): 256 MiB,
// d = 1000, m = 16: AC 102 -> 62.5, WM 99 -> 62.5 (4.3 TB/s of text; while all
// waves stream, 6.3 TB/s: the rest is the start and the wait for the slowest
// wave); 128 MiB, d = 10k, m = 16, AC 366 -> 49; 64 MiB, d = 100k, m = 16, WM
// 3554 -> 74; 64 MiB, d = 1000, m = 8 with counts, WM 421 -> 72; 128 MiB,
// lengths 8-32, AC 134 -> 62; 32 MiB, lengths 8-32, WM 2110 -> 26.
#include "mpm_gram.h"

#include <cmath>
#include <functional>
#include <queue>

namespace mpm {

namespace {

constexpr uint32_t GBITS_OFF = LDS_CLS_OFF;         // filter bits, after the header
constexpr uint32_t BIAS = 16;                       // items hold start + BIAS

// One wave's LDS: code words ([3] the 16 characters before the block, from
// [4] on the block, then the 16 after it), 64 items (first a batch's
// candidates, then its strings to compare), and the occurrence list.
constexpr int GN = 4;                               // 16-byte pieces per lane and block
constexpr uint32_t GBLOCK = 1024 * GN;              // text bytes per wave and step
static_assert(256 / 64 * GBLOCK >= GRAM_CHUNK_MIN, "workspace bound");
constexpr uint32_t WV_ITEMS = (64 * GN + 8) * 4;
constexpr uint32_t WV_HITS = WV_ITEMS + 64 * 8;

// LDS bytes of one wave's buffers in a batched launch of lds_bytes per
// workgroup, beside an index's bits.
__host__ __device__ constexpr uint32_t batch_wave_bytes(uint32_t lds_bytes, uint32_t bit_bytes)
{
    return (lds_bytes - GBITS_OFF - bit_bytes) / 16 & ~15u;
}

// Write the pairs of up to 64 occurrences (one per active lane, in lane
// order) from output slot o on; o moves past them.
__device__ __forceinline__ void write_hits(mpm_match *out_, uint64_t cap, uint64_t &o, bool active,
                                           uint32_t pos, uint32_t u, const IdMap &im)
{
    GLB_AS v2u *out = (GLB_AS v2u *)out_;
    uint32_t b = 0, e = 0;
    if (active)
        im.span(u, b, e);
    uint32_t total;
    const uint32_t pre = wave_excl_sum(e - b, total);
    uint64_t q = o + pre;
    for (uint32_t j = b; j < e && q < cap; ++j, ++q)
        out[q] = v2u{pos, im.id(j)};
    o += total;
}

// A descriptor at a uniform address that no launch writes, by scalar loads.
template <class T>
__device__ __forceinline__ T uniform_load(const T *p)
{
    typedef const __attribute__((address_space(4))) uint32_t *words;
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (uint32_t k = 0; k < sizeof(T) / 4; ++k)
        w[k] = ((words)(uintptr_t)p)[k];
    T t;
    __builtin_memcpy(&t, w, sizeof t);
    return t;
}

// One wave's blocks [b0, b1). direct = false: count, keep the first `hcap`
// occurrences in LDS; nh and nid (ids, summed over lanes) come back. direct =
// true: write every pair from slot o on.
template <int TL, bool Var, bool Pair = false>
struct GramScan {
    static constexpr uint32_t T = 1u << TL;
    static constexpr uint32_t NS = (16u * GN) >> TL;  // samples per lane and block
    static constexpr uint32_t NM = (NS + 31) / 32;          // words of sample bits
    GramDev a;
    View text;
    IdMap im;
    uint32_t wv;    // LDS offset of this wave's buffers
    uint32_t hcap;
    uint32_t amask, bsh, wmask, pmask;

    __device__ __forceinline__ void bind(const GramDev &dev, const uint8_t *t, uint64_t n)
    {
        a = dev;
        text.lo = (uint32_t)((uintptr_t)t & 15u);
        text.p = (glb_cptr<uint8_t>)(t - text.lo);
        text.hi = n + text.lo;
        im.uoff = (glb_cptr<uint32_t>)a.uoff;
        im.uids = (glb_cptr<uint32_t>)a.uids;
        im.lds_uoff = 0;
        im.lds_uids = 0;
        im.dupfree = 0;
        im.n_single = a.n_single;
        wmask = (1u << (2 * a.q - 5)) - 1u;
        amask = wmask << 2;
        bsh = 2 * a.q - 3;
        pmask = ((1u << (2 * a.q - 2)) - 1u) << 2;
    }

    // Whether the len >= 4 bytes at view position s are string (row, len):
    // whole 16-, 8- or 4-byte pieces, the last one ending with the string.
    __device__ __forceinline__ bool equal(uint64_t s, uint32_t row, uint32_t len) const
    {
        glb_cptr<uint8_t> t = text.p + s, q = (glb_cptr<uint8_t>)a.rows + (uint64_t)row * 16;
        if (len < 16) {
            if (len < 8)
                return *(const GLB_AS u32_any *)t == *(const GLB_AS u32_any *)q &&
                       *(const GLB_AS u32_any *)(t + len - 4) == *(const GLB_AS u32_any *)(q + len - 4);
            return *(const GLB_AS u64_any *)t == *(const GLB_AS u64_any *)q &&
                   *(const GLB_AS u64_any *)(t + len - 8) == *(const GLB_AS u64_any *)(q + len - 8);
        }
        for (uint32_t j = 0;; j += 16) {
            j = min(j, len - 16);
            const v4u d = *(const GLB_AS v4u_any *)(t + j) ^ *(const GLB_AS v4u_any *)(q + j);
            if (d.x | d.y | d.z | d.w)
                return false;
            if (j == len - 16)
                return true;
        }
    }

    // Codes of the 16 characters from `off` before the sample on.
    __device__ __forceinline__ static uint32_t window_code(uint32_t code, uint32_t prev, uint32_t off)
    {
        return off ? __builtin_amdgcn_alignbit(code, prev, 32u - 2u * off) : code;
    }

    __device__ __forceinline__ void emit(bool direct, bool hit, uint64_t sv, uint32_t u, uint32_t &nh, uint32_t &nid,
                                         uint32_t &last, mpm_match *out, uint64_t cap, uint64_t &o) const
    {
        const uint32_t pos = (uint32_t)(sv - text.lo);
        uint64_t bal = __ballot(hit);
        if (bal == 0)
            return;
        if constexpr (Var) {
            // longer strings come first at a start: drop the others
            const uint64_t lower = bal & ((1ull << (threadIdx.x & 63)) - 1ull);
            const uint32_t src = lower ? 63u - (uint32_t)__clzll((long long)lower) : 0u;
            const uint32_t before = (uint32_t)__shfl((int)pos, (int)src, 64);
            const uint32_t top = (uint32_t)__shfl((int)pos, 63 - (int)__clzll((long long)bal), 64);
            if (hit && pos == (lower ? before : last))
                hit = false;
            last = top;
            bal = __ballot(hit);
        }
        if (direct) {
            write_hits(out, cap, o, hit, pos, u, im);
        } else {
            const uint32_t k = nh + below(bal);
            if (hit) {
                if (k < hcap)
                    lds_at<v2u>(wv + WV_HITS)[k] = v2u{pos, u};
                nid += im.count(u);
            }
            nh += (uint32_t)__popcll(bal);
        }
    }

    __device__ __forceinline__ void run(bool direct, uint64_t b0, uint64_t b1, uint32_t &nh, uint32_t &nid,
                                        mpm_match *out, uint64_t cap, uint64_t &o) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        LDS_AS uint32_t *cw = lds_at<uint32_t>(wv);
        LDS_AS uint32_t *slot = lds_at<uint32_t>(wv + WV_ITEMS);
        nh = 0;
        nid = 0;
        if (b0 >= b1)
            return;
        const uint64_t base = b0 * GBLOCK;
        uint32_t last = 0xffffffffu;  // Var: start of the last occurrence
        v4u r[GN];
        uint32_t c[GN + 1], cn[GN];  // codes of the current block (and 16 more), of the next
        text.load(base, lane, r);
        uint32_t prev = b0 ? codes16(text.piece(base - 16), a.code_shift) : 0u;
        const uint32_t after = text.fix(codes16(text.piece(b1 * GBLOCK), a.code_shift), b1 * GBLOCK);
        text.codes(base, lane, r, a.code_shift, cn);
        if (b0 + 1 < b1)
            text.load(base + GBLOCK, lane, r);
        for (uint64_t b = b0; b < b1; ++b) {
            uint32_t ct = after;
#pragma unroll
            for (int k = 0; k < GN; ++k)
                c[k] = cn[k];
            if (b + 1 < b1) {
                text.codes((b + 1) * GBLOCK, lane, r, a.code_shift, cn);
                ct = (uint32_t)__builtin_amdgcn_readfirstlane((int)cn[0]);
                if (b + 2 < b1)
                    text.load((b + 2) * GBLOCK, lane, r);
            }
            c[GN] = from_next(c[0], ct);
            // one bit per sample, the first sample in the lowest bit
            uint32_t mk[NM];
            uint32_t cnt = 0;
#pragma unroll
            for (uint32_t h = 0; h < NM; ++h)
                mk[h] = 0;
#pragma unroll
            for (uint32_t s = 0; s < NS; ++s) {
                const uint32_t k = (s * T) >> 4, sub = 2 * ((s * T) & 15);
                const uint32_t y = sub ? __builtin_amdgcn_alignbit(c[k + 1], c[k], sub - 2) : c[k] << 2;
                if constexpr (Pair) {
                    if (s & 1)
                        continue;
                    const uint32_t x = *(lds_cptr<uint32_t>)lds_at<const uint8_t>(GBITS_OFF + a.pair_off + (y & pmask));
                    mk[s >> 5] = __builtin_amdgcn_alignbit(x >> (__builtin_amdgcn_ubfe(y, bsh + 3, 4) << 1), mk[s >> 5], 2);
                    continue;
                }
                const uint32_t x = *(lds_cptr<uint32_t>)lds_at<const uint8_t>(GBITS_OFF + (y & amask));
                mk[s >> 5] = __builtin_amdgcn_alignbit(x >> ((y >> bsh) & 31u), mk[s >> 5], 1);
            }
            if (NS < 32)
                mk[0] >>= (32 - NS) & 31;
            const uint64_t v0 = b * GBLOCK + lane * (16 * GN);
            if (!text.whole<GN>(b * GBLOCK)) {
                // nothing starts past the end (where codes read as zeros)
                const uint32_t left = (uint32_t)(text.hi > v0 ? min(text.hi - v0 + T - 1, (uint64_t)16 * GN) : 0) >> TL;
#pragma unroll
                for (uint32_t h = 0; h < NM; ++h)
                    mk[h] &= left >= 32 * h + 32 ? ~0u : left > 32 * h ? (1u << (left - 32 * h)) - 1u : 0u;
            }
#pragma unroll
            for (uint32_t h = 0; h < NM; ++h)
                cnt += __popc(mk[h]);
            const uint32_t before = prev;
            prev = (uint32_t)__builtin_amdgcn_readlane((int)c[GN - 1], 63);
            if (__ballot(cnt != 0) == 0)
                continue;
#pragma unroll
            for (int k = 0; k < GN; k += 4)
                *(LDS_AS v4u *)(cw + 4 + GN * lane + k) = v4u{c[k], c[k + 1], c[k + 2], c[k + 3]};
            if (lane == 0) {
                cw[3] = before;
                cw[4 + 64 * GN] = ct;
            }
            const uint32_t incl = wave_incl_sum(cnt);
            const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            if (__builtin_expect(tot > 64, 0) && tot > a.crowd) {  // (crowd >= 64)
                // the lane's first and last candidate
                uint32_t f = 0, l = 0;
#pragma unroll
                for (uint32_t h = 0; h < NM; ++h) {
                    f = mk[NM - 1 - h] ? 32 * (NM - 1 - h) + (uint32_t)__builtin_ctz(mk[NM - 1 - h]) : f;
                    l = mk[h] ? 32 * h + 31 - (uint32_t)__builtin_clz(mk[h]) : l;
                }
                crowded(direct, hidden(b) * GBLOCK, cnt != 0, f, l, nh, nid, out, cap, o);
                // again, as they are not kept in registers over the walk
                // (of the last blocks: any block's)
                text.load(hidden(min(b + 2, b1 - 1)) * GBLOCK, lane, r);
                continue;
            }
            uint32_t rk = incl - cnt;  // place of the lane's next candidate
#pragma unroll 1
            for (uint32_t win = 0; win < tot; win += 128) {
                wave_sync();
#pragma unroll
                for (uint32_t h = 0; h < NM; ++h)
                    for (; mk[h] && rk < win + 128; mk[h] &= mk[h] - 1, ++rk)
                        slot[rk - win] = lane * NS + 32 * h + (uint32_t)__builtin_ctz(mk[h]);
                wave_sync();
                if (tot - win > 64)
                    candidates<2>(direct, b * GBLOCK, tot - win, nh, nid, last, out, cap, o);
                else
                    candidates<1>(direct, b * GBLOCK, tot - win, nh, nid, last, out, cap, o);
            }
        }
    }

    // The starting positions that a block's samples stand for, with the
    // index's automaton: each lane its own, from its first candidate to its
    // last, counted, then walked again for their pairs. For blocks with more
    // candidates than a.crowd (mpm_gram.cpp): runs of one character (poly-A;
    // N, which shares G's code) and short repeats whose grams are in the set
    // make every sample a candidate, with a chain of entries and strings to
    // compare at each, where a walk takes a table row per byte. It is bound by
    // the rows' round trips to L1 and L2. Measured, 128 MiB, d = 1000, us by
    // the candidates, with the walk here, and by the walkers of explicit
    // placements (1024 positions per lane): a tenth of the text in runs of N,
    // G^m in the set, m = 16: 1246, 149, 84, m = 24: 1891, 194, 115; all A, A^16
    // in the set: 3126, 1022, 2541; lengths 8-32 with 50 strings of one head of
    // nine A, on A: 4854, 139, 85, on records with poly-A tails: 779, 487, 116
    // (490 with 64 positions per lane): there the table outgrows the L1. (Four
    // bytes per turn are 7 % faster here and cost the batch 1 % more for their
    // code.)
    // Texts without such blocks: 256 MiB, m = 16, 62.1 -> 61.7; lengths 8-32,
    // 128 MiB, 62.2 -> 62.1; the batch of 256 texts 109 -> 111.
    __device__ __forceinline__ void crowded(bool direct, uint64_t base, bool any, uint32_t fs, uint32_t ls,
                                            uint32_t &nh, uint32_t &nid, mpm_match *out, uint64_t cap,
                                            uint64_t &o) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        const GramWalk w = uniform_load(a.walk);
        glb_cptr<uint8_t> img = (glb_cptr<uint8_t>)a.walk - w.self;
        glb_cptr<uint16_t> cls = (glb_cptr<uint16_t>)(img + w.cls);
        const int64_t first = (int64_t)base - (int64_t)(T - 1);  // the wave's first start
        // Positions from here on are relative to it. The lane's starts [s0, s1],
        // those of its first to its last candidate.
        const int32_t s0 = (int32_t)(64 * lane + T * fs), s1 = (int32_t)(64 * lane + T * ls + T - 1);
        glb_cptr<uint8_t> tx = text.p + first;
        const int32_t lo = (int32_t)max((int64_t)text.lo - first, -((int64_t)1 << 30));
        const int32_t end = (int32_t)min((int64_t)text.hi - first, (int64_t)1 << 30);
        const bool whole = lo <= 0 && (int32_t)(GBLOCK + w.past + 16) <= end;
        // 16 bytes at v; ok: which of them lie in the text (the others restart the walk)
        auto piece = [&](int32_t v, uint32_t &ok) {
            if (whole) {
                ok = 0xffffu;
                return *(const GLB_AS v4u_any *)(tx + v);
            }
            v4u c = {0, 0, 0, 0};
            ok = 0;
#pragma unroll 1
            for (uint32_t k = 0; k < 16; ++k) {
                const int32_t x = v + (int32_t)k;
                c = v4u{__builtin_amdgcn_alignbit(c.y, c.x, 8), __builtin_amdgcn_alignbit(c.z, c.y, 8),
                        __builtin_amdgcn_alignbit(c.w, c.z, 8), c.w >> 8};
                if (x >= lo && x < end) {
                    c.w |= (uint32_t)tx[x] << 24;
                    ok |= 1u << k;
                }
            }
            return c;
        };
        uint32_t hits = 0, ids = 0, slot = 0;
        uint64_t ob = 0;
#pragma unroll 1
        for (uint32_t pass = 0; pass < 2; ++pass) {
            uint32_t np = any ? (uint32_t)(s1 - s0 + w.past + 16) >> 4 : 0u;  // pieces, of the lane's own
            const int32_t step = Var ? -16 : 16;
            int32_t v = Var ? s0 + 16 * (int32_t)np - 16 : s0;
            uint32_t s = 0, okn = 0, entry = 0xffffffffu;
            v4u cn = {0, 0, 0, 0}, was = cn;
            if (np)
                cn = piece(v, okn);
#pragma unroll 1
            for (uint32_t j = 0; __ballot(j < np) != 0; ++j, v += step) {
                if (j >= np)
                    continue;
                v4u c = cn;
                uint32_t ok = okn;
                if (j + 1 < np)
                    cn = piece(v + step, okn);
                // The piece of before again, from the state that it left as it
                // found it and without a string: it does the same (runs and
                // repeats of 2, 4, 8 or 16 characters).
                const bool same = s == entry && ok == 0xffffu && ((c.x ^ was.x) | (c.y ^ was.y) | (c.z ^ was.z) | (c.w ^ was.w)) == 0;
                if (__ballot(!same) == 0)
                    continue;
                entry = s;
                was = c;
                // one byte per turn, the next one's column requested beside its row
                uint32_t col = cls[Var ? c.w >> 24 : c.x & 0xffu];
#pragma unroll 1
                for (uint32_t k = 0; k < 16; ++k) {
                    c = Var ? v4u{c.x << 8, __builtin_amdgcn_alignbit(c.y, c.x, 24), __builtin_amdgcn_alignbit(c.z, c.y, 24),
                                  __builtin_amdgcn_alignbit(c.w, c.z, 24)}
                            : v4u{__builtin_amdgcn_alignbit(c.y, c.x, 8), __builtin_amdgcn_alignbit(c.z, c.y, 8),
                                  __builtin_amdgcn_alignbit(c.w, c.z, 8), c.w >> 8};
                    const uint32_t off = s * w.rowb + col;
                    col = cls[Var ? c.w >> 24 : c.x & 0xffu];
                    s = w.wide ? *(glb_cptr<uint32_t>)(img + w.dfa + off) : *(glb_cptr<uint16_t>)(img + w.dfa + off);
                    const uint32_t i = Var ? 15 - k : k;
                    if (!(ok >> i & 1u))
                        s = 0;
                    if (s < w.first_term)
                        continue;
                    entry = 0xffffffffu;
                    const int32_t at = v + (int32_t)i - (Var ? 0 : (int32_t)w.past);
                    if (at > s1)
                        continue;
                    uint32_t u = s - w.first_term;
                    if (Var)
                        u = ((glb_cptr<uint32_t>)(img + w.term))[u];
                    uint32_t ib, ie;
                    im.span(u, ib, ie);
                    if (pass == 0) {
                        ++hits;
                        ids += ie - ib;
                        continue;
                    }
                    const uint32_t pos = (uint32_t)(first - (int64_t)text.lo) + (uint32_t)at;
                    if (Var)
                        ob -= ie - ib, --slot;
                    if (direct) {
                        for (uint32_t t = ib; t < ie; ++t)
                            if (ob + (t - ib) < cap)
                                ((GLB_AS v2u *)out)[ob + (t - ib)] = v2u{pos, im.id(t)};
                    } else {
                        lds_at<v2u>(wv + WV_HITS)[slot] = v2u{pos, u};
                    }
                    if (!Var)
                        ob += ie - ib, ++slot;
                }
                if (!Var && s == 0 && v + 16 > s1)  // nothing begun up to the last start
                    np = j + 1;
            }
            if (pass)
                break;
            // places of the lane's occurrences and pairs (Var: those after its last)
            const uint32_t hi = wave_incl_sum(hits), ii = wave_incl_sum(ids);
            const uint32_t th = (uint32_t)__builtin_amdgcn_readlane((int)hi, 63);
            const uint32_t ti = (uint32_t)__builtin_amdgcn_readlane((int)ii, 63);
            slot = nh + (Var ? hi : hi - hits);
            ob = o + (Var ? ii : ii - ids);
            const uint64_t o0 = o;
            nid += ids;
            nh += th;
            o += ti;
            if (th == 0 || (direct ? o0 >= cap : nh > hcap))
                break;
        }
    }

    // The first min(n, 64 K) candidates of the slots, in text order: lane l
    // takes slots l, l + 64, ... The K loads of a step are in flight together:
    // the steps are a chain of L2 round trips (two candidates per lane instead
    // of one: 64 MiB, d = 1000, m = 8 with counts, 98 -> 91 us; 64 MiB,
    // d = 100k, m = 16, 106 -> 96; the batch below 133 -> 115).
    template <int K>
    __device__ __forceinline__ void candidates(bool direct, uint64_t base, uint32_t n, uint32_t &nh, uint32_t &nid,
                                               uint32_t &last, mpm_match *out, uint64_t cap, uint64_t &o) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        LDS_AS uint32_t *cw = lds_at<uint32_t>(wv);
        LDS_AS uint32_t *slot = lds_at<uint32_t>(wv + WV_ITEMS);
        uint32_t p[K], code[K], pv[K], head[K], i[K], nm[K], fm[K], key[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            p[k] = lane + 64 * k < n ? slot[lane + 64 * k] << TL : 0u;  // sample, relative to the block
            const uint32_t wi = p[k] >> 4, sub = 2 * (p[k] & 15);
            const uint32_t A = cw[3 + wi], B = cw[4 + wi], C = cw[5 + wi];
            code[k] = __builtin_amdgcn_alignbit(C, B, sub);
            pv[k] = __builtin_amdgcn_alignbit(B, A, sub);
        }
        uint2 w[K];
#pragma unroll
        for (int k = 0; k < K; ++k)
            w[k].x = *(lds_cptr<uint32_t>)lds_at<const uint8_t>(GBITS_OFF + ((code[k] & wmask) << 2));
        if (a.rank_off) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                w[k].y = *(lds_cptr<uint32_t>)lds_at<const uint8_t>(GBITS_OFF + a.rank_off + ((code[k] & wmask) << 2));
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k)
                w[k].y = a.ranks[code[k] & wmask];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            head[k] = w[k].y + __popc(w[k].x & ((1u << ((code[k] >> (bsh - 2)) & 31u)) - 1u));
            if (lane + 64 * k >= n)
                head[k] = 0xffffffffu;
            i[k] = head[k];
            nm[k] = fm[k] = key[k] = 0;
        }
        // chain entries whose first codes agree
        bool more = true;
        while (more) {
            v4u e[K];  // key, mask, meta, next
#pragma unroll
            for (int k = 0; k < K; ++k)
                e[k] = *((glb_cptr<v4u>)a.ents + (i[k] != 0xffffffffu ? i[k] : 0u));
            more = false;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (i[k] != 0xffffffffu) {
                    if (((window_code(code[k], pv[k], e[k].z & 15u) ^ e[k].x) & e[k].y) == 0) {
                        if (nm[k] == 0) {
                            fm[k] = e[k].z;
                            key[k] = e[k].x;
                        }
                        ++nm[k];
                    }
                    i[k] = e[k].w;
                    more |= i[k] != 0xffffffffu;
                }
        }
        bool any = false, many = false;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            any |= nm[k] != 0;
            many |= nm[k] > 1;
        }
        if (__ballot(any) == 0)
            return;
        if (__ballot(many) == 0) {
            uint64_t sv[K];
            uint32_t u[K];
            bool act[K], plain[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                act[k] = nm[k] != 0;
                sv[k] = base + p[k] - (fm[k] & 15u);
                u[k] = fm[k] >> 5;
                plain[k] = fm[k] & 16u;
            }
            check<K>(direct, act, sv, u, plain, key, nh, nid, last, out, cap, o);
            return;
        }
        // lanes with several agreeing entries: deal them out in order
        LDS_AS v2u *item = lds_at<v2u>(wv + WV_ITEMS);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            uint32_t tot;
            const uint32_t pre = wave_excl_sum(nm[k], tot);
#pragma unroll 1
            for (uint32_t iw = 0; iw < tot; iw += 64) {
                wave_sync();
                uint32_t r = pre - iw;
                if (nm[k])
                    for (uint32_t j = head[k]; j != 0xffffffffu;) {
                        const v4u e = *((glb_cptr<v4u>)a.ents + j);
                        if (((window_code(code[k], pv[k], e.z & 15u) ^ e.x) & e.y) == 0) {
                            if (r < 64)
                                item[r] = v2u{p[k] + BIAS - (e.z & 15u), e.z >> 5};
                            ++r;
                        }
                        j = e.w;
                    }
                wave_sync();
                const v2u it = item[lane];
                const bool act[1] = {lane < min(64u, tot - iw)};
                const uint64_t sv[1] = {base + it.x - BIAS};
                const uint32_t u[1] = {it.y}, none[1] = {0};
                const bool plain[1] = {false};
                check<1>(direct, act, sv, u, plain, none, nh, nid, last, out, cap, o);
            }
        }
    }

    // Blocks [b0, b1): count, get the output slot of this wave's first pair
    // from place(number of ids), write the pairs.
    template <class F>
    __device__ __forceinline__ void part(uint64_t b0, uint64_t b1, mpm_match *out, uint64_t cap, F place) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        uint32_t nh, nid;
        uint64_t o = 0;
#pragma unroll 1
        for (uint32_t pass = 0; pass < 2; ++pass) {
            run(pass != 0, hidden(b0), b1, nh, nid, out, cap, o);
            if (pass)
                break;
#pragma unroll
            for (int k = 32; k >= 1; k >>= 1)
                nid += __shfl_xor(nid, k, 64);
            o = place(nid);
            if (nh == 0 || o >= cap)
                break;
            if (nh <= hcap) {
                wave_sync();
                for (uint32_t r = 0; r < nh && o < cap; r += 64) {
                    const bool act = r + lane < nh;
                    v2u h = {0, 0};
                    if (act)
                        h = lds_at<v2u>(wv + WV_HITS)[r + lane];
                    write_hits(out, cap, o, act, h.x, h.y, im);
                }
                break;
            }
        }
    }

    // The main bytes of four codes; of eight.
    __device__ __forceinline__ uint32_t bytes4(uint32_t c) const
    {
        c = (c | c << 12) & 0x000f000fu;
        c = (c | c << 6) & 0x03030303u;
        return __builtin_amdgcn_perm(0u, a.main4, c);
    }
    __device__ __forceinline__ uint64_t bytes8(uint32_t c) const
    {
        return (uint64_t)bytes4((c >> 8) & 0xffu) << 32 | bytes4(c & 0xffu);
    }

    // Whether the bytes at view positions s[] are the strings u[], all of
    // them of one length of at most 16 (two overlapping pieces V each). A
    // plain string's bytes follow from its codes.
    template <typename V, int K>
    __device__ __forceinline__ void equal_short(const uint64_t (&s)[K], const uint32_t (&u)[K], const bool (&plain)[K],
                                                const uint32_t (&key)[K], bool (&hit)[K]) const
    {
        typedef V any __attribute__((aligned(1)));
        const uint32_t tail = a.m - sizeof(V);
        V x[K][2], y[K][2];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            glb_cptr<uint8_t> t = text.p + s[k];
            x[k][0] = *(const GLB_AS any *)t;
            x[k][1] = *(const GLB_AS any *)(t + tail);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (sizeof(V) == 4) {
                y[k][0] = bytes4(key[k] & 0xffu);
                y[k][1] = bytes4((key[k] >> (2 * tail)) & 0xffu);
            } else {
                y[k][0] = bytes8(key[k]);
                y[k][1] = bytes8(key[k] >> (2 * tail));
            }
            if (hit[k] && !plain[k]) {
                glb_cptr<uint8_t> q = (glb_cptr<uint8_t>)a.rows + (uint64_t)u[k] * 16;
                y[k][0] = *(const GLB_AS any *)q;
                y[k][1] = *(const GLB_AS any *)(q + tail);
            }
            hit[k] = hit[k] && ((x[k][0] ^ y[k][0]) | (x[k][1] ^ y[k][1])) == 0;
        }
    }

    // Bytewise check of K (start, string) pairs per lane, the first ones of
    // all lanes before the second ones in text order.
    template <int K>
    __device__ __forceinline__ void check(bool direct, const bool (&act)[K], const uint64_t (&sv)[K],
                                          const uint32_t (&u)[K], const bool (&plain)[K], const uint32_t (&key)[K],
                                          uint32_t &nh, uint32_t &nid, uint32_t &last, mpm_match *out, uint64_t cap,
                                          uint64_t &o) const
    {
        bool hit[K];
        if (!Var && a.m <= 16) {
            uint64_t s[K];
            uint32_t v[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                // (a start before the text wraps below zero and fails here too)
                hit[k] = act[k] && (int64_t)sv[k] >= (int64_t)text.lo && sv[k] + a.m <= text.hi;
                s[k] = hit[k] ? sv[k] : text.lo;
                v[k] = hit[k] ? u[k] : 0u;
            }
            if (a.m < 8)
                equal_short<uint32_t, K>(s, v, plain, key, hit);
            else
                equal_short<uint64_t, K>(s, v, plain, key, hit);
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                hit[k] = false;
                if (act[k] && (int64_t)sv[k] >= (int64_t)text.lo) {
                    const uint2 st = Var ? a.strs[u[k]] : make_uint2(u[k] * ((a.m + 15) / 16), a.m);
                    hit[k] = sv[k] + st.y <= text.hi && equal(sv[k], st.x, st.y);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
            emit(direct, hit[k], sv[k], u[k], nh, nid, last, out, cap, o);
    }
};

template <int W, int TL, bool Var, bool Pair = false>
__global__ __launch_bounds__(W) void gram_kernel(GramDev a, ScanDev sd, GramShare share, uint32_t hits,
                                                 uint32_t wave_bytes)
{
    extern __shared__ __align__(16) uint8_t smem[];
    if (!lds_layout_ok(smem, sd.hdr))
        return;
    LdsHdr *const H = (LdsHdr *)lds_at<LdsHdr>(LDS_HDR_OFF);
    uint64_t &s_tile = H->tile;
    uint32_t &s_epoch = H->epoch;
    uint64_t *const s_scan = H->scan;
    uint32_t *const hdr = sd.hdr;
    constexpr uint32_t NW = W / 64;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    if (threadIdx.x == 0) {
        s_tile = take_ticket(hdr);
        s_epoch = __hip_atomic_load(&hdr[WS_EPOCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    copy_to_lds<W>(GBITS_OFF, (const uint8_t *)a.bits, a.bit_bytes);
    load_groups(a.grp);

    GramScan<TL, Var, Pair> sc;
    sc.bind(a, sd.single.text, sd.single.n);
    sc.wv = GBITS_OFF + a.bit_bytes + wave * wave_bytes;
    sc.hcap = hits;
    const uint64_t ntiles = sd.ntiles;
    const uint64_t cap = sd.single.cap;

    while (true) {
        __syncthreads();
        const uint64_t g = uniform64(s_tile);
        if (g >= ntiles)
            break;
        const uint64_t b0 = share.first(g * NW + wave), b1 = share.first(g * NW + wave + 1);
        sc.part(b0, b1, sd.single.out, cap, [&](uint32_t nid) {
            return wave_offset<W>(nid, s_scan, sd.status, g, ntiles, sd.single.total, s_epoch,
                                  &hdr[WS_ERR]);
        });
        if (gridDim.x >= ntiles)  // one chunk per workgroup
            break;
        if (threadIdx.x == 0)
            s_tile = take_ticket(hdr);
    }
    if (gridDim.x == ntiles && ntiles <= WIDE_CHUNKS) {
        if (threadIdx.x == 0 && s_tile + 1 == ntiles)
            finish_wide(hdr, s_epoch);
        return;
    }
    finish_launch(hdr, s_epoch);
}

// Batched texts. A wave takes a piece: parts (runs of blocks) of one or more
// texts of an index, of about equal expected time in every piece
// (plan_gram_batch). Sixteen pieces of an index are a ticket; the workgroup
// copies the index's bits to LDS, and its waves don't wait for each other
// until the next ticket: each looks back over the parts of its own texts.
// A piece's last part, which the next piece may go on from, is run first, so
// that a piece that starts inside a text finds the counts before it early.
// (Workgroup chunks of one text each, as the walkers have, leave the chip idle
// for short texts; with one text per wave the short ones still took a good part
// of the waves, 198 us for the batch below.)
//
// Measured on 256 EST-shaped texts of 1 KiB to 4 MiB (120 MB) and eight sets
// of 115 to 4648 strings of 8 to 32 characters, replayed graph: 298 us by
// the walkers, 106 here.
template <int TL>
__device__ __forceinline__ void batch_part(const GramDev &dev, const TextDesc &td, uint64_t g, const GramPart &part,
                                           uint32_t wv, uint32_t hits, uint32_t epoch, uint32_t *hdr, uint64_t *status)
{
    GramScan<TL, false> sc;
    sc.bind(dev, td.text, td.n);
    sc.wv = wv;
    sc.hcap = hits;
    const uint64_t first = td.tile_begin, last = first + td.ntiles - 1;
    uint64_t *const total = td.total;
    const uint64_t b0 = part.b0, b1 = b0 + part.nb;
    sc.part(b0, b1, td.out, td.cap, [&](uint32_t nid) {
        const uint64_t agg = __builtin_amdgcn_readfirstlane(nid);
        const uint64_t o = uniform64(look_back(status, g, first, agg, epoch, &hdr[WS_ERR]));
        if (g == last && (threadIdx.x & 63u) == 0)
            *total = o + agg;
        return o;
    });
}

__global__ __launch_bounds__(1024) void gram_batch_kernel(GramBatchDev bd)
{
    extern __shared__ __align__(16) uint8_t smem[];
    if (!lds_layout_ok(smem, bd.hdr))
        return;
    LdsHdr *const H = (LdsHdr *)lds_at<LdsHdr>(LDS_HDR_OFF);
    uint64_t &s_tile = H->tile;
    uint32_t &s_epoch = H->epoch;
    constexpr uint32_t NW = 1024 / 64;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0)
        s_epoch = __hip_atomic_load(&bd.hdr[WS_EPOCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t loaded = 0xffffffffu;
    while (true) {
        if (threadIdx.x == 0)
            s_tile = take_ticket(bd.hdr);
        __syncthreads();
        const uint64_t t = uniform64(s_tile);
        if (t >= bd.ntickets)
            break;
        const uint32_t epoch = __builtin_amdgcn_readfirstlane(s_epoch);
        const uint2 range = uniform_load((const uint2 *)bd.pieces + t * NW + wave);
        const uint32_t ix = uniform_load(bd.tickets + t);
        const GramDev dev = uniform_load(bd.idx + ix);
        if (ix != loaded) {
            copy_to_lds<1024>(GBITS_OFF, (const uint8_t *)dev.bits, dev.bit_bytes);
            load_groups(bd.idx[ix].grp);
            loaded = ix;
        }
        __syncthreads();
        const uint32_t wave_bytes = batch_wave_bytes(bd.lds_bytes, dev.bit_bytes);
        const uint32_t wv = GBITS_OFF + dev.bit_bytes + wave * wave_bytes;
        const uint32_t hits = (wave_bytes - WV_HITS) / 8;
#pragma unroll 1
        for (uint32_t k = range.y; k-- > range.x;) {
            const GramPart p = uniform_load(bd.parts + k);
            const BatchText bt = uniform_load(bd.texts + p.text);
            uint64_t t0 = 0;
            if (bt.cost)
                t0 = wall_clock64();
            switch (dev.t_log) {
            case 0: batch_part<0>(dev, bt.td, k, p, wv, hits, epoch, bd.hdr, bd.status); break;
            case 1: batch_part<1>(dev, bt.td, k, p, wv, hits, epoch, bd.hdr, bd.status); break;
            case 2: batch_part<2>(dev, bt.td, k, p, wv, hits, epoch, bd.hdr, bd.status); break;
            case 3: batch_part<3>(dev, bt.td, k, p, wv, hits, epoch, bd.hdr, bd.status); break;
            default: batch_part<4>(dev, bt.td, k, p, wv, hits, epoch, bd.hdr, bd.status); break;
            }
            // a timed request: a wave's time on a part counts as a sixteenth
            // of a workgroup's
            if (bt.cost && (threadIdx.x & 63u) == 0) {
                const float us = (float)(wall_clock64() - t0) * bd.us_per_tick;
                atomicAdd(&bt.cost[0], us / (float)(gridDim.x * NW));
                atomicMax((uint32_t *)&bt.cost[1], __float_as_uint(us));  // order of >= 0 floats
            }
        }
        __syncthreads();
    }
    finish_launch(bd.hdr, s_epoch);
}

template <int W>
const void *pick(uint32_t tl, bool var)
{
#define MPM_GRAM_PICK(TL) \
    case TL: return var ? (const void *)gram_kernel<W, TL, true> : (const void *)gram_kernel<W, TL, false>;
    switch (tl) {
        MPM_GRAM_PICK(0)
        MPM_GRAM_PICK(1)
        MPM_GRAM_PICK(2)
        MPM_GRAM_PICK(3)
        MPM_GRAM_PICK(4)
    }
#undef MPM_GRAM_PICK
    return nullptr;
}

const void *kernel_of(uint32_t W, uint32_t tl, bool var, bool pair)
{
    if (W == 1024 && tl == 0 && pair)
        return var ? (const void *)gram_kernel<1024, 0, true, true> : (const void *)gram_kernel<1024, 0, false, true>;
    return W == 256 ? pick<256>(tl, var) : pick<1024>(tl, var);
}

}  // namespace

// LDS bytes of the tables: the bits, the grams before each word where those
// pay for their copy (small workgroups share one of 32 KiB, q = 9, between four
// waves only), the two-position answers in the largest workgroups.
static uint32_t lds_tables(const mpm_index::Gram &G, uint32_t W)
{
    if (!G.ranked || (W == 256 && G.q > 8))
        return G.bit_bytes;
    return 2 * G.bit_bytes + (W == 1024 ? G.pair_bytes : 0);
}

// Whether automatic placement runs an index through the filter.
bool gram_takes(const mpm_index *ix, const mpm_variant *v, uint64_t n)
{
    if ((!ix->gram.ok && !ix->direct.ok) || n < 64)
        return false;
    return !v || (v->placement == MPM_PLACE_AUTO && !(v->flags & ~(uint32_t)MPM_VARIANT_DENSE));
}

// Launch shape for a text of n bytes that starts lo bytes past a 16-byte
// boundary; false when the filter cannot run it.
bool gram_config(const mpm_index *ix, const mpm_variant *v, uint64_t n, uint32_t lo, GramCfg *g)
{
    const mpm_index::Gram &G = ix->gram;
    // (where the builder kept a direct-address table it is the faster scan)
    g->direct = ix->direct.ok;
    if (g->direct && direct_config(ix, v, n, lo, g))
        return true;
    g->direct = false;
    if (!G.ok)
        return false;
    const DeviceLimits lim = limits();
    // Workgroups of 1024 threads share one copy of the bits between 16 waves;
    // texts that would leave CUs without work are cut finer.
    const uint64_t nblocks = (n + lo + GBLOCK - 1) / GBLOCK;
    const uint32_t W = nblocks >= 16ull * lim.cus ? 1024 : 256;
    const uint32_t nw = W / 64;
    // the occurrence lists: all the LDS that is left to 16 waves (their
    // registers admit no second workgroup), 256 occurrences per wave of a
    // small workgroup
    auto hits_of = [&](uint32_t tables_w) {
        const uint32_t room = ((uint32_t)lim.max_lds - GBITS_OFF - lds_tables(G, tables_w)) / nw;
        return room < WV_HITS + 16 * 8 ? 0u : std::min<uint32_t>((room - WV_HITS) / 8, W == 1024 ? 1024 : 256) & ~1u;
    };
    // The two-position answers where the shorter lists still hold the expected
    // occurrences of one round (1 GiB, d = 1000, m = 8, 16 rounds with them and
    // 7 without: 1.97 against 2.02 TB/s; 64 MiB, one round: 72.5 against 75 us).
    const uint64_t each = (nblocks + (uint64_t)lim.cus * nw - 1) / ((uint64_t)lim.cus * nw);
    const bool pair = W == 1024 && G.pair_bytes && 0.6 * hits_of(W) >= (double)GBLOCK * G.hit * (double)each;
    g->tables_w = W == 1024 && !pair ? GRAM_BATCH_W : W;
    const uint32_t hits = hits_of(g->tables_w), tables = lds_tables(G, g->tables_w);
    if (hits == 0)
        return false;
    g->nblocks = nblocks;
    g->W = W;
    g->hits = hits;
    g->wave_bytes = WV_HITS + 8 * hits;
    g->lds_bytes = GBITS_OFF + tables + nw * g->wave_bytes;
    if (g->lds_bytes > (uint32_t)lim.max_lds)
        return false;
    const void *k = kernel_of(W, G.t_log, ix->var != 0, pair);
    if (g->lds_bytes > 65536)
        (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)g->lds_bytes);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, (int)W, g->lds_bytes) != hipSuccess || nb <= 0)
        nb = 1;
    const uint64_t slots = (uint64_t)nb * lim.cus;
    // One round of chunks, as each round waits for its first text and its
    // offsets, unless the expected occurrences would not fit the lists.
    uint64_t blocks = (nblocks + slots * nw - 1) / (slots * nw);
    const double fit = 0.6 * hits / (GBLOCK * G.hit);
    blocks = std::max<uint64_t>(1, std::min<uint64_t>(blocks, fit > 4096 ? 4096 : (uint64_t)fit));
    // The blocks are spread evenly over whole rounds of chunks (64 MiB and
    // 12 KB, 4.001 blocks per wave, d = 100k, m = 16: 80.4 us when 3,278 waves
    // took five each, 75.0 now; 32 MiB and 7 bytes, lengths 8-32: 29.9 -> 26.9).
    g->nchunks = (nblocks + blocks * nw - 1) / (blocks * nw);
    g->nchunks = std::min((g->nchunks + slots - 1) / slots * slots, (nblocks + nw - 1) / nw);
    g->share = gram_share(nblocks, g->nchunks * nw);
    uint64_t grid = v && v->grid ? v->grid : slots;
    g->grid = (uint32_t)std::max<uint64_t>(1, std::min(grid, g->nchunks));
    // a wave's count of ids stays in 32 bits
    return (uint64_t)(blocks * GBLOCK + 16) * std::max<uint64_t>(1, ix->max_dup) < (1ull << 32);
}

GramDev gram_dev(const mpm_index *ix, uint32_t W)
{
    const mpm_index::Gram &G = ix->gram;
    GramDev a;
    const uint8_t *img = ix->d_image;
    a.bits = (const uint32_t *)(img + G.off_bits);
    a.ranks = a.bits + G.bit_bytes / 4;
    a.ents = (const GramEnt *)(img + G.off_ents);
    a.strs = (const uint2 *)(img + G.off_strs);
    a.rows = img + G.off_rows;
    id_csr(ix, &a.uoff, &a.uids);
    a.q = G.q;
    a.t_log = G.t_log;
    a.code_shift = G.code_shift;
    a.bit_bytes = lds_tables(G, W);
    a.rank_off = a.bit_bytes > G.bit_bytes ? G.bit_bytes : 0;
    a.pair_off = a.bit_bytes > 2 * G.bit_bytes ? 2 * G.bit_bytes : 0;
    a.main4 = G.main4;
    a.m = ix->m;
    a.n_single = ix->n_single;
    a.crowd = G.crowd;
    a.walk = (const GramWalk *)(img + G.off_walk);
    a.grp = id_groups(ix);
    return a;
}

mpm_status gram_launch(const mpm_index *ix, const GramCfg &g, const ScanDev &sd, void *stream)
{
    if (g.direct)
        return direct_launch(ix, g, sd, stream);
    GramDev a = gram_dev(ix, g.tables_w);
    ScanDev s = sd;
    s.ntiles = g.nchunks;
    GramShare share = g.share;
    uint32_t hits = g.hits, wave_bytes = g.wave_bytes;
    void *args[] = {&a, &s, &share, &hits, &wave_bytes};
    const hipError_t e = hipLaunchKernel(kernel_of(g.W, ix->gram.t_log, ix->var != 0, a.pair_off != 0), dim3(g.grid), dim3(g.W),
                                         args, g.lds_bytes, (hipStream_t)stream);
    if (e != hipSuccess)
        return fail(MPM_EHIP, "scan launch: %s", hipGetErrorString(e));
    return MPM_OK;
}

// Whether a batched request runs through the filter. (Sets without one whose
// single scans use direct addressing stay with the walkers.)
bool gram_batch_takes(const mpm_index *ix, const mpm_variant *v, uint64_t n)
{
    return ix->gram.ok && !ix->var && n < (1ull << 32) && gram_takes(ix, v, n) &&
           GBITS_OFF + lds_tables(ix->gram, GRAM_BATCH_W) + 16 * (WV_HITS + 16 * 8) <= (uint32_t)limits().max_lds &&
           (uint64_t)(GBLOCK + 16) * std::max<uint64_t>(1, ix->max_dup) < (1ull << 32);
}

// Blocks of a batched text (whatever its alignment).
static uint64_t batch_blocks(uint64_t n) { return (n + 15 + GBLOCK - 1) / GBLOCK; }

// Cut the texts (those of an index together) into pieces for one wave each.
// A block takes a wave about 1.5 us for the sparsest sets, 0.85 us per unit of
// the filter's cost and 300 us per occurrence and byte (timed requests of 9 to
// 23 MB, costs 1.6 to 17: 1.6 to 39 us per block), a part's first load and
// offset about 2 us more. Of the piece lengths around the average load of a
// wave the one is taken whose tickets, longest first, end earliest; one round
// in most cases, but the occurrence lists bound the blocks of a part, and
// with them a dense set's pieces.
void plan_gram_batch(const std::vector<const mpm_index *> &index, std::vector<BatchText> *texts,
                     GramPieces *out, uint32_t grid_req, uint32_t *grid, uint32_t *lds_bytes)
{
    const DeviceLimits lim = limits();
    const uint32_t lds = (uint32_t)lim.max_lds & ~15u;
    const uint64_t slots = grid_req ? grid_req : std::max(1, lim.cus);  // workgroups of 1024 threads: one per CU
    const double part_us = 2.0, ticket_us = 4.0;
    std::vector<double> w;       // us per block
    std::vector<uint64_t> most;  // blocks of a part
    std::vector<std::vector<uint32_t>> of(index.size());
    for (const mpm_index *ix : index) {
        const mpm_index::Gram &G = ix->gram;
        w.push_back(std::max(1.5, 0.85 * G.cost + 300.0 * G.hit));
        const double fit = 0.6 * ((batch_wave_bytes(lds, lds_tables(G, GRAM_BATCH_W)) - WV_HITS) / 8) / (GBLOCK * G.hit);
        const uint64_t ids = ((1ull << 32) - 1) / std::max<uint64_t>(1, ix->max_dup);  // a part's count of ids: 32 bits
        most.push_back(std::max<uint64_t>(1, std::min<uint64_t>(fit > 4096 ? 4096 : (uint64_t)fit, (ids - 16) / GBLOCK)));
    }
    double sum = 0;
    for (size_t i = 0; i < texts->size(); i++) {
        const BatchText &bt = (*texts)[i];
        of[bt.index].push_back((uint32_t)i);
        sum += w[bt.index] * (double)batch_blocks(bt.td.n) + part_us;
    }
    // The pieces of index k, each at most len long where its parts allow:
    // piece() starts one, part(text, b0, nb) adds to it. No piece has two
    // parts of one text (the later one would wait for the earlier).
    auto cut = [&](uint32_t k, double len, auto piece, auto part) {
        double room = 0;
        for (uint32_t i : of[k]) {
            const uint64_t nb = batch_blocks((*texts)[i].td.n);
            for (uint64_t b = 0; b < nb;) {
                if (b || room < part_us + w[k]) {
                    piece();
                    room = len;
                }
                const uint64_t c = room < part_us + w[k] ? 1 : (uint64_t)((room - part_us) / w[k]);
                const uint64_t take = std::min({c, most[k], nb - b});
                part(i, b, take);
                room -= part_us + w[k] * (double)take;
                b += take;
            }
        }
    };
    // End of the last ticket; order: indexes, those of the longest tickets first.
    std::vector<uint32_t> order(index.size());
    auto plan = [&](double len) {
        std::vector<uint64_t> pieces(index.size(), 0);
        std::vector<double> longest(index.size(), 0.0);
        for (uint32_t k = 0; k < index.size(); k++) {
            double cur = 0;
            cut(k, len, [&] { pieces[k]++; cur = 0; },
                [&](uint32_t, uint64_t, uint64_t take) {
                    cur += part_us + w[k] * (double)take;
                    longest[k] = std::max(longest[k], cur);
                });
            order[k] = k;
        }
        std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return longest[x] > longest[y]; });
        std::priority_queue<double, std::vector<double>, std::greater<double>> busy;
        double end = 0;
        for (uint32_t k : order)
            for (uint64_t t = 0; t < (pieces[k] + 15) / 16; t++) {
                double at = 0;
                if (busy.size() >= slots) {
                    at = busy.top();
                    busy.pop();
                }
                busy.push(at + ticket_us + longest[k]);
                end = std::max(end, at + ticket_us + longest[k]);
            }
        return end;
    };
    const double mean = sum / (16.0 * (double)slots);
    double best = 1e300, len = mean;
    for (int k = -8; k <= 12; k++) {
        const double l = mean * exp2(k / 8.0), end = plan(l);
        if (end < best) {
            best = end;
            len = l;
        }
    }
    (void)plan(len);
    for (uint32_t k : order) {
        std::vector<uint32_t> first;
        cut(k, len, [&] { first.push_back((uint32_t)out->parts.size()); },
            [&](uint32_t i, uint64_t b0, uint64_t take) {
                TextDesc &td = (*texts)[i].td;
                if (b0 == 0) {
                    td.tile_begin = out->parts.size();
                    td.ntiles = 0;
                }
                td.ntiles++;
                out->parts.push_back(GramPart{i, (uint32_t)b0, (uint32_t)take});
            });
        const uint32_t end = (uint32_t)out->parts.size();
        for (size_t j = 0; j < (first.size() + 15) / 16 * 16; j++) {
            const uint32_t lo = j < first.size() ? first[j] : end, hi = j + 1 < first.size() ? first[j + 1] : end;
            out->pieces.push_back(make_uint2(lo, hi));
        }
        out->tickets.resize(out->pieces.size() / 16, k);
    }
    *grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(slots, out->tickets.size()));
    *lds_bytes = lds;
}

mpm_status launch_gram_batch(const GramBatchDev &bd, uint32_t grid, void *stream)
{
    const void *k = (const void *)gram_batch_kernel;
    if (bd.lds_bytes > 65536)
        (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bd.lds_bytes);
    GramBatchDev b = bd;
    void *args[] = {&b};
    const hipError_t e = hipLaunchKernel(k, dim3(grid), dim3(1024), args, bd.lds_bytes, (hipStream_t)stream);
    if (e != hipSuccess)
        return fail(MPM_EHIP, "batch launch: %s", hipGetErrorString(e));
    return MPM_OK;
}

}  // namespace mpm
