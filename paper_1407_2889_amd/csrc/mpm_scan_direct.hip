// Direct-address scan for short patterns against large sets.
//
// With m <= 8 characters of a four-letter alphabet a window is an index, and
// a position costs LDS reads at an address that needs no earlier result,
// where the automaton walks a chain of m dependent reads and Wu-Manber a
// bucket. (Aho-Corasick: the depth-m states addressed by their labels.
// Wu-Manber: HASH with a block as long as the window.) The ids lie in window
// order, so the table needs only the number of ids of each window, four bits,
// and the first id slot of every eight windows: 64 KiB for m = 8; a window's
// own slot is that plus a sum of nibbles (one v_dot8).
//
// A wave takes 4 KiB of text, 64 contiguous bytes per lane, packed to 2-bit
// codes. The first pass counts, each lane over its own bytes. Once the
// chunk's offset is known a second pass over the same text (by then in the
// caches) takes 256 positions per round, four per lane: a prefix sum gives
// every lane its place in the round's output, the lanes put (position, id
// slot) there in LDS, and the wave then writes 64 consecutive pairs at a time,
// whole cache lines, each lane gathering one id.
//
// Bytes that share a code with a more frequent pattern byte (N beside G), and
// bytes of no pattern, make a window "odd". Odd windows take nothing from the
// table; the few strings that hold such bytes themselves have a bit table
// over the same codes, and windows that pass it are compared byte by byte.
// In a run of N that is every window: each lane then looks up its own, two in
// flight (32 MiB, d = 10k, m = 8, N^8 in the set, a tenth in runs of N: 1894 ->
// 319 us, the dense-output walkers 213; a list of 64 windows at a time, as for
// the few of other texts, costs its round trips 64 times per block and pass).
//
// Measured against the dense-output walkers (EST-shaped text, m = 8, us, before
// and after): 64 MiB, d = 10k 398 -> 189, d = 100k (92 M pairs) 856 -> 368;
// 16 MiB, d = 30k 492 -> 65; 4 MiB, d = 30k 133 -> 39. No unit alone bounds it
// (d = 100k, counters): sixteen waves of a CU share four SIMDs, an instruction
// takes one of them four cycles, and a round of 256 positions has 200 to 300,
// 48 % of the issue slots; the L2 serves 60 M requests, an id per pair, about
// 58 % of its rate; the LDS is active a quarter of the time (d = 100k with odd strings looked up round by round,
// four runs of ids in flight and branches around each item: 390). Keeping the
// first pass's strings in registers (64 unrolled rounds) or their id counts as
// scalar thresholds measured 586 to 860 us for d = 100k.
#include "mpm_gram.h"

namespace mpm {

namespace {

constexpr uint32_t DBLOCK = 4096;  // text bytes per wave and step
static_assert(1024 / 64 * DBLOCK >> 4 >= GRAM_CHUNK_MIN, "workspace bound");
constexpr uint32_t DTAB_OFF = LDS_CLS_OFF;
// One wave's LDS: code words (from [4] on the block, [260] the 16 characters
// after it); a bit per position that takes its ids from the table; a bit per
// odd window that may be an odd string; the items of a round; the block's odd
// strings (position, first id, number of ids).
constexpr uint32_t DW_KEEP = 264 * 4;
constexpr uint32_t DW_ODD = DW_KEEP + 512;
constexpr uint32_t DW_ITEMS = DW_ODD + 512;
constexpr uint32_t DITEMS = 512;
constexpr uint32_t DW_LIST = DW_ITEMS + 4 * (DITEMS + 64);
constexpr uint32_t DW_BYTES = DW_LIST + 3 * 64 * 4;

// Bit per byte of c that is not the main byte of its code.
__device__ __forceinline__ uint32_t odd4(uint32_t w, uint32_t sh, uint32_t main4)
{
    const uint32_t x = w ^ __builtin_amdgcn_perm(0u, main4, (w >> sh) & 0x03030303u);
    const uint32_t t = ((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) >> 7) & 0x01010101u;
    return __builtin_amdgcn_udot4(t, 0x08040201u, 0u, false);
}

__device__ __forceinline__ uint32_t odd16(const v4u c, uint32_t sh, uint32_t main4)
{
    return odd4(c.x, sh, main4) | odd4(c.y, sh, main4) << 4 | odd4(c.z, sh, main4) << 8 |
           odd4(c.w, sh, main4) << 12;
}

struct DirectScan {
    DirectDev a;
    View T;
    uint32_t wv;     // LDS offset of this wave's buffers
    uint32_t obits;  // LDS offset of the odd strings' bits
    uint64_t last;   // last starting position
    uint32_t split;  // log2 of the waves that share a block's positions
    uint32_t amask;  // byte offsets of the table's words

    // Ids [s, s + n) of the odd strings with these codes at view positions v,
    // where `on` (n = 0: none); the others stay as they are. The K lookups'
    // loads are in flight together.
    template <int K>
    __device__ __forceinline__ void odd_strings(const uint64_t (&v)[K], const uint32_t (&code)[K], const bool (&on)[K],
                                                uint32_t (&s)[K], uint32_t (&n)[K]) const
    {
        const uint64_t keep = a.m == 8 ? ~0ull : (1ull << (8 * a.m)) - 1ull;
        uint2 w[K];
        uint64_t t[K], t2[K];
        uint32_t i[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint64_t at = T.inside(on[k] ? v[k] : T.lo);
            w[k] = a.odd_words[on[k] ? code[k] >> 5 : 0u];
            t[k] = *(const GLB_AS u64_any *)(T.p + at);
            t2[k] = *(const GLB_AS u64_any *)(T.p + at + 8);
        }
        bool more = false;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t d = 8 * (uint32_t)(v[k] - T.inside(v[k]));  // the window lies inside the piece
            t[k] = (d == 0 ? t[k] : d < 64 ? t[k] >> d | t2[k] << (64 - d) : t2[k] >> ((d - 64) & 63)) & keep;
            i[k] = on[k] ? w[k].y + __popc(w[k].x & ((1u << (code[k] & 31u)) - 1u)) : 0xffffffffu;
            if (on[k])
                n[k] = 0;
            more |= on[k];
        }
        while (more) {
            OddEnt e[K];
#pragma unroll
            for (int k = 0; k < K; ++k)
                e[k] = a.odd_ents[i[k] != 0xffffffffu ? i[k] : 0u];
            more = false;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (i[k] != 0xffffffffu) {
                    const bool eq = e[k].bytes == t[k];
                    if (eq) {
                        s[k] = e[k].first;
                        n[k] = e[k].count;
                    }
                    i[k] = eq ? 0xffffffffu : e[k].next;
                    more |= i[k] != 0xffffffffu;
                }
        }
    }
    __device__ __forceinline__ bool odd_bit(uint32_t code) const
    {
        return lds_at<const uint32_t>(obits)[code >> 5] >> (code & 31u) & 1u;
    }

    __device__ __forceinline__ uint32_t code_at(uint32_t p) const
    {
        LDS_AS uint32_t *cw = lds_at<uint32_t>(wv);
        const uint32_t wi = 4 + (p >> 4);
        return __builtin_amdgcn_alignbit(cw[wi + 1], cw[wi], 2 * (p & 15u)) & cmask();
    }

    // Of a block's odd windows (one bit per position of the lane) those with an
    // odd string's codes: their bits, tot their number in the wave.
    __device__ __forceinline__ uint64_t odd_hits(uint64_t odd, uint32_t &incl, uint32_t &tot) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        uint64_t hit = 0;
        for (uint64_t q = odd; q; q &= q - 1) {
            const uint32_t j = (uint32_t)__builtin_ctzll(q);
            if (odd_bit(code_at(64 * lane + j)))
                hit |= 1ull << j;
        }
        incl = wave_incl_sum((uint32_t)__popcll(hit));
        tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        return hit;
    }

    // At most 64 of them, as there usually are: one per lane, positions to the
    // list; s, n: this lane's string.
    __device__ __forceinline__ void odd_few(uint64_t vb, uint64_t hit, uint32_t incl, uint32_t tot, uint32_t &s,
                                            uint32_t &n) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        LDS_AS uint32_t *list = lds_at<uint32_t>(wv + DW_LIST);
        uint32_t at = incl - (uint32_t)__popcll(hit);
        wave_sync();
        for (uint64_t q = hit; q; q &= q - 1, ++at)
            list[at] = 64 * lane + (uint32_t)__builtin_ctzll(q);
        wave_sync();
        s = n = 0;
        if (lane < tot) {
            const uint32_t p = list[lane];
            const uint64_t v[1] = {vb + p};
            const uint32_t code[1] = {code_at(p)};
            const bool on[1] = {true};
            uint32_t s1[1] = {0}, n1[1] = {0};
            odd_strings<1>(v, code, on, s1, n1);
            s = s1[0];
            n = n1[0];
        }
    }

    // Units [u0, u1) of a wave: unit u is part u mod 2^split of block
    // u >> split, the positions of as many lanes' bytes.
    __device__ __forceinline__ bool in_part(uint64_t u, uint32_t lane) const
    {
        return lane >> (6 - split) == ((uint32_t)u & ((1u << split) - 1u));
    }

    // The block at vb: its codes (c[4]: the first ones of the next lane),
    // into LDS too; keep: positions that take their ids from the table; odd:
    // odd windows inside the text.
    __device__ __forceinline__ void block(uint64_t vb, const v4u (&r)[4], uint32_t (&c)[5], uint64_t &keep,
                                          uint64_t &odd) const
    {
        const uint32_t lane = threadIdx.x & 63u, m = a.m, sh = a.code_shift;
        const uint64_t v0 = vb + lane * 64;
        uint32_t q[4];
        T.codes(vb, lane, r, sh, q);
        odd = 0;  // bytes, then windows
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t x = odd16(r[k], sh, a.main4);
            if (!T.whole<4>(vb)) {
                const int64_t d = (int64_t)(v0 + 16 * k - T.inside(v0 + 16 * k));
                x = d >= 16 ? 0u : d >= 0 ? x >> d : (x << -d) & 0xffffu;
            }
            odd |= (uint64_t)x << (16 * k);
            c[k] = q[k];
        }
        uint32_t ct = 0, to = 0;  // the 16 characters after the block
        if (vb + DBLOCK < T.hi) {
            const uint64_t v = vb + DBLOCK;
            const v4u t = T.piece(v);
            ct = T.fix(codes16(t, sh), v);
            to = odd16(t, sh, a.main4) >> (uint32_t)(v - T.inside(v));
        }
        c[4] = from_next(c[0], ct);
        LDS_AS uint32_t *cw = lds_at<uint32_t>(wv);
        wave_sync();
        *(LDS_AS v4u *)(cw + 4 + 4 * lane) = v4u{c[0], c[1], c[2], c[3]};
        if (lane == 0)
            cw[260] = ct;
        // spread each odd byte over the m starts up to it
        uint64_t hi = from_next((uint32_t)odd, to) & 0xffffu;
        uint32_t span = 1;
        while (2 * span <= m) {
            odd |= odd >> span | hi << (64 - span);
            hi |= hi >> span;
            span *= 2;
        }
        if (span < m)
            odd |= odd >> (m - span) | hi << (64 - (m - span));
        // starts outside the text report nothing
        uint64_t none = 0;
        if (vb < T.lo || vb + DBLOCK - 1 > last) {
            if (v0 < T.lo)
                none = (1ull << (T.lo - v0)) - 1ull;  // lo < 16
            if (v0 + 63 > last)
                none |= v0 > last ? ~0ull : ~0ull << (last - v0) << 1;
        }
        keep = ~(odd | none);
        odd &= ~none;
    }

    // Number of ids of units [b0, b1).
    __device__ __forceinline__ uint32_t count(uint64_t b0, uint64_t b1) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        uint32_t sum = 0;
        if (b0 >= b1)
            return 0;
        v4u r[4];
        T.load((b0 >> split) * DBLOCK, lane, r);
        for (uint64_t b = b0; b < b1; ++b) {
            const uint64_t vb = (b >> split) * DBLOCK;
            uint32_t c[5];
            uint64_t keep, odd;
            block(vb, r, c, keep, odd);
            if (b + 1 < b1)
                T.load(((b + 1) >> split) * DBLOCK, lane, r);
            if (!in_part(b, lane))
                keep = odd = 0;
#pragma unroll
            for (uint32_t s = 0; s < 64; ++s) {
                const uint32_t k = s >> 4, sub = 2 * (s & 15);
                const uint32_t x = sub ? __builtin_amdgcn_alignbit(c[k + 1], c[k], sub) : c[k];
                const uint32_t w = *(lds_cptr<uint32_t>)lds_at<const uint8_t>(DTAB_OFF + ((x >> 1) & amask));
                const uint32_t kh = s < 32 ? (uint32_t)keep : (uint32_t)(keep >> 32);
                sum = __umul24(__builtin_amdgcn_ubfe(w, x << 2, 4), __builtin_amdgcn_ubfe(kh, s & 31, 1)) + sum;
            }
            if (a.odd_bytes) {
                wave_sync();
                uint32_t incl, tot;
                uint64_t hit = odd_hits(odd, incl, tot);
                if (tot > 64) {
                    // a run of odd characters: each lane its own, two at a time
                    while (hit) {
                        uint64_t v[2];
                        uint32_t code[2], s[2], n[2];
                        bool on[2];
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            const uint32_t p = 64 * lane + (hit ? (uint32_t)__builtin_ctzll(hit) : 0u);
                            on[k] = hit != 0;
                            v[k] = vb + p;
                            code[k] = code_at(p);
                            s[k] = n[k] = 0;
                            hit &= hit - 1;
                        }
                        odd_strings<2>(v, code, on, s, n);
                        sum += n[0] + n[1];
                    }
                } else if (tot) {
                    uint32_t s, n;
                    odd_few(vb, hit, incl, tot, s, n);
                    sum += n;
                }
            }
        }
        return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(sum), 63);
    }

    __device__ __forceinline__ uint32_t cmask() const { return (1u << (2 * a.m)) - 1u; }

    // The pairs of a round's first `many` <= 64 K items.
    template <int K>
    __device__ __forceinline__ static void write_items(GLB_AS v2u *at, LDS_AS uint32_t *item, glb_cptr<uint32_t> ids,
                                                       uint32_t many, uint32_t pos)
    {
        const uint32_t lane = threadIdx.x & 63u;
        // (the last lanes of the last run write the last pair again)
        uint32_t it[K], id[K], at_[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            at_[k] = min(lane + 64 * k, many - 1);
            it[k] = item[at_[k]];
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
            id[k] = ids[it[k] >> 8];
#pragma unroll
        for (int k = 0; k < K; ++k)
            at[at_[k]] = v2u{pos + (it[k] & 255u), id[k]};
    }

    // The pairs of units [b0, b1) from output slot o on.
    __device__ __forceinline__ void write(uint64_t b0, uint64_t b1, mpm_match *out_, uint64_t cap, uint64_t o) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        LDS_AS uint32_t *cw = lds_at<uint32_t>(wv);
        LDS_AS uint32_t *item = lds_at<uint32_t>(wv + DW_ITEMS), *list = lds_at<uint32_t>(wv + DW_LIST);
        GLB_AS v2u *out = (GLB_AS v2u *)out_;
        glb_cptr<uint32_t> ids = (glb_cptr<uint32_t>)a.ids;
        v4u r[4];
        T.load((b0 >> split) * DBLOCK, lane, r);
        for (uint64_t b = b0; b < b1; ++b) {
            const uint64_t vb = (b >> split) * DBLOCK;
            uint32_t c[5];
            uint64_t keep, odd;
            block(vb, r, c, keep, odd);
            if (b + 1 < b1)
                T.load(((b + 1) >> split) * DBLOCK, lane, r);
            // the block's odd strings; more than the list holds are looked up
            // again where they are needed
            uint32_t nodd = 0;
            if (a.odd_bytes) {
                wave_sync();
                uint32_t incl;
                odd = odd_hits(in_part(b, lane) ? odd : 0, incl, nodd);
                if (nodd && nodd <= 64) {
                    uint32_t s, n;
                    odd_few(vb, odd, incl, nodd, s, n);
                    list[64 + lane] = s;
                    list[128 + lane] = n;
                }
                lds_at<uint64_t>(wv + DW_ODD)[lane] = odd;
            }
            lds_at<uint64_t>(wv + DW_KEEP)[lane] = keep;
            wave_sync();
#pragma unroll 1
            for (uint32_t i = ((uint32_t)b & ((1u << split) - 1u)) << (4 - split), e = i + (16u >> split); i < e; ++i) {
                // positions 256 i + 4 lane + k of the block
                const uint32_t wi = 4 + 16 * i + (lane >> 2);
                const uint32_t x = __builtin_amdgcn_alignbit(cw[wi + 1], cw[wi], 8 * (lane & 3u));
                const uint32_t bit = 32 * i + (lane >> 1), nb = 4 * (lane & 1u);
                const uint32_t kp = (uint32_t)lds_at<const uint8_t>(wv + DW_KEEP)[bit] >> nb;
                uint32_t s[4], n[4];
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    const uint32_t y = x >> (2 * k), off = (y >> 1) & amask;
                    const uint32_t w = *(lds_cptr<uint32_t>)lds_at<const uint8_t>(DTAB_OFF + off);
                    const uint32_t base = *(lds_cptr<uint32_t>)lds_at<const uint8_t>(DTAB_OFF + a.table_bytes + off);
                    const uint32_t f = (y << 2) & 31u;
                    s[k] = __builtin_amdgcn_udot8(w & ((1u << f) - 1u), 0x11111111u, base, false);
                    n[k] = __builtin_amdgcn_ubfe(w, f, 4) & (uint32_t)__builtin_amdgcn_sbfe((int)kp, k, 1);
                }
                if (nodd) {
                    const uint32_t od = ((uint32_t)lds_at<const uint8_t>(wv + DW_ODD)[bit] >> nb) & 15u;
                    if (__ballot(od != 0)) {
                        if (nodd <= 64) {
                            for (uint32_t j = 0; j < nodd; ++j) {
                                const uint32_t rel = list[j] - (256 * i + 4 * lane);
#pragma unroll
                                for (uint32_t k = 0; k < 4; ++k)
                                    if (rel == k) {
                                        s[k] = list[64 + j];
                                        n[k] = list[128 + j];
                                    }
                            }
                        } else {
#pragma unroll
                            for (uint32_t k = 0; k < 4; k += 2) {
                                const uint64_t v = vb + 256 * i + 4 * lane + k;
                                const uint64_t vs[2] = {v, v + 1};
                                const uint32_t code[2] = {(x >> (2 * k)) & cmask(), (x >> (2 * k + 2)) & cmask()};
                                const bool on[2] = {(od >> k & 1u) != 0, (od >> k & 2u) != 0};
                                uint32_t s2[2] = {s[k], s[k + 1]}, n2[2] = {n[k], n[k + 1]};
                                odd_strings<2>(vs, code, on, s2, n2);
                                s[k] = s2[0], s[k + 1] = s2[1];
                                n[k] = n2[0], n[k + 1] = n2[1];
                            }
                        }
                    }
                }
                const uint32_t mine = n[0] + n[1] + n[2] + n[3];
                const uint32_t incl = wave_incl_sum(mine);
                const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                const uint32_t pos = (uint32_t)(vb + 256 * i - T.lo);
                const uint64_t deep = __ballot(max(max(n[0], n[1]), max(n[2], n[3])) > 2);
                for (uint32_t win = 0; win < total; win += DITEMS) {
                    wave_sync();
                    int32_t q = (int32_t)(incl - mine - win);  // of [0, DITEMS): this window's place
                    if (total <= DITEMS) {
#pragma unroll
                        for (uint32_t k = 0; k < 4; ++k) {
                            // (lanes without an item write to a spare slot:
                            // a select costs less than a branch)
                            const uint32_t v = s[k] << 8 | (4 * lane + k);
                            item[n[k] > 0 ? q : DITEMS + lane] = v;
                            item[n[k] > 1 ? q + 1 : DITEMS + lane] = v + 256;
                            if (deep)
                                for (uint32_t t = 2; t < n[k]; ++t)
                                    item[q + t] = v + 256 * t;
                            q += n[k];
                        }
                    } else {
#pragma unroll
                        for (uint32_t k = 0; k < 4; ++k) {
                            // (the ids of this window alone: an odd string may have thousands)
                            const int32_t te = min((int32_t)n[k], (int32_t)DITEMS - q);
                            for (int32_t t = max(0, -q); t < te; ++t)
                                item[q + t] = (s[k] + (uint32_t)t) << 8 | (4 * lane + k);
                            q += (int32_t)n[k];
                        }
                    }
                    wave_sync();
                    // pairs of this window to write (the capacity cuts the list)
                    const uint64_t room = cap - o > win ? cap - o - win : 0;
                    const uint32_t many = (uint32_t)min((uint64_t)min(total - win, DITEMS), room);
                    GLB_AS v2u *at = out + o + win;
                    // the ids of all runs of 64 pairs requested together
                    if (many > 384)
                        write_items<8>(at, item, ids, many, pos);
                    else if (many > 256)
                        write_items<6>(at, item, ids, many, pos);
                    else if (many > 128)
                        write_items<4>(at, item, ids, many, pos);
                    else if (many)
                        write_items<2>(at, item, ids, many, pos);
                }
                o += total;
                if (o >= cap)
                    return;
            }
        }
    }
};

constexpr int W = 1024;
__global__ __launch_bounds__(W) void direct_kernel(DirectDev a, ScanDev sd, GramShare share, uint32_t split)
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
    copy_to_lds<W>(DTAB_OFF, (const uint8_t *)a.table, 2 * a.table_bytes);
    DirectScan sc;
    sc.obits = DTAB_OFF + 2 * a.table_bytes;
    copy_to_lds<W>(sc.obits, (const uint8_t *)a.odd_bits, a.odd_bytes);
    sc.a = a;
    sc.wv = sc.obits + a.odd_bytes + wave * DW_BYTES;
    const uint64_t addr = (uint64_t)(uintptr_t)sd.single.text;
    sc.T.lo = (uint32_t)(addr & 15u);
    sc.T.p = (glb_cptr<uint8_t>)(sd.single.text - sc.T.lo);
    sc.T.hi = sd.single.n + sc.T.lo;
    sc.last = sc.T.hi - a.m;
    sc.split = split;
    sc.amask = ((1u << (2 * a.m - 3)) - 1u) << 2;

    while (true) {
        __syncthreads();
        const uint64_t g = uniform64(s_tile);
        if (g >= sd.ntiles)
            break;
        const uint64_t b0 = share.first(g * NW + wave), b1 = share.first(g * NW + wave + 1);
        const uint32_t n = sc.count(hidden(b0), b1);
        const uint64_t o = wave_offset<W>(n, s_scan, sd.status, g, sd.ntiles, sd.single.total, s_epoch,
                                          &hdr[WS_ERR]);
        if (n && o < sd.single.cap)
            sc.write(hidden(b0), b1, sd.single.out, sd.single.cap, o);
        if (gridDim.x >= sd.ntiles)  // one chunk per workgroup
            break;
        if (threadIdx.x == 0)
            s_tile = take_ticket(hdr);
    }
    if (gridDim.x == sd.ntiles && sd.ntiles <= WIDE_CHUNKS) {
        if (threadIdx.x == 0 && s_tile + 1 == sd.ntiles)
            finish_wide(hdr, s_epoch);
        return;
    }
    finish_launch(hdr, s_epoch);
}

}  // namespace

// Launch shape for a text of n bytes that starts lo bytes past a 16-byte boundary.
bool direct_config(const mpm_index *ix, const mpm_variant *v, uint64_t n, uint32_t lo, GramCfg *g)
{
    const mpm_index::Direct &D = ix->direct;
    const DeviceLimits lim = limits();
    // Texts of fewer blocks than the GPU has waves share each block between
    // up to sixteen waves: a block's sixteen rounds take about 20 us one
    // after another (4 MiB, d = 10k: 35 us with four waves, 52 with one).
    const uint64_t nblocks = (n + lo + DBLOCK - 1) / DBLOCK;
    const uint32_t nw = W / 64;
    g->split = 0;
    while (g->split < 4 && nblocks << g->split <= 8ull * lim.cus)
        g->split++;
    g->W = W;
    g->nblocks = nblocks << g->split;
    g->hits = 0;
    g->wave_bytes = DW_BYTES;
    g->lds_bytes = DTAB_OFF + 2 * D.table_bytes + D.odd_bytes + nw * DW_BYTES;
    if (g->lds_bytes > (uint32_t)lim.max_lds)
        return false;
    (void)hipFuncSetAttribute((const void *)direct_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)g->lds_bytes);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)direct_kernel, W, g->lds_bytes) !=
            hipSuccess ||
        nb <= 0)
        nb = 1;
    const uint64_t slots = (uint64_t)nb * lim.cus;
    const uint64_t units = std::min<uint64_t>(256, (g->nblocks + slots * nw - 1) / (slots * nw));
    g->nchunks = (g->nblocks + units * nw - 1) / (units * nw);
    g->nchunks = std::min((g->nchunks + slots - 1) / slots * slots, (g->nblocks + nw - 1) / nw);
    g->share = gram_share(g->nblocks, g->nchunks * nw);
    const uint64_t grid = v && v->grid ? v->grid : slots;
    g->grid = (uint32_t)std::max<uint64_t>(1, std::min(grid, g->nchunks));
    // a wave's count of ids stays in 32 bits
    return (units * DBLOCK + 16) * std::max<uint64_t>(1, ix->max_dup) < (1ull << 32);
}

mpm_status direct_launch(const mpm_index *ix, const GramCfg &g, const ScanDev &sd, void *stream)
{
    const mpm_index::Direct &D = ix->direct;
    DirectDev a;
    memset(&a, 0, sizeof a);
    const uint8_t *img = ix->d_image;
    a.table = (const uint32_t *)(img + D.off_table);
    a.odd_bits = (const uint32_t *)(img + D.off_bits);
    a.odd_words = (const uint2 *)(img + D.off_words);
    a.odd_ents = (const OddEnt *)(img + D.off_ents);
    a.ids = (const uint32_t *)(img + D.off_ids);
    a.table_bytes = D.table_bytes;
    a.odd_bytes = D.odd_bytes;
    a.m = ix->m;
    a.code_shift = D.code_shift;
    a.main4 = D.main4;
    ScanDev s = sd;
    s.ntiles = g.nchunks;
    GramShare share = g.share;
    uint32_t split = g.split;
    void *args[] = {&a, &s, &share, &split};
    const hipError_t e = hipLaunchKernel((const void *)direct_kernel, dim3(g.grid), dim3(g.W), args, g.lds_bytes,
                                         (hipStream_t)stream);
    if (e != hipSuccess)
        return fail(MPM_EHIP, "scan launch: %s", hipGetErrorString(e));
    return MPM_OK;
}

}  // namespace mpm
