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
//      ds_read, two shifts, one v_alignbit to collect the bit.
//   3. The block's candidates, in text order, are dealt to the lanes 64 at a
//      time; each walks its gram's chain of (string, offset) entries and
//      compares the codes of the string's first 16 characters.
//   4. What remains is compared byte by byte, 16 bytes per step; occurrences
//      go to a list in LDS in text order (ballots keep the order).
//   5. Per chunk: wave counts -> workgroup offsets -> decoupled look-back, as
//      the walkers do, then the wave writes its pairs 64 at a time. A wave
//      whose list overflows runs its part again and writes as it goes.
//
// Steps 1 and 2 cost about 1 + 6 / t vector instructions per byte of a lane,
// step 3 about 120 per 64 candidates: for 1,000 strings of 16 characters
// (t = 8, q = 9, one candidate per 260 bytes) that is below what HBM asks for.
//
// Measured (EST-shaped text, walkers before, filter after, us): 256 MiB,
// d = 1000, m = 16: AC 102 -> 67, WM 100 -> 67 (4.0 TB/s of text); 128 MiB,
// d = 10k, m = 16, AC 366 -> 48; 64 MiB, d = 100k, m = 16, WM 3577 -> 109;
// 64 MiB, d = 1000, m = 8 with counts, WM 422 -> 99; 128 MiB, lengths 8-32,
// AC 135 -> 69; 32 MiB, lengths 8-32, WM 2132 -> 30.
#include "mpm_gram.h"

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

// One wave's blocks [b0, b1). direct = false: count, keep the first `hcap`
// occurrences in LDS; nh and nid (ids, summed over lanes) come back. direct =
// true: write every pair from slot o on.
template <int TL, bool Var>
struct GramScan {
    static constexpr uint32_t T = 1u << TL;
    static constexpr uint32_t NS = (16u * GN) >> TL;  // samples per lane and block
    static constexpr uint32_t NM = (NS + 31) / 32;          // words of sample bits
    GramDev a;
    View text;
    IdMap im;
    uint32_t wv;    // LDS offset of this wave's buffers
    uint32_t hcap;
    uint32_t amask, bsh, wmask;

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
            uint32_t tot;
            const uint32_t pre = wave_excl_sum(cnt, tot);
#pragma unroll 1
            for (uint32_t win = 0; win < tot; win += 64) {
                wave_sync();
                uint32_t rk = pre - win;  // below 64: this window's slot
#pragma unroll
                for (uint32_t h = 0; h < NM; ++h)
                    for (uint32_t mm = mk[h]; mm; mm &= mm - 1, ++rk)
                        if (rk < 64)
                            slot[rk] = lane * NS + 32 * h + (uint32_t)__builtin_ctz(mm);
                wave_sync();
                const bool active = lane < tot - win;
                uint32_t p = 0, code = 0, pv = 0;
                if (active) {
                    p = slot[lane] << TL;  // sample, relative to the block
                    const uint32_t wi = p >> 4, sub = 2 * (p & 15);
                    const uint32_t A = cw[3 + wi], B = cw[4 + wi], C = cw[5 + wi];
                    code = __builtin_amdgcn_alignbit(C, B, sub);
                    pv = __builtin_amdgcn_alignbit(B, A, sub);
                }
                candidates(direct, b * GBLOCK, active, p, code, pv, nh, nid, last, out, cap, o);
            }
        }
    }

    // One batch of candidates, one per active lane in text order.
    __device__ __forceinline__ void candidates(bool direct, uint64_t base, bool active, uint32_t p, uint32_t code,
                                               uint32_t pv, uint32_t &nh, uint32_t &nid, uint32_t &last,
                                               mpm_match *out, uint64_t cap, uint64_t &o) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        uint32_t head = 0xffffffffu;
        if (active) {
            const uint2 w = a.words[code & wmask];
            head = w.y + __popc(w.x & ((1u << ((code >> (bsh - 2)) & 31u)) - 1u));
        }
        // chain entries whose first codes agree
        uint32_t nm = 0, fm = 0;
        for (uint32_t i = head; i != 0xffffffffu;) {
            const v4u e = *((glb_cptr<v4u>)a.ents + i);  // key, mask, meta, next
            if (((window_code(code, pv, e.z & 15u) ^ e.x) & e.y) == 0) {
                if (nm == 0)
                    fm = e.z;
                ++nm;
            }
            i = e.w;
        }
        if (__ballot(nm != 0) == 0)
            return;
        const bool single = __ballot(nm > 1) == 0;
        LDS_AS v2u *item = lds_at<v2u>(wv + WV_ITEMS);
        uint32_t tot = 0, pre = 0;
        if (!single)
            pre = wave_excl_sum(nm, tot);
        uint32_t iw = 0;
#pragma unroll 1
        do {
            bool act = nm != 0;
            v2u it = {p + BIAS - (fm & 15u), fm >> 4};
            if (!single) {
                // lanes with several agreeing entries: deal them out in order
                wave_sync();
                uint32_t k = pre - iw;
                if (nm)
                    for (uint32_t i = head; i != 0xffffffffu;) {
                        const v4u e = *((glb_cptr<v4u>)a.ents + i);
                        if (((window_code(code, pv, e.z & 15u) ^ e.x) & e.y) == 0) {
                            if (k < 64)
                                item[k] = v2u{p + BIAS - (e.z & 15u), e.z >> 4};
                            ++k;
                        }
                        i = e.w;
                    }
                wave_sync();
                act = lane < min(64u, tot - iw);
                it = item[lane];
            }
            check(direct, act, base + it.x - BIAS, it.y, nh, nid, last, out, cap, o);
            iw += 64;
        } while (iw < tot);
    }

    // Bytewise check of one (start, string) per active lane, in text order.
    __device__ __forceinline__ void check(bool direct, bool act, uint64_t sv, uint32_t u, uint32_t &nh, uint32_t &nid,
                                          uint32_t &last, mpm_match *out, uint64_t cap, uint64_t &o) const
    {
        bool hit = false;
        // (a start before the text wraps below zero and fails here too)
        if (act && (int64_t)sv >= (int64_t)text.lo) {
            const uint2 st = a.strs[u];
            hit = sv + st.y <= text.hi && equal(sv, st.x, st.y);
        }
        emit(direct, hit, sv, u, nh, nid, last, out, cap, o);
    }
};

template <int W, int TL, bool Var>
__global__ __launch_bounds__(W) void gram_kernel(GramDev a, ScanDev sd, uint32_t blocks, uint64_t nblocks,
                                                 uint32_t hits, uint32_t wave_bytes)
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
    const uint32_t lane = threadIdx.x & 63u;

    if (threadIdx.x == 0) {
        s_tile = take_ticket(hdr);
        s_epoch = __hip_atomic_load(&hdr[WS_EPOCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    copy_to_lds<W>(GBITS_OFF, (const uint8_t *)a.bits, a.bit_bytes);
    load_groups(a.grp);

    GramScan<TL, Var> sc;
    sc.a = a;
    const uint64_t addr = (uint64_t)(uintptr_t)sd.single.text;
    sc.text.lo = (uint32_t)(addr & 15u);
    sc.text.p = (glb_cptr<uint8_t>)(sd.single.text - sc.text.lo);
    sc.text.hi = sd.single.n + sc.text.lo;
    sc.im.uoff = (glb_cptr<uint32_t>)a.uoff;
    sc.im.uids = (glb_cptr<uint32_t>)a.uids;
    sc.im.lds_uoff = 0;
    sc.im.lds_uids = 0;
    sc.im.dupfree = 0;
    sc.im.n_single = a.n_single;
    sc.wv = GBITS_OFF + a.bit_bytes + wave * wave_bytes;
    sc.hcap = hits;
    sc.wmask = (1u << (2 * a.q - 5)) - 1u;
    sc.amask = sc.wmask << 2;
    sc.bsh = 2 * a.q - 3;
    const uint64_t ntiles = sd.ntiles;
    const uint64_t cap = sd.single.cap;

    while (true) {
        __syncthreads();
        const uint64_t g = uniform64(s_tile);
        if (g >= ntiles)
            break;
        const uint64_t b0 = min((g * NW + wave) * blocks, nblocks);
        const uint64_t b1 = min(b0 + blocks, nblocks);
        uint32_t nh, nid;
        uint64_t o = 0;
#pragma unroll 1
        for (uint32_t pass = 0; pass < 2; ++pass) {
            sc.run(pass != 0, hidden(b0), b1, nh, nid, sd.single.out, cap, o);
            if (pass)
                break;
#pragma unroll
            for (int k = 32; k >= 1; k >>= 1)
                nid += __shfl_xor(nid, k, 64);
            o = wave_offset<W>(nid, s_scan, sd.status, g, ntiles, sd.single.total, s_epoch | GRAM_EPOCH,
                               &hdr[WS_ERR]);
            if (nh == 0 || o >= cap)
                break;
            if (nh <= hits) {
                wave_sync();
                for (uint32_t r = 0; r < nh && o < cap; r += 64) {
                    const bool act = r + lane < nh;
                    v2u h = {0, 0};
                    if (act)
                        h = lds_at<v2u>(sc.wv + WV_HITS)[r + lane];
                    write_hits(sd.single.out, cap, o, act, h.x, h.y, sc.im);
                }
                break;
            }
        }
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

const void *kernel_of(uint32_t W, uint32_t tl, bool var)
{
    return W == 256 ? pick<256>(tl, var) : pick<1024>(tl, var);
}

}  // namespace

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
    // The direct-address scan costs the same whatever the candidates; past a
    // filter cost of about 18 it is the faster one (64 MiB, m = 8: d = 5000,
    // cost 16.7, filter 155 us, direct 186; d = 6000, 18.4, 201 and 189).
    g->direct = !G.ok || (ix->direct.ok && G.cost > 18.0);
    if (g->direct)
        return direct_config(ix, v, n, lo, g);
    const DeviceLimits lim = limits();
    // Workgroups of 1024 threads share one copy of the bits between 16 waves;
    // texts that would leave CUs without work are cut finer.
    const uint64_t nblocks = (n + lo + GBLOCK - 1) / GBLOCK;
    const uint32_t W = nblocks >= 16ull * lim.cus ? 1024 : 256;
    const uint32_t nw = W / 64;
    // the occurrence lists: all the LDS that is left to 16 waves (their
    // registers admit no second workgroup), 256 occurrences per wave of a
    // small workgroup
    const uint32_t room = (uint32_t)lim.max_lds - GBITS_OFF - G.bit_bytes;
    if (room / nw < WV_HITS + 16 * 8)
        return false;
    uint32_t hits = (room / nw - WV_HITS) / 8;
    hits = std::min<uint32_t>(hits, W == 1024 ? 1024 : 256) & ~1u;
    g->nblocks = nblocks;
    g->W = W;
    g->hits = hits;
    g->wave_bytes = WV_HITS + 8 * hits;
    g->lds_bytes = GBITS_OFF + G.bit_bytes + nw * g->wave_bytes;
    if (g->lds_bytes > (uint32_t)lim.max_lds)
        return false;
    const void *k = kernel_of(W, G.t_log, ix->var != 0);
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
    g->blocks = (uint32_t)blocks;
    g->nchunks = (nblocks + blocks * nw - 1) / (blocks * nw);
    uint64_t grid = v && v->grid ? v->grid : slots;
    g->grid = (uint32_t)std::max<uint64_t>(1, std::min(grid, g->nchunks));
    // a wave's count of ids stays in 32 bits
    return (uint64_t)(blocks * GBLOCK + 16) * std::max<uint64_t>(1, ix->max_dup) < (1ull << 32);
}

mpm_status gram_launch(const mpm_index *ix, const GramCfg &g, const ScanDev &sd, void *stream)
{
    if (g.direct)
        return direct_launch(ix, g, sd, stream);
    const mpm_index::Gram &G = ix->gram;
    GramDev a;
    const uint8_t *img = ix->d_image;
    a.bits = (const uint32_t *)(img + G.off_bits);
    a.words = (const uint2 *)(img + G.off_words);
    a.ents = (const GramEnt *)(img + G.off_ents);
    a.strs = (const uint2 *)(img + G.off_strs);
    a.rows = img + G.off_rows;
    id_csr(ix, &a.uoff, &a.uids);
    a.q = G.q;
    a.t_log = G.t_log;
    a.code_shift = G.code_shift;
    a.bit_bytes = G.bit_bytes;
    a.m = ix->m;
    a.n_single = ix->n_single;
    a.grp = id_groups(ix);
    ScanDev s = sd;
    s.ntiles = g.nchunks;
    uint32_t blocks = g.blocks, hits = g.hits, wave_bytes = g.wave_bytes;
    uint64_t nblocks = g.nblocks;
    void *args[] = {&a, &s, &blocks, &nblocks, &hits, &wave_bytes};
    const hipError_t e = hipLaunchKernel(kernel_of(g.W, G.t_log, ix->var != 0), dim3(g.grid), dim3(g.W),
                                         args, g.lds_bytes, (hipStream_t)stream);
    if (e != hipSuccess)
        return fail(MPM_EHIP, "scan launch: %s", hipGetErrorString(e));
    return MPM_OK;
}

}  // namespace mpm
