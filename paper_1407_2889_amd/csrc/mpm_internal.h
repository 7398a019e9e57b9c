// Internal declarations shared by the host builders (mpm_host.cpp) and the
// scan kernels (mpm_scan.hip). Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/mpm.h"

namespace mpm {

// ---------------------------------------------------------------------------
// Kernel-argument descriptors (passed by value)
// ---------------------------------------------------------------------------

// Bytes at the start of a scan kernel's LDS before the matching tables: the
// per-workgroup header (with the id groups below) and the byte-class map.
static const uint32_t LDS_FIXED_BYTES = 1536;

// Distinct strings numbered by their id count: strings below n_single have
// one id (at CSR slot u); then groups k < n of strings sharing a count: group
// k holds strings [u0[k], u0[k + 1]) with cnt[k] ids each, the first one's
// ids from CSR slot off[k]. Strings from u0[n] on (past the groups kept
// here) read the CSR offsets.
static const int ID_GROUPS = 8;
struct IdGroups {
    uint32_t n;
    uint32_t u0[ID_GROUPS + 1];
    uint32_t cnt[ID_GROUPS];
    uint32_t off[ID_GROUPS];
};

// Dense Aho-Corasick table. Row s holds `cp` entries: column 0 is the class of
// bytes that occur in no pattern (always leads to the root), columns 1..cp-1
// the pattern bytes in ascending order. States are numbered breadth-first, so
// the depth-m states (one per distinct pattern string, in ascending string
// order) are the last `n_unique` rows: state s is terminal iff
// s >= first_term, and then u = s - first_term is the string's rank.
struct AcDev {
    const void *dfa;        // uint16 or uint32 entries
    const uint8_t *cls;     // 256 uint16 entries: byte offset of the column within a row
    const uint32_t *uoff;   // n_unique + 1: CSR offsets into uids
    const uint32_t *uids;   // d: ascending pattern ids per distinct string
    uint32_t n_states;
    uint32_t first_term;
    uint32_t cp;            // columns per row
    uint32_t m;
    uint32_t dfa_bytes;     // bytes of the table (multiple of 16)
    uint32_t dupfree;       // every distinct string has exactly one id
    uint32_t n_single;      // distinct strings below this have one id each
    IdGroups grp;           // id count groups of the other strings
    uint32_t hot_states;    // hot placement: rows [0, hot_states) in LDS
    uint32_t hot_bytes;     // bytes of those rows (multiple of 16)
    // Goto rows (same numbering and columns as the table, all-ones for a
    // missing transition) followed by the supply link of every state, for
    // the supply-link walk; go_bytes = 0 when the index has none.
    const void *go;
    uint32_t go_bytes;      // goto rows and supply links (multiple of 16)
    uint32_t sup_off;       // byte offset of the supply links within go
    // Byte classes without a lookup table, usable when the pattern bytes
    // have distinct 3-bit codes (b >> swar_shift) & 7: perm_byte selects, per
    // code, the only byte with that code that is a pattern byte (or a byte
    // whose code differs, for unused codes); perm_col gives its column's byte
    // offset (0 for unused codes). Bytes that are not their code's pattern
    // byte take column 0.
    uint32_t swar_ok;
    uint32_t swar_shift;
    uint32_t perm_byte_lo, perm_byte_hi, perm_col_lo, perm_col_hi;
    // Sets of different lengths: the table is the automaton of the reversed
    // strings, walked from a range's end to its start; a state s >=
    // first_term reports string term_u[s - first_term] (null for one length).
    const uint32_t *term_u;
    uint32_t m_max;         // longest string (m: the shortest)
};

// Wu-Manber tables. Characters map to 2-bit codes (c >> code_shift) & 3; a
// string of k characters hashes to sum_j code(c_j) << 2j (first character
// in the low bits). SHIFT is stored per block hash as a uint16: the shift
// when positive, else 0x8000 | bucket. Bucket b lists, in ascending order,
// the distinct strings whose last block hashes to that value
// (bu[boff[b] .. boff[b+1])), each with a filter key: the hash of the
// key_len characters just before its last block.
struct WmDev {
    const uint8_t *tables;  // shift16 | boff | bkey | bu, contiguous (table_bytes)
    uint32_t off_boff, off_bkey, off_bu;  // byte offsets inside `tables`
    const uint8_t *pats;    // distinct strings, n_unique * m bytes, ascending
    const uint32_t *uoff;
    const uint32_t *uids;
    uint32_t B;
    uint32_t code_shift;
    uint32_t m;
    uint32_t key_len;
    uint32_t table_bytes;
    uint32_t dupfree;
    uint32_t n_single;
    uint32_t shift_bytes;   // bytes of SHIFT at the start of `tables` (multiple of 16)
    IdGroups grp;
    // Sets of different lengths (var != 0): m is the shortest length, the
    // window; string u is pats[upoff[u] .. upoff[u + 1]) and buckets list
    // longer strings first. Null for one length.
    const uint32_t *upoff;
    uint32_t var;
};

// q-gram filter tables (mpm_gram.cpp), kept for either index kind when the
// set is sparse enough. Characters map to 2-bit codes (c >> code_shift) & 3,
// k characters to sum_j code(c_j) << 2j. Sampled text positions are the
// multiples of t = 1 << t_log; a sample is a candidate when the q-gram that
// starts there occurs in a string at one of the offsets 0 .. t - 1, which
// `bits` records (word = low 2q - 5 bits of the gram, bit = its upper five).
// Every occurrence covers a whole sampled q-gram at such an offset, because
// t + q - 1 <= m.
struct GramEnt {      // one (string, offset) of a gram
    uint32_t key;     // codes of the string's first characters (at most 16)
    uint32_t mask;    // the bits of key that count
    uint32_t meta;    // string << 5 | plain << 4 | offset; plain: the string has at most 16
                      // characters, all strings have its length, and each of them is
                      // the main byte of its code, so that key tells the bytes
    uint32_t next;    // next entry of the same gram (all ones: none)
};
struct GramWalk {     // an Aho-Corasick index's automaton, for crowded blocks; kept in the image
    uint64_t self, dfa, cls, term;  // byte offsets in the image: this struct, the table, the columns, term_u
    uint32_t rowb;        // bytes of a table row
    uint32_t first_term;
    uint32_t wide;        // 32-bit table entries
    uint32_t past;        // bytes a walk reads past its starting positions
};
struct GramDev {
    const uint32_t *bits;     // 4^q bits, copied to LDS
    const uint32_t *ranks;    // behind them: grams before each word of bits
    const GramEnt *ents;      // the first entry of gram number k at k, the others after them;
                              // a chain's offsets descend, longer strings first
    const uint2 *strs;        // per string: first 16-byte row, length
    const uint8_t *rows;      // the strings, each padded to whole 16-byte rows
    const uint32_t *uoff;
    const uint32_t *uids;
    uint32_t q, t_log, code_shift;
    uint32_t bit_bytes;       // bytes copied to LDS (multiple of 16)
    uint32_t rank_off;        // where the ranks start there (0: not copied)
    uint32_t pair_off;        // where the two-position answers start there (0: not copied)
    uint32_t main4;           // main byte of code k in byte k
    uint32_t m;               // shortest string
    uint32_t n_single;
    uint32_t crowd;           // candidates of a block past which it is walked (all ones: no automaton)
    const GramWalk *walk;
    IdGroups grp;
};

// Direct-address tables of a set with 2 <= m <= 8 (mpm_gram.cpp), for the
// strings made of each code's main byte: per window of m codes the number of
// its ids (four bits, eight windows to a word), then per word the first id
// slot of its windows; ids in window order. The other strings ("odd") have a
// bit per window code (word = code >> 5) and a chain of 8-byte strings.
struct OddEnt {
    uint64_t bytes;   // the string, zero padded
    uint32_t first;   // its ids: [first, first + count)
    uint32_t count;
    uint32_t next;    // next entry of the same code (all ones: none)
    uint32_t pad;
};
struct DirectDev {
    const uint32_t *table;      // counts, then slots: table_bytes each, copied to LDS
    const uint32_t *odd_bits;   // 4^m bits, copied to LDS
    const uint2 *odd_words;     // per word of odd_bits: (the word, codes before it)
    const OddEnt *odd_ents;
    const uint32_t *ids;
    uint32_t table_bytes, odd_bytes;  // multiples of 16; odd_bytes 0: no odd strings
    uint32_t m, code_shift;
    uint32_t main4;             // main byte of code k in byte k (a byte of another code: none)
};

// One text of a launch. Tiles of a launch are numbered globally; a text
// owns tiles [tile_begin, tile_begin + ntiles).
struct TextDesc {
    const uint8_t *text;
    uint64_t n;
    mpm_match *out;
    uint64_t cap;
    uint64_t *total;
    uint64_t tile_begin;
    uint64_t ntiles;
};

// Workspace header words (uint32): ticket counter, finished-workgroup
// counter, launch epoch, device error flag. Followed (at byte 64) by one
// uint64 look-back status word per tile, then (256-byte aligned) by the
// staging area: per workgroup, `stage_cap` slots for each of its virtual
// lanes, slot j of virtual lane v at (j * lanes + v), one (position, string)
// pair each. A lane keeps its first occurrences in registers, stages the next
// stage_cap ones there, and walks its range again only past those.
enum { WS_TICKET = 0, WS_DONE = 1, WS_EPOCH = 2, WS_ERR = 3 };
// Device error flag bits.
enum { WS_ERR_LOOKBACK = 1u, WS_ERR_LDS_LAYOUT = 2u };
static const uint64_t WS_HEADER_BYTES = 64;

struct ScanDev {
    TextDesc single;          // used when ntexts == 1
    const TextDesc *multi;    // device array when ntexts > 1
    uint32_t ntexts;
    uint32_t lane_bytes;
    uint64_t ntiles;
    uint32_t *hdr;
    uint64_t *status;
    // The distinct-string -> id CSR copied to LDS at these byte offsets
    // (0: read from global memory), with its word counts.
    uint32_t csr_uoff_lds, csr_uids_lds;
    uint32_t csr_uoff_words, csr_uids_words;
    mpm_match *stage;     // staging area (null when stage_cap is 0)
    uint32_t stage_cap;   // staged occurrences per virtual lane
    uint32_t mark_lds;    // dense output: LDS byte offset of the position marks
};

// Batched launches: one descriptor per text (in queue order) and one per
// index. kind selects the walker; BK_SWAR marks AC byte classes computed in
// registers.
enum {
    BK_AC16_LDS = 0,
    BK_AC16_GLB = 1,
    BK_AC32_GLB = 2,
    BK_WM_LDS = 3,
    BK_WM_GLB = 4,
    BK_AC16_HOT = 5,
    BK_WM_HOT = 6,
    BK_AC32_HOT = 7,
    BK_GRAM = 8,   // the q-gram filter (its own kernel and descriptors)
    BK_WALK_MASK = 0x7f,
    BK_SWAR = 0x80
};

struct BatchIndex {
    AcDev ac;
    WmDev wm;
};

struct BatchText {
    TextDesc td;
    uint32_t index;       // into the launch's BatchIndex array
    uint32_t kind;        // BK_*
    uint32_t lane_bytes;
    uint32_t pad;
    float *cost;          // per-request time share and longest chunk (null: not timed)
};

struct BatchDev {
    const BatchText *texts;
    const BatchIndex *idx;
    uint32_t ntexts;
    uint32_t pad;
    uint64_t ntiles;
    uint32_t *hdr;
    uint64_t *status;
    mpm_match *stage;     // staging area (null when stage_cap is 0)
    uint32_t stage_cap;   // staged occurrences per lane
    float us_per_tick;    // microseconds per wall-clock tick (timed requests)
};

// Filter launches: blocks [b0, b0 + nb) of a text.
struct GramPart {
    uint32_t text;        // into the launch's BatchText array
    uint32_t b0, nb;
};

struct GramBatchDev {
    const BatchText *texts;    // index: into idx; tile_begin, ntiles: the text's parts
    const GramDev *idx;
    const GramPart *parts;
    const uint2 *pieces;       // a wave's parts [x, y); 16 pieces per ticket
    const uint32_t *tickets;   // a ticket's index
    uint64_t ntickets;
    uint32_t *hdr;
    uint64_t *status;          // one word per part
    uint32_t lds_bytes;        // per workgroup
    float us_per_tick;
};

// Staged occurrences per lane: single-text scans stage a lane's whole range
// when the workspace allows; batched launches (many workspaces at once)
// stage at most this many.
static const uint32_t BATCH_STAGE_CAP = 16;

// Look-back status word: [63:38] tag, [37:36] flag, [35:0] value. The tag is
// the launch epoch with its top bit set. On a workspace that serves texts of
// different lengths, or walkers and filter scans, a status word may hold what
// an earlier scan staged there, a (position, string) pair: string numbers stay
// below 2^31, so its top bit is clear and it is no word of any epoch.
static const uint64_t ST_VAL_BITS = 36;
static const uint64_t ST_VAL_MASK = (1ull << ST_VAL_BITS) - 1;
static const uint32_t ST_TAG_BIT = 1u << 25;

}  // namespace mpm

// ---------------------------------------------------------------------------
// Host-side index
// ---------------------------------------------------------------------------
struct mpm_index {
    uint32_t algo = 0;
    uint32_t m = 0, d = 0, du = 0, max_dup = 0;
    uint32_t n_single = 0;              // distinct strings 0..n_single-1 have one id each
    std::vector<uint32_t> uoff, uids;   // distinct strings -> ids
    // Strings from n_single on come in groups sharing an id count: group k
    // starts at string grp_u0[k], its strings have grp_cnt[k] ids each, and
    // its first string's ids start at grp_off[k].
    std::vector<uint32_t> grp_u0, grp_cnt, grp_off;
    std::vector<uint8_t> upats;         // du * m, ascending strings
    // Sets of different lengths (var): m is the shortest length, m_max the
    // longest; string u is upats[upoff[u] .. upoff[u + 1]) and its id list
    // holds the ids of every pattern that is a prefix of it (those occur
    // wherever it does).
    uint32_t var = 0, m_max = 0;
    std::vector<uint32_t> upoff;
    std::vector<uint8_t> wpats;         // Wu-Manber: first m bytes of every string

    // Aho-Corasick
    uint32_t n_classes = 0;
    uint8_t class_bytes[256] = {0};
    uint16_t cls[256] = {0};         // byte -> 1 + class (0: in no pattern); up to 256 classes
    uint32_t swar_ok = 0, swar_shift = 0;
    uint8_t perm_byte[8] = {0}, perm_col[8] = {0};
    uint64_t n_states = 0;
    uint32_t state_bytes = 0;
    std::vector<uint32_t> dfa;          // n_states * (1 + n_classes)
    uint64_t first_term = 0;            // var: states from here on report a string
    std::vector<uint32_t> term_u;       // var: the string each reporting state reports

    // Wu-Manber
    uint32_t B = 0, code_shift = 0, zero_shift = 0, n_buckets = 0, key_len = 0;
    double mean_shift = 0;
    std::vector<uint8_t> shift;       // SHIFT per block hash
    std::vector<uint16_t> shift16;    // SHIFT, or 0x8000 | bucket when zero
    std::vector<uint32_t> boff, bu, bkey;

    // Device image: host copy, offsets, and the caller-owned device buffer.
    std::vector<uint8_t> image;
    uint64_t off_a = 0, off_b = 0, off_c = 0, off_d = 0, off_e = 0, off_f = 0, off_g = 0, off_h = 0;
    // Aho-Corasick goto rows and supply links (kept when asked for)
    uint32_t keep_goto = 0;
    uint64_t off_go = 0, go_bytes = 0, sup_off = 0;
    uint64_t table_bytes = 0;
    const uint8_t *d_image = nullptr;

    // q-gram filter (mpm_gram.cpp); ok = 0: the set has none
    struct Gram {
        uint32_t ok = 0, q = 0, t_log = 0, code_shift = 0, bit_bytes = 0, ranked = 0, pair_bytes = 0, main4 = 0;
        double cost = 0; // expected vector instructions per text byte (mpm_gram.cpp)
        double hit = 0;  // expected occurrences per text byte
        uint64_t off_bits = 0, off_ents = 0, off_strs = 0, off_rows = 0;
        uint32_t crowd = 0xffffffffu;
        uint64_t off_walk = 0;
    } gram;
    // direct-address table (mpm_gram.cpp); ok = 0: the set has none
    struct Direct {
        uint32_t ok = 0, code_shift = 0, main4 = 0, table_bytes = 0, odd_bytes = 0;
        uint64_t off_table = 0, off_ids = 0, off_bits = 0, off_words = 0, off_ents = 0;
    } direct;
};

namespace mpm {
void set_error(const char *fmt, ...);
mpm_status fail(mpm_status st, const char *fmt, ...);

// Launch the scan kernels (mpm_scan.hip).
struct LaunchCfg {
    uint32_t lane_bytes;
    uint32_t block_threads;
    uint32_t placement;   // resolved: LDS or GLOBAL
    uint32_t grid;        // resolved workgroup count
    uint32_t lds_bytes;   // dynamic LDS per workgroup
    bool swar;            // AC: byte classes computed in registers
    bool supply;          // AC: goto function and supply links at run time
    uint32_t ilp;         // virtual lanes per thread (1 or 2)
    uint32_t csr_lds;     // LDS byte offset of the id CSR (0: global memory)
    bool dense;           // dense output (position marks in LDS)
    uint32_t mark_lds;    // LDS byte offset of the marks (dense)
    uint32_t text_mode;   // 0: line streaming; 1: bytes from global; 2: text staged in LDS
    uint32_t text_lds;    // text_mode 2: LDS byte offset of the staged text
};
// LDS bytes of the dense output's position marks (1024 lanes x 16 positions).
static const uint32_t DENSE_MARK_BYTES = 1024 * 16 * 4;
// csr_in_lds: single-text scans may copy the id CSR to LDS (batched launches
// keep it in global memory).
mpm_status resolve_variant(const mpm_index *idx, const mpm_variant *v, uint64_t ntiles_hint,
                           LaunchCfg *cfg, bool csr_in_lds = false);
// Words of the id CSR arrays: uoff (d_unique + 1) and ids (d), each padded
// to 16 bytes.
uint32_t csr_uoff_words(const mpm_index *idx);
uint32_t csr_uids_words(const mpm_index *idx);
uint64_t tile_bytes(const LaunchCfg &cfg);
mpm_status launch_scan(const mpm_index *idx, const LaunchCfg &cfg, const ScanDev &sd,
                       void *stream);
mpm_status launch_zero_totals(uint64_t *const *d_totals_dev, uint32_t count, uint64_t *single,
                              void *stream);
// reserve: LDS bytes the launch keeps beside the tables (the hot part of an
// Aho-Corasick table shrinks by as much).
AcDev ac_dev(const mpm_index *ix, uint32_t reserve = 0);
WmDev wm_dev(const mpm_index *ix);
// Sets of different lengths (mpm_mixed.cpp, mpm_scan_var.hip).
mpm_status build_ac_rev_tables(mpm_index *ix);
const void *var_kernel(const mpm_index *ix, const LaunchCfg &c);
mpm_status var_launch(const mpm_index *ix, const LaunchCfg &c, const ScanDev &sd, void *stream);
// Text-access ladder variants (mpm_scan_ladder.hip).
const void *ladder_kernel(const mpm_index *ix, const LaunchCfg &c);
mpm_status ladder_launch(const mpm_index *ix, const LaunchCfg &c, const ScanDev &sd, void *stream);
// q-gram filter scans (mpm_gram.cpp, mpm_scan_gram.hip).
// Items (text blocks) of wave k, of a number of waves that the items are spread
// over evenly: [first(k), first(k + 1)). frac is the remainder's share in
// units of 2^-32, rounded up: first(waves) is the number of items.
struct GramShare {
    uint32_t per, frac;
    __host__ __device__ uint64_t first(uint64_t k) const { return k * per + (k * frac >> 32); }
};
inline GramShare gram_share(uint64_t items, uint64_t waves)
{
    const uint64_t rem = items % waves;
    return GramShare{(uint32_t)(items / waves), rem ? (uint32_t)((rem << 32) / waves + 1) : 0u};
}
struct GramCfg {
    uint32_t W;            // threads per workgroup
    GramShare share;       // of the waves of all chunks
    uint32_t grid;
    uint32_t lds_bytes;
    uint32_t wave_bytes;   // LDS bytes of one wave's buffers
    uint32_t hits;         // occurrences a wave keeps in LDS
    uint32_t tables_w;     // workgroup size that decides on the tables in LDS (gram_dev)
    uint64_t nblocks;      // blocks of the text
    uint64_t nchunks;
    bool direct;           // the direct-address scan
    uint32_t split;        // log2 of the waves that share a block (direct)
};
static const uint64_t GRAM_CHUNK_MIN = 4096;   // text bytes of the smallest chunk
void build_gram(mpm_index *ix);
void build_direct(mpm_index *ix);
struct DeviceLimits {
    int cus = 0;
    int max_lds = 0;
};
DeviceLimits limits();
IdGroups id_groups(const mpm_index *ix);
// The id CSR in an uploaded index's device image.
void id_csr(const mpm_index *ix, const uint32_t **uoff, const uint32_t **uids);
bool gram_takes(const mpm_index *ix, const mpm_variant *v, uint64_t n);
bool gram_config(const mpm_index *ix, const mpm_variant *v, uint64_t n, uint32_t lo, GramCfg *g);
mpm_status gram_launch(const mpm_index *ix, const GramCfg &g, const ScanDev &sd, void *stream);
// W: the launch's workgroup size; batches have workgroups of 1024 threads, but
// keep no two-position answers in LDS.
static const uint32_t GRAM_BATCH_W = 512;
GramDev gram_dev(const mpm_index *ix, uint32_t W);
struct GramPieces {
    std::vector<GramPart> parts;
    std::vector<uint2> pieces;
    std::vector<uint32_t> tickets;
};
bool gram_batch_takes(const mpm_index *ix, const mpm_variant *v, uint64_t n);
void plan_gram_batch(const std::vector<const mpm_index *> &index, std::vector<BatchText> *texts,
                     GramPieces *out, uint32_t grid_req, uint32_t *grid, uint32_t *lds_bytes);
mpm_status launch_gram_batch(const GramBatchDev &bd, uint32_t grid, void *stream);
bool direct_config(const mpm_index *ix, const mpm_variant *v, uint64_t n, uint32_t lo, GramCfg *g);
mpm_status direct_launch(const mpm_index *ix, const GramCfg &g, const ScanDev &sd, void *stream);
uint32_t batch_kind(const mpm_index *ix, const LaunchCfg &c);
// Batched launches run one kernel per walker kind (BK_*, with BK_SWAR).
uint32_t batch_grid(uint32_t kind, uint32_t W, uint32_t lds_bytes, uint64_t ntiles,
                    uint32_t grid_req);
mpm_status launch_batch(const BatchDev &bd, uint32_t kind, uint32_t W, uint32_t grid, uint32_t lds,
                        void *stream);
}  // namespace mpm
