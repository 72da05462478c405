// Internal launcher interface between the C-ABI layer (sp_api.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>
#include <stdint.h>
#include <vector>
#include "sp_common.hpp"

namespace sp {

// Segment table of a call as the FIRST parameter of its kernel: kernels that need nothing else prepared read a table of up to
// ARG_WORDS words (with the other parameters, under the 4 KB of kernel arguments) from there, larger ones from `dev`.  A launch
// that only stores the table is 5 us and the gap behind it: rotation of a 16K prompt's q and k 112.0 -> 109.9, loss over a 152K
// vocabulary 395.8 -> 390.9 (with the objective of up to 16 responses in one launch instead of two).
constexpr int ARG_WORDS = 768;
struct TabArg { const int* dev; int32_t words[ARG_WORDS]; };
inline TabArg make_tab_arg(const int32_t* words, size_t n, const int* dev) {
    TabArg t;
    t.dev = n <= (size_t)ARG_WORDS ? nullptr : dev;
    for (size_t i = 0; i < (size_t)ARG_WORDS; ++i) t.words[i] = !t.dev && i < n ? words[i] : 0;
    return t;
}
// (in the constant address space, which the compiler follows: as a generic pointer it made flat loads of what scalar loads
// serve, 0.5 ns per row of the loss, 15 % of 62 K rows of 3328 logits)
__device__ __forceinline__ const int* table_of(const TabArg& t) {
    const uint64_t at = t.dev ? (uint64_t)(uintptr_t)t.dev : (uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(TabArg, words);
    return (const int*)(const __attribute__((address_space(4))) int*)at;
}

constexpr unsigned STAGE_ROWSUM = 1u, STAGE_DKDV = 2u, STAGE_DQ = 4u;
constexpr int MAX_SETS = 4;      // tensor sets that one forward launch can serve

// Tag block at the head of every workspace (64 words).  Words 0..TAG_WORDS-1 describe the reserve a
// forward left in this workspace (magic, o and lse pointers, token count, heads, head_dim, byte offset of
// the reserve, response-rows-only flag); word TAG_FLAG_WORD is the verdict of the latest check.
constexpr int TAG_WORDS = 12;
constexpr int TAG_FLAG_WORD = 15;
constexpr uint32_t TAG_MAGIC = 0x53504152u;
struct ReserveTag { uint32_t w[TAG_WORDS]; };
// TAG_CLEAR: the workspace holds no reserve from here on.  TAG_WRITE: a forward is about to write the
// reserve that `tag` describes.  TAG_CHECK: a backward asks whether the workspace holds exactly the
// reserve `tag` describes; if not, the tag is cleared (the call is about to write into the workspace).
constexpr int TAG_CLEAR = 0, TAG_WRITE = 1, TAG_CHECK = 2;
constexpr int TAG_KEEP = -1;      // for launch_prepare: leave the tag block as it is

// What the attention kernels of a small call do themselves instead of the preparation launch: the table comes as a kernel
// argument, a wave looks its tile and its tokens' segments up in registers, and the tag block is kept by the kernels
// (forward: written by the first workgroup; backward: compared by each workgroup of the dq pass, updated by the dkdv pass).
// us, before -> after: one short group's forward 17.8 -> 15.4, two small groups' training pass 69.8 -> 66.8, one 1K prompt
// 248.9 -> 244.9, one group of 9000 tokens, 28/4 heads (1988 tiles times heads), 2419.7 -> 2411.5.  The line is at 2048 of them, beyond
// which a training pass no longer shows it (forward; training pass): 40 groups of 300, 3360 tiles times heads, 82.5 -> 80.6; 298.8 ->
// 299.1; one group of 12000, 2632, 863.6 -> 858.6; 4178.6 -> 4174.4; one of 20000, 4396, 2267 -> 2249; 9987 -> 9964.
struct SmallCall { int on; int tag_mode; ReserveTag want; uint32_t* tag; };
// Tag block maintenance by one wave (lane i = word i).  A reserve written for all rows (word 10 = 0) also serves a backward
// over response rows only (want word 10 = 1), not the reverse.
__device__ __forceinline__ bool reserve_tag_matches(const uint32_t* blk, const ReserveTag& want, int i) {
    const uint32_t have = blk[i];
    uint32_t w = 0;
#pragma unroll
    for (int k = 0; k < TAG_WORDS; ++k) if (i == k) w = want.w[k];
    bool same = i >= TAG_WORDS || have == w;
    if (i == 10) same = same || have == 0u;
    return __builtin_amdgcn_ballot_w64(!same) == 0;
}
__device__ __forceinline__ void reserve_tag_body(uint32_t* blk, const ReserveTag& want, int mode, int i) {
    if (mode == TAG_CLEAR) { blk[i] = 0u; return; }
    if (mode == TAG_WRITE) {
        uint32_t w = 0;
#pragma unroll
        for (int k = 0; k < TAG_WORDS; ++k) if (i == k) w = want.w[k];
        blk[i] = w;
        return;
    }
    const bool ok = reserve_tag_matches(blk, want, i);
    if (i < TAG_WORDS && !ok) blk[i] = 0u;
    if (i == TAG_FLAG_WORD) blk[i] = ok ? 1u : 0u;
}

// Lookups of a whole wave in a table of at most 64 groups of at most 63 responses each: a lane holds a group, or a response
// offset of the tile's group, and the searches are ballots and lane exchanges, not chains of loads.
constexpr int SMALL_CALL_TILES = 2048;      // 128-row tiles times q heads
constexpr int SMALL_GROUPS = 64, SMALL_RESPONSES = 63;
struct SmallGroup { int tok_base, Lp, Tg, G, off; };      // off: response offset `lane` of the group (lanes 0 .. G)
template <int BT>
__device__ __forceinline__ SmallGroup small_tile(const int* tab, int n_groups, int tile, int l, int& ti) {
    SmallGroup g;
    const int* e = tab + TAB_HEADER + TAB_GROUP_WORDS * min(l, n_groups - 1);
    const int tok = e[0], Lp = e[1], Tg = e[2], roff = e[3], G = e[4], before = e[BT == 256 ? TAB_TILES256 : TAB_TILES128];
    const int n = 63 - __clzll((long long)__builtin_amdgcn_ballot_w64(l < n_groups && before <= tile));   // before[0] = 0
    g.tok_base = __builtin_amdgcn_readlane(tok, n); g.Lp = __builtin_amdgcn_readlane(Lp, n);
    g.Tg = __builtin_amdgcn_readlane(Tg, n); g.G = __builtin_amdgcn_readlane(G, n);
    ti = tile - __builtin_amdgcn_readlane(before, n);
    g.off = tab[__builtin_amdgcn_readlane(roff, n) + min(l, g.G)];
    return g;
}
// the response that holds token t >= Lp (its start and end by lane): the last offset ahead of the end that is at most t
__device__ __forceinline__ void small_segment(const SmallGroup& g, int t, int& st, int& en) {
    int pos = 0;
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1) {
        const int at = pos + step, x = __shfl(g.off, at & 63, 64);
        if (at < g.G && x <= t) pos = at;
    }
    st = __shfl(g.off, pos, 64);
    en = __shfl(g.off, pos + 1, 64);
}

struct Problem {
    const void* q; const void* k; const void* v;
    const void* o; const float* lse; const void* d_o;     // backward inputs (o also fwd output)
    void* o_out; float* lse_out;                          // forward outputs
    // forward over several tensor sets that share one packing (n_sets > 1): set i reads qs/ks/vs[i]
    // and writes os/lses[i]; with n_sets <= 1 the single-set fields above are used
    int n_sets;
    const void* qs[MAX_SETS]; const void* ks[MAX_SETS]; const void* vs[MAX_SETS];
    void* os[MAX_SETS]; float* lses[MAX_SETS];
    void* dq; void* dk; void* dv;                         // backward outputs
    const int* tab;                                       // segment table (device)
    Schedule sched;                                       // tile descriptors and per-token segment bounds (device)
    int n_tiles256, n_tiles128;                           // exact tile counts of the packing
    float* Dbuf;                                          // [Hq, T_total] rowsum(dO*O) (device)
    int n_groups;
    int64_t total_tokens;
    int64_t total_responses;
    int min_prompt_len;                                   // shortest prompt of the batch
    int max_group_tokens;
    int Hq, Hkv, head_dim;
    float scale;
    int naive;                                            // forward: naive packed-causal schedule
    unsigned stages;                                      // backward: SP_BWD_STAGE_* bits to run
    int resp_only;                                        // only response rows are computed / contribute
    void* o_lo_out;                                       // forward (bf16): optional rounding residual of o
    const void* o_lo;                                     // backward (bf16): optional residual for D
    const uint32_t* o_lo_flag;                            // device word: o_lo may be used only if it is non-zero (NULL: always)
    int accumulate;                                       // backward: dk, dv += instead of =
    int dkdv_parts;                                       // row parts of a key tile in the head-split pass
    const struct KeyPieces* pieces;                       // bf16 backward: the dkdv pass in pieces of key tiles (null: not)
    const struct RowPieces* row_pieces;                   // the forward of response rows and the dq pass with key loops in parts (null: not)
    float* piece_sums;                                    // the partial sums of either
    float* dkdv_partial;                                  // bf16 backward on small problems: fp32 per-q-head partials
    float* dkdv_partial2;                                 // the second row part's
    // host copies of the per-group token counts and of the whole segment table, for grid sizing and
    // for choosing kernel shapes
    SmallCall small;
    const int* host_group_tokens;
    const int32_t* host_table;
};

hipError_t launch_fwd_bf16(const Problem& p, hipStream_t s);
hipError_t launch_bwd_bf16(const Problem& p, hipStream_t s);
hipError_t launch_fwd_f32(const Problem& p, hipStream_t s);
hipError_t launch_bwd_f32(const Problem& p, hipStream_t s);
hipError_t launch_rowsum(const Problem& p, bool f32, hipStream_t s);
// Rows that see at most EDGE_LEN keys are recomputed (sp_edge.hpp): D, and dQ, which the dq pass's row workgroups
// then do not store.
constexpr int EDGE_LEN = 64;
hipError_t launch_short_rows(const Problem& p, hipStream_t s);
hipError_t launch_rope(const void* x, void* y, int H, const void* x2, void* y2, int H2, const TabArg& tab,
                       int64_t total_tokens, int d, double base, bool inverse, bool f32, hipStream_t s);
hipError_t launch_logprob_fwd(const void* z, const int* y, float* logp, float* lse, const TabArg& tab,
                              int64_t total_tokens, int64_t V, bool f32, hipStream_t s);
hipError_t launch_logprob_bwd(const void* z, const int* y, const float* lse, const float* g, void* dz,
                              const TabArg& tab, int64_t total_tokens, int64_t V, bool f32, bool zero_prompt, hipStream_t s);
hipError_t launch_grpo(const float* logp, const float* old, const float* ref, const float* adv, float* g,
                       float* J, float* loss, const TabArg& tab, uint32_t* tag, int n_resp, int n_nonempty,
                       float eps_low, float eps_high, float beta, hipStream_t s);
// Order of the key tiles (Schedule): the packing's, prompt tiles first group by group, or prompt tiles first by the rows that
// see them, most first.  A dkdv workgroup of a prompt's first tile can run a hundred times as long as one of a response,
// and in the packing's order the last group's starts when the rest of the launch is nearly through.  Sorted by rows they also
// pair well on the CUs, but tiles of one group, which stream the same Q / dO rows, no longer run side by side.  dkdv
// stage of 90 packings (10 to 7000 workgroups), geometric mean over the packing's order: group by group 0.906, by rows 0.896.
// By rows over group by group: up to 1500 workgroups 0.73 .. 1.03, mean 0.955; 1600 to 2000 0.93 .. 1.07; beyond,
// 1.00 .. 1.12 (64 groups of 1000 tokens: 28/4 heads, 2048 workgroups 936 and 990 us, packing's order 1178; 32/8 heads, 4096,
// 1057 and 1183, 1188).  As built, 100 other packings: 0.903.  Four long prompts with 16 answers (32/8) 3690 -> 3556 us, 64
// short ones (28/4) 4000 -> 3110.  Up to 256 workgroups all start at once, and one group's tiles are in order already.
constexpr int KEYS_AS_PACKED = 0, KEYS_BY_GROUP = 1, KEYS_BY_ROWS = 2;
inline int key_order(const Problem& p) {
    const int64_t wgs = (int64_t)p.n_tiles128 * (p.dkdv_partial ? p.Hq : p.Hkv);
    if (wgs <= 256 || p.n_groups == 1) return KEYS_AS_PACKED;
    return wgs <= 1536 && p.n_groups <= 256 ? KEYS_BY_ROWS : KEYS_BY_GROUP;    // (a tile's place by rows is a loop over the groups)
}

hipError_t launch_prepare(const int32_t* host_words, int n_words, int* dev_tab, uint32_t* tag_block, const ReserveTag& tag,
                          int tag_mode, bool with_schedule, int n_groups, int64_t total_tokens, int n256, int n128,
                          const Schedule& sched, int key_order, hipStream_t s);

// The threshold of sp_attn_set_small_shape_steps(), or < 0: the rule of use_small_shape().
int small_shape_steps();

inline TabArg small_table(const Problem& p) {
    return p.small.on ? make_tab_arg(p.host_table, (size_t)p.host_table[2], nullptr) : make_tab_arg(p.host_table, 0, nullptr);
}

// Calls whose kernels look everything up themselves (SmallCall)
inline bool use_small_call(const Problem& p, size_t words, int max_responses) {
    return words <= (size_t)ARG_WORDS && p.n_groups <= SMALL_GROUPS && max_responses <= SMALL_RESPONSES &&
           (int64_t)p.n_tiles128 * p.Hq <= SMALL_CALL_TILES;
}

// Number of (row tile of `bm` rows, 64-key tile) pairs of one q head that hold an allowed pair, and of row tiles (host
// arithmetic on the segment table).  With one q head per kv head these are the steps and the workgroups that run; with
// more, a workgroup spans fewer rows (wave_rows() in sp_common.hpp) and skips most of what only other rows see.  Key tiles are
// counted from multiples of 64, where the kernels walk a response from its first key on, and rows of the prompt are counted
// in response-rows mode too, which does not run them: it is a measure of the packing, not of the call.
inline void key_steps(const Problem& p, int bm, int64_t& steps, int64_t& tiles) {
    const int32_t* tab = p.host_table;
    steps = 0; tiles = 0;
    for (int g = 0; g < p.n_groups; ++g) {
        const int32_t* e = tab + TAB_HEADER + TAB_GROUP_WORDS * g;
        const int Lp = e[1], Tg = e[2], G = e[4];
        const int32_t* roff = tab + e[3];
        for (int t0 = 0; t0 < Tg; t0 += bm, ++tiles) {
            const int t1 = t0 + bm < Tg ? t0 + bm : Tg;
            const int n1 = ((Lp < t1 ? Lp : t1) + 63) / 64;
            steps += n1;
            if (t1 > Lp) {
                const int first = t0 > Lp ? t0 : Lp;          // first response row: its segment start opens the range
                int lo = 0, hi = G;
                while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (roff[mid] <= first) lo = mid; else hi = mid; }
                const int k2b = roff[lo] / 64 > n1 ? roff[lo] / 64 : n1;
                steps += (t1 + 63) / 64 - k2b;
            }
        }
    }
}

// Which workgroup shape the forward and the dq pass take: four waves where row tiles of 128 rows need more than 3 % fewer
// steps than tiles of 256.  Those are not the steps that run (with four to seven q heads per kv head the shapes differ by 1 to
// 3 % of them); the share says how short and ragged a packing's segments are, and with that how much of a workgroup's life is
// fixed cost, which the four-wave shape hides behind the CU's other workgroup.  Its price is twice the tile copies
// per MFMA and a barrier per step.  Both shapes timed on 9 workloads and 51 drawn packings, 354 to 265 K tokens, 28/4 to
// 40/8 and 4/2 heads (time with eight waves over time with four; forward, dq pass):
//   no more than 3 % saved    0.97 .. 1.01, 1.00 .. 1.03      (16K prompt and short answers 0.971, 0.996)
//   3 to 8 % saved            0.95 .. 1.34, 1.01 .. 1.32      (response rows under an 8K prompt 0.954, 1.023)
//   more                      1.02 .. 1.40, 1.02 .. 1.38
// The shape taken is on average 0.1 % (forward) and 0.04 % (dq) from the faster one, at worst 4.8 % (the response rows).
// The knob, when set, replaces the rule by a threshold on the mean number of steps of a 256-row tile.
inline bool use_small_shape(const Problem& p) {
    int64_t s256, t256, s128, t128;
    key_steps(p, 256, s256, t256);
    const int knob = small_shape_steps();
    if (knob >= 0) return t256 > 0 && (double)s256 / (double)t256 < (double)knob;
    key_steps(p, 128, s128, t128);
    return 0.5 * (double)s128 * 1.03 < (double)s256;
}


// Packings that the bandwidth-shaped bf16 rowsum kernel takes (its per-head sums of 16 tokens fit its LDS)
inline bool rowsum_fast_path(const Problem& p) { return p.head_dim == 128 && (size_t)p.Hq * 16 * sizeof(float) <= 32768; }

inline int count_tiles(const Problem& p, int bm) {
    int n = 0;
    for (int g = 0; g < p.n_groups; ++g) n += (p.host_group_tokens[g] + bm - 1) / bm;
    return n;
}

// Small problems leave most CUs idle in the dkdv pass (one workgroup per 128 keys and kv head):
// below this many workgroups the pass is split over the q heads of each kv head, through fp32
// partial sums in the workspace.  Both the workspace size and the launch use this rule.
inline bool dkdv_head_split(int64_t total_tokens, int n_groups, int Hq, int Hkv) {
    return Hq > Hkv && (total_tokens / 128 + n_groups) * Hkv <= 192;
}

// Where it is split over the q heads, the pass is over when the workgroup of the first key tile is, which walks every row of
// its group.  Packings that leave CUs idle all the same can use a second set of partial sums (sp_attn_row_parts_bytes()); whether
// tiles of at least eight steps (512 rows) are cut into two row parts as well is then decided by the longest tile's
// steps: what is gained is half of them, what is paid is a workgroup's fixed cost (five steps) and the sums.  Training passes, us, one part
// and two (workgroups, longest tile's steps):
//   56, 14   66.4  60.6      104, 24   99.9  88.7      168, 24  107.8 102.3      116, 57  194.1 163.9      188, 22  105.1 105.3
//   196, 13  76.2  82.7      256, 14   83.4  89.7      280, 19   88.1  95.4      308, 22  105.6 116.9       76, 3    44.5  46.0
inline int64_t head_split_wgs(int64_t total_tokens, int n_groups, int Hq) { return (total_tokens / 128 + n_groups) * Hq; }
// (By the totals alone, as callers size workspaces by them; both sets within 30 MB, the range that was measured.)
inline int dkdv_max_parts(int64_t total_tokens, int n_groups, int Hq, int Hkv) {
    return dkdv_head_split(total_tokens, n_groups, Hq, Hkv) && head_split_wgs(total_tokens, 1, Hq) <= 224 &&
           2 * 2 * (int64_t)Hq * total_tokens * 128 * 4 <= (int64_t)30 << 20 ? 2 : 1;
}
constexpr int PART_STEPS = 8, PIECE_STEPS = 8;
inline int dkdv_parts(const Problem& p) {
    if (dkdv_max_parts(p.total_tokens, p.n_groups, p.Hq, p.Hkv) < 2) return 1;
    int most = 0;                                              // of a group's first tile: no other has more
    for (int g = 0; g < p.n_groups; ++g) {
        const int32_t* e = p.host_table + TAB_HEADER + TAB_GROUP_WORDS * g;
        const int steps = p.resp_only && e[1] == e[2] ? 0 : (e[2] + 63) / 64 - (p.resp_only ? e[1] / 64 : 0);
        if (steps > most) most = steps;
    }
    return most >= PART_STEPS && head_split_wgs(p.total_tokens, p.n_groups, p.Hq) <= 9 * most ? 2 : 1;
}

// Key tiles in pieces: of the packings that use it, the dkdv pass takes a list of (tile, part of its row tiles and q heads), sorted by length,
// from the kernel arguments behind the table.  word: tile | part << 16 | parts << 24.  Pieces of a tile with several parts lie next
// to one another ahead of all others and leave partial sums in the slot of their place in the list; a second launch adds them (sums: two
// words for each such tile, its first slot | parts << 16 | keys - 1 << 24 and its first packed token).
constexpr int PIECE_TILES = 640, PIECE_SLOTS = 384;       // most key tiles; most slots, all kv heads
constexpr size_t PIECE_SLOT_BYTES = 2 * 128 * 128 * 4;    // dK and dV of a key tile, float32
struct KeyPieces { std::vector<uint32_t> words, sums; int n_slots = 0; bool no_room = false; };      // no_room: shorter pieces did not fit the list
// slots of a kv head that a call can use, by its totals
inline int piece_slots(int64_t total_tokens, int n_groups, int Hq, int Hkv) {
    const int64_t tiles = total_tokens / 128 + n_groups, rows = total_tokens / 64 + n_groups;
    if (tiles > PIECE_TILES || Hkv < 1 || Hq % Hkv != 0) return 0;
    const int64_t by_work = tiles * rows * (Hq / Hkv) / PIECE_STEPS, cap = PIECE_SLOTS / Hkv;
    return (int)(by_work < cap ? by_work : cap);
}
inline size_t piece_bytes(int64_t total_tokens, int n_groups, int Hq, int Hkv) {
    return (size_t)piece_slots(total_tokens, n_groups, Hq, Hkv) * Hkv * PIECE_SLOT_BYTES;
}
// the pieces of a call (none where whole key tiles are as good, or `cost` steps of a workgroup worse), at most `slots` with partial sums
KeyPieces plan_key_pieces(const Problem& p, int slots, size_t max_words, int cost);

// Key loops of the dq pass, and of a forward of response rows, in parts: of the packings that use it, both take a list of (tile of 128 rows, workgroup of the tile,
// part of its key tiles) from the kernel arguments behind the table, one of four-wave workgroups, longest first.  Workgroups with
// several parts leave unnormalised float32 sums in slots, in the order of the list, where they lie next to one another from first_slot on, and a second
// launch brings them together.  word: tile | workgroup << 10 | part << 16 | parts << 24; sums: three words for each such
// workgroup, its first slot | parts << 16, the packed token of its tile's first row, and its number within the tile, counted from the first rows.
constexpr int ROW_PIECE_TILES = 1024, ROW_SUMS = 240;     // most tiles (and 64 q heads per kv head); most workgroups with parts, per kv head
constexpr size_t ROW_SLOT_BYTES = 4 * (32 * 128 + 32 * 4) * 4;        // four items: 32 rows of 128 columns, four numbers per row
struct RowPieces { std::vector<uint32_t> words, sums; int first_slot = 0, n_slots = 0; };
struct RowSums { uint32_t w[3 * ROW_SUMS]; };
struct RowPieceArgs { int at, first_slot, n_slots; float* slots; Div rep, kv_heads; };      // at: word of the table argument at which the list starts
struct RowPiece { int tile, hr, part, parts, slot; };
__device__ __forceinline__ RowPiece row_piece(const int* tab, const RowPieceArgs& a, const Item& it) {
    const unsigned w = (unsigned)tab[a.at + it.tile];
    return RowPiece{(int)(w & 1023), (int)(w >> 10 & 63), (int)(w >> 16 & 255), (int)(w >> 24), it.tile - a.first_slot};
}
struct RowItem { int first, parts, kvh, w, tok, head; };
__device__ __forceinline__ RowItem row_item(const RowSums& list, const RowPieceArgs& a) {
    unsigned kvh, h;
    const unsigned n = divmod(blockIdx.x >> 2, a.kv_heads, kvh);
    RowItem it{(int)(list.w[3 * n] & 0xffff), (int)(list.w[3 * n] >> 16), (int)kvh, (int)(blockIdx.x & 3), 0, 0};
    it.tok = (int)list.w[3 * n + 1] + 32 * (int)divmod(4 * list.w[3 * n + 2] + it.w, a.rep, h);       // as wave_rows()
    it.head = (int)(kvh * a.rep.d + h);
    return it;
}
__device__ __forceinline__ const float* row_slot(const RowPieceArgs& a, const RowItem& it) {
    return a.slots + ((int64_t)it.kvh * a.n_slots + it.first) * (int64_t)(ROW_SLOT_BYTES / 4) + it.w * (int)(ROW_SLOT_BYTES / 16);
}
RowPieces plan_row_pieces(const Problem& p, size_t slots, size_t max_words);
inline RowPieceArgs row_piece_args(const Problem& p) {
    return RowPieceArgs{p.small.on ? p.host_table[2] : 0, p.row_pieces->first_slot, p.row_pieces->n_slots, p.piece_sums, make_div(p.Hq / p.Hkv), make_div(p.Hkv)};
}
inline RowSums row_sums(const RowPieces& r) {
    RowSums s{};
    for (size_t i = 0; i < r.sums.size(); ++i) s.w[i] = r.sums[i];
    return s;
}
// the table argument with a list behind the table
inline TabArg with_list(TabArg t, const Problem& p, const std::vector<uint32_t>& list) {
    const size_t at = p.small.on ? (size_t)p.host_table[2] : 0;
    for (size_t i = 0; i < list.size(); ++i) t.words[at + i] = (int32_t)list[i];
    return t;
}

// Rows (keys) per workgroup of a float32 kernel (0 forward, 1 dq, 2 dkdv): 16, 4 or 1 (rule and reasons: sp_f32.hip).
int f32_rows(const Problem& p, int kernel);

// Waves per workgroup (8 or 4) of a dkdv pass that is not split over the q heads (rule and reasons: sp_bwd.hip).
int dkdv_waves(const Problem& p);

}  // namespace sp
