// Shared device-side definitions for the shared-prompt attention kernels (gfx950 only).
//
// Packed layout and mask follow Section 4.3 of the paper: a group is
// [prompt | resp_1 | ... | resp_G]; query t may attend key s iff s <= t and
// (s is a prompt token or s lies in t's own response).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Segment table (int32 words, device memory, written by sp_upload_table):
//   [0] n_groups   [1] total_tokens   [2] table_words   [3] reserved
//   group g at 4 + 8*g : { tok_base, prompt_len, T_g, roff_idx, G, tiles256_before, tiles128_before, reserved }
//   roff_idx points at G+1 group-local offsets: roff[0] = prompt_len,
//   roff[i+1] = roff[i] + len(resp_i), roff[G] = T_g.
//   tilesB_before = sum over earlier groups of ceil(T_g / B): the kernels number their work
//   tiles (B rows or keys) group by group and find a tile's group by bisection on this word.
// ---------------------------------------------------------------------------
constexpr int TAB_HEADER = 4;
constexpr int TAB_GROUP_WORDS = 8;
constexpr int TAB_TILES256 = 5;        // word of the group entry: 256-row tiles before this group
constexpr int TAB_TILES128 = 6;        // 128-key tiles before this group
constexpr int TAB_CHUNK_WORDS = 960;   // words carried by one upload launch (kernarg limit 4 KB)

struct TabChunk { int32_t w[TAB_CHUNK_WORDS]; };
constexpr int PREP_WORDS = 896;        // largest table that travels beside the other arguments of the one-launch preparation
struct PrepChunk { int32_t w[PREP_WORDS]; };

struct GroupDesc {
    int tok_base;       // first packed token of the group
    int Lp;             // prompt length
    int Tg;             // tokens in the group
    int G;              // number of responses
    const int* roff;    // G+1 group-local response offsets
};

__device__ __forceinline__ GroupDesc load_group(const int* __restrict__ tab, int g) {
    const int* e = tab + TAB_HEADER + TAB_GROUP_WORDS * g;
    GroupDesc d;
    d.tok_base = e[0]; d.Lp = e[1]; d.Tg = e[2]; d.roff = tab + e[3]; d.G = e[4];
    return d;
}

// Start of the segment that owns group-local token t: 0 for a prompt token, the first
// token of its response otherwise.  Requires 0 <= t < Tg.  With this value the mask is
//   allowed(t, s) = (s <= t) && (s < Lp || s >= seg_start(t)).
__device__ __forceinline__ int seg_start(const GroupDesc& d, int t) {
    if (t < d.Lp) return 0;
    int lo = 0, hi = d.G;              // invariant: roff[lo] <= t, (hi == G or roff[hi] > t)
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (d.roff[mid] <= t) lo = mid; else hi = mid;
    }
    return d.roff[lo];
}

// One past the last token of the segment that owns t (prompt: Lp).
__device__ __forceinline__ int seg_end(const GroupDesc& d, int t) {
    if (t < d.Lp) return d.Lp;
    int lo = 0, hi = d.G;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (d.roff[mid] <= t) lo = mid; else hi = mid;
    }
    return d.roff[lo + 1];
}

// Segment bounds [st, en) of N group-local response tokens at once (every t[n] must satisfy
// Lp <= t[n] < Tg; for a prompt token the caller substitutes its own bounds).  One descending-step
// search over the response offsets per token, all N advanced in lock-step with unconditional
// loads, so the N dependent load chains overlap instead of following one another.  st is the last
// accepted offset; en is the last rejected one (the probes that fail come at ever smaller indices,
// the last of them is the accepted index + 1), so neither needs a load after the search.
template <int N>
__device__ __forceinline__ void seg_bounds(const GroupDesc& d, const int (&t)[N], int (&st)[N], int (&en)[N]) {
    int pos[N];
#pragma unroll
    for (int n = 0; n < N; ++n) { pos[n] = 0; st[n] = d.Lp; en[n] = d.Tg; }
    for (int step = d.G > 0 ? 1 << (31 - __clz(d.G)) : 0; step >= 1; step >>= 1) {
        int val[N];
#pragma unroll
        for (int n = 0; n < N; ++n) val[n] = d.roff[pos[n] + step < d.G ? pos[n] + step : 0];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const bool in = pos[n] + step < d.G;
            if (in && val[n] <= t[n]) { pos[n] += step; st[n] = val[n]; }
            else if (in) en[n] = val[n];
        }
    }
}

// Group that owns packed token tok (0 <= tok < total_tokens): bisection on tok_base.
__device__ __forceinline__ int find_group_of_token(const int* __restrict__ tab, int64_t tok) {
    int lo = 0, hi = tab[0];           // invariant: tok_base[lo] <= tok, (hi == n_groups or tok_base[hi] > tok)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tab[TAB_HEADER + TAB_GROUP_WORDS * mid] <= tok) lo = mid; else hi = mid;
    }
    return lo;
}

// Work-tile lookup: tiles of BT rows (256) or keys (128) are numbered group by group.  Returns
// the group and the tile's index inside it (0 .. ceil(T_g / BT) - 1), or g_out = -1 when the
// tile number lies past the last group.  Bisection on the group entries' running tile counts,
// so a batch of many small groups costs log2(n_groups) dependent scalar loads per workgroup.
template <int BT>
__device__ __forceinline__ void find_tile(const int* __restrict__ tab, int n_groups, int tile, int& g_out, int& idx_out) {
    static_assert(BT == 256 || BT == 128, "the table carries running tile counts for 256 and 128 only");
    constexpr int W = BT == 256 ? TAB_TILES256 : TAB_TILES128;
    int lo = 0, hi = n_groups;         // passed in (a kernel argument): one load less at the head of the chain
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tab[TAB_HEADER + TAB_GROUP_WORDS * mid + W] <= tile) lo = mid; else hi = mid;
    }
    const int* e = tab + TAB_HEADER + TAB_GROUP_WORDS * lo;
    const int idx = tile - e[W];
    const int nt = (e[2] + BT - 1) / BT;
    g_out = idx < nt ? lo : -1;
    idx_out = idx;
}

// Schedule: what the MFMA kernels' prologues would otherwise look up in the table through chains of
// dependent loads, written once per call by a small kernel (sp_f32.hip: schedule_kernel).
//   TileDesc  per work tile (one array for tiles of 256, one for tiles of 128 rows or keys): its group
//             and index inside the group, and the group's first token, prompt length and token count.
//             key_tiles: the tiles of 128 in the order in which the dkdv pass takes them (key_order() in sp_launch.hpp)
//   key_lo[tok]  first key of its own segment that token tok may attend besides the prompt
//                (group-local; 0 for a prompt token): the mask is s <= t && (s < Lp || s >= key_lo[t])
//   row_hi[tok]  one past the last row that sees token tok as a key (group-local): the group's end for
//                a prompt token, the end of its response otherwise
struct TileDesc { int g, ti, tok_base, Lp, Tg, pad0, pad1, pad2; };
struct Schedule { const TileDesc* tiles256; const TileDesc* tiles128; const TileDesc* key_tiles; const int* key_lo; const int* row_hi; };

// Division by a number that a launch knows: the quotient by the reciprocal floor(2^32 / d) is the exact one or one less.
// (A plain division is some 25 instructions, vector ones among them even where both numbers are uniform, and a workgroup's
// place and its rows take eight.  Training passes, us: two small groups 70.9 -> 70.2, one 1K prompt 249 -> 246, 64 short prompts with 16 answers 8294 -> 8263.)
struct Div { unsigned d, m; };
__host__ inline Div make_div(int d) { return Div{(unsigned)d, d == 1 ? 0xffffffffu : (unsigned)((1ull << 32) / (unsigned)d)}; }
__host__ __device__ __forceinline__ unsigned divmod(unsigned x, const Div& v, unsigned& rest) {
    unsigned q = (unsigned)(((uint64_t)x * v.m) >> 32);
    rest = x - q * v.d;
    if (rest >= v.d) { ++q; rest -= v.d; }
    return q;
}

// Map a flat block index to (tile, kv head, q head of the kv head) so that the blocks an XCD receives
// (blocks are dealt round-robin over the 8 XCDs, each with a private L2) share one
// kv head, and q heads of the same tile sit next to each other.
struct ItemMap { Div rep, kv_per_x, heads; int n_tiles, per_kv, log_nx; };      // log_nx: XCDs that share a kv head, -1: other counts
__host__ inline ItemMap make_item_map(int n_tiles, int Hq, int Hkv) {
    const int rep = Hq / Hkv;
    ItemMap m{make_div(rep), make_div(Hkv % 8 == 0 ? Hkv / 8 : 1), make_div(Hq), n_tiles, n_tiles * rep, -1};
    if (Hkv % 8 == 0) m.log_nx = 0;
    else if (8 % Hkv == 0) m.log_nx = Hkv == 4 ? 1 : Hkv == 2 ? 2 : 3;
    return m;
}
struct Item { int tile, kvh, hr; };
// Returns false when the block has no work.
__host__ __device__ __forceinline__ bool decode_item(int bid, const ItemMap& m, Item& it) {
    unsigned hr, r;
    if (m.log_nx < 0) {
        it.tile = (int)divmod((unsigned)bid, m.heads, r);
        it.kvh = (int)divmod(r, m.rep, hr);
        it.hr = (int)hr;
        return it.tile < m.n_tiles;
    }
    const unsigned x = bid & 7, j = (unsigned)bid >> 3;
    if (m.log_nx == 0) {
        const unsigned rest = divmod(j, m.rep, hr);
        it.hr = (int)hr;
        it.tile = (int)divmod(rest, m.kv_per_x, r);
        it.kvh = (int)(x + 8 * r);
        return it.tile < m.n_tiles;
    }
    const unsigned n = (j << m.log_nx) + (x & ((1u << m.log_nx) - 1));
    it.kvh = (int)(x >> m.log_nx);
    it.tile = (int)divmod(n, m.rep, hr);
    it.hr = (int)hr;
    return n < (unsigned)m.per_kv;
}

// Rows of a workgroup of NW waves.  A row tile of 32 NW rows x the rep = Hq / Hkv q heads that share a kv head
// is cut into rep workgroups, not one per head: its NW x rep items (32 rows of one head) are numbered row block
// first, head second, and workgroup i takes items i NW .. i NW + NW - 1, one per wave.  All items read the same
// K/V tiles, so a tile is copied for as many rows as before, but the workgroup spans about 32 NW / rep rows
// instead of 32 NW, and a wave rides along through fewer tiles that only other rows of the workgroup see (past its own
// diagonal, other responses' keys).  Against one head per workgroup (executed steps and time, one box):
//   64 groups of 128 + 16 x 256 tokens, 28 / 4 heads   -15 %   fwd 2.88 -> 2.63 ms, dq pass 4.04 -> 3.60 ms
//   64 groups of 1000 tokens, 32 / 8 heads             -13 %   fwd 0.88 -> 0.84 ms, dq pass 1.27 -> 1.15 ms
//   4 x (4096 + 16 x 320), 32 / 8                       -2 %   fwd 1.97 -> 1.94 ms, dq pass 2.81 -> 2.74 ms
//   16384 + 32 x 160, 40 / 8                            -1 %   fwd 4.04 -> 4.00 ms, dq pass 5.72 -> 5.55 ms
// With one q head per kv head the two cuts are the same.
struct WaveRows {
    int head;           // q head of this wave
    int tw0;            // its first row (group-local)
    int t0, t1;         // rows of the workgroup
};
template <int NW>
__device__ __forceinline__ WaveRows wave_rows(const TileDesc& td, const Item& it, const Div& rep, int w) {
    const int i = (int)rep.d - 1 - it.hr;                    // last rows first: they carry the most work
    const int base = ((td.Tg + 32 * NW - 1) / (32 * NW) - 1 - td.ti) * (32 * NW);
    unsigned h, r;
    WaveRows wr;
    wr.tw0 = base + 32 * (int)divmod((unsigned)(i * NW + w), rep, h);
    wr.head = it.kvh * (int)rep.d + (int)h;
    wr.t0 = base + 32 * (int)divmod((unsigned)(i * NW), rep, r);
    wr.t1 = min(base + 32 * (int)divmod((unsigned)(i * NW + NW - 1), rep, r) + 32, td.Tg);
    return wr;
}

__host__ __device__ inline int grid_for_items(int n_tiles, int Hq, int Hkv) {
    const int rep = Hq / Hkv;
    if (Hkv % 8 == 0) return 8 * (n_tiles * rep * (Hkv / 8));
    if (8 % Hkv == 0) { const int nx = 8 / Hkv; return 8 * ((n_tiles * rep + nx - 1) / nx); }
    return n_tiles * Hq;
}

// ---------------------------------------------------------------------------
// LDS tiles: rows of 128 bf16 (256 B = 16 granules of 16 B).  Granule g of row r is
// stored at granule slot g ^ swz(r).  swz permutes 0..15 over 16 consecutive rows
// (conflict-free b128 reads of one granule column by 16 rows) and its two high bits
// differ over 4 consecutive rows (conflict-free transposed b64 reads of a 4-row x
// 4-granule block).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

__device__ __forceinline__ int tile_off(int row, int granule) {   // byte offset
    return row * 256 + ((granule ^ swz(row)) << 4);
}

typedef __attribute__((address_space(3))) char lds_char;

__device__ __forceinline__ bf16x8 lds_read_row8(const char* tile, int row, int granule) {
    return *reinterpret_cast<const bf16x8*>(tile + tile_off(row, granule));
}

// Transposed read feeding an MFMA operand whose in-lane (contraction) index runs over
// tile ROWS: the lane receives rows row4 .. row4+3 at column col (one bf16 each).
// Lanes of a 16-lane group must pass: row = row4 + (j >> 2), col4 = colbase + 4*(j & 3)
// with j = lane & 15; lane j then receives column colbase + j.
__device__ __forceinline__ s16x4 lds_read_tr4(const char* tile, int row, int col4) {
    const char* p = tile + tile_off(row, col4 >> 3) + ((col4 & 4) << 1);
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4*)(p));
}

// The same two reads at an LDS byte address
__device__ __forceinline__ bf16x8 lds_at_row8(unsigned addr) {
    return *(__attribute__((address_space(3))) const bf16x8*)(uintptr_t)addr;
}
__device__ __forceinline__ s16x4 lds_at_tr4(unsigned addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)addr);
}

// the n lowest bits set (none for n <= 0, all from 32 on)
__device__ __forceinline__ unsigned low_bits(int n) { return n <= 0 ? 0u : 0xffffffffu >> (32 - min(n, 32)); }
// Masks a 32 x 32 score block: S[r], of row (or key) 8 (r / 4) + 4 (lane / 32) + r % 4 of the block, becomes -inf unless
// bit 8 (r / 4) + r % 4 of `bits` is set.  Two instructions per score; comparing each index took five, or a branch.
__device__ __forceinline__ void mask16(f32x16& S, unsigned bits) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const unsigned keep = (unsigned)__builtin_amdgcn_sbfe((int)bits, 8 * (r >> 2) + (r & 3), 1);
        S[r] = __uint_as_float((__float_as_uint(S[r]) & keep) | (0xff800000u & ~keep));
    }
}

__device__ __forceinline__ bf16x8 cat4(s16x4 a, s16x4 b) {
    s16x8 r = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Round 8 floats to bf16 (round-to-nearest-even, hardware v_cvt_pk_bf16_f32).
__device__ __forceinline__ bf16x8 pack8(float a0, float a1, float a2, float a3,
                                        float a4, float a5, float a6, float a7) {
    bf16x8 r;
    r[0] = (__bf16)a0; r[1] = (__bf16)a1; r[2] = (__bf16)a2; r[3] = (__bf16)a3;
    r[4] = (__bf16)a4; r[5] = (__bf16)a5; r[6] = (__bf16)a6; r[7] = (__bf16)a7;
    return r;
}

// acc + the dot product of eight bf16 pairs, two at a time (v_dot2_f32_bf16)
__device__ __forceinline__ float dot8(bf16x8 a, bf16x8 b, float acc) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int e = 0; e < 8; e += 2)
        acc = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{a[e], a[e + 1]}, bf16x2{b[e], b[e + 1]}, acc, false);
    return acc;
}

__device__ __forceinline__ float xor32(float x) { return __shfl_xor(x, 32, 64); }

// max / sum of x over the lane pair (l, l ^ 32) with one v_permlane32_swap: after the swap
// one result holds the low-half value and the other the high-half value in every lane.
__device__ __forceinline__ float pair_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Asynchronous global -> LDS copy of 16 bytes per lane (global_load_lds_dwordx4): lane i of
// the wave writes LDS bytes [lds_base + 16*i, +16).  lds_base must be wave-uniform.
// Written as inline assembly so that the compiler does not place a conservative
// "wait for all global loads" in front of every later LDS read; the kernels order the
// copy against its readers themselves with wait_vm0() followed by a workgroup barrier.
// M0 (the LDS base of the copy) is overwritten.  It cannot be named as a clobber: the compiler
// treats M0 as a reserved register (it rejects the clobber as undefined behaviour) and writes it
// itself immediately before each of its own uses, never keeping a value in it across statements;
// gfx9 LDS instructions do not read M0 and nothing else in these kernels uses it.
__device__ __forceinline__ void async_copy16(const void* gptr, char* lds_base) {
    const unsigned lds_addr = __builtin_amdgcn_readfirstlane(
        (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_base);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(gptr), "s"(lds_addr) : "memory");
}
// Same copy with the global address split into a wave-uniform 64-bit base (scalar registers)
// and a 32-bit per-lane byte offset, and the LDS destination given as a byte address: a kernel
// keeps the lane part constant and advances only the scalar base from tile to tile.
__device__ __forceinline__ void async_copy16_sm(uint64_t sbase, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}
// 4-byte variant: lane i writes LDS bytes [lds_base + 4*i, +4).
__device__ __forceinline__ void async_copy4(const void* gptr, char* lds_base) {
    const unsigned lds_addr = __builtin_amdgcn_readfirstlane(
        (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_base);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :: "v"(gptr), "s"(lds_addr) : "memory");
}
// wait until every global load (including global -> LDS copies) of this wave has landed
__device__ __forceinline__ void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0F70); }

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

}  // namespace sp
