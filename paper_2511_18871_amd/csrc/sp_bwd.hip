// Backward shared-prompt attention, bf16 MFMA path (gfx950).  Two deterministic passes
// after D = rowsum(dO * O):
//
//  dq pass   -- a workgroup owns a tile of query rows (like the forward) and streams the
//               keys that those rows may see: S^T = K Q^T, dP^T = V dO^T,
//               dS^T = P^T * (dP^T - D), dQ^T += K^T dS^T.
//  dkdv pass -- a workgroup owns a tile of keys of one kv head and streams every query
//               row that sees them, for each q head of the kv head: for a PROMPT key tile
//               that is the later prompt rows and all rows of all G responses, which is
//               where the prompt's dK/dV accumulate over the responses (Section 4.3,
//               grad L_shared = sum_k grad L_k).  S = Q K^T, dP = dO V^T,
//               dV^T += dO^T P, dK^T += Q^T dS.  Accumulation stays in registers, so no
//               atomics are needed and results are bitwise repeatable.
//
// The S/dP recomputation runs in both passes (7 contractions instead of 5); in exchange
// neither pass exchanges dS between lanes or accumulates through memory.
#include "sp_common.hpp"
#include "sp_launch.hpp"
#include "sp_edge.hpp"
#include <algorithm>
#include <type_traits>
#include <vector>

namespace sp {
namespace {

constexpr int TILE_BYTES = 64 * 256;   // 64 rows x 128 bf16

struct BwdArgs {
    const __bf16* q; const __bf16* k; const __bf16* v; const __bf16* d_o;
    // planes read by the dkdv pass: -D (the initial value of its dP accumulators) and L2 = lse * log2(e), written by the
    // rowsum stage (or the dq pass, below)
    const float* lse; float* nD; float* L2;
    // dq pass with the rowsum stage folded in: D = rowsum(dO * (o + residual)) is formed in the prologue from
    // the dO rows the pass loads anyway, and the two planes are written for the dkdv pass
    int fused_rowsum;
    const __bf16* o; const __bf16* o_lo; const uint32_t* lo_flag;
    __bf16* dq; __bf16* dk; __bf16* dv;
    SmallCall small;
    int64_t T_total;
    Schedule sched;      // tile descriptors and per-token segment bounds, written by the schedule kernel of the call
    ItemMap items;       // of the pass
    int n_groups, Hq, Hkv;
    float scale, c;      // c = scale * log2(e)
    int resp_only;       // only response rows are computed (dq) / contribute (dk, dv)
    int accumulate;      // dk, dv are added to what the output buffers hold
    // dkdv pass on small problems: one workgroup per (key tile, Q head) instead of per (key tile,
    // kv head); the per-q-head partial sums go to `partial` in fp32 and a second kernel adds them
    int rep;             // q heads per kv head
    Div kv_heads, rep_div;
    int head_split;      // row parts of a key tile: 0 (not split), 1 or 2
    float* partial;      // [2 (dK, dV)][rep][T_total][Hkv][128] fp32 of the first row part
    float* partial2;     // the same of the second
    RowPieceArgs rows;   // dq pass with key loops in parts
    int pieces_at;       // dkdv pass in pieces: word of the table argument at which their list starts
    int n_slots;         // pieces of tiles with several parts
    float* piece_sums;   // [kv head][slot][dK, dV][128 keys][128]
};

static_assert(sizeof(TabArg) + sizeof(BwdArgs) + sizeof(EdgeArgs) + 8 <= 4096 && sizeof(RowSums) + sizeof(BwdArgs) <= 4096 &&
              2 * PIECE_SLOTS * 4 + sizeof(BwdArgs) <= 4096, "kernel arguments");

// ------------------------------------------------------------------------------------
// dq pass
// ------------------------------------------------------------------------------------
//
// Two shapes of workgroup, as in the forward (and the same items: 32 rows of one q head per wave, wave_rows()).
// NW = 8: a ring of three slots of a whole 64-key tile
// (K and V: 96 KB), one workgroup per CU, one barrier per tile.  NW = 4: a ring of four slots of HALF
// a tile (32 keys of K and V: 64 KB), one barrier per half, two workgroups per CU: for packings whose key
// loops are short, where a workgroup's fixed costs (a quarter of its life with one workgroup per CU) then
// overlap with the other workgroup's loop and fewer rows ride along through tiles they cannot see.
// Bound: bf16 MFMA (24 per wave, 32 rows and 32 keys; 16 LDS reads and about 100 vector instructions beside them).  The
// loop holds neither address arithmetic nor spills: a turn is a whole turn of the ring, so that slots are constants, the
// operand addresses are whole sums in registers, the mask is a word of bits per lane, the operand ring runs through M
// and D, and dP starts at -D.  One box, before -> after, us: 16K prompt with 32 answers 5440 -> 5190, four long prompts
// 2750 -> 2515, 64 groups of a short prompt and 16 answers 3640 -> 3110, 64 groups of 1000 tokens 1100 -> 990, response
// rows under an 8K prompt 630 -> 545.
// On short key loops a quarter of a wave's life was the prologue: six waits for memory behind one another (descriptor, segment
// starts, reserve flag, q and dO, o and its residual, first keys), now two, and D by dot products of pairs (64 instructions for
// 320).  With the forward's key tiles and addresses, us: 64 groups of a short prompt and 16 answers 2782 -> 2679, 64 groups of
// 1000 tokens 981 -> 957, two small groups 20.6 -> 19.8, four long prompts 2442 -> 2434, 16K prompt 5192 -> 5225.
template <int NW, bool SMALL, bool PIECES>          // SMALL, PIECES: as in the forward
__global__ __launch_bounds__(NW * 64, 2) void bwd_dq_kernel(TabArg table, BwdArgs a, EdgeArgs edge, int short_blocks, int row_blocks) {
    constexpr int BM = 32 * NW, BN = 64;
    constexpr int RD = 3;                       // LDS operand ring depth (prefetch distance RD - 1 MFMAs)
    constexpr int NE1 = 5;                      // elements of a half's vector work done under the previous D stage
    static_assert(NW == 8 || NW == 4, "the copy split below assumes eight or four waves");
    constexpr int NSLOT = NW == 8 ? 3 : 4;
    constexpr int SLOT_BYTES = NW == 8 ? 2 * TILE_BYTES : TILE_BYTES;       // [K | V] of 64 keys, or of 32
    constexpr int V_OFF = SLOT_BYTES / 2;                                    // where V starts inside a slot
    // (one slot more than the ring: the rows come in through all but slot 0, into which the first keys are copied meanwhile)
    __shared__ __attribute__((aligned(1024))) char lds[NSLOT + 1][SLOT_BYTES];

    // Workgroups ahead of the row tiles' (a multiple of 8, so that those keep their XCDs) or, NW = 8, behind them: the rows
    // that see at most EDGE_LEN keys, two waves per (segment, q head).  As a launch of their own they had the chip to
    // themselves for 7 to 10 us of latency (37 us for 2048 pairs); beside row tiles, us for both, before -> after: two small
    // groups 28.4 -> 21.2, one 1K prompt 93 -> 88, 64 groups of 1000 tokens 1048 -> 1034, four long prompts 2553 -> 2545,
    // 16K prompt 5331 -> 5323 (ahead: 5350; the 64 groups behind: 1050).
    constexpr int PAIRS = NW == 8 ? 3 : 2;          // that the LDS holds
    static_assert(PAIRS * EDGE_LDS <= NSLOT * SLOT_BYTES && 2 * PAIRS <= NW, "short rows do not fit");
    const int sb = (int)blockIdx.x - (NW == 8 ? row_blocks : 0), rb = (int)blockIdx.x - (NW == 8 ? 0 : short_blocks);
    if (NW == 8 ? sb >= 0 : rb < 0) {
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = min(w >> 1, PAIRS - 1);
        if constexpr (SMALL) edge.tab = table_of(table);
        for (int64_t p0 = (int64_t)PAIRS * sb; p0 < edge.n_pairs; p0 += (int64_t)PAIRS * short_blocks) {
            short_rows_body<true>(edge, w < 2 * PAIRS ? p0 + i : edge.n_pairs, w & 1, &lds[0][0] + EDGE_LDS * i);
            __syncthreads();
        }
        return;
    }
    Item item;
    if (!decode_item(rb, a.items, item)) return;
    RowPiece piece{item.tile, item.hr, 0, 1, 0};
    if constexpr (PIECES) { piece = row_piece(table_of(table), a.rows, item); item.hr = piece.hr; item.tile = piece.tile; }
    TileDesc td;
    SmallGroup sg;
    if constexpr (SMALL) {
        int ti;
        sg = small_tile<BM>(table_of(table), a.n_groups, item.tile, threadIdx.x & 63, ti);
        td = TileDesc{0, ti, sg.tok_base, sg.Lp, sg.Tg, 0, 0, 0};
    } else {
        td = (BM == 256 ? a.sched.tiles256 : a.sched.tiles128)[item.tile];
    }
    GroupDesc gd;
    gd.tok_base = td.tok_base; gd.Lp = td.Lp; gd.Tg = td.Tg; gd.G = 0; gd.roff = nullptr;
    const int Lp = gd.Lp, Tg = gd.Tg;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const WaveRows wr = wave_rows<NW>(td, item, PIECES ? a.rows.rep : a.items.rep, w);
    const int head = wr.head;
    const int t0 = wr.t0, t1 = wr.t1;
    const int64_t T_total = a.T_total;
    if (t0 >= Tg || (a.resp_only && t1 <= Lp)) return;      // past the group's end, or prompt rows only

    const int c = l & 31, hh = l >> 5, j = l & 15, c16 = (l >> 4) & 1;

    const int tw0 = wr.tw0;
    const int t = tw0 + c;
    const bool valid = t < Tg;
    const int tm = valid ? t : -1;
    const bool wave_valid = tw0 < Tg;
    const int tw1 = min(tw0 + 31, Tg - 1);
    // What the rows' own words say is loaded ahead of everything and looked at behind the issue of the rows: a wait for each
    // of them in turn was a quarter of the prologue.
    const int64_t row_word = (int64_t)head * T_total + gd.tok_base + min(t, Tg - 1);
    int st_word, b2_word;
    if constexpr (SMALL) {
        const int first = max(t0, Lp);                     // as in the forward
        int s1, e1;
        small_segment(sg, hh == 0 ? t : first, s1, e1);
        b2_word = first < Tg ? __builtin_amdgcn_readlane(s1, 32) : 0;
        s1 = __shfl(s1, c, 64);
        st_word = t >= Lp ? s1 : 0;
    } else {
        st_word = a.sched.key_lo[gd.tok_base + min(t, Tg - 1)];
        b2_word = a.sched.key_lo[gd.tok_base + min(max(t0, Lp), Tg - 1)];
    }
    const float lse_word = a.lse[row_word], nD_word = a.fused_rowsum ? 0.f : a.nD[row_word];
    const bool have_lo = a.fused_rowsum && a.o_lo != nullptr;
    const uint32_t lo_word = !have_lo || a.lo_flag == nullptr ? 1u : SMALL ? (uint32_t)reserve_tag_matches(a.small.tag, a.small.want, l) : *a.lo_flag;

    auto sgpr64 = [](const void* p) -> uint64_t {
        const uint64_t b = (uint64_t)(uintptr_t)p;
        return ((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
               (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    };
    auto lds_u32 = [](char* p) -> unsigned {
        return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)p);
    };

    const int kvh = item.kvh;
    const int64_t kv_stride = (int64_t)a.Hkv * 128;
    const __bf16* kbase = a.k + ((int64_t)gd.tok_base * a.Hkv + kvh) * 128;
    const __bf16* vbase = a.v + ((int64_t)gd.tok_base * a.Hkv + kvh) * 128;

    // Tile copy global -> LDS, issued by the first wave of each SIMD (w < 4): those waves are
    // served first by the instruction arbiter and would otherwise idle at the barrier.  Wave w
    // copies chunks 4w .. 4w+3 (4 rows each) of the K tile and of the V tile.  Rows past the
    // group's end re-read its last row (those keys are always masked; values must be finite).
    const unsigned stride_b = (unsigned)(kv_stride * 2);
    // (NW = 4: every wave is the first of its SIMD within the workgroup; wave w copies chunks 2w, 2w+1 of the
    // 32 rows of K and of V of a half.)
    const bool copier = w < 4;
    constexpr int NCH = NW == 8 ? 4 : 2;        // chunks of K (and of V) a copying wave moves per slot
    unsigned voff[NCH];
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
        const int row = 4 * (NCH * (w & 3) + u) + (l >> 4);
        voff[u] = row * stride_b + (((l & 15) ^ swz(row)) << 4);
    }
    const uint64_t kbase_s = sgpr64(kbase), vbase_s = sgpr64(vbase);
    unsigned m0slot[NSLOT];
#pragma unroll
    for (int i = 0; i < NSLOT; ++i) m0slot[i] = lds_u32(lds[i]) + 1024u * NCH * (w & 3);
    // copies a slot's keys, from key0 on
    auto copy_keys = [&](int key0, int slot) {
        constexpr int ROWS = NW == 8 ? BN : 32;
        const uint64_t off = (uint64_t)(unsigned)key0 * stride_b;
        const unsigned m0 = m0slot[slot];
        if (key0 + ROWS <= Tg) {
#pragma unroll
            for (int u = 0; u < NCH; ++u) async_copy16_sm(kbase_s + off, voff[u], m0 + 1024u * u);
#pragma unroll
            for (int u = 0; u < NCH; ++u) async_copy16_sm(vbase_s + off, voff[u], m0 + V_OFF + 1024u * u);
        } else {
            const int last = Tg - 1 - key0;
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                const int row = 4 * (NCH * (w & 3) + u) + (l >> 4);
                const unsigned vo = min(row, last) * stride_b + (((l & 15) ^ swz(row)) << 4);
                async_copy16_sm(kbase_s + off, vo, m0 + 1024u * u);
                async_copy16_sm(vbase_s + off, vo, m0 + V_OFF + 1024u * u);
            }
        }
    };
    // the first keys under a prompt are known without a look at the rows' segments
    const int n1 = (min(Lp, t1) + BN - 1) / BN;
    const bool early = n1 > 0 && (!PIECES || piece.part == 0);
    if (copier && early) copy_keys(0, 0);

    // The wave's rows of q and dO (and of o and its residual for the folded rowsum) in MFMA operand layout.
    // Loaded straight from memory in that layout an instruction touches 32 rows and uses 32 bytes of each,
    // and the 32 such instructions of a wave are bound by the address unit: a quarter of a 128-row workgroup's
    // life on short key loops.  They come in like the K/V tiles instead: copied row-contiguous (four whole
    // rows per instruction) into the wave's own share of the not yet used tile ring, swizzled, and read back
    // with the operand reads of a K tile.  The share holds TPR tensors of 32 rows at a time; the others are loaded
    // meanwhile, row-contiguous too, into registers that the accumulators need only later, and pass through the share
    // afterwards: the prologue waits for memory once.  Rows past the
    // end of the group read the group's last row: their scores are all masked (P = dS = 0 whatever q and dO
    // hold, and a non-finite dO there only reaches dq rows that are not stored).
    constexpr int SHARE = NSLOT * SLOT_BYTES / NW;          // 16 KB (NW = 4), 12 KB (NW = 8)
    constexpr int TPR = SHARE / 8192;
    char* const stg = &lds[1][0] + SHARE * w;
    const int rbase = min(tw0, Tg - 1), rlast = Tg - 1 - rbase;
    auto stage_rows = [&](const __bf16* tensor, int slot) {
        const uint64_t sb = sgpr64(tensor + ((int64_t)(gd.tok_base + rbase) * a.Hq + head) * 128);
        const unsigned m0 = lds_u32(stg) + 8192u * slot;
        const unsigned row_bytes = (unsigned)a.Hq * 256u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int row = 4 * u + (l >> 4);
            async_copy16_sm(sb, (unsigned)min(row, rlast) * row_bytes + (((l & 15) ^ swz(row)) << 4), m0 + 1024u * u);
        }
    };
    auto load_rows = [&](const __bf16* tensor, i32x4 (&r)[8]) {
        const char* const p = reinterpret_cast<const char*>(tensor + ((int64_t)(gd.tok_base + rbase) * a.Hq + head) * 128);
        const unsigned row_bytes = (unsigned)a.Hq * 256u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int row = 4 * u + (l >> 4);
            r[u] = *reinterpret_cast<const i32x4*>(p + ((unsigned)min(row, rlast) * row_bytes + (((l & 15) ^ swz(row)) << 4)));
        }
    };
    auto put_rows = [&](const i32x4 (&r)[8], int slot) {
#pragma unroll
        for (int u = 0; u < 8; ++u) *reinterpret_cast<i32x4*>(stg + 8192 * slot + 1024 * u + 16 * l) = r[u];
    };
    auto read_rows = [&](int slot, bf16x8 (&r)[8]) {
        asm volatile("" ::: "memory");              // the reads stay behind the wait for the copies
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) r[ks] = lds_read_row8(stg + 8192 * slot, c, 2 * ks + hh);
    };
    auto lds_reads_done = [] { __builtin_amdgcn_s_waitcnt(0xC07F); };     // lgkmcnt(0): the share may be overwritten

    bf16x8 qreg[8], goreg[8];
    float Lq = 0.f, Dq = 0.f;
    {
        i32x4 gotmp[8], otmp[8], ltmp[8];
        stage_rows(a.q, 0);
        if constexpr (TPR == 2) stage_rows(a.d_o, 1);
        else load_rows(a.d_o, gotmp);
        if (a.fused_rowsum) load_rows(a.o, otmp);
        if (have_lo) load_rows(a.o_lo, ltmp);
        wait_vm0();
        read_rows(0, qreg);
        if constexpr (TPR == 2) {
            read_rows(1, goreg);
        } else {
            lds_reads_done();
            put_rows(gotmp, 0);
            read_rows(0, goreg);
        }
        if (a.fused_rowsum) {
            // The arithmetic of rowsum_bf16_kernel, operation for operation, so that a backward in one call
            // and a staged one agree bit for bit: that kernel gives a row to 16 lanes of 8 elements each
            // (lane `sub` = elements 8 sub .. 8 sub + 7: dO . o, then dO . residual, dot8()) and adds the lanes in an
            // xor-shuffle tree (8, 4, 2, 1).  This lane holds the chunks sub = 2 ks + hh, so the first three
            // levels are sums inside the lane and the last one is the exchange with the row's other lane.
            const bool use_lo = have_lo && __builtin_amdgcn_readfirstlane((int)lo_word) != 0;
            bf16x8 oreg[8], lreg[8];
            float ch[8];
            lds_reads_done();
            put_rows(otmp, 0);
            if (TPR == 2 && use_lo) put_rows(ltmp, 1);
            read_rows(0, oreg);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) ch[ks] = dot8(goreg[ks], oreg[ks], 0.f);
            if (use_lo) {
                if constexpr (TPR == 1) {
                    lds_reads_done();
                    put_rows(ltmp, 0);
                }
                read_rows(TPR - 1, lreg);
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) ch[ks] = dot8(goreg[ks], lreg[ks], ch[ks]);
            }
            const float x0 = ch[0] + ch[4], x1 = ch[1] + ch[5], x2 = ch[2] + ch[6], x3 = ch[3] + ch[7];
            const float y0 = x0 + x2, y1 = x1 + x3;
            Dq = pair_sum(y0 + y1);
        } else {
            Dq = -nD_word;
        }
        // in response-rows mode what prompt rows hold takes no part; the dkdv pass, which loads the planes of the 64 rows around
        // the prompt's end, gets zeros
        const bool idle = a.resp_only && t < Lp;
        if (!valid || idle) Dq = 0.f;
        Lq = valid && !idle ? lse_word * LOG2E : 0.f;
        if (a.fused_rowsum && hh == 0 && (!PIECES || piece.part == 0)) {
            if (valid) a.L2[row_word] = Lq;
            if (valid && idle) a.nD[row_word] = 0.f;
            if (a.resp_only && (tw0 & 32) && tw0 <= Lp && Lp < tw0 + 32) {      // first half of those 64 rows: of another workgroup
                const int64_t before = (int64_t)head * T_total + gd.tok_base + t - 32;
                a.L2[before] = 0.f;
                a.nD[before] = 0.f;
            }
        }
        // the shares overlap the ring slots that the first tile copies (of other waves, too) are about to fill
        lds_reads_done();
        __syncthreads();
    }
    // first own-segment key of this lane's row and of the workgroup's first response row (0 on the prompt)
    const int st = valid ? st_word : 0;
    const int b2 = __builtin_amdgcn_readfirstlane(b2_word);
    // lanes 0..31 hold the wave's rows in order: the last valid row's start comes from its lane
    const int st_last = wave_valid ? __builtin_amdgcn_readlane(st, tw1 - tw0) : 0;

    // key tiles as in the forward: n1 from the group's first key on, then from k2 on
    const int k2 = max(n1 * BN, b2);
    const int tiles = n1 + (t1 <= Lp ? 0 : max(t1 - k2 + BN - 1, 0) / BN);
    const int from = PIECES ? tiles * piece.part / piece.parts : 0;       // this workgroup's first tile, and how many it walks
    const int total = (PIECES ? tiles * (piece.part + 1) / piece.parts : tiles) - from;
    auto key_at = [&](int it) { return it + from < n1 ? (it + from) * BN : k2 + (it + from - n1) * BN; };
    // NW = 8: `it` counts 64-key tiles; NW = 4: halves of them (32 keys), each into a slot of its own.  The second half of a
    // group's last tile may lie wholly past the group's end: it is then read from the group's last row on
    auto issue = [&](int it, int slot) {
        if (!copier || it >= (NW == 8 ? total : 2 * total)) return;
        copy_keys(min(NW == 8 ? key_at(it) : key_at(it >> 1) + 32 * (it & 1), Tg - 1), slot);
    };

    f32x16 acc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    const float cs = a.c;
    float dsum = 0.f;      // sum over this lane's keys of P (dP - D): what D lacks to an O-free, fp32 evaluation of it
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    f32x16 nD16;           // dP accumulates on top of -D: dS = P acc, and sum P acc = sum P dP - D (sum P = 1)
#pragma unroll
    for (int r = 0; r < 16; ++r) nD16[r] = -Dq;
    asm volatile("" : "+v"(nD16));
    // Work is cut into halves of 32 keys (two per 64-key tile).  For half h a wave runs
    //   M(h): S^T, dP^T of the half (16 MFMAs);  V(h): P^T = exp2(S^T c - L), dS^T = P^T (dP^T - D)
    //   (16 elements of vector work);  D(h): dQ^T += K^T dS^T (8 MFMAs),
    // software-pipelined so that the vector work always sits between MFMAs of other halves:
    // V(h) is spread over the slices of D(h-1) (its first NE1 elements) and M(h+1) (the rest).
    // Each slice is {LDS read for the MFMA RD-1 ahead, one MFMA, a piece of vector work}, fenced.
    // Masking is done beforehand on S (masked score = -inf gives P = 0 and dS = 0), so the
    // pipeline body is the same for every tile; what the last stage computes of the half past the last one is
    // not used.
    const int H = 2 * total;
    auto s0_of = [&](int h) { return key_at(h >> 1) + 32 * (h & 1); };
    auto needs_mask = [&](int h) -> bool {
        if (h >= H) return false;
        if (!wave_valid) return true;
        const int s0 = s0_of(h);
        return !((s0 + 31 <= tw0) && (s0 + 32 <= Lp || s0 >= st_last));
    };
    auto mask = [&](int h, f32x16& S) {
        const int s0 = s0_of(h);
        mask16(S, (low_bits(min(Lp, tm + 1) - s0) | (low_bits(tm + 1 - s0) & ~low_bits(st - s0))) >> (4 * hh));
    };
    // LDS addresses of the operands within slot 0, opaque so that they are kept as whole sums (see the dkdv pass); `at`
    // = the slot's and the half's offset, a constant of the code
    unsigned rowA[8], trA[4][2];
    {
        const unsigned lds0 = lds_u32(&lds[0][0]);
#pragma unroll
        for (int i = 0; i < 8; ++i) { rowA[i] = lds0 + tile_off(c, 2 * i + hh); asm volatile("" : "+v"(rowA[i])); }
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                const int col4 = 32 * db + 16 * c16 + 4 * (j & 3);
                trA[db][part] = lds0 + tile_off(4 * hh + (j >> 2) + 8 * part, col4 >> 3) + ((col4 & 4) << 1);
                asm volatile("" : "+v"(trA[db][part]));
            }
    }
    // operand of slice i of a stage: 0..15 those of M, K rows then V rows; 16..23 those of D, slice 16 + i of D: db = i % 4,
    // 16-key step i / 4 (read transposed; four MFMAs in a row share their operand of dS, as in the forward).  They pass through one ring of RD registers, read RD - 1 slices ahead.
    auto fetch = [&](int atM, int atD, int i) -> bf16x8 {
        if (i < 16) return lds_at_row8(rowA[i & 7] + atM + ((i & 8) ? V_OFF : 0));
        const int n = i - 16, at = atD + 4096 * (n >> 2);
        return cat4(lds_at_tr4(trA[n & 3][0] + at), lds_at_tr4(trA[n & 3][1] + at));
    };
    bf16x8 ring[RD];
    auto pack2 = [&](float x, float y) -> unsigned {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        bf16x2 v = {(__bf16)x, (__bf16)y};
        return __builtin_bit_cast(unsigned, v);
    };
    float tprev = 0.f;
    // vector work on element r: the exponential is issued in one slice and consumed in the next
    auto v_issue = [&](f32x16& S, int r) {
        const float tcur = __builtin_amdgcn_exp2f(__builtin_fmaf(S[r], cs, -Lq));
        return tcur;
    };
    auto v_consume = [&](f32x16& S, f32x16& P, int r, float p) {
        dsum = __builtin_fmaf(p, P[r], dsum);
        S[r] = p * P[r];
        asm volatile("" : "+v"(dsum), "+v"(S[r]));
    };
    // One pipeline stage for half h: Sc/Pc hold S, dP of half h (elements < NE1 already turned
    // into dS), Sn/Pn receive half h+1.
    auto stage = [&](int h, f32x16& Sc, f32x16& Pc, f32x16& Sn, f32x16& Pn,
                     auto m_tag, auto d_tag, auto off_tag, auto next_tag) {
        constexpr int atM = decltype(m_tag)::value, atD = decltype(d_tag)::value;
        constexpr int OFF = decltype(off_tag)::value;       // ring position of this stage's first operand
        unsigned pk[8];
        // M(h+1) with the rest of V(h)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            ring[(i + RD - 1 + OFF) % RD] = fetch(atM, atD, i + RD - 1);
            if (i & 8) Pn = mfma32(ring[(i + OFF) % RD], goreg[i & 7], i == 8 ? nD16 : Pn);
            else Sn = mfma32(ring[(i + OFF) % RD], qreg[i & 7], i == 0 ? zero16 : Sn);
            float tcur = 0.f;
            if (NE1 + i < 16) { tcur = v_issue(Sc, NE1 + i); asm volatile("" : "+v"(tcur)); }
            if (i >= 1 && NE1 + i - 1 < 16) v_consume(Sc, Pc, NE1 + i - 1, tprev);
            tprev = tcur;
            if (i >= 12) {
#pragma unroll
                for (int q = 2 * (i - 12); q < 2 * (i - 12) + 2; ++q) {
                    pk[q] = pack2(Sc[2 * q], Sc[2 * q + 1]);
                    asm volatile("" : "+v"(pk[q]));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (needs_mask(h + 1)) mask(h + 1, Sn);
        const float dsum_h = dsum;
        __builtin_amdgcn_sched_barrier(0);
        // D(h) with the first NE1 elements of V(h+1); the ring runs on into the next stage where its tile is resident (NEXT)
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        const bf16x8 db8[2] = {__builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]}),
                               __builtin_bit_cast(bf16x8, u32x4{pk[4], pk[5], pk[6], pk[7]})};
        constexpr int NEXT = decltype(next_tag)::value;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i + RD - 1 < 8) ring[(16 + i + RD - 1 + OFF) % RD] = fetch(atM, atD, 16 + i + RD - 1);
            else if (NEXT >= 0) ring[(16 + i + RD - 1 + OFF) % RD] = fetch(NEXT, 0, i + RD - 1 - 8);
            acc[i & 3] = mfma32(ring[(16 + i + OFF) % RD], db8[i >> 2], acc[i & 3]);
            float tcur = 0.f;
            if (i < NE1) { tcur = v_issue(Sn, i); asm volatile("" : "+v"(tcur)); }
            if (i >= 1 && i - 1 < NE1) v_consume(Sn, Pn, i - 1, tprev);
            tprev = tcur;
            __builtin_amdgcn_sched_barrier(0);
        }
        if (h + 1 >= H) dsum = dsum_h;          // the half past the last one (stale LDS) contributes to nothing
    };

    f32x16 SA, PA, SB, PB;
    if (total > 0) {
        if (!early) {
            issue(0, 0);
            wait_vm0();
            __syncthreads();
        }
        issue(1, 1);
        if constexpr (NW == 4) issue(2, 2);
        // M(0) and the first NE1 elements of V(0), unpipelined
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i & 8) PA = mfma32(fetch(0, 0, i), goreg[i & 7], i == 8 ? nD16 : PA);
            else SA = mfma32(fetch(0, 0, i), qreg[i & 7], i == 0 ? zero16 : SA);
        }
        if (needs_mask(0)) mask(0, SA);
#pragma unroll
        for (int r = 0; r < NE1; ++r) v_consume(SA, PA, r, v_issue(SA, r));
        // the first operands of a stage behind a barrier are fetched ahead of the issue of the next copies
        auto prime = [&](int atM) {
#pragma unroll
            for (int i = 0; i < RD - 1; ++i) ring[i] = fetch(atM, 0, i);
            __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (NW == 8) {
        // tile `it` lives in slot it % 3; a turn of the loop is a turn of the ring
        auto tile_stages = [&](int it, auto slot_tag) {
            constexpr int S = decltype(slot_tag)::value, S1 = (S + 1) % 3, S2 = (S + 2) % 3, HALF = 32 * 256;
            constexpr int A0 = S * SLOT_BYTES, A1 = A0 + HALF, A2 = S1 * SLOT_BYTES;       // halves 2 it, 2 it + 1, 2 it + 2
            wait_vm0();
            __syncthreads();
            prime(A1);
            issue(it + 2, S2);              // into the slot of tile it-1, which every wave has left
            stage(2 * it, SA, PA, SB, PB, std::integral_constant<int, A1>{}, std::integral_constant<int, A0>{},
                  std::integral_constant<int, 0>{}, std::integral_constant<int, A2>{});
            stage(2 * it + 1, SB, PB, SA, PA, std::integral_constant<int, A2>{}, std::integral_constant<int, A1>{},
                  std::integral_constant<int, 24 % RD>{}, std::integral_constant<int, -1>{});
        };
        for (int it = 0; it < total; it += 3) {
            tile_stages(it, std::integral_constant<int, 0>{});
            if (it + 1 >= total) break;
            tile_stages(it + 1, std::integral_constant<int, 1>{});
            if (it + 2 >= total) break;
            tile_stages(it + 2, std::integral_constant<int, 2>{});
        }
        } else {
        // Half h lives in slot h % 4.  Stage h reads the slots of h + 1 (M) and h (D); at the barrier in
        // front of it every wave has left stage h - 1, whose D read the slot of h - 1 = the slot of h + 3,
        // which is issued then: two stages ahead of the M that needs it.
        // (Leaving the half issued at the previous barrier in flight across the barrier, vmcnt(4) instead of
        // vmcnt(0), measured the same: the other workgroup of the CU covers the wait.)
        auto half_stage = [&](int h, auto slot_tag, f32x16& Sc, f32x16& Pc, f32x16& Sn, f32x16& Pn) {
            constexpr int S = decltype(slot_tag)::value, A0 = S * SLOT_BYTES, A1 = ((S + 1) & 3) * SLOT_BYTES;
            wait_vm0();
            __syncthreads();
            prime(A1);
            issue(h + 3, (S + 3) & 3);
            stage(h, Sc, Pc, Sn, Pn, std::integral_constant<int, A1>{}, std::integral_constant<int, A0>{},
                  std::integral_constant<int, 0>{}, std::integral_constant<int, -1>{});
        };
        for (int h = 0; h < H; h += 4) {
            half_stage(h, std::integral_constant<int, 0>{}, SA, PA, SB, PB);
            half_stage(h + 1, std::integral_constant<int, 1>{}, SB, PB, SA, PA);
            if (h + 2 >= H) break;
            half_stage(h + 2, std::integral_constant<int, 2>{}, SA, PA, SB, PB);
            half_stage(h + 3, std::integral_constant<int, 3>{}, SB, PB, SA, PA);
        }
        }
    }

    // D + sum_s P (dP - D) = sum_s P dP equals rowsum(dO * O) exactly, but does not inherit the bf16 rounding of O.
    // Publish it for the dkdv pass (this workgroup owns these rows of D, so overwriting is safe).
    dsum = pair_sum(dsum);
    const bool store = valid && !(a.resp_only && t < Lp);
    // rows that see at most EDGE_LEN keys are written by the workgroups above (fp32 dS): not stored here
    const bool short_row = (t < Lp ? 0 : Lp) + t - st + 1 <= EDGE_LEN;
    if constexpr (PIECES)
        if (piece.parts > 1) {
            float* const slot = a.rows.slots + ((int64_t)item.kvh * a.rows.n_slots + piece.slot) * (int64_t)(ROW_SLOT_BYTES / 4) + w * (ROW_SLOT_BYTES / 16);
#pragma unroll
            for (int n = 0; n < 16; ++n)
                *reinterpret_cast<f32x4*>(slot + 128 * c + 32 * (n >> 2) + 8 * (n & 3) + 4 * hh) =
                    f32x4{acc[n >> 2][4 * (n & 3)], acc[n >> 2][4 * (n & 3) + 1], acc[n >> 2][4 * (n & 3) + 2], acc[n >> 2][4 * (n & 3) + 3]};
            if (hh == 0) *reinterpret_cast<f32x4*>(slot + 4096 + 4 * c) = f32x4{dsum, Dq, 0.f, store && !short_row ? 1.f : 0.f};
            return;
        }
    if (store && !short_row && hh == 0) a.nD[(int64_t)head * T_total + gd.tok_base + t] = -(Dq + dsum);
    // dQ leaves in whole rows: staged in the wave's share of the ring (every wave has left it), 16 lanes to a row, four rows
    // per instruction; stored from the accumulators an instruction touched 32 rows (64 groups of a short prompt and 16
    // answers 3158 -> 2935 us, 64 groups of 1000 tokens 1017 -> 969, four long prompts 2503 -> 2483)
    int lz = l;
    asm volatile("" : "+v"(lz));
    const uint64_t keep = __builtin_amdgcn_ballot_w64(store && !short_row);        // bit = the row's low lane
    const unsigned putA = lds_u32(stg) + 256u * (lz & 31) + 8u * (lz >> 5) + (swz(lz & 31) << 4);      // as in the forward
    const unsigned getA = lds_u32(stg) + 256u * (lz >> 4) + (((lz & 15) ^ ((lz >> 4) << 2)) << 4);
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 16; ++n) {
        f32x16& x = acc[n >> 2];
        const int r = 4 * (n & 3);
        *(__attribute__((address_space(3))) u32x2*)(uintptr_t)(putA ^ (n << 4)) =
            u32x2{pack2(x[r] * a.scale, x[r + 1] * a.scale), pack2(x[r + 2] * a.scale, x[r + 3] * a.scale)};
    }
    bf16x8 x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = lds_at_row8((getA ^ ((i & 3) << 4)) + 1024u * i);
    __bf16* const p0 = a.dq + ((int64_t)(gd.tok_base + tw0 + (lz >> 4)) * a.Hq + head) * 128 + 8 * (lz & 15);
    const int64_t stride = (int64_t)4 * a.Hq * 128;
    if ((unsigned)keep == 0xffffffffu) {
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<bf16x8*>(p0 + i * stride) = x[i];
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if ((keep >> (4 * i + (lz >> 4))) & 1) *reinterpret_cast<bf16x8*>(p0 + i * stride) = x[i];
    }
}

// Adds up the parts of an item's dQ (32 rows of one q head) and of what D lacks: a workgroup per item, 8 threads to a row, 16 columns each.
__global__ __launch_bounds__(256) void dq_pieces_kernel(RowSums list, BwdArgs a) {
    const RowItem it = row_item(list, a.rows);
    const float* const slot = row_slot(a.rows, it);
    const int r = threadIdx.x >> 3, d0 = 16 * (threadIdx.x & 7);
    if (slot[4096 + 4 * r + 3] == 0.f) return;             // not a row to store
    float dsum = 0.f, x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = 0.f;
    for (int p = 0; p < it.parts; ++p) {
        const float* const s = slot + p * (int64_t)(ROW_SLOT_BYTES / 4);
        dsum += s[4096 + 4 * r];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const f32x4 y = *reinterpret_cast<const f32x4*>(s + 128 * r + d0 + 4 * n);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * n + e] += y[e];
        }
    }
    bf16x8 y[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e >> 3][e & 7] = (__bf16)(x[e] * a.scale);
    __bf16* const out = a.dq + ((int64_t)(it.tok + r) * a.Hq + it.head) * 128 + d0;
    *reinterpret_cast<bf16x8*>(out) = y[0];
    *reinterpret_cast<bf16x8*>(out + 8) = y[1];
    if (d0 == 0) a.nD[(int64_t)it.head * a.T_total + it.tok + r] = -(slot[4096 + 4 * r + 1] + dsum);
}

// ------------------------------------------------------------------------------------
// dkdv pass
// ------------------------------------------------------------------------------------
// A workgroup owns 128 keys of one kv head and streams Q/dO row tiles through a double buffer.
// Bound: bf16 MFMA (32 per wave and 32 rows x 32 keys).  Two shapes:
//   NW = 4: wave w owns 32 keys and every row, in tiles of 32 rows.  Its K rows stay in 32 registers and its V rows in
//     LDS in the order the lanes read them: 64.5 KB of LDS, TWO workgroups per CU that do not wait for one another, so
//     that one's barriers, first loads, stores and steps without work (other responses' rows) lie under the other's MFMAs.
//   NW = 8: wave w owns key block w & 3 and the row half w >> 2 of tiles of 64 rows, K and V in LDS, one workgroup per
//     CU; the two halves' partial sums are added through LDS at the end, in a fixed order.  Half as many steps per
//     workgroup: where the longest one counts (dkdv_head_split, and by dkdv_waves()).
// The LDS addresses of a step's operands are whole sums in registers plus constants (two steps per turn of the loop, one
// per buffer); left to the compiler they were 25 additions per step, and K did not fit the registers.
// 8 -> 4 waves with these addresses, one box: 16K prompt with 32 answers 7.67 -> 7.24 ms, 64 groups of a short prompt
// and 16 answers 4.44 -> 3.95 ms, 64 groups of 1000 tokens 1.33 -> 1.07 ms, response rows under an 8K prompt 0.77 -> 0.67 ms.

// Row parts of a key tile of `steps` 64-row tiles in the head-split pass (see dkdv_parts())
__device__ __forceinline__ int row_parts(const BwdArgs& a, int steps) { return a.head_split == 2 && steps >= PART_STEPS ? 2 : 1; }

// PIECES: part `part` of `parts` of the tile's steps (row tile, q head); the sums go to `sums` where there are several
template <int NW, bool SMALL, bool PIECES>
__device__ __forceinline__ void dkdv_body(const BwdArgs& a, const SmallGroup& sg, const TileDesc td, const int kvh, const int hr_only, const int part,
                                          const int parts, float* const sums) {
    const int ti = td.ti;
    constexpr int BNK = 128, BQ = 8 * NW;
    constexpr bool K_REG = NW == 4;                 // the wave's K rows stay in registers, only V in LDS
    constexpr int QT_BYTES = BQ * 256;              // a Q (or dO) tile
    constexpr int CH = BQ / (4 * NW);               // 4-row chunks of a Q (or dO) tile that a wave copies
    // NW = 8: [K | V] of the 128 keys, swizzled rows.  NW = 4: the eight V operands of each wave in lane order
    __shared__ __attribute__((aligned(1024))) char dkdv_ldsKV[K_REG ? 128 * 256 : 2 * 128 * 256];
    __shared__ __attribute__((aligned(1024))) char dkdv_lds[2][2 * QT_BYTES];                // [buffer][Q | dO]
    __shared__ __attribute__((aligned(256))) float dkdv_ldsLD[2][2][BQ];                     // [buffer][L2 | -D][row]
    __shared__ int dkdv_ldsEnd[K_REG ? BNK : 1];    // e_s of the tile's keys, below
    constexpr int RD = 3;      // LDS operand ring depth (prefetch distance RD - 1 MFMAs)
    const int s0 = ti * BNK;
    GroupDesc gd;
    gd.tok_base = td.tok_base; gd.Lp = td.Lp; gd.Tg = td.Tg; gd.G = 0; gd.roff = nullptr;
    const int Lp = gd.Lp, Tg = gd.Tg;
    const int64_t T_total = a.T_total;

    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int c = l & 31, hh = l >> 5, j = l & 15, c16 = (l >> 4) & 1;
    const int kb = NW == 8 ? w & 3 : (w + ti) & 3, qh = w >> 2;

    // this lane's key (a column of S) and the rows [s, e_s) that may see it
    const int s = s0 + 32 * kb + c;
    const bool valid = s < Tg;
    const int ws0 = s0 + 32 * kb;                      // wave's first key
    const bool wave_valid = ws0 < Tg;
    const int ws1 = min(ws0 + 31, Tg - 1);             // wave's last valid key
    const int s1 = min(s0 + BNK, Tg);
    // rows [s, e_s) see this lane's key; row_end: where the rows that see any key of the tile end (the
    // group's end if the tile holds a prompt key, else the end of its last key's response)
    int e_s, row_end;
    if constexpr (SMALL) {
        int b1, e1;
        small_segment(sg, hh == 0 ? s : s1 - 1, b1, e1);
        row_end = s0 < Lp ? Tg : __builtin_amdgcn_readlane(e1, 32);
        e1 = __shfl(e1, c, 64);
        e_s = !valid ? 0 : s < Lp ? Tg : e1;
    } else {
        e_s = valid ? a.sched.row_hi[gd.tok_base + s] : 0;
        row_end = __builtin_amdgcn_readfirstlane(s0 < Lp ? Tg : a.sched.row_hi[gd.tok_base + s1 - 1]);
    }
    // smallest / largest row bound e_s over the wave's keys (prompt keys: Tg; response keys: the
    // end of their response, non-decreasing in s); lanes 0..31 hold the wave's keys in order
    const int e_min = !wave_valid ? 0 : (ws1 < Lp ? Tg : __builtin_amdgcn_readlane(e_s, max(ws0, Lp) - ws0));
    const int e_max = !wave_valid ? 0 : (ws0 < Lp ? Tg : __builtin_amdgcn_readlane(e_s, ws1 - ws0));

    // with only response rows contributing, the rows start at the end of the prompt
    const int row_lo = a.resp_only ? Lp : 0;
    // (four waves: a step that masks reads e_s back; held in a register it was spilled, and its reload waited for the
    // tile copies.  Eight waves have the register: 1 % of the pass)
    if (K_REG && hh == 0) dkdv_ldsEnd[32 * kb + c] = e_s;
    // (no tile at all under a prompt without response rows: the one that its end cuts holds no row that takes part, and nothing
    // writes L2 and -D of its rows)
    int qt0 = max(s0, row_lo) / BQ, qt1 = row_end > row_lo ? (row_end + BQ - 1) / BQ : qt0;
    if (NW == 8 && !PIECES && a.head_split) {          // this workgroup's row part, the later rows first
        const int n = row_parts(a, qt1 - qt0), mid = (qt0 + qt1) / 2;
        if (part >= n) return;
        if (n == 2) { if (part == 0) qt0 = mid; else qt1 = mid; }
    }
    const int rep_all = a.rep;
    const int rep = NW == 8 && !PIECES && a.head_split ? 1 : rep_all;        // q heads this workgroup walks
    const int64_t q_stride = (int64_t)a.Hq * 128;
    const int64_t kv_stride = (int64_t)a.Hkv * 128;

    bf16x8 kreg[8];                                   // NW = 4 only
    // K/V of the tile -> LDS (64 chunks of 4 rows; 8 per wave).  Keys past the group's end
    // re-read its last row; such lanes are masked everywhere (e_s = 0).
    {
        const __bf16* kb_ = a.k + ((int64_t)gd.tok_base * a.Hkv + kvh) * 128;
        const __bf16* vb_ = a.v + ((int64_t)gd.tok_base * a.Hkv + kvh) * 128;
        if constexpr (!K_REG) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int ci = w * 8 + u;              // 0..31 K, 32..63 V
                const int row = 4 * (ci & 31) + (l >> 4);
                const int gran = (l & 15) ^ swz(row);
                const int sk = min(s0 + row, Tg - 1);
                const __bf16* src = (ci < 32 ? kb_ : vb_) + (int64_t)sk * kv_stride + gran * 8;
                async_copy16(src, &dkdv_ldsKV[ci * 1024]);
            }
        } else {
            // this wave's 32 rows of V, then of K, row-contiguous through its quarter of the Q/dO buffers and from
            // there in operand layout to their place
            char* const stg = &dkdv_lds[0][0] + 8192 * w;
#pragma unroll
            for (int which = 0; which < 2; ++which) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int row = 4 * u + (l >> 4);
                    const int sk = min(ws0 + row, Tg - 1);
                    async_copy16((which == 0 ? vb_ : kb_) + (int64_t)sk * kv_stride + ((l & 15) ^ swz(row)) * 8, stg + 1024 * u);
                }
                wait_vm0();
                asm volatile("" ::: "memory");
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const bf16x8 x = lds_read_row8(stg, c, 2 * ks + hh);
                    if (which == 0) *reinterpret_cast<bf16x8*>(&dkdv_ldsKV[1024 * (8 * w + ks) + 16 * l]) = x;
                    else kreg[ks] = x;
                }
                __builtin_amdgcn_s_waitcnt(0xC07F);    // lgkmcnt(0): the buffers may be overwritten
                asm volatile("" ::: "memory");
            }
            __syncthreads();
        }
    }
    // Row tiles are walked from the LAST one down to the workgroup's own keys: workgroups that
    // start together (they share a kv head and an XCD) then stream the same Q/dO tiles at the
    // same time, so all but the first read of a tile hit that XCD's L2.
    // The q heads of the kv head are the inner loop, for the same reason.
    // Step `it` = (row tile qt1 - 1 - it / rep, q head it % rep).  Its Q/dO tile is copied
    // asynchronously into buffer it & 1: wave w copies chunks 2w, 2w+1 (4 rows each) of Q and of
    // dO, from a scalar tile base plus a constant per-lane offset.  (The copies wait on HBM, and a
    // wave that queues more than a few of them stalls at issue, so all eight waves share them.)
    // Rows past the group's end re-read its last row; they are masked (t < e_s <= Tg fails).
    const unsigned qstride_b = (unsigned)(q_stride * 2);
    unsigned voff[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int row = 4 * (CH * w + u) + (l >> 4);
        voff[u] = row * qstride_b + (((l & 15) ^ swz(row)) << 4);
    }
    auto sgpr64 = [](const void* p) -> uint64_t {
        const uint64_t b = (uint64_t)(uintptr_t)p;
        return ((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
               (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    };
    auto lds_u32 = [](const void* p) -> unsigned {
        return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)p);
    };
    // first q head of this workgroup, token 0 of the group
    const int head0 = kvh * rep_all + hr_only;          // first q head this workgroup walks
    const uint64_t qbase_s = sgpr64(a.q + ((int64_t)gd.tok_base * a.Hq + head0) * 128);
    const uint64_t gbase_s = sgpr64(a.d_o + ((int64_t)gd.tok_base * a.Hq + head0) * 128);
    const uint64_t l2_s = sgpr64(a.L2), nd_s = sgpr64(a.nD);       // (selected per lane, not loaded per lane and step)
    const unsigned m0buf[2] = {lds_u32(dkdv_lds[0]) + 1024u * CH * w, lds_u32(dkdv_lds[1]) + 1024u * CH * w};
    const unsigned tile_bytes = BQ * qstride_b;
    auto issue_tile = [&](int qt, int hr, int buf) {
        const uint64_t off = (uint64_t)(unsigned)qt * tile_bytes + (unsigned)hr * 256u;
        const unsigned m0 = m0buf[buf];
        if (qt * BQ + BQ <= Tg) {
#pragma unroll
            for (int u = 0; u < CH; ++u) async_copy16_sm(qbase_s + off, voff[u], m0 + 1024u * u);
#pragma unroll
            for (int u = 0; u < CH; ++u) async_copy16_sm(gbase_s + off, voff[u], m0 + QT_BYTES + 1024u * u);
        } else {
            const int last = Tg - 1 - qt * BQ;
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const int row = 4 * (CH * w + u) + (l >> 4);
                const unsigned vo = min(row, last) * qstride_b + (((l & 15) ^ swz(row)) << 4);
                async_copy16_sm(qbase_s + off, vo, m0 + 1024u * u);
                async_copy16_sm(gbase_s + off, vo, m0 + QT_BYTES + 1024u * u);
            }
        }
        if constexpr (NW == 4) {      // wave 0: L2 of the 32 rows in its low lanes, -D in its high lanes
            if (w == 0) {
                const int head = head0 + hr;
                const int t = min(qt * BQ + c, Tg - 1);
                const float* src = (const float*)(uintptr_t)(hh == 0 ? l2_s : nd_s) + (int64_t)head * T_total + gd.tok_base + t;
                async_copy4(src, reinterpret_cast<char*>(&dkdv_ldsLD[buf][0][0]));
            }
        } else if (w < 2) {        // wave 0: L2 of the 64 rows, wave 1: -D (the first wave of a SIMD has slack)
            const int head = head0 + hr;
            const int t = min(qt * BQ + l, Tg - 1);
            const float* src = (w == 0 ? a.L2 : a.nD) + (int64_t)head * T_total + gd.tok_base + t;
            async_copy4(src, reinterpret_cast<char*>(&dkdv_ldsLD[buf][w][0]));
        }
    };

    f32x16 dkacc[4], dvacc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dkacc[db][r] = 0.f; dvacc[db][r] = 0.f; }
    const float cs = a.c;
    // LDS addresses of the operands within buffer 0, opaque so that they are kept as sums: row operands of Q (dO: + QT_BYTES),
    // transposed operands of Q, rows + 8 part of the block's first 16 rows (last 16: + 4096, the swizzle repeats)
    unsigned rowA[8], trA[4][2];
    const unsigned lds0 = lds_u32(dkdv_lds[0]);
#pragma unroll
    for (int i = 0; i < 8; ++i) { rowA[i] = lds0 + tile_off(32 * qh + c, 2 * i + hh); asm volatile("" : "+v"(rowA[i])); }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            const int col4 = 32 * db + 16 * c16 + 4 * (j & 3);
            trA[db][part] = lds0 + tile_off(32 * qh + 4 * hh + (j >> 2) + 8 * part, col4 >> 3) + ((col4 & 4) << 1);
            asm volatile("" : "+v"(trA[db][part]));
        }
    unsigned opB = lds_u32(dkdv_ldsKV) + (K_REG ? 8192 * w + 16 * l : 0);
    asm volatile("" : "+v"(opB));
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const char* ldsK = dkdv_ldsKV;
    const char* ldsV = dkdv_ldsKV + 128 * 256;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

    // dP accumulates on top of -D, so that dS = P acc is one multiplication per element and D of the rows occupies no
    // registers of its own; S starts from zero and L2 is subtracted within the exponent's fma.  (S seeded with -lse / scale
    // in the same way saves 1.5 % of the pass under responses of 30 to 600 tokens and nothing elsewhere, but each of its
    // partial sums rounds at the magnitude of lse / scale, which doubles the error of P on ordinary inputs, and
    // -lse / scale leaves float32 under a scale of 1e-30.)
    // Within a step the vector work is folded under the MFMAs: the exponentials of the first 8
    // rows run under the dP MFMAs (S is complete by then), those of the last 8 rows under the
    // first half of the dV/dK MFMAs (which only need the first 8 rows of P and dS).  Masking is
    // applied to S beforehand (score -inf gives P = 0 and dS = 0).
    // Rows that see only a few keys carry weights P of order one, and a key's dK / dV can be made up almost
    // entirely of a handful of such terms, whose bf16 roundings of P and dS then do not average out.  The
    // steps that hold such rows (the first EDGE_LEN rows of a prompt; under a shorter prompt, conservatively,
    // every step with response rows: with only the row tiles that hold short rows, dK and dV of 2 x (60 + 26 x 60..85) tokens
    // were off from float64 by 2.0e-3 instead of 1.66e-3) are therefore swept a second time after the main sweep, with P and dS
    // replaced by what their rounding dropped, P - bf16(P) and dS - bf16(dS) (rounded to bf16 in turn): the
    // two sweeps together carry P and dS into dV and dK to about 2^-17.  The second sweep is the same code
    // with another packing function, outside the main loop, so it costs that loop neither registers nor time.
    auto sweep = [&](auto lo_tag, const int q_hi, const int q_lo) {      // row tiles q_hi - 1 down to q_lo
    constexpr bool LO = decltype(lo_tag)::value;
    auto pack2 = [&](float x, float y) -> unsigned {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        bf16x2 v = {(__bf16)x, (__bf16)y};
        if (LO) v = bf16x2{(__bf16)(x - (float)v[0]), (__bf16)(y - (float)v[1])};
        return __builtin_bit_cast(unsigned, v);
    };
    int n_steps = max(q_hi - q_lo, 0) * rep;
    int qt = q_hi - 1, hr = 0;                // step 0
    if constexpr (PIECES) {
        const int from = n_steps * part / parts;
        n_steps = n_steps * (part + 1) / parts - from;
        unsigned r;
        qt -= (int)divmod((unsigned)from, a.rep_div, r);
        hr = (int)r;
    }
    int qt_n = qt, hr_n = hr + 1;             // step 1
    if (hr_n == rep) { hr_n = 0; --qt_n; }
    if (n_steps > 0) issue_tile(qt, hr, 0);
    auto step = [&](const int it, auto buf_tag) {
        constexpr int buf = decltype(buf_tag)::value;
        wait_vm0();
        __syncthreads();
        constexpr int offQ = buf * 2 * QT_BYTES, offG = offQ + QT_BYTES;
        const float* ldsL = dkdv_ldsLD[buf][0];
        const float* ldsD = dkdv_ldsLD[buf][1];
        const int r0 = qt * BQ + 32 * qh;              // this wave's 32 rows
        const int qt_n_issue = qt_n, hr_n_issue = hr_n;
        qt = qt_n; hr = hr_n;
        if (++hr_n == rep) { hr_n = 0; --qt_n; }
        // no row of this wave's half sees any key of this wave
        const bool skip = !wave_valid || r0 + 31 < max(ws0, row_lo) || r0 >= e_max ||
                          (LO && !(r0 < min(Lp, EDGE_LEN) || (Lp < EDGE_LEN && r0 + 31 >= Lp)));   // or: no short row here

        // The LDS operands of the step's 32 MFMAs pass through one pair of rings, read RD - 1 MFMAs ahead
        // without a break between the four products (a product that primed rings of its own would start with
        // an exposed LDS round trip).  Slice i: 0..7 S = Q K^T, 8..15 dP = dO V^T, 16..23 and 24..31 the dV / dK
        // updates for the first and the last 16 rows of the block (A operand only: P and dS are in registers).
        auto ldt = [&](int mm, int i, int part) {       // dV for even i, dK for odd i; db = i / 2
            return lds_at_tr4(trA[i >> 1][part] + ((i & 1) ? offQ : offG) + 4096 * mm);
        };
        auto fetchA = [&](int i) -> bf16x8 {
            if (i < 8) return lds_at_row8(rowA[i] + offQ);
            if (i < 16) return lds_at_row8(rowA[i - 8] + offG);
            return cat4(ldt((i - 16) >> 3, i & 7, 0), ldt((i - 16) >> 3, i & 7, 1));
        };
        auto fetchB = [&](int i) -> bf16x8 {            // NW = 4: i >= 8 only
            if (K_REG) return lds_at_row8(opB + 1024 * (i & 7));
            return lds_read_row8(i < 8 ? ldsK : ldsV, 32 * kb + c, 2 * (i & 7) + hh);
        };
        bf16x8 ra[RD], rb[RD];
        auto advance = [&](int i) {                      // fetch the operands of slice i + RD - 1
            const int n = i + RD - 1;
            if (n < 32) ra[n % RD] = fetchA(n);
            if (n < 16 && (n >= 8 || !K_REG)) rb[n % RD] = fetchB(n);
        };
        // rows of a plane in accumulator layout: the initial value of a product over this wave's 32 rows
        auto rows16 = [&](const float* plane, int gq, f32x16& acc) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(&plane[32 * qh + 8 * gq + 4 * hh]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * gq + e] = x[e];
        };
        f32x16 sacc, pacc;
        f32x4 Lr[2];                                     // L2 of rows 8 gq + 4 hh .. + 3 of the block, in Lr[gq & 1]
        auto rowsL = [&](int gq) { Lr[gq & 1] = *reinterpret_cast<const f32x4*>(&ldsL[32 * qh + 8 * gq + 4 * hh]); };
        // the first operands are fetched ahead of the issue of the next tile's copies, which every wave takes
        // part in whether it has work in this step or not
        if (!skip) {
#pragma unroll
            for (int i = 0; i < RD - 1; ++i) { ra[i] = fetchA(i); if (!K_REG) rb[i] = fetchB(i); }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (it + 1 < n_steps) issue_tile(qt_n_issue, hr_n_issue, buf ^ 1);
        if (skip) return;
#pragma unroll
        for (int i = 0; i < 8; ++i) {       // S = Q K^T
            advance(i);
            if (i < 2) rowsL(i);                         // (both planes two slices later: 1 % of the pass)
            if (i >= 2 && i < 6) rows16(ldsD, i - 2, pacc);
            sacc = mfma32(ra[i % RD], K_REG ? kreg[i] : rb[i % RD], i == 0 ? zero16 : sacc);
            __builtin_amdgcn_sched_barrier(0);
        }
        // every row of the half sees every key of the wave
        const bool full = r0 >= max(ws1, row_lo) && ws0 + 31 < Tg && r0 + 32 <= e_min;
        if (!full) {
            int lane;                                    // again, so that nothing of the mask lives across steps
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(lane));
            const int key = 32 * kb + (lane & 31), end = K_REG ? dkdv_ldsEnd[key] : e_s;
            mask16(sacc, (low_bits(end - r0) & ~low_bits(max(s0 + key, row_lo) - r0)) >> (4 * (lane >> 5)));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {       // dP - D = dO V^T on top of -D, with the exponentials of rows 0..7 of the block
            advance(8 + i);
            pacc = mfma32(ra[(8 + i) % RD], rb[(8 + i) % RD], pacc);
            sacc[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], cs, -Lr[i >> 2][i & 3]));      // P
            asm volatile("" : "+v"(sacc[i]));
            if (i == 3) rowsL(2);
            __builtin_amdgcn_sched_barrier(0);
        }
        unsigned pp[8], dd[8];       // packed bf16 pairs of P and dS: [4 * mm + r / 2]
#pragma unroll
        for (int r = 0; r < 8; ++r) pacc[r] *= sacc[r];                                  // dS
#pragma unroll
        for (int q = 0; q < 4; ++q) { pp[q] = pack2(sacc[2 * q], sacc[2 * q + 1]); dd[q] = pack2(pacc[2 * q], pacc[2 * q + 1]); }
        __builtin_amdgcn_sched_barrier(0);
        // dV^T += dO^T P, dK^T += Q^T dS
        {   // first 16 rows of the block (mm = 0), with the exponentials and dS of rows 8..15
            const bf16x8 p8 = __builtin_bit_cast(bf16x8, u32x4{pp[0], pp[1], pp[2], pp[3]});
            const bf16x8 d8 = __builtin_bit_cast(bf16x8, u32x4{dd[0], dd[1], dd[2], dd[3]});
            float tprev = 0.f;
            rowsL(3);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                advance(16 + i);
                const bf16x8 A = ra[(16 + i) % RD];
                if (i & 1) dkacc[i >> 1] = mfma32(A, d8, dkacc[i >> 1]);
                else dvacc[i >> 1] = mfma32(A, p8, dvacc[i >> 1]);
                float tcur = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[8 + i], cs, -Lr[i >> 2][i & 3]));
                asm volatile("" : "+v"(tcur));
                if (i >= 1) {
                    sacc[8 + i - 1] = tprev;
                    pacc[8 + i - 1] *= tprev;
                    asm volatile("" : "+v"(pacc[8 + i - 1]));
                }
                tprev = tcur;
                __builtin_amdgcn_sched_barrier(0);
            }
            sacc[15] = tprev;
            pacc[15] *= tprev;
        }
#pragma unroll
        for (int q = 4; q < 8; ++q) { pp[q] = pack2(sacc[2 * q], sacc[2 * q + 1]); dd[q] = pack2(pacc[2 * q], pacc[2 * q + 1]); }
        __builtin_amdgcn_sched_barrier(0);
        {   // last 16 rows of the block (mm = 1)
            const bf16x8 p8 = __builtin_bit_cast(bf16x8, u32x4{pp[4], pp[5], pp[6], pp[7]});
            const bf16x8 d8 = __builtin_bit_cast(bf16x8, u32x4{dd[4], dd[5], dd[6], dd[7]});
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                advance(24 + i);
                const bf16x8 A = ra[(24 + i) % RD];
                if (i & 1) dkacc[i >> 1] = mfma32(A, d8, dkacc[i >> 1]);
                else dvacc[i >> 1] = mfma32(A, p8, dvacc[i >> 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // two steps a turn: the buffer is a constant of the code, and the LDS addresses need no arithmetic per step
    for (int it = 0; it < n_steps; it += 2) {
        step(it, std::integral_constant<int, 0>{});
        if (it + 1 < n_steps) step(it + 1, std::integral_constant<int, 1>{});
    }
    };
    sweep(std::false_type{}, qt1, qt0);
    {   // the steps that can hold short rows: row tile 0 under a prompt of at least EDGE_LEN tokens, else all
        const int f_hi = Lp >= EDGE_LEN ? min(qt1, EDGE_LEN / BQ) : qt1;
        if (f_hi > qt0) {
            __syncthreads();                       // every wave has left the main sweep's last buffer
            sweep(std::true_type{}, f_hi, qt0);
        }
    }

    const int64_t orow = ((int64_t)(gd.tok_base + (valid ? s : 0)) * a.Hkv + kvh) * 128 + 4 * hh;
    if constexpr (NW == 4) {
        if (!valid) return;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const f32x16* acc = pass == 0 ? dkacc : dvacc;
            __bf16* out = pass == 0 ? a.dk : a.dv;
            const float mul = pass == 0 ? a.scale : 1.0f;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    bf16x4 x;
                    bf16x4 old = {0, 0, 0, 0};
                    if (a.accumulate) old = *reinterpret_cast<const bf16x4*>(out + orow + 32 * db + 8 * gq);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = (__bf16)(acc[db][4 * gq + e] * mul + (float)old[e]);
                    *reinterpret_cast<bf16x4*>(out + orow + 32 * db + 8 * gq) = x;
                }
        }
        return;
    }
    wait_vm0();                                // the K and V copies of a workgroup without steps
    // add the two row halves: waves 4..7 park their partial sums in LDS (the Q/dO buffers,
    // 16 KB per wave), waves 0..3 add them and write the result.  dK first, then dV.
    float* xch = reinterpret_cast<float*>(&dkdv_lds[0][0]) + (size_t)kb * 4096 + l * 4;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        f32x16* acc = pass == 0 ? dkacc : dvacc;
        __bf16* out = pass == 0 ? a.dk : a.dv;
        const float mul = pass == 0 ? a.scale : 1.0f;
        __syncthreads();
        if (qh == 1) {
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    f32x4 x = {acc[db][4 * gq], acc[db][4 * gq + 1], acc[db][4 * gq + 2], acc[db][4 * gq + 3]};
                    *reinterpret_cast<f32x4*>(xch + (db * 4 + gq) * 256) = x;
                }
        }
        __syncthreads();
        if (qh == 0 && valid) {
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const f32x4 y = *reinterpret_cast<const f32x4*>(xch + (db * 4 + gq) * 256);
                    if (PIECES && parts > 1) {
                        const f32x4 z = {acc[db][4 * gq] + y[0], acc[db][4 * gq + 1] + y[1], acc[db][4 * gq + 2] + y[2],
                                         acc[db][4 * gq + 3] + y[3]};
                        *reinterpret_cast<f32x4*>(sums + (pass * 128 + 32 * kb + c) * 128 + 4 * hh + 32 * db + 8 * gq) = z;
                        continue;
                    }
                    if (!PIECES && a.head_split) {      // fp32 partial sum of this q head; scaled and rounded by the reduce kernel
                        float* sums = (part == 0 ? a.partial : a.partial2) + ((int64_t)pass * rep_all + hr_only) * T_total * a.Hkv * 128;
                        const f32x4 z = {acc[db][4 * gq] + y[0], acc[db][4 * gq + 1] + y[1], acc[db][4 * gq + 2] + y[2],
                                         acc[db][4 * gq + 3] + y[3]};
                        *reinterpret_cast<f32x4*>(sums + orow + 32 * db + 8 * gq) = z;
                        continue;
                    }
                    bf16x4 x;
                    bf16x4 old = {0, 0, 0, 0};
                    if (a.accumulate) old = *reinterpret_cast<const bf16x4*>(out + orow + 32 * db + 8 * gq);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = (__bf16)((acc[db][4 * gq + e] + y[e]) * mul + (float)old[e]);
                    *reinterpret_cast<bf16x4*>(out + orow + 32 * db + 8 * gq) = x;
                }
        }
    }
}

template <int NW, bool SMALL, bool PIECES>
__global__ __launch_bounds__(64 * NW, 2) void bwd_dkdv_kernel(TabArg table, BwdArgs a) {
    if (SMALL && blockIdx.x == 0 && threadIdx.x < 64 && a.small.tag_mode != TAG_KEEP)       // (the dq pass is through)
        reserve_tag_body(a.small.tag, a.small.want, a.small.tag_mode, threadIdx.x);
    Item item;           // per (key tile, q head) where the pass is split over the q heads, else per (key tile, kv head)
    if (!decode_item(blockIdx.x, a.items, item)) return;
    TileDesc td;
    SmallGroup sg;
    unsigned piece = (unsigned)item.tile;
    if constexpr (PIECES) piece = (unsigned)table_of(table)[a.pieces_at + item.tile];
    const int tile = PIECES ? (int)(piece & 0xffff) : item.tile;
    if constexpr (SMALL) {
        int ti;
        sg = small_tile<128>(table_of(table), a.n_groups, tile, threadIdx.x & 63, ti);
        td = TileDesc{0, ti, sg.tok_base, sg.Lp, sg.Tg, 0, 0, 0};
    } else {
        td = a.sched.key_tiles[tile];
    }
    if constexpr (PIECES) {
        dkdv_body<NW, SMALL, true>(a, sg, td, item.kvh, 0, (int)(piece >> 16 & 0xff), (int)(piece >> 24),
                                   a.piece_sums + ((int64_t)item.kvh * a.n_slots + item.tile) * (int64_t)(PIECE_SLOT_BYTES / 4));
        return;
    }
    const int two = NW == 8 && a.head_split == 2 ? 1 : 0;          // (q head, row part)
    dkdv_body<NW, SMALL, false>(a, sg, td, item.kvh, item.hr >> two, item.hr & two, 1, nullptr);
}

// Second stage of the head-split dkdv pass: dk = scale * sum_hr partial[0][hr], dv = sum_hr
// partial[1][hr], summed in a fixed order (bitwise repeatable), rounded once, optionally added
// to what the outputs hold.  One thread per 4 consecutive elements.
__global__ __launch_bounds__(256) void dkdv_reduce_kernel(const float* __restrict__ partial, __bf16* __restrict__ dk,
                                                          __bf16* __restrict__ dv, int64_t n4, int rep, float scale,
                                                          int accumulate) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const int64_t plane = n4 * 4;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int hr = 0; hr < rep; ++hr) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(partial + ((int64_t)pass * rep + hr) * plane + 4 * i);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += x[e];
        }
        __bf16* out = (pass == 0 ? dk : dv) + 4 * i;
        const float mul = pass == 0 ? scale : 1.0f;
        bf16x4 old = {0, 0, 0, 0};
        if (accumulate) old = *reinterpret_cast<const bf16x4*>(out);
        bf16x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (__bf16)(acc[e] * mul + (float)old[e]);
        *reinterpret_cast<bf16x4*>(out) = r;
    }
}

// The same where key tiles may have two row parts: over the parts of the key's tile and the q heads.  Looking the tile up costs
// 1.7 us, so a pass without row parts takes the kernel above.  A workgroup takes RK keys of a tile and one kv head, a thread 4 consecutive elements.
constexpr int RK = 8;
template <bool SMALL>
__global__ __launch_bounds__(256) void dkdv_reduce_parts_kernel(TabArg table, BwdArgs a) {
    const int part = blockIdx.x & (128 / RK - 1);
    unsigned kvh;
    const int tile = (int)divmod(blockIdx.x / (128 / RK), a.kv_heads, kvh);
    SmallGroup sg;
    TileDesc td;
    int row_end;
    if constexpr (SMALL) {
        int ti, b1, e1;
        sg = small_tile<128>(table_of(table), a.n_groups, tile, threadIdx.x & 63, ti);
        td = TileDesc{0, ti, sg.tok_base, sg.Lp, sg.Tg, 0, 0, 0};
        small_segment(sg, min(128 * ti + 128, td.Tg) - 1, b1, e1);
        row_end = 128 * ti < td.Lp ? td.Tg : e1;
    } else {
        td = a.sched.key_tiles[tile];
        row_end = 128 * td.ti < td.Lp ? td.Tg : a.sched.row_hi[td.tok_base + min(128 * td.ti + 128, td.Tg) - 1];
    }
    row_end = __builtin_amdgcn_readfirstlane(row_end);
    const int s0 = 128 * td.ti;
    const int row_lo = a.resp_only ? td.Lp : 0;
    const int parts = row_parts(a, row_end > row_lo ? (row_end + 63) / 64 - max(s0, row_lo) / 64 : 0);
    const int s = s0 + RK * part + (threadIdx.x >> 5);
    if (s >= td.Tg) return;
    const int64_t plane = a.T_total * a.Hkv * 128, i = ((int64_t)(td.tok_base + s) * a.Hkv + kvh) * 128 + 4 * (threadIdx.x & 31);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int n = 0; n < parts; ++n) {
            const float* const sums = (n == 0 ? a.partial : a.partial2) + (int64_t)pass * a.rep * plane + i;
            for (int hr = 0; hr < a.rep; ++hr) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(sums + hr * plane);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += x[e];
            }
        }
        __bf16* out = (pass == 0 ? a.dk : a.dv) + i;
        const float mul = pass == 0 ? a.scale : 1.0f;
        bf16x4 old = {0, 0, 0, 0};
        if (a.accumulate) old = *reinterpret_cast<const bf16x4*>(out);
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (__bf16)(acc[e] * mul + (float)old[e]);
        *reinterpret_cast<bf16x4*>(out) = y;
    }
}

// The same for key tiles in pieces: a workgroup adds up PK keys of a tile with several parts and one kv head, a thread 4
// consecutive elements of dK and of dV, parts in order.
struct PieceSums { uint32_t w[2 * PIECE_SLOTS]; };
constexpr int PK = 8;
__global__ __launch_bounds__(256) void dkdv_pieces_kernel(PieceSums tiles, BwdArgs a) {
    unsigned kvh;
    const unsigned n = divmod(blockIdx.x / (128 / PK), a.kv_heads, kvh);
    const uint32_t w = tiles.w[2 * n];
    const int first = (int)(w & 0xffff), parts = (int)(w >> 16 & 0xff), keys = (int)(w >> 24) + 1;
    const int key = PK * (int)(blockIdx.x & (128 / PK - 1)) + (int)(threadIdx.x >> 5);
    if (key >= keys) return;
    const float* const sums = a.piece_sums + ((int64_t)kvh * a.n_slots + first) * (int64_t)(PIECE_SLOT_BYTES / 4) + 128 * key + 4 * (threadIdx.x & 31);
    const int64_t i = (((int64_t)tiles.w[2 * n + 1] + key) * a.Hkv + kvh) * 128 + 4 * (threadIdx.x & 31);
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 4
    for (int p = 0; p < parts; ++p)
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(sums + (int64_t)p * (int64_t)(PIECE_SLOT_BYTES / 4) + pass * 128 * 128);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[pass][e] += x[e];
        }
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        __bf16* const out = (pass == 0 ? a.dk : a.dv) + i;
        const float mul = pass == 0 ? a.scale : 1.0f;
        bf16x4 old = {0, 0, 0, 0};
        if (a.accumulate) old = *reinterpret_cast<const bf16x4*>(out);
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (__bf16)(acc[pass][e] * mul + (float)old[e]);
        *reinterpret_cast<bf16x4*>(out) = y;
    }
}

}  // namespace

// Eight waves walk a key tile 1.2 times as fast as four that have the CU to themselves, but two workgroups of four
// share a CU at 0.7 of that speed each.  Which shape ends first depends on how the tiles fall onto the CUs: workgroups go
// round the XCDs and within an XCD round its four shader engines, in order, and a group's first tiles are its longest.
// The launch is therefore played through on the host, for one XCD (the others get the same mixture), with the times that
// the two shapes take on an idle chip, us per row tile and q head.
// Measured on 439 packings of 96 to 2600 workgroups (both shapes; one to 40 groups, 4/4 to 40/8 heads): the shape taken is
// 0.3 % from the faster one on average (0.4 % on 138 more, drawn afterwards); four waves throughout 10 %, eight waves 2.9 %, a line by the number of
// workgroups alone up to 24 % (a group of 9152 tokens, 28/4 heads, 288 workgroups: 1592 us with four waves, 1281 with
// eight; nine groups of 1000, as many workgroups: 292 and 323).  What is played is the packing's order; the launch itself
// starts prompt tiles first (key_order()), which gains more than the choice of a shape: there, on 75 packings of more than 256
// workgroups, the shape taken is 1.8 % from the faster one on average, four waves throughout 7.8 %, eight 7.2 %.
int dkdv_waves(const Problem& p) {
    constexpr int SE = 4, CUS = 8;                             // of an XCD
    const int n_wgs = count_tiles(p, 128) * p.Hkv;
    if (n_wgs <= 8 * SE * CUS) return 8;                       // no CU gets a second workgroup
    const bool many = n_wgs > 2048;
    const int rep = p.Hq / p.Hkv;
    std::vector<float> w8, w4;                                 // time of each key tile's workgroup
    double sum = 0.;
    float longest = 0.f;
    for (int g = 0; g < p.n_groups; ++g) {
        const int32_t* e = p.host_table + TAB_HEADER + TAB_GROUP_WORDS * g;
        const int Lp = e[1], Tg = e[2];
        const int32_t* roff = p.host_table + e[3];
        for (int s0 = 0, j = 0; s0 < Tg; s0 += 128) {
            const int last = (s0 + 128 < Tg ? s0 + 128 : Tg) - 1, from = p.resp_only && Lp > s0 ? Lp : s0;
            int to = Tg;                                       // one past the last row that sees a key of the tile
            if (s0 >= Lp) { while (roff[j + 1] <= last) ++j; to = roff[j + 1]; }
            const int n32 = to > from ? (to + 31) / 32 - from / 32 : 0, n64 = to > from ? (to + 63) / 64 - from / 64 : 0;
            const float t4 = 5.f + 0.77f * (float)(n32 * rep);
            sum += t4;
            longest = std::max(longest, t4);
            if (many) continue;
            w8.push_back(6.f + 1.24f * (float)(n64 * rep));
            w4.push_back(t4);
        }
    }
    // many workgroups: even, unless one is longer than what a CU gets in all
    if (many) return sum * p.Hkv < 256. * longest ? 8 : 4;
    std::vector<int> tiles;                                    // of XCD 0, in order
    const ItemMap items = make_item_map((int)w8.size(), p.Hkv, p.Hkv);
    for (int bid = 0, grid = grid_for_items((int)w8.size(), p.Hkv, p.Hkv); bid < grid; bid += 8) {
        Item it;
        if (decode_item(bid, items, it)) tiles.push_back(it.tile);
    }
    float end8 = 0.f, end4 = 0.f;
    for (int se = 0; se < SE; ++se) {
        float busy[CUS] = {};
        for (size_t i = se; i < tiles.size(); i += SE) {
            float* cu = std::min_element(busy, busy + CUS);
            *cu += w8[tiles[i]];
            end8 = std::max(end8, *cu);
        }
        float left[CUS][2] = {}, now = 0.f;                    // work left of the residents of each CU
        for (size_t i = se;;) {
            for (int fill = 0; fill < 2; ++fill)               // an empty CU first
                for (int c = 0; c < CUS && i < tiles.size(); ++c) {
                    if (left[c][0] > 0.f && left[c][1] > 0.f) continue;
                    if (fill == 0 && (left[c][0] > 0.f || left[c][1] > 0.f)) continue;
                    left[c][left[c][0] > 0.f] = w4[tiles[i]];
                    i += SE;
                }
            float dt = 1e30f;
            auto speed = [&](int c) { return left[c][0] > 0.f && left[c][1] > 0.f ? 0.7f : 1.f; };
            for (int c = 0; c < CUS; ++c)
                for (int k = 0; k < 2; ++k)
                    if (left[c][k] > 0.f) dt = std::min(dt, left[c][k] / speed(c));
            if (dt == 1e30f) break;
            now += dt;
            for (int c = 0; c < CUS; ++c) {
                const float done = dt * speed(c) * 1.0001f + 1e-3f;        // the one that sets dt ends in any rounding
                for (int k = 0; k < 2; ++k) left[c][k] = left[c][k] > done ? left[c][k] - done : 0.f;
            }
        }
        end4 = std::max(end4, now);
    }
    return end4 < end8 ? 4 : 8;
}

// Key tiles in pieces.  The pass ends with its longest workgroup, and a prompt's first key tile is seen by every row of its group: few
// groups, and short prompts above all, left most CUs waiting for it.  Tiles longer than some length are therefore cut into equal parts
// (of their row tiles and q heads), and that length is the one at which a launch of pieces, longest first, each to the CU that is
// free first, is through soonest.  Whole tiles (or, where the pass is split over the q heads, those) are played in the same way; they stay
// where pieces do not gain a tenth on them (four waves to a workgroup walk whole tiles faster than is played here), and are
// not played at all where the longest is within a quarter of an even share.  Backward passes, us, before -> after (prompt x answers, q / kv heads): 2 x (60 + 26 x 85), 32/8 (two sweeps,
// as prompts are short) 436 -> 132; 100 + 10 x 400, 4/2 117 -> 52; 2 x (560 + 27 x 840), 28/4 4757 -> 2552; 35 + 22 x 470,
// 32/8 2121 -> 516; 1024 + 8 x 256, 28/4 182 -> 170 (sums of prompt tiles only); 650 + 4 x (9 x 84), 32/8 258 -> 234; on 52 drawn
// packings of 1e8 to 2e11 operations 1.17 times as fast on average, on 18 larger ones 1.20, at worst 0.98.
namespace {
// When workgroups of `lens` steps, `copies` of each, longest first, are through: each goes to the place that is free first.
// That place's time never falls, so places are counted by the time at which they are free, and one look over the times serves all workgroups
// (and lengths are sorted by counting).  The longest plan of 3000 drawn packings, on the host, a sort and a heap -> counts: 1150 -> 180 us.
struct Play {
    std::vector<int> of_len, at;                     // kept from one play to the next
    int operator()(const std::vector<int>& lens, int places, int copies, double* half = nullptr) {
        int longest = 0;
        int64_t all = 0;
        for (int n : lens) { longest = std::max(longest, n); all += n; }
        of_len.assign((size_t)longest + 1, 0);
        at.assign((size_t)(all * copies / places + longest + 1), 0);      // (a workgroup starts at the mean or before)
        for (int n : lens) of_len[(size_t)n] += copies;
        at[0] = places;
        int first = 0, end = 0;
        for (int n = longest; n >= 0; --n)
            for (int left = of_len[(size_t)n]; left > 0;) {
                while (at[(size_t)first] == 0) ++first;
                const int now = std::min(left, at[(size_t)first]);
                at[(size_t)first] -= now;
                at[(size_t)(first + n)] += now;
                end = std::max(end, first + n);
                left -= now;
            }
        if (half) {
            int t = 0;
            for (int before = at[0]; before <= places / 2; before += at[(size_t)t]) ++t;
            *half = t;
        }
        return end;
    }
};
// CUs over which the workgroups of a kv head go, and kv heads that share them (ItemMap)
void cus_of(const Problem& p, int& cus, int& copies) {
    const bool by_xcd = p.Hkv % 8 == 0 || 8 % p.Hkv == 0;
    cus = !by_xcd ? 256 : p.Hkv % 8 == 0 ? 32 : 32 * (8 / p.Hkv);
    copies = !by_xcd ? p.Hkv : p.Hkv % 8 == 0 ? p.Hkv / 8 : 1;
}
}  // namespace

KeyPieces plan_key_pieces(const Problem& p, int slots, size_t max_words, int cost) {
    // steps' worth of time: of a workgroup without steps, of storing partial sums, of the launch that adds them up
    constexpr int FIXED = 5, STORE = 2, SUM_STEPS = 3;
    KeyPieces out;
    const int rep = p.Hq / p.Hkv;
    struct Tile { int steps, id, tok, keys; };
    std::vector<Tile> tiles;
    tiles.reserve((size_t)p.n_tiles128);
    int longest = 0;
    int64_t all = 0;
    for (int g = 0; g < p.n_groups; ++g) {
        const int32_t* e = p.host_table + TAB_HEADER + TAB_GROUP_WORDS * g;
        const int Lp = e[1], Tg = e[2];
        const int32_t* roff = p.host_table + e[3];
        for (int s0 = 0, j = 0; s0 < Tg; s0 += 128) {
            const int s1 = std::min(s0 + 128, Tg), from = p.resp_only && Lp > s0 ? Lp : s0;
            int to = Tg;
            if (s0 >= Lp) { while (roff[j + 1] < s1) ++j; to = roff[j + 1]; }
            const int q0 = from / 64, q1 = to > (p.resp_only ? Lp : 0) ? (to + 63) / 64 : q0;
            const int lo = std::max((Lp >= EDGE_LEN ? std::min(q1, 1) : q1) - q0, 0);
            const int steps = rep * (std::max(q1 - q0, 0) + lo);
            tiles.push_back(Tile{steps, (int)tiles.size(), e[0] + s0, s1 - s0});
            longest = std::max(longest, steps);
            all += steps + FIXED;
        }
    }
    int bins, copies;
    cus_of(p, bins, copies);
    const double even = (double)copies * (double)all / bins;
    if (longest + FIXED <= 1.25 * even) return out;
    // A launch is played in units of one step, of more where the longest tile (many q heads per kv head) has more than MOST: the plan of 40 + 130 x 600
    // tokens, 128 / 1 heads, took 2.1 ms on the host, 64 / 1 0.7
    constexpr int MOST = 2048;
    const int unit = std::max((longest + MOST - 1) / MOST, 1);
    Play play;
    auto through = [&](const std::vector<int>& lens) { return unit * play(lens, bins, copies); };
    auto parts_of = [&](int steps, int len) { return steps <= len ? 1 : std::min((steps + len - 1) / len, 255); };
    std::vector<int> lens;
    lens.reserve(tiles.size() + (size_t)slots);
    auto cut = [&](int max_len, int each) {                    // (each: a tile's workgroups of equal share, whatever its length)
        lens.clear();
        int64_t n_slots = 0;
        for (const Tile& t : tiles) {
            const int parts = max_len ? parts_of(t.steps, max_len) : each * (each > 1 && t.steps / rep >= PART_STEPS ? p.dkdv_parts : 1);
            if (parts > 1) n_slots += parts;
            if (max_len && lens.size() + parts > max_words) out.no_room = true;
            if (max_len && (n_slots > slots || out.no_room)) return false;
            const int len = (t.steps + parts - 1) / parts + (parts > 1 ? STORE : 0) + FIXED;
            lens.insert(lens.end(), (size_t)parts, unit == 1 ? len : (len + unit - 1) / unit);
        }
        return max_len == 0 || n_slots > 0;
    };
    // whole tiles, or one workgroup per q head and row part, then pieces of falling length
    cut(0, p.dkdv_partial ? rep : 1);
    int best = through(lens) - (p.dkdv_partial ? 0 : SUM_STEPS), len = 0;
    if (!p.dkdv_partial) best = best * 9 / 10;
    best -= cost;
    if (best <= std::max<double>(2 + STORE + FIXED, even)) return out;      // no pieces can be through sooner
    for (int l = longest * 3 / 4; l >= 3; l = std::min(l * 7 / 8, l - 1)) {
        if (!cut(l, 1)) break;
        const int end = through(lens);
        if (end < best) { best = end - best / 50; len = l; }
        if (l + FIXED < 0.5 * even) break;
    }
    if (len == 0) return out;
    std::sort(tiles.begin(), tiles.end(), [&](const Tile& a, const Tile& b) {
        const int pa = parts_of(a.steps, len), pb = parts_of(b.steps, len);
        if ((pa > 1) != (pb > 1)) return pa > 1;
        const int64_t x = (int64_t)a.steps * pb, y = (int64_t)b.steps * pa;
        return x != y ? x > y : a.id < b.id;
    });
    for (const Tile& t : tiles) {
        const int parts = parts_of(t.steps, len);
        if (parts > 1) {
            out.sums.push_back((uint32_t)out.words.size() | (uint32_t)parts << 16 | (uint32_t)(t.keys - 1) << 24);
            out.sums.push_back((uint32_t)t.tok);
            out.n_slots += parts;
        }
        for (int i = 0; i < parts; ++i) out.words.push_back((uint32_t)t.id | (uint32_t)i << 16 | (uint32_t)parts << 24);
    }
    return out;
}

// Key loops of the dq pass, and of a forward of response rows, in parts, planned in the same way for four-wave workgroups, two to a CU.  Few rows under
// long prompts leave CUs without a workgroup, or a last round of workgroups that are half as many as the places.  Either all workgroups
// longer than some length are cut into equal parts, or only those that no full round takes, whichever is through sooner; neither unless it
// gains a twentieth and the launch that brings the sums together, which up to LEAST steps cannot be.  Forward and dq pass, us, whole -> in parts
// (prompt x answers, response rows only, q / kv heads): 3 x (10500 + 17 x 40), 4/2 259 -> 66 and 310 -> 77; 2 x (2260 + 58), 28/4
// 51 -> 26; 8192 + 16 x 160, 40/8 (760 workgroups in 512 places) 439 -> 400 and 568 -> 553; on 66 drawn packings forward and backward
// 1.06 times as fast on average (forwards of all rows in parts too, which made o depend on the entry point).  Two waves of one workgroup to an item, without a second launch, walked in step and took 13 to 30 % longer.
RowPieces plan_row_pieces(const Problem& p, size_t slots, size_t max_words) {
    // steps' worth of time: of a workgroup without steps, of storing sums, of the launch that brings them together
    constexpr int FIXED = 4, STORE = 1, SUM_STEPS = 8, LEAST = 16;       // (up to LEAST steps there is nothing to gain)
    RowPieces out;
    const int rep = p.Hq / p.Hkv;
    int places, copies;
    cus_of(p, places, copies);
    places *= 2;
    if (p.n_tiles128 > ROW_PIECE_TILES || rep > 64 || (size_t)p.n_tiles128 * rep > max_words) return out;
    struct Wg { int steps, word, tok, i; };
    std::vector<Wg> wgs;
    wgs.reserve((size_t)p.n_tiles128 * rep);
    int longest = 0, tile = 0;
    int64_t all = 0;
    for (int g = 0; g < p.n_groups; ++g) {
        const int32_t* e = p.host_table + TAB_HEADER + TAB_GROUP_WORDS * g;
        const int Lp = e[1], Tg = e[2];
        const int32_t* roff = p.host_table + e[3];
        const int n = (Tg + 127) / 128;
        for (int ti = 0; ti < n; ++ti, ++tile) {
            const int base = (n - 1 - ti) * 128;               // as wave_rows()
            for (int hr = 0; hr < rep; ++hr) {
                const int i = rep - 1 - hr, t0 = base + 32 * (4 * i / rep), t1 = std::min(base + 32 * ((4 * i + 3) / rep) + 32, Tg);
                if (t0 >= Tg || (p.resp_only && t1 <= Lp)) continue;
                const int n1 = (std::min(Lp, t1) + 63) / 64;
                int steps = n1;
                if (t1 > Lp) {
                    const int32_t* const after = std::upper_bound(roff, roff + e[4], std::max(t0, Lp));      // behind the row's segment start
                    steps += std::max(t1 - std::max(n1 * 64, (int)after[-1]) + 63, 0) / 64;
                }
                wgs.push_back(Wg{steps, tile | hr << 10, e[0] + base, i});
                longest = std::max(longest, steps);
                all += steps + FIXED;
            }
        }
    }
    const double even = (double)copies * (double)all / places;
    if (8 * longest < even || longest <= LEAST) return out;
    std::sort(wgs.begin(), wgs.end(), [](const Wg& a, const Wg& b) { return a.steps != b.steps ? a.steps > b.steps : a.word < b.word; });
    // the `whole` longest stay whole, others longer than `len` are cut
    auto parts_of = [&](size_t n, int whole, int len) {
        const int steps = wgs[n].steps;
        return (int)n < whole || steps <= len ? 1 : std::min((steps + len - 1) / len, 255);
    };
    Play play;
    std::vector<int> lens;
    lens.reserve(max_words);
    auto end_of = [&](int whole, int len) {
        lens.clear();
        size_t n_slots = 0, n_sums = 0;
        for (size_t n = 0; n < wgs.size(); ++n) {
            const int parts = parts_of(n, whole, len);
            if (parts > 1) { n_slots += parts; ++n_sums; }
            if (n_slots > slots || n_sums > (size_t)ROW_SUMS || lens.size() + parts > max_words) return 1e30;
            lens.insert(lens.end(), (size_t)parts, (wgs[n].steps + parts - 1) / parts + (parts > 1 ? STORE : 0) + FIXED);
        }
        double half;               // when half of the places are empty: from then on workgroups are alone on their CUs, 1.44 times as fast
        const double end = play(lens, places, copies, &half);
        return half + 0.69 * (end - half) + (n_slots ? SUM_STEPS : 0);
    };
    const int n_wgs = (int)wgs.size(), rounds = n_wgs - n_wgs % std::max(places / copies, 1);
    double best = 0.95 * end_of(n_wgs, longest);
    int whole = 0, len = 0;
    for (const int w : {0, rounds}) {
        if (w == n_wgs || (w == 0 && rounds == 0 && whole)) continue;
        for (const int q : {2, 3, 4, 6, 8, 12, 16}) {
            const int l = (wgs[w].steps + q - 1) / q;
            if (l < 3) break;
            const double end = end_of(w, l);
            if (end < best) { best = 0.98 * end; whole = w; len = l; }
        }
        if (rounds == 0) break;
    }
    if (len == 0) return out;
    // longest first, pieces next to one another
    const int cut = (wgs[whole].steps + parts_of(whole, whole, len) - 1) / parts_of(whole, whole, len);
    auto put = [&](auto which) {
        for (size_t n = 0; n < wgs.size(); ++n) {
            const int parts = parts_of(n, whole, len);
            if (which(parts, wgs[n].steps))
                for (int i = 0; i < parts; ++i) out.words.push_back((uint32_t)wgs[n].word | (uint32_t)i << 16 | (uint32_t)parts << 24);
        }
    };
    put([&](int parts, int steps) { return parts == 1 && steps >= cut; });
    out.first_slot = (int)out.words.size();
    put([](int parts, int) { return parts > 1; });
    put([&](int parts, int steps) { return parts == 1 && steps < cut; });
    for (size_t n = 0; n < wgs.size(); ++n) {
        const int parts = parts_of(n, whole, len);
        if (parts == 1) continue;
        out.sums.push_back((uint32_t)out.n_slots | (uint32_t)parts << 16);
        out.sums.push_back((uint32_t)wgs[n].tok);
        out.sums.push_back((uint32_t)wgs[n].i);
        out.n_slots += parts;
    }
    return out;
}

hipError_t launch_bwd_bf16(const Problem& p, hipStream_t s) {
    hipError_t e = hipSuccess;
    // A call that runs both the rowsum and the dq stage folds the first into the second (the dq pass has
    // the dO rows in registers anyway): one pass over o and dO less (in response-rows mode, where the separate pass read the prompt rows too: 2560 rows under an 8K prompt, forward and backward 1707 -> 1632 us).  Not
    // for head counts that the layout of rowsum_bf16_kernel (whose arithmetic the fold repeats) does not take.
    const bool fused = (p.stages & STAGE_ROWSUM) && (p.stages & STAGE_DQ) && rowsum_fast_path(p);
    if ((p.stages & STAGE_ROWSUM) && !fused) {
        e = launch_rowsum(p, false, s);
        if (e != hipSuccess) return e;
    }
    BwdArgs a{};
    a.fused_rowsum = fused; a.o = (const __bf16*)p.o; a.o_lo = (const __bf16*)p.o_lo; a.lo_flag = p.o_lo_flag;
    a.q = (const __bf16*)p.q; a.k = (const __bf16*)p.k; a.v = (const __bf16*)p.v; a.d_o = (const __bf16*)p.d_o;
    a.lse = p.lse; a.nD = p.Dbuf; a.L2 = p.Dbuf + (int64_t)p.Hq * p.total_tokens;
    a.dq = (__bf16*)p.dq; a.dk = (__bf16*)p.dk; a.dv = (__bf16*)p.dv;
    a.small = p.small; a.T_total = p.total_tokens; a.sched = p.sched; a.n_groups = p.n_groups; a.Hq = p.Hq; a.Hkv = p.Hkv; a.scale = p.scale; a.c = p.scale * LOG2E;
    a.resp_only = p.resp_only; a.accumulate = p.accumulate;
    const TabArg table = small_table(p);
    if (p.stages & STAGE_DQ) {
        // short key loops: the four-wave shape, two workgroups per CU (the forward's rule, see bwd_dq_kernel)
        const RowPieces* const pieces = p.row_pieces;
        const bool small = pieces || use_small_shape(p);
        const int n_tiles = pieces ? (int)pieces->words.size() : count_tiles(p, small ? 128 : 256), per_kv = pieces ? p.Hkv : p.Hq;
        const int grid = grid_for_items(n_tiles, per_kv, p.Hkv);
        a.items = make_item_map(n_tiles, per_kv, p.Hkv);
        if (pieces) a.rows = row_piece_args(p);
        const EdgeArgs edge = edge_args(p);
        const int shorts = (edge_blocks(edge, small ? 2 : 3) + 7) & ~7, total = grid + shorts;
        auto launch = [&](auto small_call) {
            constexpr bool S = decltype(small_call)::value;
            if (pieces) hipLaunchKernelGGL((bwd_dq_kernel<4, S, true>), dim3(total), dim3(256), 0, s, with_list(table, p, pieces->words), a, edge, shorts, grid);
            else if (small) hipLaunchKernelGGL((bwd_dq_kernel<4, S, false>), dim3(total), dim3(256), 0, s, table, a, edge, shorts, grid);
            else hipLaunchKernelGGL((bwd_dq_kernel<8, S, false>), dim3(total), dim3(512), 0, s, table, a, edge, shorts, grid);
        };
        if (p.small.on) launch(std::true_type{}); else launch(std::false_type{});
        if (pieces) hipLaunchKernelGGL(dq_pieces_kernel, dim3((unsigned)(pieces->sums.size() / 3 * p.Hkv * 4)), dim3(256), 0, s, row_sums(*pieces), a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (p.stages & STAGE_DKDV) {
        auto launch = [&](int waves, int grid) {
            auto go = [&](auto small_call) {
                constexpr bool S = decltype(small_call)::value;
                if (p.pieces) {
                    hipLaunchKernelGGL((bwd_dkdv_kernel<8, S, true>), dim3(grid), dim3(512), 0, s, with_list(table, p, p.pieces->words), a);
                } else if (waves == 8) hipLaunchKernelGGL((bwd_dkdv_kernel<8, S, false>), dim3(grid), dim3(512), 0, s, table, a);
                else hipLaunchKernelGGL((bwd_dkdv_kernel<4, S, false>), dim3(grid), dim3(256), 0, s, table, a);
            };
            if (p.small.on) go(std::true_type{}); else go(std::false_type{});
        };
        const int n_tiles = count_tiles(p, 128);
        a.rep = p.Hq / p.Hkv;
        a.rep_div = make_div(a.rep);
        a.kv_heads = make_div(p.Hkv);
        a.head_split = p.dkdv_partial && !p.pieces ? p.dkdv_parts : 0;
        a.partial = p.dkdv_partial; a.partial2 = p.dkdv_partial2;
        if (p.pieces) {
            const int n = (int)p.pieces->words.size();
            a.pieces_at = p.small.on ? p.host_table[2] : 0;
            a.n_slots = p.pieces->n_slots;
            a.piece_sums = p.piece_sums;
            a.items = make_item_map(n, p.Hkv, p.Hkv);
            launch(8, grid_for_items(n, p.Hkv, p.Hkv));
            PieceSums sums{};
            std::copy(p.pieces->sums.begin(), p.pieces->sums.end(), sums.w);
            hipLaunchKernelGGL(dkdv_pieces_kernel, dim3((unsigned)(p.pieces->sums.size() / 2 * p.Hkv * (128 / PK))), dim3(256), 0, s, sums, a);
        } else if (a.head_split) {
            const int items = p.Hq * p.dkdv_parts;
            a.items = make_item_map(n_tiles, items, p.Hkv);
            launch(8, grid_for_items(n_tiles, items, p.Hkv));
            const int64_t n4 = p.total_tokens * p.Hkv * 32;
            const dim3 rg((unsigned)(n_tiles * p.Hkv * (128 / RK)));
            if (p.dkdv_parts == 1)
                hipLaunchKernelGGL(dkdv_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, a.partial, a.dk, a.dv,
                                   n4, p.Hq / p.Hkv, p.scale, a.accumulate);
            else if (p.small.on) hipLaunchKernelGGL(dkdv_reduce_parts_kernel<true>, rg, dim3(256), 0, s, table, a);
            else hipLaunchKernelGGL(dkdv_reduce_parts_kernel<false>, rg, dim3(256), 0, s, table, a);
        } else {
            const int grid = grid_for_items(n_tiles, p.Hkv, p.Hkv);
            a.items = make_item_map(n_tiles, p.Hkv, p.Hkv);
            launch(dkdv_waves(p), grid);
        }
        e = hipGetLastError();
    }
    return e;
}

}  // namespace sp
