// Forward shared-prompt attention, bf16 MFMA path (gfx950).
//
// One workgroup owns eight (or four) items of one group and one kv head, an item being 32 consecutive
// packed query rows of one of the q heads that read this kv head; a wave owns one item (wave_rows() in
// sp_common.hpp).  Keys/values stream through LDS in tiles of 64 keys.  Per tile a wave computes S^T = K Q^T (keys x queries) so that every lane
// holds scores of ONE query (column) and the online softmax needs a single
// cross-lane exchange, then O^T += V^T P^T with V read transposed from LDS.
//
// The mask of Section 4.3 (modification 3) is never materialised: with
// st(t) = first token of t's own segment (0 on the prompt),
//     allowed(t, s) = (s <= t) && (s < Lp || s >= st(t)).
// The key loop visits [0, min(Lp, t1)) and, for tiles holding response rows,
// [st(first response row), t1); everything else is wholly masked and skipped
// (the three terms of the section's complexity split).  Tiles that lie entirely in
// the allowed region skip the mask arithmetic.
#include "sp_common.hpp"
#include "sp_launch.hpp"
#include <type_traits>

namespace sp {
namespace {

constexpr int BN = 64;                 // keys per LDS tile
constexpr float P_LIMIT = 16384.0f;     // bound on a lane's per-tile sum of exponentials (2^14)
constexpr int TILE_BYTES = BN * 256;   // 64 rows x 128 bf16

struct FwdArgs {
    // one entry per tensor set; the sets share the packing, the schedule and the launch
    const __bf16* q[MAX_SETS]; const __bf16* k[MAX_SETS]; const __bf16* v[MAX_SETS];
    __bf16* o[MAX_SETS]; float* lse[MAX_SETS];
    int blocks_per_set;
    Schedule sched; // tile descriptors and per-token segment bounds, written by the schedule kernel of the call
    ItemMap items;
    int n_groups, T_total, Hq, Hkv;
    float c;        // softmax_scale * log2(e)
    float m_none;   // reference point of a row that has not seen a key yet: finite, as is its product with c, -1e30 where float32 holds that
    int naive;
    int resp_only;  // compute and write response rows only
    SmallCall small;
    RowPieceArgs pieces;
    __bf16* o_lo;   // optional (single-set launches): o_fp32 - bf16(o), rounded to bf16, same layout as o
};

static_assert(sizeof(TabArg) + sizeof(FwdArgs) <= 4096 && sizeof(RowSums) + sizeof(FwdArgs) <= 4096, "kernel arguments");

// ------------------------------------------------------------------------------------
// Hand-scheduled software-pipelined forward.  Step j of a wave holds the MFMAs of two tiles and
// the vector-ALU work of a third:
//   O^T += V(j-1)^T P(j-1)^T  (16 MFMAs),  S(j+1) = K(j+1) Q^T  (16 MFMAs),
//   P(j) = exp2(S(j) c - m c), its row sums and its bf16 packing  (32 scores per lane).
// The step is written as 32 slices of {LDS operand read for the MFMA two slices ahead, one
// MFMA, the vector work of one score}, fenced so the compiler keeps that order: while MFMAs
// stream, a SIMD takes about five other vector instructions per MFMA for free, which is what a
// slice holds.  So that the exponentials can be spread this evenly they are taken against the
// reference point m the row had before the tile (see `step`).  Two steps run per workgroup
// barrier; the K and V tiles of the following two steps are copied into LDS meanwhile.
// ------------------------------------------------------------------------------------
//
// Two shapes of workgroup.  NW = 8: eight items, four K and four V buffers (128 KB of LDS), one workgroup
// per CU: the shape for long key loops.  NW = 4: four items, two K and two V buffers (64 KB), one step
// per barrier, TWO workgroups per CU: each workgroup's fixed costs (table lookups, first loads,
// epilogue, the gap before the next dispatch) then overlap with the other's key loop, which is what
// batches of short groups need, where a workgroup runs only a handful of steps.
// The loop holds no address arithmetic (operand addresses are whole sums in registers, buffers are constants) and no
// spills, the mask is a word of bits per lane, and the loop ends with the last barrier interval instead of the last turn of
// the buffer ring.  One box, before -> after, us: 64 groups of a short prompt and 16 answers 2674 -> 2349, 64 groups of
// 1000 tokens 874 -> 789, three sets of eight 2K prompts 7560 -> 7290, four long prompts 1922 -> 1886, one short group
// 17.9 -> 14.6, 16K prompt with 32 answers 4020 -> 3997.
// Short key loops are bound by instruction issue, not by memory (64 groups of a short prompt and 16 answers, one wave's life of
// 37 K cycles: lookups 4.7, first copies 3.4, 5.8 steps of 3.5, last product 1.8, stores 5.8; 2.9 TB/s).  The rows' own
// segments are therefore walked from their first key on, not from the multiple of 64 below it (a quarter of a step less),
// and what follows the loop takes its addresses from those of the loop or by one xor each (200 of 900 vector instructions
// outside the loop).  One box, before -> after, us: that packing 2410 -> 2308, 64 groups of 1000 tokens 805 -> 784, one short group
// 14.8 -> 14.0; three sets of eight 2K prompts and the 16K prompt within what runs differ.
// NAIVE = the measurement baseline (every tile at or below the packed diagonal, mask applied element by
// element): a separate instantiation, so that it shows under its own name in kernel traces and its
// branches cost the product kernel nothing.
// SMALL = a call whose kernels look everything up themselves (SmallCall); as a run-time branch it cost the others 0.5 to 1 %.
// PIECES = key loops in parts (RowPieces): a workgroup walks part of its key tiles and leaves unnormalised sums to fwd_pieces_kernel.
template <int NW, bool NAIVE, bool SMALL, bool PIECES>
__global__ __launch_bounds__(NW * 64, 2) void fwd_kernel(TabArg table, FwdArgs a) {      // two waves per SIMD in either shape
    constexpr int BM = 32 * NW;
    constexpr int NB = NW == 8 ? 4 : 2;            // K buffers = V buffers
    constexpr int RD = 3;      // LDS operand ring depth (prefetch distance RD - 1 MFMAs)
    __shared__ __attribute__((aligned(1024))) char ldsKb[NB][TILE_BYTES];      // K tile t lives in ldsKb[t % NB]
    __shared__ __attribute__((aligned(1024))) char ldsVb[NB][TILE_BYTES];      // V tile t in ldsVb[t % NB]

    // blocks are dealt set-major; blocks_per_set is a multiple of 8, so the block -> XCD mapping
    // of a set does not depend on how many sets the launch carries
    const int bid = blockIdx.x, bps = a.blocks_per_set, set = (bid >= bps) + (bid >= 2 * bps) + (bid >= 3 * bps);
    static_assert(MAX_SETS == 4, "sets are counted by comparisons");
    const __bf16* const aq = a.q[set]; const __bf16* const ak = a.k[set]; const __bf16* const av = a.v[set];
    __bf16* const ao = a.o[set]; float* const alse = a.lse[set];
    if (SMALL && bid == 0 && threadIdx.x < 64 && a.small.tag_mode != TAG_KEEP)
        reserve_tag_body(a.small.tag, a.small.want, a.small.tag_mode, threadIdx.x);
    Item item;
    if (!decode_item(bid - set * bps, a.items, item)) return;
    RowPiece piece{item.tile, item.hr, 0, 1, 0};
    if constexpr (PIECES) { piece = row_piece(table_of(table), a.pieces, item); item.hr = piece.hr; item.tile = piece.tile; }
    // the tile's descriptor: one 32-byte load instead of a bisection over the groups and the group's entry
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
    const WaveRows wr = wave_rows<NW>(td, item, PIECES ? a.pieces.rep : a.items.rep, w);
    const int head = wr.head;
    const int t0 = wr.t0, t1 = wr.t1;
    const int T_total = a.T_total;
    if (t0 >= Tg || (a.resp_only && t1 <= Lp)) return;      // past the group's end, or prompt rows only

    const int c = l & 31, hh = l >> 5, j16 = l & 15, c16 = (l >> 4) & 1;

    const int tw0 = wr.tw0;
    const int t = tw0 + c;
    const bool valid = t < Tg;
    const int tm = valid ? t : -1;
    const bool wave_valid = tw0 < Tg;
    const int tw1 = min(tw0 + 31, Tg - 1);
    // first own-segment key of this lane's row and of the workgroup's first response row (0 on the prompt)
    int st = 0, b2;
    if constexpr (SMALL) {
        const int first = max(t0, Lp);                     // as a lane's token, so that one search serves both
        int s1, e1;
        small_segment(sg, hh == 0 ? t : first, s1, e1);
        b2 = first < Tg ? __builtin_amdgcn_readlane(s1, 32) : 0;
        s1 = __shfl(s1, c, 64);
        st = valid && t >= Lp ? s1 : 0;
    } else {
        st = valid ? a.sched.key_lo[gd.tok_base + t] : 0;
        b2 = __builtin_amdgcn_readfirstlane(a.sched.key_lo[gd.tok_base + min(max(t0, Lp), Tg - 1)]);
    }
    // lanes 0..31 hold the wave's rows in order: the last valid row's start comes from its lane
    const int st_last = wave_valid ? __builtin_amdgcn_readlane(st, tw1 - tw0) : 0;

    bf16x8 qreg[8];
    {
        // rows past the end of the group read the group's last row instead: every score of such a
        // row is masked and nothing of it is stored, and without a select on the loaded value the
        // wait for these loads moves down to the first MFMA, behind the issue of the tile copies
        const __bf16* qp = aq + ((int64_t)(gd.tok_base + min(t, Tg - 1)) * a.Hq + head) * 128 + 8 * hh;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
    }

    // key tiles: n1 from the group's first key on, then those of the rows' own segments, from k2 on: the first key of the
    // first response row's segment, unless the prompt's last tile holds it
    const int n1 = ((NAIVE ? t1 : min(Lp, t1)) + BN - 1) / BN;
    const int k2 = max(n1 * BN, b2);
    const int tiles = n1 + (NAIVE || t1 <= Lp ? 0 : max(t1 - k2 + BN - 1, 0) / BN);
    const int from = PIECES ? tiles * piece.part / piece.parts : 0;       // this workgroup's first tile, and how many it walks
    const int total = (PIECES ? tiles * (piece.part + 1) / piece.parts : tiles) - from;
    auto key_at = [&](int it) { return it + from < n1 ? (it + from) * BN : k2 + (it + from - n1) * BN; };

    const int kvh = item.kvh;
    const int64_t kv_stride = (int64_t)a.Hkv * 128;
    const __bf16* kbase = ak + ((int64_t)gd.tok_base * a.Hkv + kvh) * 128;
    const __bf16* vbase = av + ((int64_t)gd.tok_base * a.Hkv + kvh) * 128;

    // Tile copy global -> LDS.  The first wave of each SIMD (w < 4) is served first by the
    // instruction arbiter and reaches the workgroup barrier well ahead of its partner, so those
    // four waves issue all the copies: wave w copies chunks 4w .. 4w+3 (4 rows each) of a 64-row
    // tile.  The per-lane byte offset inside a tile is constant; only the scalar tile base moves.
    // The tile that crosses the end of the group re-reads the group's last row for the rows past it.
    const unsigned stride_b = (unsigned)(kv_stride * 2);
    const bool copier = w < 4;
    unsigned voff[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int row = 4 * (4 * (w & 3) + u) + (l >> 4);
        voff[u] = row * stride_b + (((l & 15) ^ swz(row)) << 4);
    }
    auto sgpr64 = [](const void* p) -> uint64_t {       // a wave-uniform pointer, kept in scalar registers
        const uint64_t b = (uint64_t)(uintptr_t)p;
        return ((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
               (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    };
    const uint64_t kbase_s = sgpr64(kbase), vbase_s = sgpr64(vbase);
    auto lds_u32 = [](char* p) -> unsigned {
        return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)p);
    };
    const unsigned chunk0 = 4096u * (w & 3);
    unsigned m0K[NB], m0V[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) { m0K[b] = lds_u32(ldsKb[b]) + chunk0; m0V[b] = lds_u32(ldsVb[b]) + chunk0; }
    auto issue = [&](uint64_t base_s, unsigned m0dst, int it) {
        if (!copier || it >= total) return;
        const int key0 = key_at(it);
        const uint64_t tb = base_s + (uint64_t)(unsigned)key0 * stride_b;
        if (key0 + BN <= Tg) {
#pragma unroll
            for (int u = 0; u < 4; ++u) async_copy16_sm(tb, voff[u], m0dst + 1024u * u);
        } else {
            const int last = Tg - 1 - key0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int row = 4 * (4 * (w & 3) + u) + (l >> 4);
                const unsigned vo = min(row, last) * stride_b + (((l & 15) ^ swz(row)) << 4);
                async_copy16_sm(tb, vo, m0dst + 1024u * u);
            }
        }
    };
    // true when some (row, key) pair of this wave in tile `it` is masked; tiles past the end
    // of the key range (the pad step of an odd-length loop) are masked entirely
    // the first n_full tiles (whole prompt tiles at or below the wave's first row) never need it
    const int n_full = (!wave_valid || NAIVE) ? 0 : __builtin_amdgcn_readfirstlane(min(min(Lp, tw0 + 1) / BN, n1));
    auto needs_mask = [&](int it) -> bool {
        if (it + from < n_full && (!PIECES || it < total)) return false;
        if (it >= total || !wave_valid || NAIVE) return true;
        const int s0 = key_at(it);
        return !((s0 + BN - 1 <= tw0) && (s0 + BN <= Lp || s0 >= st_last));
    };

    f32x16 oacc[4], sA[2], sB[2];
    unsigned pbA[16], pbB[16]; // P of a tile as packed bf16 pairs, [8*kb + r/2]; the two alternate from step to step
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) { pbA[i] = 0u; pbB[i] = 0u; }
    float m = -INFINITY, lsum = 0.f, lsr = 0.f;
    const float cs = a.c;
    const f32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

    // LDS addresses of the operands within buffer 0, opaque so that they are kept as whole sums; what is added to them
    // below is a constant (the swizzle repeats every 16 rows)
    unsigned rowA[8], trA[4][2];
#pragma unroll
    for (int i = 0; i < 8; ++i) { rowA[i] = lds_u32(ldsKb[0]) + tile_off(c, 2 * i + hh); asm volatile("" : "+v"(rowA[i])); }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int col4 = 32 * db + 16 * c16 + 4 * (j16 & 3);
            trA[db][half] = lds_u32(ldsVb[0]) + tile_off(4 * hh + (j16 >> 2) + 8 * half, col4 >> 3) + ((col4 & 4) << 1);
            asm volatile("" : "+v"(trA[db][half]));
        }
    // operand fetchers, all indices compile-time
    // (QK: the two key blocks in turn, so that pairs of MFMAs share their operand of Q and none waits for its predecessor: under
    // random operands the clock is what the power allows.  16K prompt 3750 -> 3720 us, three sets of eight 2K prompts 7355 -> 7298)
    auto ldK = [&](int buf, int i) -> bf16x8 {         // MFMA i of QK: kb = i % 2, ks = i / 2
        return lds_at_row8(rowA[i >> 1] + TILE_BYTES * buf + 8192 * (i & 1));
    };
    auto ldV = [&](int buf, int i) -> bf16x8 {         // MFMA i of PV: kb = i / 8, mm = (i / 4) % 2, db = i % 4
        const int at = TILE_BYTES * buf + 4096 * (i >> 2);
        return cat4(lds_at_tr4(trA[i & 3][0] + at), lds_at_tr4(trA[i & 3][1] + at));
    };
    auto pbop = [&](const unsigned (&pbw)[16], int kb, int mm) -> bf16x8 {
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        u32x4 x = {pbw[8 * kb + 4 * mm], pbw[8 * kb + 4 * mm + 1], pbw[8 * kb + 4 * mm + 2], pbw[8 * kb + 4 * mm + 3]};
        return __builtin_bit_cast(bf16x8, x);
    };
    auto sum2 = [&](unsigned packed, float acc) -> float {       // acc + both bf16 halves of `packed`
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, packed), one, acc, false);
    };
    auto pack2 = [&](float x, float y) -> unsigned {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        bf16x2 v = {(__bf16)x, (__bf16)y};
        return __builtin_bit_cast(unsigned, v);
    };

    // the first S = K Q^T, ahead of the pipeline
    auto qk_plain = [&](f32x16 (&S)[2]) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            S[i & 1] = mfma32(ldK(0, i), qreg[i >> 1], i < 2 ? zero16 : S[i & 1]);
    };
    auto mask = [&](int it, f32x16 (&S)[2]) {
        const int s0 = it < total ? key_at(it) : 0;
        const int tme = it < total ? tm : -1;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int k0 = s0 + 32 * kb;
            mask16(S[kb], (low_bits(min(Lp, tme + 1) - k0) | (low_bits(tme + 1 - k0) & ~low_bits(st - k0))) >> (4 * hh));
        }
    };

    // one pipeline step for tile j (R = j & 3 selects the LDS buffers): Scur holds S(j), Snext receives S(j+1).
    // Every wave runs every step: tiles it cannot see are handled by the mask (P = 0), the
    // first step multiplies the zero P against a zero-filled V buffer, and the last step's
    // S(j+1) is computed from a stale K buffer and never used.
    //
    // The exponentials of S(j) are taken against the reference point m that the row had BEFORE
    // this tile, so they do not wait for the tile's row maximum and can be spread evenly, one
    // element per MFMA slice, over the 32 MFMAs of the step (16 of O += V(j-1) P(j-1), then 16
    // of S(j+1) = K(j+1) Q^T).  The softmax is shift-invariant, so any finite reference gives
    // the same O and LSE; what has to hold is that the exponentials stay in range.  That is
    // checked after the fact: if a lane's 32 exponentials sum to more than P_LIMIT = 2^14 (or
    // to inf/NaN), the wave takes the exact row maximum as the new reference, rescales O and
    // the row sum, and recomputes this tile's P -- a rare path, taken a few times per row.
    // The LDS operands of the step's 32 MFMAs pass through one ring of RD registers that is read RD - 1
    // MFMAs ahead without a break between the two products: a product that primed its own ring would
    // start with an exposed LDS round trip.  Between the two steps of a barrier interval the ring is
    // carried over as well (BRIDGE: the last slices fetch the first operands of the next step, whose V
    // tile is resident; SECOND: the step finds them there): only the first step behind a barrier primes.
    // (Priming right behind the barrier, ahead of the issue of the tile copies, measured the same.)
    bf16x8 ring[RD];
    auto step = [&](int j, auto par_tag, auto second_tag, auto bridge_tag, f32x16 (&Scur)[2], f32x16 (&Snext)[2],
                    const unsigned (&pbw)[16], unsigned (&pnew)[16]) {
        constexpr int R = decltype(par_tag)::value;
        constexpr bool SECOND = decltype(second_tag)::value, BRIDGE = decltype(bridge_tag)::value;
        constexpr int OFF = SECOND ? 32 % RD : 0;     // ring position of this step's first operand
        if (__builtin_expect(needs_mask(j), 0)) mask(j, Scur);
        __builtin_amdgcn_sched_barrier(0);
        const float mc = m * cs;
        float tsum = 0.f;          // this lane's half of the tile's row sum
        float tsr = 0.f;           // the same sum over the bf16-rounded exponentials (what the MFMA multiplies V by)
        float pe[32];
        // vector-ALU slice e: exponential of element e; the sum and the bf16 packing consume
        // elements issued in earlier slices, so nothing waits on a transcendental just issued
        auto valu = [&](int e) {
            pe[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(Scur[e >> 4][e & 15], cs, -mc));
            asm volatile("" : "+v"(pe[e]));
            if (e >= 1) { tsum += pe[e - 1]; asm volatile("" : "+v"(tsum)); }
            if (e >= 2 && (e & 1) == 0) { pnew[(e - 2) >> 1] = pack2(pe[e - 2], pe[e - 1]); asm volatile("" : "+v"(pnew[(e - 2) >> 1])); }
            if (e >= 3 && (e & 1) == 1) { tsr = sum2(pnew[(e - 3) >> 1], tsr); asm volatile("" : "+v"(tsr)); }
        };
        // operand of slice i: 0..15 the V^T pieces of O^T += V(j-1)^T P(j-1)^T, 16..31 the K rows of
        // S(j+1) = K(j+1) Q^T, 32.. the next step's first V^T pieces
        auto fetch = [&](int i) -> bf16x8 {
            if (i < 16) return ldV((R + NB - 1) % NB, i);            // V(j-1)
            if (i < 32) return ldK((R + 1) % NB, i - 16);            // K(j+1)
            return ldV(R % NB, i - 32);                              // V(j), the next step's
        };
        if (!SECOND) {
#pragma unroll
            for (int i = 0; i < RD - 1; ++i) ring[i] = fetch(i);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            if (i + RD - 1 < 32 || BRIDGE) ring[(i + RD - 1 + OFF) % RD] = fetch(i + RD - 1);
            if (i < 16)     // P operand outermost so that its registers die early
                oacc[i & 3] = mfma32(ring[(i + OFF) % RD], pbop(pbw, i >> 3, (i >> 2) & 1), oacc[i & 3]);
            else
                Snext[i & 1] = mfma32(ring[(i + OFF) % RD], qreg[(i - 16) >> 1], i < 18 ? zero16 : Snext[i & 1]);
            valu(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        tsum += pe[31];
        pnew[15] = pack2(pe[30], pe[31]);
        tsr = sum2(pnew[15], tsr);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(tsum <= P_LIMIT)) != 0, 0)) {
            float mx = Scur[0][0];
#pragma unroll
            for (int e = 1; e < 32; ++e) mx = fmaxf(mx, Scur[e >> 4][e & 15]);
            mx = pair_max(mx);
            const float mnew = fmaxf(m, mx);          // m is always finite
            const float alpha = __builtin_amdgcn_exp2f((m - mnew) * cs);
            lsum *= alpha;
            lsr *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
            m = mnew;
            const float mc2 = mnew * cs;
            tsum = 0.f;
            tsr = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(Scur[q >> 3][(2 * q) & 15], cs, -mc2));
                const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(Scur[q >> 3][((2 * q) & 15) + 1], cs, -mc2));
                tsum += p0 + p1;
                pnew[q] = pack2(p0, p1);
                tsr = sum2(pnew[q], tsr);
            }
        }
        lsum += tsum;
        lsr += tsr;
    };

    // Zero-fill every V buffer that is multiplied against P = 0 before a copy has filled it: the last
    // buffer stands for V(-1) in the first step, and the padded step of an odd count of steps (NW = 8) may find a
    // buffer that no copy has filled.  LDS keeps what earlier
    // workgroups left there (bit patterns that may read as inf or NaN), and 0 * NaN would reach O.
#pragma unroll
    for (int b = 1; b < NB; ++b)
        if (b == NB - 1 || total <= b)
            for (int i = tid; i < TILE_BYTES / 16; i += 64 * NW)
                reinterpret_cast<i32x4*>(ldsVb[b])[i] = i32x4{0, 0, 0, 0};
    if constexpr (NB == 4) {
        issue(kbase_s, m0K[0], 0);
        issue(kbase_s, m0K[1], 1);
        issue(kbase_s, m0K[2], 2);
        issue(vbase_s, m0V[0], 0);
    } else {
        issue(kbase_s, m0K[0], 0);
        issue(kbase_s, m0K[1], 1);
    }
    wait_vm0();
    __syncthreads();
    qk_plain(sA);
    {   // exact row maximum of the first tile as the initial reference point
        if (needs_mask(0)) mask(0, sA);
        float mx = sA[0][0];
#pragma unroll
        for (int e = 1; e < 32; ++e) mx = fmaxf(mx, sA[e >> 4][e & 15]);
        mx = pair_max(mx);
        // A row that sees nothing in this tile (without a prompt: a later response's rows against the first
        // response's keys; PIECES: any row whose keys end ahead of the piece's) starts from a finite sentinel far below any score:
        // the first tile in which it does see a key then overflows the after-check and takes that
        // tile's exact maximum.  (Starting from 0 would let a row whose scores all lie below about
        // -126 / log2(e) underflow to a zero sum.)
        m = (mx == -INFINITY) ? a.m_none : mx;
    }
    int vlast = NB - 1;        // buffer of the last step's V tile
    if constexpr (NB == 4) {
        // Two steps per workgroup barrier: with four K and four V buffers the tiles of the next two
        // steps are copied while these two run.  At the barrier before steps j, j+1 (j even) the tiles
        // V(j-1), V(j), K(j+1), K(j+2) are resident and V(j+1), V(j+2), K(j+3), K(j+4) are issued into
        // the four buffers that the previous two steps read last.  Buffer indices are compile-time, so a turn of the
        // loop is four steps, left after two of them where they are the last; a padded step is fully masked.
        for (int j = 0; j < total; j += 4) {
            wait_vm0();
            __syncthreads();
            issue(vbase_s, m0V[1], j + 1);
            issue(vbase_s, m0V[2], j + 2);
            issue(kbase_s, m0K[3], j + 3);
            issue(kbase_s, m0K[0], j + 4);
            step(j, std::integral_constant<int, 0>{}, std::false_type{}, std::true_type{}, sA, sB, pbA, pbB);
            step(j + 1, std::integral_constant<int, 1>{}, std::true_type{}, std::false_type{}, sB, sA, pbB, pbA);
            if (j + 2 >= total) { vlast = 1; break; }
            wait_vm0();
            __syncthreads();
            issue(vbase_s, m0V[3], j + 3);
            issue(vbase_s, m0V[0], j + 4);
            issue(kbase_s, m0K[1], j + 5);
            issue(kbase_s, m0K[2], j + 6);
            step(j + 2, std::integral_constant<int, 2>{}, std::false_type{}, std::true_type{}, sA, sB, pbA, pbB);
            step(j + 3, std::integral_constant<int, 3>{}, std::true_type{}, std::false_type{}, sB, sA, pbB, pbA);
        }
    } else {
        // One step per barrier.  At the barrier before step j the tiles V(j-1) and K(j+1) are resident
        // (issued a whole step earlier); V(j) and K(j+2) are issued into the buffers that step j-1 read
        // last (V(j-2), and K(j), from which S(j) has been formed).
        for (int j = 0; j < total; j += 2) {
            wait_vm0();
            __syncthreads();
            issue(vbase_s, m0V[0], j);
            issue(kbase_s, m0K[0], j + 2);
            step(j, std::integral_constant<int, 0>{}, std::false_type{}, std::false_type{}, sA, sB, pbA, pbB);
            if (j + 1 >= total) {              // an odd count of steps: P of the last one is in the other registers
#pragma unroll
                for (int i = 0; i < 16; ++i) pbA[i] = pbB[i];
                vlast = 0;
                break;
            }
            wait_vm0();
            __syncthreads();
            issue(vbase_s, m0V[1], j + 1);
            issue(kbase_s, m0K[1], j + 3);
            step(j + 1, std::integral_constant<int, 1>{}, std::false_type{}, std::false_type{}, sB, sA, pbB, pbA);
        }
    }
    wait_vm0();
    __syncthreads();
    // lane indices re-derived behind an opaque barrier: the addresses of everything behind the loop are
    // loop-invariant, and hoisted above the main loop they would cost it registers (they were spilled)
    int lz = l;
    asm volatile("" : "+v"(lz));
    {   // P of the last step that ran (eight waves: the padded one of an odd count) and its V tile
        unsigned tv[4][2];
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int half = 0; half < 2; ++half) tv[db][half] = trA[db][half] + TILE_BYTES * vlast;
        auto ldVz = [&](int i, int half) -> s16x4 { return lds_at_tr4(tv[i & 3][half] + 4096 * (i >> 2)); };
        s16x4 rg[RD][2];
#pragma unroll
        for (int i = 0; i < RD - 1; ++i) { rg[i][0] = ldVz(i, 0); rg[i][1] = ldVz(i, 1); }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i + RD - 1 < 16) { rg[(i + RD - 1) % RD][0] = ldVz(i + RD - 1, 0); rg[(i + RD - 1) % RD][1] = ldVz(i + RD - 1, 1); }
            oacc[i & 3] = mfma32(cat4(rg[i % RD][0], rg[i % RD][1]), pbop(pbA, i >> 3, (i >> 2) & 1), oacc[i & 3]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // O is normalised by the sum of the ROUNDED weights, the ones V was actually multiplied by:
    // a row dominated by one key then returns that key's V exactly, whatever the reference point.
    // LSE uses the unrounded sum.
    const float ltot = pair_sum(lsum);
    const float lrt = pair_sum(lsr);
    const bool store = valid && !(a.resp_only && t < Lp);
    if constexpr (PIECES)
        if (piece.parts > 1) {
            float* const slot = a.pieces.slots + ((int64_t)item.kvh * a.pieces.n_slots + piece.slot) * (int64_t)(ROW_SLOT_BYTES / 4) + w * (ROW_SLOT_BYTES / 16);
#pragma unroll
            for (int n = 0; n < 16; ++n)
                *reinterpret_cast<f32x4*>(slot + 128 * c + 32 * (n >> 2) + 8 * (n & 3) + 4 * hh) =
                    f32x4{oacc[n >> 2][4 * (n & 3)], oacc[n >> 2][4 * (n & 3) + 1], oacc[n >> 2][4 * (n & 3) + 2], oacc[n >> 2][4 * (n & 3) + 3]};
            if (hh == 0) *reinterpret_cast<f32x4*>(slot + 4096 + 4 * c) = f32x4{m, ltot, lrt, store ? 1.f : 0.f};
            return;
        }
    // The K buffers are free from here on (every wave has passed the last barrier and only the last V buffer
    // is still read).  A lane holds 16 pieces of 8 bytes of its row; written to memory directly, one
    // store instruction would touch 32 rows.  Each wave therefore stages its own 32 rows x 256 B in
    // its own 8 KB of LDS (swizzled like the operand tiles: two-way conflicts on the 8-byte writes,
    // which is their minimum, none on the 16-byte reads) and stores whole rows: 16 lanes per row,
    // four rows per instruction.  No workgroup barrier: a wave reads back only what it wrote.
    // Addresses: a granule's place is the row's base with the granule and the row's swizzle xored in, one instruction per access.
    const float inv = 1.0f / lrt;
    const unsigned stage = lds_u32(ldsKb[0]) + 8192u * w;
    const unsigned putA = stage + 256u * (lz & 31) + 8u * (lz >> 5) + (swz(lz & 31) << 4);
    const unsigned getA = stage + 256u * (lz >> 4) + (((lz & 15) ^ ((lz >> 4) << 2)) << 4);
    const bool whole = tw0 + 32 <= Tg && !(a.resp_only && tw0 < Lp);
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    auto store_rows = [&](__bf16* dst, const unsigned (&x)[32]) {
#pragma unroll
        for (int n = 0; n < 16; ++n)
            *(__attribute__((address_space(3))) u32x2*)(uintptr_t)(putA ^ (n << 4)) = u32x2{x[2 * n], x[2 * n + 1]};
        // all eight reads first, then the stores (one LDS round trip instead of eight); the rows of one lane lie
        // four rows apart, so one 64-bit address and a constant stride serve all of them
        bf16x8 y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = lds_at_row8((getA ^ ((i & 3) << 4)) + 1024u * i);
        __builtin_amdgcn_sched_barrier(0);
        __bf16* const p0 = dst + ((int64_t)(gd.tok_base + tw0 + (lz >> 4)) * a.Hq + head) * 128 + 8 * (lz & 15);
        const int64_t stride = (int64_t)4 * a.Hq * 128;
        if (whole) {
#pragma unroll
            for (int i = 0; i < 8; ++i) *reinterpret_cast<bf16x8*>(p0 + i * stride) = y[i];
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int tr = tw0 + 4 * i + (lz >> 4);
                if (tr < Tg && !(a.resp_only && tr < Lp)) *reinterpret_cast<bf16x8*>(p0 + i * stride) = y[i];
            }
        }
    };
    unsigned ob[32];         // o in pairs: [8 db + 2 gq + e / 2]
#pragma unroll
    for (int n = 0; n < 32; ++n) {
        f32x16& x = oacc[n >> 3];
        const int r = 2 * (n & 7);
        x[r] *= inv; x[r + 1] *= inv;
        ob[n] = pack2(x[r], x[r + 1]);
    }
    store_rows(ao, ob);
    if (a.o_lo) {            // what the rounding of o dropped: lets the backward form D from an unrounded o
        // x - bf16(x), which is exact, element by element: as dot products of the pair with {-1, 0} and {0, -1}, half the
        // instructions, an infinite o made its neighbour's residual NaN
#pragma unroll
        for (int n = 0; n < 32; ++n) {
            const f32x16& x = oacc[n >> 3];
            const int r = 2 * (n & 7);
            ob[n] = pack2(x[r] - __uint_as_float(ob[n] << 16), x[r + 1] - __uint_as_float(ob[n] & 0xffff0000u));
        }
        store_rows(a.o_lo, ob);
    }
    if (store && hh == 0)
        alse[(int64_t)head * T_total + gd.tok_base + t] = (m * cs + __log2f(ltot)) * LN2;
}

// Brings the parts of an item's sums (32 rows of one q head) to one reference point, as a workgroup without parts ends: a workgroup per item, 8 threads to a
// row, 16 columns each.
__global__ __launch_bounds__(256) void fwd_pieces_kernel(RowSums list, FwdArgs a) {
    const RowItem it = row_item(list, a.pieces);
    const float* const slot = row_slot(a.pieces, it);
    const int r = threadIdx.x >> 3, d0 = 16 * (threadIdx.x & 7);
    float m = -INFINITY, l = 0.f, lr = 0.f, x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = 0.f;
    if (slot[4096 + 4 * r + 3] == 0.f) return;             // not a row to store
    for (int p = 0; p < it.parts; ++p) m = fmaxf(m, slot[p * (int64_t)(ROW_SLOT_BYTES / 4) + 4096 + 4 * r]);
    for (int p = 0; p < it.parts; ++p) {
        const float* const s = slot + p * (int64_t)(ROW_SLOT_BYTES / 4);
        const f32x4 st = *reinterpret_cast<const f32x4*>(s + 4096 + 4 * r);
        const float f = __builtin_amdgcn_exp2f((st[0] - m) * a.c);
        l += st[1] * f;
        lr += st[2] * f;
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const f32x4 y = *reinterpret_cast<const f32x4*>(s + 128 * r + d0 + 4 * n);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * n + e] += y[e] * f;
        }
    }
    const float inv = 1.0f / lr;
    const int64_t at = ((int64_t)(it.tok + r) * a.Hq + it.head) * 128 + d0;
    bf16x8 o[2], lo[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        x[e] *= inv;
        o[e >> 3][e & 7] = (__bf16)x[e];
        lo[e >> 3][e & 7] = (__bf16)(x[e] - (float)o[e >> 3][e & 7]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        *reinterpret_cast<bf16x8*>(a.o[0] + at + 8 * i) = o[i];
        if (a.o_lo) *reinterpret_cast<bf16x8*>(a.o_lo + at + 8 * i) = lo[i];
    }
    if (d0 == 0) a.lse[0][(int64_t)it.head * a.T_total + it.tok + r] = (m * a.c + __log2f(l)) * LN2;
}

}  // namespace

hipError_t launch_fwd_bf16(const Problem& p, hipStream_t s) {
    FwdArgs a{};
    const int n_sets = p.n_sets > 1 ? p.n_sets : 1;
    for (int i = 0; i < n_sets; ++i) {
        const bool multi = p.n_sets > 1;
        a.q[i] = (const __bf16*)(multi ? p.qs[i] : p.q); a.k[i] = (const __bf16*)(multi ? p.ks[i] : p.k);
        a.v[i] = (const __bf16*)(multi ? p.vs[i] : p.v);
        a.o[i] = (__bf16*)(multi ? p.os[i] : p.o_out); a.lse[i] = multi ? p.lses[i] : p.lse_out;
    }
    a.n_groups = p.n_groups; a.T_total = (int)p.total_tokens; a.sched = p.sched; a.small = p.small;
    const TabArg table = small_table(p);
    a.Hq = p.Hq; a.Hkv = p.Hkv; a.c = p.scale * LOG2E; a.m_none = fmaxf(-1e30f / a.c, -3e38f); a.naive = p.naive; a.resp_only = p.resp_only;
    a.o_lo = n_sets == 1 ? (__bf16*)p.o_lo_out : nullptr;
    // Short key loops: the four-wave shape, two workgroups per CU (see fwd_kernel).  The naive baseline keeps
    // the eight-wave shape whatever the packing (its loops are long by construction).
    const RowPieces* const pieces = p.row_pieces;
    const bool small = !p.naive && (pieces || use_small_shape(p));
    const int bm = small ? 128 : 256;
    const int n_tiles = pieces ? (int)pieces->words.size() : count_tiles(p, bm), per_kv = pieces ? p.Hkv : p.Hq;
    a.items = make_item_map(n_tiles, per_kv, p.Hkv);
    a.blocks_per_set = grid_for_items(n_tiles, per_kv, p.Hkv);
    if (pieces) a.pieces = row_piece_args(p);
    if (a.blocks_per_set % 8 != 0) a.blocks_per_set += 8 - a.blocks_per_set % 8;
    const dim3 grid(a.blocks_per_set * n_sets);
    auto launch = [&](auto small_call) {
        constexpr bool S = decltype(small_call)::value;
        if (p.naive) hipLaunchKernelGGL((fwd_kernel<8, true, S, false>), grid, dim3(512), 0, s, table, a);
        else if (pieces) hipLaunchKernelGGL((fwd_kernel<4, false, S, true>), grid, dim3(256), 0, s, with_list(table, p, pieces->words), a);
        else if (small) hipLaunchKernelGGL((fwd_kernel<4, false, S, false>), grid, dim3(256), 0, s, table, a);
        else hipLaunchKernelGGL((fwd_kernel<8, false, S, false>), grid, dim3(512), 0, s, table, a);
    };
    if (p.small.on) launch(std::true_type{}); else launch(std::false_type{});
    if (pieces) hipLaunchKernelGGL(fwd_pieces_kernel, dim3((unsigned)(pieces->sums.size() / 3 * p.Hkv * 4)), dim3(256), 0, s, row_sums(*pieces), a);
    return hipGetLastError();
}

}  // namespace sp
