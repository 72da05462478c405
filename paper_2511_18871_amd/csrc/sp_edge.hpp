// Exact treatment of the short rows of the backward (bf16 path, gfx950).
//
// The main backward kernels round P and dS to bf16 before the second contraction.  Over a row
// with many keys those roundings average out; a row that sees a handful of keys carries weights of
// order one, so its dQ is a sum of a few large terms whose roundings do not average, and together
// with the bf16 rounding of the output they were the largest relative error of the gradients.
// The mask of Section 4.3 makes those rows easy to name: row t sees n(t) = t + 1 keys on the
// prompt and Lp + (t - st(t)) + 1 in a response, so they are the first rows of each prompt and,
// under a prompt shorter than EDGE, the first rows of each response.  For every row with
// n(t) <= EDGE this kernel recomputes, from the definitions and in fp32,
//   D = sum_s P_s dP_s      (used by the rowsum stage in place of rowsum(dO * O)), and
//   dQ = scale * sum_s dS_s K_s with dS carried into the contraction as a bf16 pair (value +
//        remainder: two MFMAs, error 2^-17); the dq pass does not store those rows.
// (The same rows' contributions to dK / dV get their remainders added inside the dkdv pass.)
//
// Work item = (segment, q head): a segment is a group's prompt or one of its responses.  An item has
// at most EDGE rows and EDGE keys, so every product is 64 x 64 x 128 or smaller.  Its K and V rows come into LDS
// row-contiguous and swizzled like the tiles of the main passes, which serves both the row operands and the transposed
// ones.  Bound by latency (two waves, a dozen loads each, three short products in sequence).  With every operand read
// from global memory in MFMA layout, K^T as 2-byte gathers: 64 prompts, 28 heads 54.4 -> 35.2 us; one prompt, 40
// heads 11.2 -> 8.9 us (one box).
#pragma once
#include "sp_common.hpp"
#include "sp_launch.hpp"

namespace sp {

constexpr int EDGE = EDGE_LEN;       // 64: two 32-wide MFMA blocks each way

// Segment of a response item: items enumerate the table's response-offset words (a group's G + 1
// words: its prompt's word, j = 0, then one per response); the group is the one whose words hold it.
__device__ __forceinline__ void edge_item_segment(const int* __restrict__ tab, int n_groups, int item, int& g, int& j) {
    const int word = TAB_HEADER + TAB_GROUP_WORDS * n_groups + item;
    int lo = 0, hi = n_groups;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tab[TAB_HEADER + TAB_GROUP_WORDS * mid + 3] <= word) lo = mid; else hi = mid;
    }
    g = lo;
    j = word - tab[TAB_HEADER + TAB_GROUP_WORDS * g + 3];
}

// value + remainder as two bf16 octets (elements e0 .. e0+7 of x)
__device__ __forceinline__ void split8(const f32x16& x, int e0, bf16x8& hi, bf16x8& lo) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const __bf16 h = (__bf16)x[e0 + i];
        hi[i] = h;
        lo[i] = (__bf16)(x[e0 + i] - (float)h);
    }
}

struct EdgeArgs {
    const __bf16* q; const __bf16* k; const __bf16* v; const __bf16* d_o; const float* lse;
    float* nD;                       // the plane of -D
    __bf16* dq;
    const int* tab;
    int64_t T_total;
    int n_groups, Hq, Hkv;
    float scale;
    int n_prompts;                   // prompt items (one per group); the response items follow
    int64_t n_pairs;                 // (item, q head) pairs of both
};
constexpr int64_t EDGE_MAX_BLOCKS = 1 << 22;  // more pairs than that go round the workgroups
constexpr int EDGE_LDS = 2 * EDGE * 256;      // K and V rows of a pair

// Rows of one pair that see at most EDGE keys: D, and with WITH_DQ their dQ.  128 threads: wave rb of them owns rows
// 32 rb .. 32 rb + 31 of the item (lane c = row, S^T orientation: a lane holds one row's scores for 16 keys of a 32-key
// block).  Every thread of the workgroup calls it (it holds a barrier); pairs past the last have no rows.
template <bool WITH_DQ>
__device__ __forceinline__ void short_rows_body(const EdgeArgs& a, int64_t pair, int rb, char* lds) {
    char* const ldsK = lds;
    char* const ldsV = lds + EDGE * 256;
    const bool some = pair < a.n_pairs;
    const int item = some ? (int)(pair / a.Hq) : 0, h = some ? (int)(pair - (int64_t)item * a.Hq) : 0;
    const int Hq = a.Hq, Hkv = a.Hkv;
    const int64_t T_total = a.T_total;
    const float scale = a.scale;
    int g = item, j = 0;                             // prompt items: found directly
    if (item >= a.n_prompts) edge_item_segment(a.tab, a.n_groups, item - a.n_prompts, g, j);
    const GroupDesc gd = load_group(a.tab, g);
    // (a response item's j = 0 is its group's prompt: not its work)
    const bool mine = some && j <= gd.G && (j > 0 || item < a.n_prompts);
    const int seg0 = !mine || j == 0 ? 0 : gd.roff[j - 1], seg1 = !mine ? 0 : j == 0 ? gd.Lp : gd.roff[j];
    const int base_keys = j == 0 ? 0 : gd.Lp;        // prompt keys that every row of this segment sees
    const int n_rows = min(seg1 - seg0, EDGE - base_keys);               // rows with at most EDGE keys
    const int l = threadIdx.x & 63, c = l & 31, hh = l >> 5;
    const int n_keys = base_keys + n_rows;           // keys seen by the last of these rows
    const int kvh = h / (Hq / Hkv);
    // key number x (0 .. n_keys - 1) -> group-local token: the prompt's keys, then the segment's own
    auto key_tok = [&](int x) { x = min(x, n_keys - 1); return x < base_keys ? x : seg0 + (x - base_keys); };
    const int r = 32 * rb + c;                       // this lane's row within the segment
    const int64_t tok = gd.tok_base + min(seg0 + max(min(r, n_rows - 1), 0), gd.Tg - 1);     // a row of the group in any case
    // K and V rows of the 32-key blocks in use -> LDS, 4 rows per copy (keys past n_keys repeat the last one)
    for (int ci = rb; n_rows > 0 && ci < (n_keys > 32 ? 16 : 8); ci += 2) {
        const int row = 4 * ci + (l >> 4);
        const int64_t off = ((gd.tok_base + (int64_t)key_tok(row)) * Hkv + kvh) * 128 + ((l & 15) ^ swz(row)) * 8;
        async_copy16(a.k + off, ldsK + 1024 * ci);
        async_copy16(a.v + off, ldsV + 1024 * ci);
    }
    const __bf16* qr = a.q + (tok * Hq + h) * 128 + 8 * hh;
    const __bf16* gr = a.d_o + (tok * Hq + h) * 128 + 8 * hh;
    bf16x8 qf[8], gf[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        qf[ks] = *reinterpret_cast<const bf16x8*>(qr + 16 * ks);
        gf[ks] = *reinterpret_cast<const bf16x8*>(gr + 16 * ks);
    }
    const float L = a.lse[(int64_t)h * T_total + tok];
    wait_vm0();
    __syncthreads();
    if (32 * rb >= n_rows) return;
    const f32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    f32x16 P[2], dP[2];                              // per 32-key block; element e: key 32 kb + 8 (e / 4) + 4 hh + e % 4
    float acc = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        P[kb] = zero16; dP[kb] = zero16;
        if (32 * kb >= n_keys) continue;
        f32x16 S = zero16;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            S = mfma32(lds_read_row8(ldsK, 32 * kb + c, 2 * ks + hh), qf[ks], S);
            dP[kb] = mfma32(lds_read_row8(ldsV, 32 * kb + c, 2 * ks + hh), gf[ks], dP[kb]);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int x = 32 * kb + 8 * (e >> 2) + 4 * hh + (e & 3);
            const bool ok = r < n_rows && x <= base_keys + r;
            P[kb][e] = ok ? __expf(S[e] * scale - L) : 0.f;
            acc += P[kb][e] * dP[kb][e];
        }
    }
    const float Dr = pair_sum(acc);                  // both lanes of a row hold its D
    if (r < n_rows && hh == 0) a.nD[(int64_t)h * T_total + tok] = -Dr;      // the plane holds -D
    if (!WITH_DQ) return;

    // dQ^T (d x rows) = scale * K^T (d x keys) dS^T (keys x rows), dS = P (dP - D) in fp32, fed as value + remainder
    f32x16 dqa[4] = {zero16, zero16, zero16, zero16};
    const int j16 = l & 15, c16 = (l >> 4) & 1;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        if (32 * kb >= n_keys) continue;
        f32x16 dS;
#pragma unroll
        for (int e = 0; e < 16; ++e) dS[e] = P[kb][e] * (dP[kb][e] - Dr);
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
            bf16x8 hi, lo;
            split8(dS, 8 * mm, hi, lo);
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                const int row4 = 32 * kb + 16 * mm + 4 * hh + (j16 >> 2), col4 = 32 * db + 16 * c16 + 4 * (j16 & 3);
                const bf16x8 A = cat4(lds_read_tr4(ldsK, row4, col4), lds_read_tr4(ldsK, row4 + 8, col4));
                dqa[db] = mfma32(A, hi, dqa[db]);
                dqa[db] = mfma32(A, lo, dqa[db]);
            }
        }
    }
    if (r < n_rows) {
        __bf16* op = a.dq + (tok * Hq + h) * 128 + 4 * hh;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                bf16x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = (__bf16)(dqa[db][4 * gq + e] * scale);
                *reinterpret_cast<bf16x4*>(op + 32 * db + 8 * gq) = x;
            }
    }
}

// workgroups for all pairs at `per_block` pairs each
inline int edge_blocks(const EdgeArgs& a, int per_block) {
    const int64_t n = (a.n_pairs + per_block - 1) / per_block;
    return (int)(n < EDGE_MAX_BLOCKS ? n : EDGE_MAX_BLOCKS);
}

inline EdgeArgs edge_args(const Problem& p) {
    EdgeArgs a{};
    a.q = (const __bf16*)p.q; a.k = (const __bf16*)p.k; a.v = (const __bf16*)p.v; a.d_o = (const __bf16*)p.d_o;
    a.lse = p.lse; a.nD = p.Dbuf; a.dq = (__bf16*)p.dq; a.tab = p.tab; a.T_total = p.total_tokens;
    a.n_groups = p.n_groups; a.Hq = p.Hq; a.Hkv = p.Hkv; a.scale = p.scale;
    a.n_prompts = p.resp_only ? 0 : p.n_groups;      // in response-rows mode prompt rows take no part
    // responses: their first rows qualify only under a prompt shorter than EDGE
    const int64_t responses = p.min_prompt_len < EDGE && p.total_responses > 0 ? p.n_groups + p.total_responses : 0;
    a.n_pairs = (a.n_prompts + responses) * p.Hq;
    return a;
}

}  // namespace sp
